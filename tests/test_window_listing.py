"""The window scorer's kernel as compiled: no integer remainders among the arithmetic of its keys."""
import os
import subprocess

from paper_2605_06676_amd import build as B
from tests.test_lds_copies import functions


def test_places_in_the_window_take_no_integer_division(tmp_path):
    listing = tmp_path / "kernel.s"
    flags = [f for f in B.FLAGS if f != "-shared"]
    subprocess.run([B.HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(B.CSRC, "score_window.hip"), "-o", str(listing)],
                   check=True, capture_output=True, text=True)
    text = listing.read_text()
    names = [n for n in functions(text) if "score_window_kernel" in n]
    assert len(names) == 8
    for name in names:
        body = text[text.index("\n" + name + ":"):]
        body = body[:body.index(".Lfunc_end")]
        # every division by a number that is not constant begins with this reciprocal; the block's place in its head and
        # the window's reciprocal are three of them, whatever the number of rows
        assert body.count("v_rcp_iflag_f32") <= 3, (name, body.count("v_rcp_iflag_f32"))
