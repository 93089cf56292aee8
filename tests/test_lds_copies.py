"""Direct copies from memory to LDS must have landed before a barrier publishes them.

A wave's copies are counted by its vector-memory counter, and a workgroup barrier orders LDS reads and writes but
waits for no copy by itself.  The kernels that use them are compiled here and every path through their code is
followed: no barrier may be reached with a copy in flight."""
import os
import re
import subprocess

import pytest

from paper_2605_06676_amd import build as B

COPY = re.compile(r"^(global_load_lds|buffer_load_\w+ .*\blds\b)")
BRANCH = re.compile(r"^s_(c?branch\w*)\s+(\S+)")


def functions(text):
    """name -> list of (label or None, instruction or None), in order, for every function of the listing."""
    out, name, body = {}, None, []
    for line in text.splitlines():
        line = line.split(";")[0].rstrip()
        label = re.match(r"^([\w.$]+):", line)
        if label and not label.group(1).startswith("."):
            name, body = label.group(1), []
            out[name] = body
        elif label and label.group(1).startswith(".Lfunc_end"):
            name = None
        elif name is not None and label:
            body.append((label.group(1), None))
        elif name is not None and line.startswith("\t") and not line.strip().startswith("."):
            body.append((None, line.strip()))
    return out


def barriers_with_a_copy_in_flight(body):
    """Positions of the barriers that some path reaches after a copy without a wait for all vector memory."""
    at_label = {label: i for i, (label, _) in enumerate(body) if label}
    seen, todo, bad, n_copies = set(), [(0, False)], set(), 0
    while todo:
        i, flying = todo.pop()
        while i < len(body) and (i, flying) not in seen:
            seen.add((i, flying))
            ins = body[i][1]
            if ins is None:
                i += 1
                continue
            if COPY.match(ins):
                flying = True
                n_copies += 1
            elif ins.startswith("s_waitcnt") and re.search(r"vmcnt\(0\)", ins):
                flying = False
            elif ins.startswith("s_barrier") and flying:
                bad.add(i)
            elif ins.startswith("s_endpgm"):
                break
            jump = BRANCH.match(ins)
            if jump:
                if jump.group(1) == "branch":
                    i = at_label[jump.group(2)]
                    continue
                todo.append((at_label[jump.group(2)], flying))
            i += 1
    return bad, n_copies


def test_the_check_itself():
    loop = "k:\n.L0:\n\t{}s_barrier\n\tglobal_load_lds_dword v0, s[0:1]\n\ts_cbranch_scc1 .L0\n\ts_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier\n\ts_endpgm\n"
    for wait, expected in (("", 1), ("s_waitcnt lgkmcnt(0)\n\t", 1), ("s_waitcnt vmcnt(0)\n\t", 0)):
        bad, copies = barriers_with_a_copy_in_flight(functions(loop.format(wait))["k"])
        assert len(bad) == expected and copies > 0, wait


@pytest.mark.parametrize("source,kernel", [("masked_attn.hip", "masked_attn_fwd_kernel"),
                                           ("masked_attn_bwd.hip", "masked_attn_bwd_dkv_kernel"),
                                           ("masked_attn_bwd.hip", "masked_attn_bwd_dq_kernel")])
def test_no_barrier_with_a_copy_in_flight(tmp_path, source, kernel):
    listing = tmp_path / "kernel.s"
    flags = [f for f in B.FLAGS if f != "-shared"]
    subprocess.run([B.HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(B.CSRC, source), "-o", str(listing)],
                   check=True, capture_output=True, text=True)
    names = [(n, b) for n, b in functions(listing.read_text()).items() if kernel in n and any(x[1] for x in b)]
    assert names
    for name, body in names:
        bad, copies = barriers_with_a_copy_in_flight(body)
        assert copies > 0, name
        assert not bad, f"{name}: {len(bad)} barriers reached with a copy in flight"
