"""The sampler's carry chains keep the wait states of gfx950 (CPU: the kernel is compiled
to assembly, no GPU).  A vector instruction that reads a carry mask needs two wait states after
the vector instruction that wrote it.  The compiler inserts them into its own code and does
not look into inline assembly, so the whole file is scanned: straight-line code between
labels, an s_nop of N for N + 1 states, any other instruction for one."""
import os
import re
import subprocess

import pytest

from paper_2503_12749_amd import build

READS_LAST = re.compile(r"v_(addc|subb|subbrev)_co_u32|v_cndmask_b32")
WRITES_SECOND = re.compile(r"v_(add|addc|sub|subb|subrev|subbrev)_co_u32|v_mad_[ui]64|v_div_scale")
MASK = re.compile(r"vcc|s\[\d+:\d+\]|s\d+")


def _short_waits(text):
    """(line number, line) of every carry read less than two wait states after its write."""
    bad, now, written = [], 0, {}
    for number, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].strip()
        if line.endswith(":"):
            written = {}
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ") if " " in line else line.partition("\t")
        args = [a.strip() for a in re.split(r",(?![^\[]*\])", rest)]
        now += int(args[0], 0) + 1 if op == "s_nop" else 1
        if READS_LAST.match(op) and args[-1] in written and now - written[args[-1]] < 3:
            bad.append((number, line))
        masks = [a for a in args[:2] if MASK.fullmatch(a)]
        if op.startswith("v_cmp"):
            written[masks[0] if masks and masks[0] == args[0] else "vcc"] = now
        elif WRITES_SECOND.match(op):
            written[args[1]] = now
        elif op.startswith("s_") and args:
            written.pop(args[0], None)
    return bad


def test_scan_finds_a_chain_without_waits():
    """The scan itself, on the smallest chains of either kind."""
    chain = "v_add_co_u32 v0, vcc, v1, v2\n{}v_addc_co_u32 v3, vcc, v4, v5, vcc\n"
    assert _short_waits(chain.format("")) and _short_waits(chain.format("s_nop 0\n"))
    assert not _short_waits(chain.format("s_nop 1\n"))
    assert not _short_waits(chain.format("v_mov_b32 v9, v8\ns_nop 0\n"))
    other = "v_mad_u64_u32 v[0:1], s[4:5], s1, v2, v[3:4]\n{}v_addc_co_u32 v6, vcc, 0, v6, s[4:5]\n"
    assert _short_waits(other.format("s_mov_b32 s9, 0\n"))
    assert not _short_waits(other.format("s_mov_b32 s9, 0\ns_mov_b32 s8, 0\n"))


def test_sampler_carries_are_waited_for(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "sample.txt"
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, "sample.hip"), "-o", str(out)], check=True,
                   stderr=subprocess.DEVNULL)
    text = out.read_text()
    assert len(re.findall(r"v_mad_u64_u32", text)) > 100  # the generator's products
    assert _short_waits(text) == []
