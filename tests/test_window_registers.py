"""Registers of the window kernels: what is spilled is waited for when it is read back, and with it everything that was asked for since, the next row's
loads among them.  So no kernel that a rule chooses uses scratch memory, by the compiler's resource report."""
import os
import re
import subprocess

from paper_2301_08984_amd import build as B


def scratch_bytes(source, tmp_path):
    """{(template arguments): bytes of scratch per lane} of the kernels of a source file"""
    r = subprocess.run(["hipcc", *B.FLAGS, *B.EXTRA_FLAGS.get(source, []), "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(B.CSRC, source), "-o", os.path.join(tmp_path, "k.o")], check=True, capture_output=True, text=True)
    out = {}
    for block in r.stderr.split("Function Name: ")[1:]:
        args = re.search(r"kernelI((?:L[ib]\d+E)+)E", block.split()[0])
        out[tuple(int(x) for x in re.findall(r"L[ib](\d+)E", args.group(1)))] = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", block).group(1))
    return out


def test_forward(tmp_path):
    scratch = scratch_bytes("win_fwd.hip", tmp_path)
    assert len(scratch) == 9 * 8  # blocks of 16 tokens, regions, bias, statistics
    assert {k: v for k, v in scratch.items() if v} == {}


def test_backward(tmp_path):
    """12 bytes at most: an address that only the start and the end of a work-group use, or one reload in two rows."""
    scratch = scratch_bytes("win_bwd.hip", tmp_path)
    assert len(scratch) == 9 * 8  # blocks of 16 tokens, regions, bias, gate
    assert {k: v for k, v in scratch.items() if v > 12} == {}
