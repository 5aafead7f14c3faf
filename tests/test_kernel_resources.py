"""What the compiler needs for the sampling kernels: registers kept in scratch memory.  A kernel of 1024 threads has
128 registers per thread; the ones that loop over rows spill every address of the loop if it is left to the compiler,
and the recursion over whole rows did so with the running target in registers (326 spilled, 1.7 times the time)."""
import os
import re
import subprocess

import pytest

from paper_2510_25739_amd import build

SPILLS = 64   # per-thread values that one row's pass reloads once; beyond that the entries themselves are spilled


def test_sampling_kernels_keep_their_entries_in_registers(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    cmd = [build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(build.CSRC, "sampling.hip"), "-o", str(tmp_path / "sampling.o")]
    report = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    spills = {name: int(n) for name, n in re.findall(r"Function Name: (\S+).*?VGPRs Spill: (\d+)", report, flags=re.S)}
    assert any("multi_verify_kernel" in k for k in spills) and any("multi_verify_greedy_kernel" in k for k in spills)
    assert {k: n for k, n in spills.items() if n > SPILLS} == {}
    assert all(n <= 1 for k, n in spills.items() if "multi_verify_kernel" not in k), spills


def test_draft_kernel_of_one_round_does_not_carry_a_second(tmp_path):
    # The output projection of a draft micro-step holds the weights of two rounds of jobs.  Slices of one round have a
    # kernel without the second one's registers and barriers: with an empty second job 12 and 16 sequences took 2 to 3 %
    # longer.  A job is 2 strips of 10 tiles a wave at the XL widths, 3 of 6 at the B widths: 80 and 72 registers of a lane.
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    cmd = [build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(build.CSRC, "stream.hip"), "-o", str(tmp_path / "stream.o")]
    report = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    use = {name: int(n) for name, n in re.findall(r"Function Name: (\S+draft_stream_kernel\S+).*? VGPRs: (\d+)", report, flags=re.S)}
    one, pair = [n for k, n in use.items() if "ELb0E" in k], [n for k, n in use.items() if "ELb1E" in k]
    assert len(one) == 2 and len(pair) == 2 and max(one) <= min(pair) - 60, use


def test_draft_chain_keeps_its_weights_in_registers(tmp_path):
    # A lane of the chain keeps 52 registers of weights at the XL widths, 32 at the B widths, and 4, 8 or 16 entries of a row while
    # it draws.  What is spilled today, XL and 16 entries: 30, of which 16 are four tiles that a workgroup that draws saves
    # around the call and seven pairs are addresses, two of them read back in a micro-step.  One more tile is four.
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    cmd = [build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(build.CSRC, "chain.hip"), "-o", str(tmp_path / "chain.o")]
    report = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    spills = {(int(t), int(e)): int(n) for t, e, n in
              re.findall(r"Function Name: \S+draft_chain_kernelILi(\d+)ELi(\d+)E.*?VGPRs Spill: (\d+)", report, flags=re.S)}
    assert set(spills) == {(t, e) for t in (6, 10) for e in (4, 8, 16)}
    most = {(10, 16): 30, (10, 8): 4, (6, 16): 8}
    assert {k: n for k, n in spills.items() if n >= most.get(k, 0) + 4} == {}


def test_assembly_that_writes_m0_says_so():
    # the compiler does not look into an asm block: it has to be told that what it last put into M0 is gone
    blocks = []
    for src in build.SOURCES:
        text = open(os.path.join(build.CSRC, src)).read()
        blocks += [b for b in re.findall(r"asm(?: volatile)?\((.*?)\);\n", text, flags=re.S) if "_b32 m0" in b]
    assert blocks and all('"m0"' in b.rpartition(":")[2] for b in blocks), blocks
