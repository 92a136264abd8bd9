"""Host-side logic that needs no GPU: the one-GPU contract of bench.py and the CU-mask builder."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""


@pytest.mark.parametrize("style", ["contiguous", "interleaved"])
@pytest.mark.parametrize("counts", [[64, 64, 64, 64], [48, 48, 48, 48, 64], [128, 128], [8, 8, 8, 8, 224], [256]])
def test_cu_masks_partition_the_device(style, counts):
    from paper_2206_08482_amd.instances import cu_masks
    masks = cu_masks(256, counts, style)
    ints = [sum(w << (32 * i) for i, w in enumerate(m)) for m in masks]
    assert [bin(x).count("1") for x in ints] == counts
    for i in range(len(ints)):
        for j in range(i):
            assert ints[i] & ints[j] == 0                      # disjoint
    assert sum(ints) == (1 << sum(counts)) - 1 if style == "contiguous" else True
    for x in ints:      # every instance keeps compute units on each of the 8 dies (bit index mod 8 = die)
        per_die = [sum((x >> b) & 1 for b in range(d, 256, 8)) for d in range(8)]
        assert min(per_die) >= 1 and max(per_die) - min(per_die) == 0      # and the same number on every die


def test_cu_masks_reject_counts_that_are_not_whole_rows():
    from paper_2206_08482_amd.instances import cu_masks
    with pytest.raises(ValueError):
        cu_masks(256, [60, 60], "contiguous")                  # not a multiple of 8: some die would get fewer CUs
    with pytest.raises(ValueError):
        cu_masks(256, [128, 136], "contiguous")                # more than the device has


def test_kernel_attributes_are_set_per_device():
    """The dynamic-LDS limit of a kernel belongs to one device; a process may hold instances on several.  Every launcher
    goes through allow_lds, which keeps a set of devices per kernel."""
    csrc = os.path.join(ROOT, "paper_2206_08482_amd", "csrc")
    with_call = [f for f in sorted(os.listdir(csrc)) if "hipFuncSetAttribute" in open(os.path.join(csrc, f)).read()]
    assert with_call == ["core.hip"]


def test_inline_assembly_names_the_registers_it_writes():
    """Instructions that take an LDS address from m0 are preceded by a write of m0 in the same statement, and the compiler is told of it."""
    csrc = os.path.join(ROOT, "paper_2206_08482_amd", "csrc")
    in_statements = everywhere = 0
    for f in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, f)).read()
        everywhere += text.count("global_load_lds")
        for stmt in re.findall(r"asm volatile\((.*?)\);", text, re.S):
            loads, writes = stmt.count("global_load_lds"), len(re.findall(r"\bs_\w+ m0\b", stmt))
            in_statements += loads
            assert writes == loads, (f, stmt)
            if writes:
                assert re.search(r':[^:]*"m0"[^:]*$', stmt), (f, stmt)
    assert in_statements == everywhere > 0
