"""Barriers of the LDS pipelines, checked in the kernel sources (CPU).

A stage that direct loads (global_load_lds) refill has to be read completely first, in every
wave: the barrier in front of the refill waits for the wave's LDS reads itself (stage_barrier),
since the compiler does not see the direct loads as LDS writes.  Only a pipeline's first barrier,
behind the prologue's loads (`wait_vm((pro - 1) * ...)`), has no reads before it.
"""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2101_06385_amd", "csrc")


def _code(path):
    with open(path) as f:
        return re.sub(r"//[^\n]*", "", f.read())


SOURCES = {os.path.basename(p): _code(p) for p in sorted(glob.glob(os.path.join(CSRC, "*.h")) +
                                                         glob.glob(os.path.join(CSRC, "*.hip")))}
PIPELINES = [n for n, s in SOURCES.items() if re.search(r"wait_vm(<\w+>)?\([^;]*\);\s*(__syncthreads|stage_barrier)", s)]


def test_the_pipelines_are_found():
    assert {"k_square_sk.h", "k_square_f64.hip", "k_square_f32.hip", "k_adjoint.hip"} <= set(PIPELINES)


@pytest.mark.parametrize("name", PIPELINES)
def test_refilled_stages_wait_for_their_reads(name):
    waits = re.findall(r"wait_vm(?:<[^;>]*>)?\(([^;]*)\);\s*(\w+)\(", SOURCES[name])
    assert any(barrier == "stage_barrier" for _, barrier in waits)
    for outstanding, barrier in waits:
        assert barrier != "__syncthreads" or "pro - 1" in outstanding, (name, outstanding)


def test_stage_barrier_waits_for_lds_reads():
    defs = [(n, m) for n, s in SOURCES.items() for m in re.findall(r"void stage_barrier\(\)\s*\{([^}]*)\}", s)]
    assert len(defs) == 1, defs
    assert re.search(r"lgkmcnt\(0\).*s_barrier", defs[0][1])
