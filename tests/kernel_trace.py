"""Names of the kernels that a call launches on the GPU, for tests of the dispatch: results alone
do not show which kernel made them."""
import re

import pytest
import torch


def traced(fn):
    """Kernels launched by fn(), in order, as 'name<template arguments>' without their namespace;
    None where the profiler sees no kernel, so that a parity test still checks its results."""
    fn()                                   # first-use work of the runtime stays out of the trace
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    names = [e.name for e in sorted(prof.events(), key=lambda e: e.time_range.start)]
    return [m.group(1) for m in (re.search(r"(\w+_kernel(?:<[^(]*>)?)\(", n) for n in names) if m] or None


def kernels(fn):
    """The same for tests that are about nothing else."""
    names = traced(fn)
    if names is None:
        pytest.skip("the profiler saw no kernel")
    return names
