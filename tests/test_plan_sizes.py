"""Workspace sizes and plan names that callers of the automatic prefill hold.

A caller may have stored a size, and the no-allocation call takes what fits its
64 MiB, so neither may depend on the tiling of the kernel that runs.
"""
import pytest

import paper_2310_18780_amd as lh


@pytest.mark.parametrize(
    "shape, size, plans",
    [
        ((12, 3240, 16, 10752), 60134400, ("mfma", "mfma")),
        ((8, 1712, 32, 2944), 53030912, ("mfma", "mfma")),
        ((5, 1904, 32, 6016), 58978304, ("mfma", "mfma")),
        ((8, 664, 64, 8192), 37056512, ("mfma", "scan")),
        ((3, 1136, 64, 36288), 63397888, ("mfma", "scan")),
    ],
)
def test_sizes_within_the_static_scratch_stay_within_it(shape, size, plans):
    assert lh.workspace_bytes(*shape) == size < 64 << 20
    assert tuple(lh.prefill_plan(*shape, io=io) for io in ("f32", "bf16")) == plans
