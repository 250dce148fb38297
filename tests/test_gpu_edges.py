"""GPU parity at the sizes where a kernel or a launch rule changes its way:
streams, perms and decodes byte-identical to the CPU oracle's."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import Oracle
from test_gpu_parity import check_parity, gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bbx():
    import paper_2404_02826_amd as b
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    b.load()
    return b


@pytest.fixture(scope="module")
def orc():
    return Oracle()


# Nodes of the fused pairs that start off a 16-byte boundary, with room for
# the slots before them, exactly filling the capacity with them, and too large
# for them (single loads); one wavefront (1,024 slots) and four (4,096).
@pytest.mark.parametrize("n", [2 * 513, 2 * 1019 + 1, 2 * 1020, 2 * 1021, 2 * 1023, 2 * 2049 + 1,
                               2 * 4092, 2 * 4093, 4 * 4095 + 1])
@pytest.mark.parametrize("kind,dims,eb", [("cosmology", 3, 1e-4), ("ties", 3, 1e-2),
                                          ("cosmology", 2, 1e-3), ("cosmology", 3, 1e-6)])
def test_fused_pair_alignment(bbx, orc, n, kind, dims, eb):
    dtype = np.float64 if eb < 1e-5 else np.float32  # 32-bit codes
    pts = gen(kind, n, dims, dtype, seed=n)
    for want_perm in (False, True):
        check_parity(orc, bbx, pts, eb, "rel", 32, want_perm=want_perm)
