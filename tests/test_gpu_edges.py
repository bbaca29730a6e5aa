"""GPU parity at the sizes where the kernels' splits begin and end, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import spion_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_2309_12578_amd as sp
    sp.load()
    return sp


def _same_pattern(sp, A, block, filt, mode, value, flags=0, variant="CF"):
    ref = oracle.generate_pattern(A, block, filt, mode, value, variant=variant)
    pat = sp.generate_pattern(torch.from_numpy(A).cuda(), block, filt, mode, value, flags=flags)
    n = ref["nnzb"]
    assert pat.nnzb == n and int(pat.nnzb_dev.item()) == n
    for name in ("pool_sum", "fl_out", "row_ptr", "col_ptr"):
        assert np.array_equal(getattr(pat, name).cpu().numpy(), ref[name]), name
    for name in ("col_idx", "row_idx", "bsr_pos"):
        assert np.array_equal(getattr(pat, name).cpu().numpy()[:n], ref[name]), name


# 1 .. 64 block rows: one workgroup, rows of one word (of which waves own four, the fill takes eight);
# above: several kernels, words of 64 columns, fill pieces of 32 rows; block 16 / 32 / 64: four / two / one
# block side by side in a wave of the convolution, the last of them beyond the matrix
@pytest.mark.parametrize("nb,block", [(1, 16), (3, 32), (5, 16), (31, 32), (63, 16), (64, 16), (65, 16), (96, 16),
                                      (127, 32), (129, 16), (33, 64), (193, 16)])
@pytest.mark.parametrize("ties", [False, True])
def test_pattern_at_the_edges_of_the_splits(sp, nb, block, ties):
    L = nb * block
    rng = np.random.default_rng(nb * 100 + block)
    if ties:
        A = (rng.integers(0, 4, size=(L, L)) / 4.0).astype(np.float32)
        A = np.repeat(np.repeat(A[::block, ::block], block, axis=0), block, axis=1)   # few distinct pooled sums
    else:
        A = (rng.random((L, L), dtype=np.float32) ** 6).astype(np.float32)
    A = np.ascontiguousarray(A)
    p_max = 2 * block - 1
    _same_pattern(sp, A, block, min(31, p_max), si.T_QUANTILE, 0.8)
    _same_pattern(sp, A, block, 1, si.T_MEAN_KSTD, 0.5)
    _same_pattern(sp, A, block, p_max, si.T_ABS, float(A.mean()) * p_max)
    _same_pattern(sp, A, block, 5, si.T_QUANTILE, 0.9, flags=sp.SPION_PATTERN_NO_FILL, variant="C")
