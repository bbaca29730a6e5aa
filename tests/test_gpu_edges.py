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
    sp.binding._native()   # tests use it by name, in any order
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
# above: several kernels, words of 64 columns, fill pieces of 64 steps (rows + words of 32 - 1); block 16 / 32 / 64: four / two / one
# block side by side in a wave of the convolution, the last of them beyond the matrix
@pytest.mark.parametrize("nb,block", [(1, 16), (3, 32), (5, 16), (31, 32), (63, 16), (64, 16), (65, 16), (96, 16),
                                      (125, 16), (126, 16), (127, 32), (129, 16), (33, 64),
                                      (193, 16)])
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


# One and two cells a thread of the kernel that counts; bins: negative values, 0, octaves below and above the first that
# is divided, its edges, one value throughout, ties at the rank
@pytest.mark.parametrize("nb", [65, 255, 300])
@pytest.mark.parametrize("kind", ["octaves", "edges", "near", "equal"])
@pytest.mark.parametrize("q", [0.0, 0.37, 0.9, 1.0])
def test_quantile_of_large_grids(sp, nb, kind, q):
    rng = np.random.default_rng(nb)
    n = nb * nb
    if kind == "octaves":
        pool = (rng.choice((-1, 1, 1, 1), n) * (2.0 ** rng.uniform(0, 58.9, n))).astype(np.int64)
        pool[rng.integers(0, n, 50)] = 0
    elif kind == "edges":
        edges = [s * ((1 << e) + d) for e in (1, 31, 32, 33, 58) for d in (-1, 0, 1, (1 << e) >> 7, ((1 << e) >> 7) - 1) for s in (-1, 1)]
        pool = rng.choice(np.array(edges, dtype=np.int64), n)
    elif kind == "near":
        pool = (1 << 40) + rng.integers(0, 1 << 30, n)
    else:
        pool = np.full(n, 12345, dtype=np.int64)
    L, block = nb * 16, 16
    dev = torch.from_numpy(pool.reshape(nb, nb)).cuda()
    z = lambda m, t=torch.int32: torch.zeros(m, dtype=t, device="cuda")
    fl, nnzb = z((nb, nb), torch.uint8), z(1)
    ws = torch.empty(sp.spion_pattern_workspace_bytes(L, block), dtype=torch.uint8, device="cuda")
    sp.spion_pattern(None, L, block, 1, sp.SPION_T_QUANTILE, q, fl, z(nb + 1), z(n), z(nb + 1), z(n), z(n), nnzb, dev, ws,
                     flags=sp.SPION_PATTERN_FROM_POOL | sp.SPION_PATTERN_NO_FILL)
    t = np.sort(pool)[int(np.floor(q * (n - 1)))]
    want = (pool.reshape(nb, nb) > t) | np.eye(nb, dtype=bool)
    assert np.array_equal(fl.cpu().numpy().astype(bool), want) and int(nnzb.item()) == want.sum()


# The first of the two ordered sums is taken in any order while the magnitudes stay below 2^53: just below, at and above it, with
# odd numbers behind a large one (which round in the ordered sum), of both signs; the waves that have rows, all of them
@pytest.mark.parametrize("nb", [1, 4, 5, 16, 63, 64])
@pytest.mark.parametrize("kind", ["below", "at", "above", "signed", "signed above", "huge"])
def test_mean_and_std_of_pools_around_the_bound_of_exact_sums(sp, nb, kind):
    rng = np.random.default_rng(nb)
    n = nb * nb
    pool = rng.integers(1, (1 << 53) // n, n) | 1
    total = (1 << 53) + {"below": -1, "at": 0, "above": 1 + n // 2}.get(kind, 0)
    if kind in ("below", "at", "above"):
        pool[0] += total - int(pool.sum())
    elif kind == "huge":
        pool = rng.integers(-(1 << 61), 1 << 61, n) | 1
    else:
        pool *= rng.choice((-1, 1), n)
        pool[0] += (1 << 53) - int(np.abs(pool).sum()) - 1 if kind == "signed" else (1 << 53)
    s = q = 0.0
    for x in pool.tolist():
        s += float(x)
    mean = s / n
    for x in pool.tolist():
        q += (float(x) - mean) ** 2
    t = mean + 0.5 * float(np.sqrt(q / n))
    dev = torch.from_numpy(pool.reshape(nb, nb)).cuda()
    z = lambda m, t=torch.int32: torch.zeros(m, dtype=t, device="cuda")
    fl, nnzb = z((nb, nb), torch.uint8), z(1)
    ws = torch.empty(sp.spion_pattern_workspace_bytes(nb * 16, 16), dtype=torch.uint8, device="cuda")
    sp.spion_pattern(None, nb * 16, 16, 1, sp.SPION_T_MEAN_KSTD, 0.5, fl, z(nb + 1), z(n), z(nb + 1), z(n), z(n), nnzb, dev, ws,
                     flags=sp.SPION_PATTERN_FROM_POOL | sp.SPION_PATTERN_NO_FILL)
    want = (pool.astype(np.float64).reshape(nb, nb) > t) | np.eye(nb, dtype=bool)
    assert np.array_equal(fl.cpu().numpy().astype(bool), want) and int(nnzb.item()) == want.sum()


def _attention(sp, Q, K, V, dO, fl, block, dtype, heads, flags=0):
    """Relative errors (2-norm and max) of O, dQ, dK, dV of the given heads against the fp64 oracle."""
    from test_gpu_parity import _run_attention_case
    return _run_attention_case(sp, Q, K, V, dO, fl, block, dtype, flags=flags, heads=heads)


def _attention_of_unlike_heads(sp, one, BH, fl, block, dtype, flags=0):
    """One head of Q, K, V, dO in BH forms that powers of two tell apart, so that their results are the first one's, multiplied,
    to the bit: that one against the fp64 oracle, the others against it.  Heads up to 104 apart are unlike."""
    from test_gpu_parity import TOL, _dev, _pattern_from_mask, _rel_errors, _torch_dtype
    h = np.arange(BH)
    sq, sv, sdo = 2.0 ** (h % 3), 2.0 ** (h % 7), 2.0 ** (h % 5)   # K the inverse of Q's: the scores stay
    Q, K, V, dO = [_dev(t, _torch_dtype(dtype)) for t in one]
    by = lambda f: torch.from_numpy(f.astype(np.float32)).cuda().view(1, BH, 1, 1)
    many = lambda t, f: (t * by(f).to(t.dtype)).contiguous()
    q, k, v, do = many(Q, sq), many(K, 1 / sq), many(V, sv), many(dO, sdo)
    pat = _pattern_from_mask(sp, fl, block)
    O, LSE = sp.attn_fwd(q, k, v, pat, flags=flags)
    dQ, dK, dV = sp.attn_bwd(q, k, v, O, do, LSE, pat, flags=flags)
    for name, x, f in (("O", O, sv), ("dQ", dQ, sv * sdo / sq), ("dK", dK, sv * sdo * sq), ("dV", dV, sdo)):
        assert torch.equal(x, x[:, :1] * by(f).to(x.dtype)), name
    assert torch.equal(LSE, LSE[:, :1].expand_as(LSE))
    P = oracle.upsample(fl, block)
    oflags = oracle.ATTN_PAPER_DENOM if flags & sp.SPION_ATTN_PAPER_DENOM else 0
    rO, rLSE = oracle.attn_fwd(one[0], one[1], one[2], P, flags=oflags)
    for name, x, ref in zip(("O", "dQ", "dK", "dV"), (O, dQ, dK, dV), (rO, *oracle.attn_bwd(*one, P, flags=oflags))):
        errors = _rel_errors(x[0, :1].float().cpu().numpy(), ref)
        assert max(errors) <= TOL[dtype], (name, errors)
    lse, fin = LSE[0, :1].cpu().numpy(), np.isfinite(rLSE)
    assert np.array_equal(np.isneginf(lse), np.isneginf(rLSE))
    assert np.abs(lse[fin] - rLSE[fin]).max() <= TOL[dtype] * max(np.abs(rLSE[fin]).max(), 1.0)


def _one_head(rng, L, dtype):
    return [si.round_to_dtype(rng.standard_normal((1, L, 64), dtype=np.float32), dtype) for _ in range(4)]


def _dense_reference(q, k, v, do, fl, block):
    """O, dQ, dK and dV of one head, in plain torch on the GPU: fp32 for bf16 tensors, fp64 for fp32."""
    keep = torch.from_numpy(fl).cuda().bool().repeat_interleave(block, 0).repeat_interleave(block, 1)
    q, k, v, do = [t.double() if t.dtype == torch.float32 else t.float() for t in (q, k, v, do)]
    P = torch.softmax((q @ k.T * 0.125).masked_fill_(~keep, float("-inf")), dim=1).nan_to_num_(0.0)   # rows that keep nothing
    O = P @ v
    dS = P * (do @ v.T - (do * O).sum(1, keepdim=True))
    return O, dS @ k * 0.125, dS.T @ q * 0.125, P.T @ do


@pytest.mark.parametrize("block", [32, 64])
def test_forward_scores_that_run_away_from_the_first_block(sp, block):
    """Scores of later blocks far above everything in the block a row starts with (and, in other rows, far
    below): the running sums are rescaled in the middle of the walk, once or several times."""
    nb, BH, d = 6, 2, 64
    L = nb * block
    rng = np.random.default_rng(block)
    Q, K, V = [rng.standard_normal((BH, L, d), dtype=np.float32) for _ in range(3)]
    Q[:, :, 0] = 8.0
    for j in range(nb):                                     # scores 8 * K[..., 0] / 8: -60, -10, 0, 25, 70, 150
        K[:, j * block:(j + 1) * block, 0] = (-60.0, -10.0, 0.0, 25.0, 70.0, 150.0)[j]
    Q, K, V = [si.round_to_dtype(t, "bf16") for t in (Q, K, V)]
    fl = np.tril(np.ones((nb, nb), dtype=np.uint8)) | np.eye(nb, k=2, dtype=np.uint8)
    fl[1, :] = 1
    # O and LSE only: with probabilities this close to 0 and 1 the gradients are differences of nearly equal
    # bf16 numbers
    from test_gpu_parity import _pattern_from_mask
    q, k, v = [torch.from_numpy(t).cuda().to(torch.bfloat16).view(1, BH, L, d) for t in (Q, K, V)]
    O, LSE = sp.attn_fwd(q, k, v, _pattern_from_mask(sp, fl, block))
    rO, rLSE = oracle.attn_fwd(Q, K, V, oracle.upsample(fl, block))
    x = O.float().cpu().numpy().reshape(BH, L, d)
    assert np.linalg.norm(x - rO) <= 2e-2 * np.linalg.norm(rO) and np.abs(x - rO).max() <= 2e-2 * np.abs(rO).max()
    assert np.abs(LSE.cpu().numpy().reshape(BH, L) - rLSE).max() <= 1e-3 * np.abs(rLSE).max()


@pytest.mark.parametrize("block", [32, 64])
def test_forward_sums_that_add_up_beyond_their_bound(sp, block):
    """Every block but a row's first scores 14.6 above it, 2^21 times the probability: no score is out of bounds, the running
    sum (2^26 or 2^27 a block) passes 2^30 after 8 to 16 blocks, and the row goes on against a reference above all its scores."""
    nb, BH, d = 32, 1, 64                                   # as many block rows as no row is cut with
    L = nb * block
    rng = np.random.default_rng(block)
    Q, K, V = [rng.standard_normal((BH, L, d), dtype=np.float32) for _ in range(3)]
    Q[:, :, 0] = 8.0
    K[:, :, 0] = 14.6
    K[:, :block, 0] = 0.0                                   # where block row 0 starts; row 2 starts high
    Q, K, V = [si.round_to_dtype(t, "bf16") for t in (Q, K, V)]
    fl = np.eye(nb, dtype=np.uint8)
    fl[0, :] = 1
    fl[2, 0:30] = 1
    from test_gpu_parity import _pattern_from_mask
    q, k, v = [torch.from_numpy(t).cuda().to(torch.bfloat16).view(1, BH, L, d) for t in (Q, K, V)]
    O, LSE = sp.attn_fwd(q, k, v, _pattern_from_mask(sp, fl, block))
    rO, rLSE = oracle.attn_fwd(Q, K, V, oracle.upsample(fl, block))
    x = O.float().cpu().numpy().reshape(BH, L, d)
    assert np.linalg.norm(x - rO) <= 2e-2 * np.linalg.norm(rO) and np.abs(x - rO).max() <= 2e-2 * np.abs(rO).max()
    assert np.abs(LSE.cpu().numpy().reshape(BH, L) - rLSE).max() <= 1e-3 * np.abs(rLSE).max()


def test_forward_more_rows_than_run_at_once(sp):
    # 130 x 16 workgroups of block 32: rows are started in the order of their length class, long ones first
    nb, BH, block, d = 130, 16, 32, 64
    rng = np.random.default_rng(4)
    Q, K, V, dO = [si.round_to_dtype(rng.standard_normal((BH, nb * block, d), dtype=np.float32), "bf16") for _ in range(4)]
    fl = si.random_block_mask(nb, 0.02, seed=3)
    fl[[0, 63, 64, 129], :] = 1
    fl[64, 64] = 0
    fl[100, :] = 0
    _attention(sp, Q, K, V, dO, fl, block, "bf16", [0, 9])


# fp32: 16 rows a forward workgroup below 2048 workgroups of 32 rows, 32 from there on; more backward workgroups than run
# at once, so that the rows of more than twice the mean go first (block 64: a row's two workgroups together), at head counts that
# do not divide over the XCDs; bf16 of block 16 likewise; the forward's rows by length from half as many workgroups again as run
# at once and more than 32 block rows; one long row, one without a diagonal block, an empty one
@pytest.mark.parametrize("dtype,block,BH,nb", [("f32", 32, 63, 32), ("f32", 32, 64, 32), ("f32", 64, 15, 24), ("f32", 64, 43, 24),
                                               ("f32", 16, 21, 40), ("bf16", 16, 37, 44), ("f32", 32, 24, 40), ("f32", 64, 11, 36),
                                               ("f32", 32, 61, 34)])
def test_generic_kernels_rows_by_length(sp, dtype, block, BH, nb):
    rng = np.random.default_rng(BH)
    Q, K, V, dO = [si.round_to_dtype(rng.standard_normal((BH, nb * block, 64), dtype=np.float32), dtype) for _ in range(4)]
    fl = si.random_block_mask(nb, 0.35, seed=nb)
    fl[[nb // 2, nb - 1], :] = 1
    fl[nb // 2, nb // 2] = 0
    fl[3, :] = 0
    _attention(sp, Q, K, V, dO, fl, block, dtype, [0, BH // 2, BH - 1])


# bf16: rows of more than four times the mean (and 24) are cut into pieces that other workgroups take; of 33 to 64 block rows
# that all run at once, those of twice the mean (and 12): two pieces and many; more pieces than there is
# room for (32 a head), a helper for each, for several, two a head (130 heads); no diagonal block, in the first piece or a later
# one; the last row; an empty row beside them; 32 block rows: none cut
@pytest.mark.parametrize("block", [32, 64])
@pytest.mark.parametrize("BH,nb,longs", [(1, 65, (65,)), (1, 70, (25, 24)), (3, 80, (80, 37, 25, 24)), (2, 130, (130, 64, 65, 129)),
                                         (64, 72, (72, 72, 72, 30)), (130, 66, (60, 26)), (5, 33, (33, 13, 12)), (5, 32, (32, 30))])
@pytest.mark.parametrize("denom", [False, True])
def test_long_rows_in_pieces(sp, block, BH, nb, longs, denom):
    rng = np.random.default_rng(nb + BH)
    Q, K, V, dO = [si.round_to_dtype(rng.standard_normal((BH, nb * block, 64), dtype=np.float32), "bf16") for _ in range(4)]
    K[:, : block] += 3.0   # scores that run away from those of the other pieces
    K = si.round_to_dtype(K, "bf16")
    fl = np.eye(nb, dtype=np.uint8)
    rows = rng.choice(nb, len(longs), replace=False)
    for r, n in zip(rows, longs):
        fl[r] = 0
        fl[r, rng.choice(nb, n, replace=False)] = 1
    fl[(rows[0] + 1) % nb] *= rows[0] + 1 == rows[-1]
    _attention(sp, Q, K, V, dO, fl, block, "bf16", sorted({0, BH // 2, BH - 1}), flags=sp.SPION_ATTN_PAPER_DENOM if denom else 0)


# bf16, above 64 block rows: the forward's rows of more than twice the mean are cut where the mean is 7 blocks and at most two rounds of
# rows run (1024 or 2048 at once), if they outlast the launch as well; the backward's where the mean is 8.  Rows at the forward's line, one above
# it, far above it and without a diagonal block; means on both sides of the lines, one round, two, one row more
@pytest.mark.parametrize("block,BH,nb,mean", [(64, 1, 65, 8), (32, 3, 65, 7), (64, 3, 65, 6), (64, 21, 97, 8), (64, 22, 97, 8), (32, 41, 99, 9),
                                              (32, 42, 99, 9), (32, 2, 255, 20), (64, 2, 65, 10)])
def test_long_rows_in_pieces_where_rows_are_many_blocks(sp, block, BH, nb, mean):
    rng = np.random.default_rng(nb + mean)
    one = _one_head(rng, nb * block, "bf16")
    longest = max(2 * mean if mean < 10 else 3 * mean // 2, 2 * (BH * nb * mean // (1024 if block == 64 else 2048)))
    lengths = np.full(nb, mean)
    for r, n in ((0, longest), (nb - 1, longest + 1), (9, min(nb - 1, 3 * longest))):
        lengths[r] = n
    fewer = np.setdiff1d(np.arange(nb), (0, nb - 1, 9))
    for i in range(lengths.sum() - nb * mean):   # the mean stays
        lengths[fewer[i % len(fewer)]] -= 1
    fl = np.zeros((nb, nb), dtype=np.uint8)
    for r, n in enumerate(lengths):
        cols = np.setdiff1d(np.arange(nb), r)
        fl[r, rng.choice(cols, n - (r != 9), replace=False)] = 1
        fl[r, r] = r != 9
    assert fl.sum() == nb * mean
    _attention_of_unlike_heads(sp, one, BH, fl, block, "bf16")


# The kernels of fp32 and of block size 16: a helper for each piece and part of a block row; 16 and 32 rows a workgroup; a row of more
# pieces than there are helpers for stays whole; no diagonal block in a piece, an empty row beside them
@pytest.mark.parametrize("dtype,block", [("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 16)])
@pytest.mark.parametrize("BH,nb,longs,denom", [(1, 65, (65,), True), (3, 80, (80, 37, 25, 24), False), (2, 130, (130, 64, 65, 129), True),
                                               (20, 70, (70, 60), False)])
def test_long_rows_in_pieces_of_the_generic_kernels(sp, dtype, block, BH, nb, longs, denom):
    rng = np.random.default_rng(nb + BH)
    Q, K, V, dO = [si.round_to_dtype(rng.standard_normal((BH, nb * block, 64), dtype=np.float32), dtype) for _ in range(4)]
    fl = np.eye(nb, dtype=np.uint8)
    rows = [nb - 1, 0, 7, nb // 2][:len(longs)]
    for r, n in zip(rows, longs):
        fl[r] = 0
        fl[r, rng.choice(nb, n, replace=False)] = 1
    fl[5, :] = 0
    _attention(sp, Q, K, V, dO, fl, block, dtype, [0, BH - 1], flags=sp.SPION_ATTN_PAPER_DENOM if denom else 0)


# Many block rows of few tiles, whose rows two waves share in the backward: long ones in pieces all the same
@pytest.mark.parametrize("dtype,block,BH,nb", [("bf16", 16, 9, 121), ("f32", 16, 9, 121), ("f32", 32, 12, 130), ("f32", 64, 24, 130)])
def test_long_rows_in_pieces_where_two_waves_share_one(sp, dtype, block, BH, nb):
    rng = np.random.default_rng(nb + BH)
    one = _one_head(rng, nb * block, dtype)
    fl = np.eye(nb, dtype=np.uint8) | np.eye(nb, k=1, dtype=np.uint8)
    for r, n in zip((nb - 1, 0, 7), (nb, 65, 44)):
        fl[r] = 0
        fl[r, rng.choice(nb, n, replace=False)] = 1
    fl[5] = 0
    _attention_of_unlike_heads(sp, one, BH, fl, block, dtype)


# fp32 backward, 16 rows a workgroup up to 800 workgroups of 32 rows (block rows, columns and chunks of all heads), from six blocks a row on up
# to 760, 32 beyond: both sides of both lines, with a row and a column that are cut
@pytest.mark.parametrize("block,BH,nb,mean,rows", [(32, 8, 38, 2, 16), (32, 9, 38, 2, 16), (32, 10, 38, 2, 32), (32, 11, 38, 2, 32), (64, 4, 38, 2, 16),
                                                   (64, 5, 38, 2, 32), (32, 8, 38, 7, 16), (32, 8, 40, 7, 32), (64, 4, 38, 7, 16), (64, 4, 40, 7, 32)])
def test_backward_around_the_line_of_16_and_32_rows(sp, block, BH, nb, mean, rows):
    rng = np.random.default_rng(nb + BH)
    fl = np.eye(nb, dtype=np.uint8)
    fl[3] = 1
    fl[:, 7] = 1
    fl[5] = 0
    if mean > 2:
        free = np.flatnonzero((fl == 0) & (np.arange(nb) != 5)[:, None])
        fl.reshape(-1)[rng.choice(free, mean * nb - int(fl.sum()), replace=False)] = 1
    kept = int(fl.sum())
    workgroups = BH * (kept // 16 + 2 * nb) * (block // 32)
    assert (workgroups <= (760 if kept > 6 * nb else 800)) == (rows == 16), workgroups
    _attention_of_unlike_heads(sp, _one_head(rng, nb * block, "f32"), BH, fl, block, "f32")


# fp32 backward: on both sides of the lines from which few waves share a row: the diagonal alone, a few blocks besides, twice as many blocks as rows; up to
# 15 block rows and with more than 2000 workgroups the last of these lines is a lower one
@pytest.mark.parametrize("block,BH,nb,kept,many", [
    (32, 10, 11, 11, False), (32, 10, 13, 13, True), (64, 10, 23, 23, False), (64, 10, 25, 25, True), (32, 10, 28, 35, False), (32, 10, 32, 40, True),
    (32, 10, 56, 112, False), (32, 10, 64, 128, True), (32, 30, 11, 19, False), (32, 30, 11, 18, True), (64, 42, 15, 24, False), (64, 42, 15, 23, True),
    (32, 30, 16, 38, False), (32, 30, 16, 25, True), (64, 24, 21, 40, False), (64, 24, 21, 32, False), (64, 24, 24, 36, False), (64, 30, 30, 60, True)])
def test_backward_around_the_lines_of_many_short_rows(sp, block, BH, nb, kept, many):
    rng = np.random.default_rng(nb)
    fl = np.eye(nb, dtype=np.uint8)
    fl.reshape(-1)[rng.choice(np.flatnonzero(fl.reshape(-1) == 0), kept - nb, replace=False)] = 1
    line = 60 if 10 * kept < 11 * nb else 120 if 2 * kept < 3 * nb else 150 if nb >= 16 and 2 * BH * nb * (block // 32) <= 2000 else 100
    assert (BH * nb * nb / (kept * (block // 16)) >= line) == many
    _attention_of_unlike_heads(sp, _one_head(rng, nb * block, "f32"), BH, fl, block, "f32")


# A row whose pieces there is no room for at first, and more rows of several pieces than helpers: larger pieces, until there is; where
# the pieces are left in memory tells that they were cut
@pytest.mark.parametrize("dtype,block,BH,nb,longs", [("bf16", 32, 2, 512, (400,)), ("bf16", 64, 1, 300, (300, 299)), ("bf16", 32, 20, 140, (100, 90, 80, 70)),
                                                     ("bf16", 16, 2, 300, (300, 280)), ("f32", 32, 1, 320, (320, 200)), ("f32", 16, 2, 512, (512,))])
def test_long_rows_of_more_pieces_than_there_is_room_for(sp, dtype, block, BH, nb, longs):
    import ctypes
    from test_gpu_parity import TOL, _pattern_from_mask, _torch_dtype
    rng = np.random.default_rng(nb)
    fl = (rng.random((nb, nb)) < 9 / nb).astype(np.uint8) | np.eye(nb, dtype=np.uint8)
    rows = (nb - 2, 70, 3, 139)[:len(longs)]
    for r, n in zip(rows, longs):
        fl[r] = 0
        fl[r, rng.choice(nb, n, replace=False)] = 1
    pat, kept, L = _pattern_from_mask(sp, fl, block), int(fl.sum()), nb * block
    gen = torch.Generator(device="cuda").manual_seed(nb)
    q, k, v, do = [torch.randn((1, BH, L, 64), generator=gen, device="cuda").to(_torch_dtype(dtype)) for _ in range(4)]
    lib = sp.load()
    lib.spion_attn_fwd_room_bytes.restype = ctypes.c_size_t
    p = sp.binding._AttnParams(1, BH, L, 64, block, sp.SPION_BF16 if dtype == "bf16" else sp.SPION_F32, 0.0, 0)
    size = lib.spion_attn_fwd_room_bytes(ctypes.byref(p), kept)
    room = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
    O, LSE = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    assert lib.spion_attn_fwd_room(ptr(q), ptr(k), ptr(v), ptr(O), ptr(LSE), ptr(pat.row_ptr), ptr(pat.col_idx), kept, ctypes.byref(p), ptr(room),
                                   ctypes.c_size_t(size), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    ws_size = sp.spion_attn_workspace_bytes(1, BH, L, 64, block, p.dtype, kept, True)
    ws = torch.full((ws_size,), 0xA5, dtype=torch.uint8, device="cuda")
    grads = sp.attn_bwd(q, k, v, O, do, LSE, pat, dQ=torch.full_like(q, float("nan")), workspace=ws)
    # behind the counters, 32 places a head: each long row leaves two pieces or more of `block` rows of 64 floats (fewer than 1 byte in 100 is 0xA5
    # by chance).  The backward's largest row at least: its steps of both sides hide the others
    piece = block * 64 * 4
    assert int((room[BH * 32 * 32:] != 0xA5).sum()) >= 0.99 * BH * len(longs) * 2 * piece
    assert int((ws[-32 * BH * piece:] != 0xA5).sum()) >= 0.99 * BH * 2 * piece
    for h in (0, BH - 1):
        for name, got, want in zip(("O", "dQ", "dK", "dV"), (O, *grads), _dense_reference(*(t[0, h] for t in (q, k, v, do)), fl, block)):
            error = torch.linalg.vector_norm(got[0, h] - want) / torch.linalg.vector_norm(want)
            assert error <= TOL[dtype], (name, h, float(error))


# bf16 backward, unsplit columns in their order and by lengths in units of 1, 2 and 4 blocks (by the rounds of workgroups); of one, two, four and more
# groups of 64, the last one full and not; columns of 0 to 16 blocks and some that are cut
@pytest.mark.parametrize("block,BH,nb", [(32, 3, 40), (32, 9, 64), (32, 24, 100), (32, 64, 65), (64, 1, 128), (64, 3, 129), (64, 9, 256), (32, 1, 257), (32, 1, 513),
                                         (64, 8, 320), (32, 1, 1024), (32, 12, 600)])
def test_backward_columns_by_length(sp, block, BH, nb):
    from test_gpu_parity import TOL, _pattern_from_mask
    rng = np.random.default_rng(nb)
    fl = (rng.random((nb, nb)) < rng.random((1, nb)) ** 2 * 12 / nb).astype(np.uint8)
    fl[:, rng.choice(nb, 3, replace=False)] |= (rng.random((nb, 3)) < min(1.0, 60 / nb)).astype(np.uint8)
    fl[:, 5] = 0
    fl[np.arange(nb), (np.arange(nb) + 6) % nb] = 1   # no row without a block
    fl[nb - 1, 5] = 0
    pat = _pattern_from_mask(sp, fl, block)
    gen = torch.Generator(device="cuda").manual_seed(BH)
    q, k, v, do = [torch.randn((1, BH, nb * block, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4)]
    nan = lambda: torch.full_like(q, float("nan"))
    O, LSE = sp.attn_fwd(q, k, v, pat)
    grads = sp.attn_bwd(q, k, v, O, do, LSE, pat, dQ=nan(), dK=nan(), dV=nan())
    assert not any(g.isnan().any() for g in grads)
    for h in sorted({0, BH // 2, BH - 1}):
        for name, got, want in zip(("O", "dQ", "dK", "dV"), (O, *grads), _dense_reference(*(t[0, h] for t in (q, k, v, do)), fl, block)):
            error = torch.linalg.vector_norm(got[0, h] - want) / torch.linalg.vector_norm(want)
            assert error <= TOL["bf16"], (name, h, float(error))


# bf16, block 16: rows are cut above 120 block rows where more workgroups than run at once (1024), above 150 where they all do
@pytest.mark.parametrize("BH,nb,cut", [(8, 128, False), (9, 120, False), (9, 121, True), (2, 150, False), (2, 151, True), (6, 170, True)])
def test_long_rows_of_block_16(sp, BH, nb, cut):
    import ctypes
    fl = np.eye(nb, dtype=np.uint8)
    fl[[3, nb - 1], :] = 1
    fl[7, : nb // 2] = 1
    fl[5, :] = 0
    lib = sp.load()
    lib.spion_attn_fwd_room_bytes.restype = ctypes.c_size_t
    p = sp.binding._AttnParams(1, BH, nb * 16, 64, 16, sp.SPION_BF16, 0.0, 0)
    assert (lib.spion_attn_fwd_room_bytes(ctypes.byref(p), int(fl.sum())) > 0) == cut
    rng = np.random.default_rng(nb)
    Q, K, V, dO = [si.round_to_dtype(rng.standard_normal((BH, nb * 16, 64), dtype=np.float32), "bf16") for _ in range(4)]
    _attention(sp, Q, K, V, dO, fl, 16, "bf16", [0, BH - 1])


@pytest.mark.parametrize("BH,nb", [(3, 160)])
def test_pieces_of_block_16_whose_scores_are_all_minus_infinity(sp, BH, nb):
    """As below, where block 16 is cut."""
    from test_gpu_parity import _pattern_from_mask
    long, without = np.eye(nb, dtype=np.uint8), np.eye(nb, dtype=np.uint8)
    long[[3, 150]] = without[[3, 150]] = 1
    without[:, 10:90] = 0
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = [torch.randn((1, BH, nb * 16, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    q = q.abs() + 0.125
    k[:, :, 10 * 16:90 * 16] = -float("inf")
    got, got_lse = sp.attn_fwd(q, k, v, _pattern_from_mask(sp, long, 16))
    want, want_lse = sp.attn_fwd(q, k, v, _pattern_from_mask(sp, without, 16))
    for row in (3, 150):
        at = slice(row * 16, (row + 1) * 16)
        # tolerances of test_pieces_whose_scores_are_all_minus_infinity
        assert torch.allclose(got[:, :, at].float(), want[:, :, at].float(), rtol=0.0, atol=2e-2)
        assert torch.allclose(got_lse[:, :, at], want_lse[:, :, at], rtol=0.0, atol=1e-2)


@pytest.mark.parametrize("dtype,block", [("bf16", 32), ("bf16", 64), ("bf16", 16), ("f32", 32)])
def test_pieces_whose_scores_are_all_minus_infinity(sp, dtype, block):
    """Keys that give scores of -infinity count nothing, also where they are all that a piece of a long row has."""
    from test_gpu_parity import _pattern_from_mask
    nb = 130
    long, without = np.eye(nb, dtype=np.uint8), np.eye(nb, dtype=np.uint8)
    long[[3, 100]] = without[[3, 100]] = 1
    without[:, 10:90] = 0
    gen = torch.Generator(device="cuda").manual_seed(3)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = [torch.randn((1, 3, nb * block, 64), generator=gen, device="cuda").to(tdt) for _ in range(3)]
    q = q.abs() + 0.125
    k[:, :, 10 * block:90 * block] = -float("inf")
    got, got_lse = sp.attn_fwd(q, k, v, _pattern_from_mask(sp, long, block))
    want, want_lse = sp.attn_fwd(q, k, v, _pattern_from_mask(sp, without, block))
    for row in (3, 100):
        at = slice(row * block, (row + 1) * block)
        # the same sums in another order: fp32 rounding of 50 blocks' scores, and one of the output
        assert torch.allclose(got[:, :, at].float(), want[:, :, at].float(), rtol=0.0, atol=2e-2 if dtype == "bf16" else 2e-5)
        assert torch.allclose(got_lse[:, :, at], want_lse[:, :, at], rtol=0.0, atol=1e-2 if dtype == "bf16" else 1e-5)


def test_long_rows_in_pieces_again_and_in_a_graph(sp):
    """Whichever piece is the last to arrive: the same bits every time, and in replays, which share their launches' tags, on other
    inputs and with other work in between."""
    from test_gpu_parity import _pattern_from_mask
    nb, block = 96, 32
    fl = np.eye(nb, dtype=np.uint8)
    fl[[5, 50], :] = 1
    pat = _pattern_from_mask(sp, fl, block)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = [torch.randn((2, 3, nb * block, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    O, LSE = [t.clone() for t in sp.attn_fwd(q, k, v, pat)]
    for _ in range(20):
        o, lse = sp.attn_fwd(q, k, v, pat)
        assert torch.equal(o, O) and torch.equal(lse, LSE)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        sp.attn_fwd(q, k, v, pat)
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        o, lse = sp.attn_fwd(q, k, v, pat)
    for i in range(5):
        for t in (q, k, v):
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
        g.replay()
        torch.cuda.synchronize()
        eager, eager_lse = sp.attn_fwd(q, k, v, pat)
        assert torch.equal(o, eager) and torch.equal(lse, eager_lse)


# The kernels of fp32 and of block size 16 share a row's tiles over the waves of a workgroup by the average number of
# tiles and the number of rows: (heads, block rows, density) for four waves a row, for few, and for rows of one
# block; with rows and columns of 0, 1, 2, 65 and more blocks, odd numbers of tiles, split columns, and head
# counts that do not divide over the XCDs.
@pytest.mark.parametrize("dtype,block", [("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 16)])
@pytest.mark.parametrize("BH,nb,density", [(1, 1, 1.0), (3, 7, 0.3), (2, 70, 0.1), (17, 33, 0.0), (64, 24, 0.05)])
def test_attention_waves_per_row(sp, dtype, block, BH, nb, density):
    d = 64
    rng = np.random.default_rng(nb + block)
    Q, K, V, dO = [si.round_to_dtype(rng.standard_normal((BH, nb * block, d), dtype=np.float32), dtype)
                   for _ in range(4)]
    fl = si.random_block_mask(nb, density, seed=nb) if density < 1.0 else np.ones((nb, nb), dtype=np.uint8)
    if nb > 5:
        fl[1, :] = fl[:, 4] = 0
    if nb > 64:
        fl[2, :] = fl[:, 3] = 1
    _attention(sp, Q, K, V, dO, fl, block, dtype, sorted({0, BH // 2, BH - 1}))


def _small_attention(sp, block=32, nb=3):
    from test_gpu_parity import _pattern_from_mask
    pat = _pattern_from_mask(sp, np.tril(np.ones((nb, nb), dtype=np.uint8)), block)
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, k, v, do = [torch.randn((1, 2, nb * block, 64), generator=gen, device="cuda") for _ in range(4)]
    return pat, q, k, v, do


def test_autograd_node_beside_the_other_transforms(sp):
    """Forward-mode and vmap are refused (there is no rule for them), saved-tensor hooks see every tensor kept."""
    pat, q, k, v, do = _small_attention(sp)
    with torch.autograd.forward_ad.dual_level():
        with pytest.raises(NotImplementedError):
            sp.sparse_attention(torch.autograd.forward_ad.make_dual(q, do), k, v, pat)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda x: sp.sparse_attention(x, k, v, pat))(torch.stack((q, q)))
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda x: sp.sparse_attention(x, k, v, pat).sum())(q)
    leaves = [t.clone().requires_grad_(True) for t in (q, k, v)]
    want = torch.autograd.grad(sp.sparse_attention(*leaves, pat), leaves, do)
    kept = []

    def pack(t):
        kept.append(tuple(t.shape))
        return t.detach().cpu()

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t.cuda()):
        o = sp.sparse_attention(*leaves, pat)
    assert sorted(kept) == sorted([tuple(q.shape)] * 4 + [tuple(q.shape[:3])])
    for a, b in zip(torch.autograd.grad(o, leaves, do), want):
        assert torch.equal(a, b)


def test_pattern_on_another_stream_right_after_the_call(sp):
    # generate_pattern has waited for the pattern, so any stream may read it without waiting for the producer's
    nb, block = 64, 16
    other = torch.cuda.Stream()
    for seed in range(5):
        A = torch.rand((nb * block, nb * block), generator=torch.Generator().manual_seed(seed)) ** 6
        pat = sp.generate_pattern(A.cuda(), block, 5, si.T_QUANTILE, 0.8)
        with torch.cuda.stream(other):
            got = [t.clone() for t in (pat.fl_out, pat.row_ptr, pat.col_ptr, pat.pool_sum)]
        ref = oracle.generate_pattern(A.numpy(), block, 5, si.T_QUANTILE, 0.8)
        other.synchronize()
        for t, name in zip(got, ("fl_out", "row_ptr", "col_ptr", "pool_sum")):
            assert np.array_equal(t.cpu().numpy(), ref[name]), name


# The backward's work items with chunks of 8, 10, 14, 16, 27 and 64 rows (by the steps each resident workgroup has to do),
# columns of as many rows as fit a chunk, one more, and of 0, 8 and 9 rows; long rows first and not
@pytest.mark.parametrize("BH,nb,density,block", [(2, 70, 0.1, 32), (16, 70, 0.12, 64), (64, 70, 0.15, 32),
                                                 (72, 130, 0.03, 32), (96, 9, 0.4, 32), (2, 100, 0.01, 64), (1, 66, 0.02, 64),
                                                 (3, 140, 0.0, 64)])
def test_backward_chunks_follow_the_work(sp, BH, nb, density, block):
    rng = np.random.default_rng(nb + BH)
    Q, K, V, dO = [si.round_to_dtype(rng.standard_normal((BH, nb * block, 64), dtype=np.float32), "bf16") for _ in range(4)]
    fl = si.random_block_mask(nb, density, seed=nb)
    for c, n in enumerate((64, 65, 16, 17, 8, 9, 27, 28, 0)):
        fl[:, c] = 0
        fl[nb - min(n, nb):, c] = n > 0
    fl[nb - 3, :] = 1
    fl[1, :] = 0
    _attention(sp, Q, K, V, dO, fl, block, "bf16", [0, BH - 1])


# 2, 7, 8, 9, 16 and 17 parts, of which eight are added up at a time; four and two waves a row (many short rows)
@pytest.mark.parametrize("dtype,block", [("f32", 16), ("f32", 32), ("bf16", 16)])
@pytest.mark.parametrize("BH", [1, 40])
def test_generic_backward_parts_of_a_column(sp, dtype, block, BH):
    nb = 260
    fl = np.eye(nb, dtype=np.uint8)
    for c, n in ((0, 17), (9, 112), (70, 128), (128, 129), (200, 256), (259, 260)):
        fl[:, c] = np.arange(nb) < n
    _attention_of_unlike_heads(sp, _one_head(np.random.default_rng(BH), nb * block, dtype), BH, fl, block, dtype)


@pytest.mark.parametrize("dtype,block", [("bf16", 32), ("bf16", 64), ("bf16", 16), ("f32", 32)])
def test_cut_columns_and_rows_again_and_in_a_graph(sp, dtype, block):
    """Backward, whichever chunk of a column or piece of a row is the last to arrive: the same bits every time, in a workspace that
    held other numbers, and in replays, which share their launches' tags, on other inputs and with other work in between."""
    from test_gpu_parity import _pattern_from_mask
    nb = 72
    fl = np.eye(nb, dtype=np.uint8)
    fl[:, [0, 40]] = 1
    fl[:33, 7] = 1
    fl[[50, 71], :] = 1   # in pieces
    pat = _pattern_from_mask(sp, fl, block)
    gen = torch.Generator(device="cuda").manual_seed(2)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, do = [torch.randn((2, 5, nb * block, 64), generator=gen, device="cuda").to(tdt) for _ in range(4)]
    dt = sp.SPION_BF16 if dtype == "bf16" else sp.SPION_F32
    ws = torch.randint(0, 256, (sp.spion_attn_workspace_bytes(2, 5, nb * block, 64, block, dt, pat.nnzb, True),),
                       generator=gen, device="cuda", dtype=torch.uint8)
    o, lse = sp.attn_fwd(q, k, v, pat)
    want = [t.clone() for t in sp.attn_bwd(q, k, v, o, do, lse, pat)]
    for _ in range(20):
        for a, b in zip(sp.attn_bwd(q, k, v, o, do, lse, pat, workspace=ws), want):
            assert torch.equal(a, b)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        sp.attn_bwd(q, k, v, o, do, lse, pat, workspace=ws)
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        got = sp.attn_bwd(q, k, v, o, do, lse, pat, workspace=ws)
    for i in range(5):
        do.copy_(torch.randn(do.shape, generator=gen, device="cuda"))
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(got, sp.attn_bwd(q, k, v, o, do, lse, pat)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,block", [("bf16", 32), ("bf16", 64), ("bf16", 16), ("f32", 32), ("f32", 64)])
def test_backward_in_workspaces_of_other_sizes(sp, dtype, block):
    """One for more kept blocks serves, and one without the room for pieces of rows, which are whole then (last bytes untouched)."""
    from test_gpu_parity import _pattern_from_mask
    nb = 80
    fl = np.eye(nb, dtype=np.uint8)
    fl[:, 3] = 1
    fl[[5, 79], :] = 1
    pat = _pattern_from_mask(sp, fl, block)
    gen = torch.Generator(device="cuda").manual_seed(block)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, do = [torch.randn((1, 3, nb * block, 64), generator=gen, device="cuda").to(tdt) for _ in range(4)]
    o, lse = sp.attn_fwd(q, k, v, pat)
    want = sp.attn_bwd(q, k, v, o, do, lse, pat)
    dt = sp.SPION_BF16 if dtype == "bf16" else sp.SPION_F32
    size = lambda kept: sp.spion_attn_workspace_bytes(1, 3, nb * block, 64, block, dt, kept, True)
    # the query's rows summed in one run instead of pieces of fp32 sums: rows of up to 80 blocks, each term rounded as before
    tol = 1e-5 if dtype == "f32" else 2.0 ** -8
    for n, same in ((size(pat.nnzb), True), (size(2000), True), (size(nb * nb), False), (size(pat.nnzb) - 256, False)):
        ws = torch.full((n + 256,), 77, dtype=torch.uint8, device="cuda")
        got = sp.attn_bwd(q, k, v, o, do, lse, pat, workspace=ws[:n])
        assert bool((ws[n:] == 77).all())
        assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
        assert torch.equal(got[0], want[0]) if same else (got[0].double() - want[0].double()).norm() <= tol * want[0].double().norm()


# Vectors of 16 bytes, one or two per thread (two from 2^20 vectors), 8 maps at a time and a remainder of 0 to 7
@pytest.mark.parametrize("L,maps,dtype", [(8, 1, "f32"), (8, 9, "bf16"), (104, 7, "bf16"), (200, 16, "f32"),
                                          (2056, 3, "f32"), (2904, 10, "bf16")])
def test_score_mean_and_distance_at_the_edges(sp, L, maps, dtype):
    gen = torch.Generator(device="cuda").manual_seed(L)
    A = torch.rand((maps, L, L), generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    want = torch.zeros((L, L), device="cuda")
    for m in range(maps):
        want += A[m].float()   # the order of the sum is the definition
    want *= torch.tensor(1.0, device="cuda") / torch.tensor(float(maps), device="cuda")
    mean = sp.score_mean(A)
    assert torch.equal(mean, want)
    prev = torch.rand((L, L), generator=gen, device="cuda")
    a, b = prev.double().norm().item(), mean.double().norm().item()
    got = sp.frobenius_distance(prev, mean).cpu().numpy()
    # sums of L^2 squares in fp64 in another order: relative error below L^2 2^-53
    assert np.allclose(got, (abs(a - b), a, b), rtol=0.0, atol=L * L * 2.0 ** -53 * (a + b))


# Output tiles of 128 x 128 and their edges, steps of 32 rows, slices of at least 128 rows (one, a last short one, many);
# sizes that are not multiples of 8 and non-contiguous or misaligned inputs take torch's product
@pytest.mark.parametrize("rows,N,M", [(1, 8, 8), (31, 128, 136), (33, 192, 64), (128, 136, 120), (129, 256, 128), (1000, 384, 128),
                                      (5000, 768, 256), (200, 12, 20), (16, 1536, 512)])
@pytest.mark.parametrize("form", ["plain", "strided", "misaligned", "bias"])
def test_projection_weight_gradient(sp, rows, N, M, form):
    from paper_2309_12578_amd.sublayer import _Projection
    gen = torch.Generator(device="cuda").manual_seed(rows + N)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)

    layer = _Projection(M, N, bias=form == "bias", device="cuda", dtype=torch.bfloat16)
    with torch.no_grad():
        for p in layer.parameters():
            p.copy_(randn(*p.shape))
    x, dy = randn(1, rows, M), randn(1, rows, N)
    if form == "strided":
        x = randn(1, M, rows).transpose(1, 2)
    if form == "misaligned":
        x = randn(rows * M + 1)[1:].view(1, rows, M)
    x.requires_grad_(True)
    y = layer(x)
    got = torch.autograd.grad(y, [x, *layer.parameters()], dy)
    w = layer.weight.detach().double()
    x64, dy64 = x.detach().double().view(rows, M), dy.double().view(rows, N)
    want = [dy64 @ w, dy64.t().contiguous() @ x64] + ([dy64.sum(0)] if form == "bias" else [])
    assert torch.equal(y, torch.nn.functional.linear(x, layer.weight, layer.bias))
    for g, r in zip(got, want):   # one rounding to bf16 (2^-9 of each value) of sums in fp32
        assert g.dtype == torch.bfloat16 and (g.double().view(r.shape) - r).norm() <= 2.0 ** -8 * r.norm()


def test_projection_beside_the_other_transforms(sp):
    from paper_2309_12578_amd.sublayer import _Projection
    layer = _Projection(64, 192, bias=False, device="cuda", dtype=torch.bfloat16)
    plain = torch.nn.Linear(64, 192, bias=False, device="cuda", dtype=torch.bfloat16)
    plain.weight = layer.weight
    x = torch.randn((4, 32, 64), device="cuda").to(torch.bfloat16).requires_grad_(True)
    ad = torch.autograd.forward_ad

    def tangent(f):
        with ad.dual_level():
            return ad.unpack_dual(f(ad.make_dual(x.detach(), x.detach()))).tangent

    def second(f):   # gradient of a gradient
        g, = torch.autograd.grad(f(x).square().sum(), f.weight, create_graph=True)
        return torch.autograd.grad(g.square().sum(), x)[0]

    def cast(f):
        with torch.autocast("cuda", dtype=torch.float16):
            return f(x)

    for call in (tangent, second, cast, lambda f: torch.func.vmap(f)(x), lambda f: torch.func.grad(lambda t: f(t).sum())(x),
                 lambda f: f(x.detach())):
        a, b = call(layer), call(plain)
        assert a.dtype == b.dtype and torch.allclose(a.float(), b.float(), rtol=2.0 ** -6, atol=2.0 ** -6 * b.float().abs().max().item())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,H,nb,block", [(1, 1, 1, 16), (3, 5, 3, 16), (2, 3, 7, 32), (2, 8, 2, 64)])
def test_sublayer_fused_and_step_by_step(sp, dtype, B, H, nb, block):
    """Head split and merge only move values: the same bits as the torch operators, which run under a mode."""
    from test_gpu_parity import _pattern_from_mask
    pat = _pattern_from_mask(sp, np.tril(np.ones((nb, nb), dtype=np.uint8)), block)
    gen = torch.Generator(device="cuda").manual_seed(H)
    mha = sp.SparseMHA(64 * H, H, device="cuda", dtype=dtype)
    mha.norm = torch.nn.LayerNorm(64 * H, device="cuda", dtype=dtype)   # the same on both sides
    E, dout = [torch.randn((B, nb * block, 64 * H), generator=gen, device="cuda").to(dtype) for _ in range(2)]
    E.requires_grad_(True)
    fused = mha(E, pat)
    d_fused, = torch.autograd.grad(fused, E, dout)

    class Watching(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    with Watching():
        steps = mha(E, pat)
    d_steps, = torch.autograd.grad(steps, E, dout.transpose(0, 1).contiguous().transpose(0, 1))
    assert fused.grad_fn is not None and torch.equal(fused, steps) and torch.equal(d_fused, d_steps)
    with torch.no_grad():
        assert torch.equal(mha(E, pat), steps)


# One block; odd heads and batches; columns of 40 rows, which are cut and added up (chunks of 16); 8 heads, which are dealt
# over the XCDs, with enough rows to be sorted by length; a row without a diagonal block and an empty one
@pytest.mark.parametrize("B,H,nb,block", [(1, 1, 1, 32), (3, 5, 4, 64), (1, 3, 40, 32), (2, 1, 40, 64), (8, 8, 34, 32), (4, 8, 34, 64)])
@pytest.mark.parametrize("denom", [False, True])
def test_heads_where_the_projections_have_them(sp, B, H, nb, block, denom):
    """The attention on [B, L, 3, H, 64] gives the bits of the attention on three tensors [B, H, L, 64]."""
    from test_gpu_parity import _pattern_from_mask
    fl = np.tril(np.ones((nb, nb), dtype=np.uint8)) if nb < 34 or H < 8 else np.eye(nb, dtype=np.uint8)
    fl[nb // 2, :] = 1
    if nb > 4:
        fl[2, 2] = 0
        fl[3, :] = 0
    pat = _pattern_from_mask(sp, fl, block)
    flags = sp.SPION_ATTN_PAPER_DENOM if denom else 0
    L = nb * block
    gen = torch.Generator(device="cuda").manual_seed(nb)
    qkv = torch.randn((B, L, 3, H, 64), generator=gen, device="cuda").to(torch.bfloat16).view(B, L, 3 * H * 64).requires_grad_(True)
    dS = torch.randn((B, L, H * 64), generator=gen, device="cuda").to(torch.bfloat16)
    S = sp.binding._host.heads_attention(qkv, H, pat.row_ptr, pat.col_idx, pat.col_ptr, pat.row_idx, pat.bsr_pos, pat.nnzb, block, flags)
    got, = torch.autograd.grad(S, qkv, dS)
    q, k, v = [t.transpose(1, 2).contiguous() for t in qkv.detach().view(B, L, 3, H, 64).unbind(2)]
    O, LSE = sp.attn_fwd(q, k, v, pat, flags=flags)
    dO = dS.view(B, L, H, 64).transpose(1, 2).contiguous()
    want = torch.stack([t.transpose(1, 2) for t in sp.attn_bwd(q, k, v, O, dO, LSE, pat, flags=flags)], 2)
    assert torch.equal(S.view(B, L, H, 64).transpose(1, 2), O)
    assert torch.equal(got.view(B, L, 3, H, 64), want)


# 33 to 64 block rows that all run at once (the forward cuts rows of twice the mean), and more (both sides cut)
@pytest.mark.parametrize("B,H,nb,block", [(1, 3, 40, 32), (2, 1, 64, 64), (1, 3, 65, 32), (2, 2, 80, 64), (1, 1, 255, 32)])
def test_long_rows_in_pieces_where_the_projections_have_the_heads(sp, B, H, nb, block):
    """As test_heads_where_the_projections_have_them, for patterns whose long rows are cut."""
    import ctypes
    from test_gpu_parity import _pattern_from_mask
    fl = np.eye(nb, dtype=np.uint8)
    fl[:, 1] = 1
    fl[7, :] = 1
    fl[nb - 1, : 7 * nb // 8] = 1
    fl[3, :] = 0
    pat = _pattern_from_mask(sp, fl, block)
    L = nb * block
    lib = sp.load()
    lib.spion_attn_fwd_room_bytes.restype = ctypes.c_size_t
    p = sp.binding._AttnParams(B, H, L, 64, block, sp.SPION_BF16, 0.0, 0)
    assert lib.spion_attn_fwd_room_bytes(ctypes.byref(p), pat.nnzb) > 0
    per_head = lambda heads: sp.spion_attn_workspace_bytes(heads, 1, L, 64, block, sp.SPION_BF16, pat.nnzb, True) / heads
    assert (per_head(B * H) > 1.1 * per_head(4000)) == (nb > 64)
    gen = torch.Generator(device="cuda").manual_seed(nb)
    qkv = torch.randn((B, L, 3, H, 64), generator=gen, device="cuda").to(torch.bfloat16).view(B, L, 3 * H * 64).requires_grad_(True)
    dS = torch.randn((B, L, H * 64), generator=gen, device="cuda").to(torch.bfloat16)
    S = sp.binding._host.heads_attention(qkv, H, pat.row_ptr, pat.col_idx, pat.col_ptr, pat.row_idx, pat.bsr_pos, pat.nnzb, block, 0)
    got, = torch.autograd.grad(S, qkv, dS)
    q, k, v = [t.transpose(1, 2).contiguous() for t in qkv.detach().view(B, L, 3, H, 64).unbind(2)]
    O, LSE = sp.attn_fwd(q, k, v, pat)
    dO = dS.view(B, L, H, 64).transpose(1, 2).contiguous()
    want = torch.stack([t.transpose(1, 2) for t in sp.attn_bwd(q, k, v, O, dO, LSE, pat)], 2)
    assert torch.equal(S.view(B, L, H, 64).transpose(1, 2), O)
    assert torch.equal(got.view(B, L, 3, H, 64), want)


# bf16 blocks of 32 and 64 have the attention work on qkv and S themselves, other types on copies
@pytest.mark.parametrize("dtype,block", [(torch.bfloat16, 32), (torch.bfloat16, 64), (torch.bfloat16, 16), (torch.float32, 32)])
def test_tensors_beside_the_attention_changed_in_place(sp, dtype, block):
    """Hooks and a replaced forward that change S or qkv in place, seen by autograd or not, against the same out of place."""
    from test_gpu_parity import _pattern_from_mask
    B, H, nb = 2, 2, 6
    pat = _pattern_from_mask(sp, np.tril(np.ones((nb, nb), dtype=np.uint8)), block)
    torch.manual_seed(block)
    mha = sp.SparseMHA(H * 64, H, device="cuda", dtype=dtype)
    E = torch.randn((B, nb * block, H * 64), device="cuda", dtype=dtype, requires_grad=True)
    dout = torch.randn_like(E)
    linear = mha.w_o.forward

    def grads(pre=None, forward=None, keep=None):
        hooks, seen = [], []
        if pre:
            hooks.append(mha.w_o.register_forward_pre_hook(lambda m, a: pre(a[0])))
        if forward:
            mha.w_o.forward = forward
        if keep:
            hooks.append(mha.w_qkv.register_forward_hook(lambda m, a, out: seen.append(out)))
        out = mha(E, pat)
        for h in hooks:
            h.remove()
        if forward:
            del mha.w_o.forward
        for t in seen:
            keep(t)
        return torch.autograd.grad(out, [E, *mha.parameters()], dout)

    def equal(a, b):
        assert all(torch.equal(x, y) for x, y in zip(a, b))

    # a factor of 1 / 2 rounds nothing
    equal(grads(lambda S: (S.mul_(0.5), None)[1]), grads(lambda S: S * 0.5))
    equal(grads(forward=lambda S: linear(S.mul_(0.5))), grads(lambda S: S * 0.5))
    equal(grads(lambda S: (S.data.mul_(0.5), None)[1]), grads(lambda S: S + (S * 0.5 - S).detach()))
    equal(grads(keep=lambda qkv: qkv.data.zero_()), grads(keep=lambda qkv: None))
    equal(grads(keep=lambda qkv: qkv.detach().zero_()), grads(keep=lambda qkv: None))


# Rows of 256, 512, 1024 and 2048 columns in registers and less; 4 rows a workgroup, 16 rows a partial of the weight's
# and bias' gradients, 512 partials at most; a width that is not a multiple of 64 is torch's
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,D", [(1, 64), (3, 192), (17, 256), (129, 320), (9000, 512), (40, 1024), (33, 1088), (16, 2048),
                                    (20, 100)])
def test_layer_norm(sp, dtype, rows, D):
    from paper_2309_12578_amd.sublayer import _Norm
    gen = torch.Generator(device="cuda").manual_seed(rows + D)
    norm = _Norm(D, device="cuda", dtype=dtype)
    x, dy = [torch.randn((1, rows, D), generator=gen, device="cuda") for _ in range(2)]
    x = (x + 5.0).to(dtype).requires_grad_(True)
    dy = dy.to(dtype)
    with torch.no_grad():
        for p in norm.parameters():
            p.copy_(torch.randn(D, generator=gen, device="cuda"))
    y = norm(x)
    got = [y, *torch.autograd.grad(y, [x, *norm.parameters()], dy)]
    x64, w64, b64 = [t.detach().double().requires_grad_(True) for t in (x, norm.weight, norm.bias)]
    y64 = torch.nn.functional.layer_norm(x64, (D,), w64, b64, norm.eps)
    want = [y64, *torch.autograd.grad(y64, [x64, w64, b64], dy.double())]
    # fp32: sums of up to 9000 values of mixed sign, statistics of values around 5: 2^-24 times a few dozen; bf16: one
    # rounding, 2^-9 of each value
    tol = 1e-5 if dtype == torch.float32 else 2.0 ** -8
    for g, r in zip(got, want):
        assert g.dtype == dtype and (g.double() - r).norm() <= tol * r.norm()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,D", [(1, 64), (129, 320), (9000, 512), (40, 1024), (16, 2048)])
def test_residual_around_layer_norm(sp, dtype, rows, D):
    """The gradient of a residual added in LayerNorm's pass; strided, alone, twice and differentiable gradients as without it."""
    from paper_2309_12578_amd.sublayer import _Norm
    gen = torch.Generator(device="cuda").manual_seed(rows + D)
    norm = _Norm(D, device="cuda", dtype=dtype)
    x, dy, dr = [torch.randn((2, rows, D), generator=gen, device="cuda").to(dtype) for _ in range(3)]
    x.requires_grad_(True)
    y = norm(x)
    r = sp.binding._host.residual(x, y)
    assert r is not x and r.data_ptr() == x.data_ptr() and r.grad_fn is y.grad_fn
    assert sp.binding._host.residual(x, y) is x and sp.binding._host.residual(x, y + 1) is x and sp.binding._host.residual(x[:1], y) is not r
    params = [x, *norm.parameters()]
    x64, w64, b64 = [t.detach().double().requires_grad_(True) for t in params]
    y64 = torch.nn.functional.layer_norm(x64, (D,), w64, b64, norm.eps)
    want = torch.autograd.grad([y64, x64 * 1], [x64, w64, b64], [dy.double(), dr.double()])
    tol = 1e-5 if dtype == torch.float32 else 2.0 ** -8   # one rounding of the sum, as in test_layer_norm
    strided = torch.stack([dr, dr], 3)[..., 0]   # added by torch, a rounding more
    for d, t in ((dr, tol), (strided, 2 * tol)):
        got = torch.autograd.grad([y, r], params, [dy, d], retain_graph=True)
        for g, w in zip(got, want):
            assert g.dtype == dtype and (g.double() - w).norm() <= t * w.norm()
    alone, = torch.autograd.grad(r, x, dr, retain_graph=True)
    assert torch.equal(alone, dr)
    with_graph, = torch.autograd.grad([y, r], x, [dy, dr], create_graph=True)
    assert with_graph.requires_grad and (with_graph.double() - want[0]).norm() <= 2 * tol * want[0].norm()
    with torch.no_grad():
        assert sp.binding._host.residual(x, norm(x)) is x


@pytest.mark.parametrize("which", [(1,), (2,), (1, 2), (0,), (0, 2)])
def test_some_gradients_of_a_residual_around_layer_norm(sp, which):
    """Any of X, weight and bias asked for without the others, by kernels, by torch's operators and batched."""
    from paper_2309_12578_amd.sublayer import _Norm
    gen = torch.Generator(device="cuda").manual_seed(7)
    norm = _Norm(128, device="cuda")
    x, dy, dr = [torch.randn((2, 8, 128), generator=gen, device="cuda") for _ in range(3)]
    x.requires_grad_(True)
    y = norm(x)
    r = sp.binding._host.residual(x, y)
    assert r.grad_fn is y.grad_fn
    every = [x, norm.weight, norm.bias]
    inputs = [every[i] for i in which]
    in64 = [t.detach().double().requires_grad_(True) for t in every]
    out64 = torch.nn.functional.layer_norm(in64[0], (128,), in64[1], in64[2], norm.eps)
    want = torch.autograd.grad([out64, in64[0] * 1], in64, [dy.double(), dr.double()])

    def same(got, factor=1.0):
        for g, i in zip(got, which):
            assert (g.double() - factor * want[i]).norm() <= 1e-5 * want[i].norm()   # as test_layer_norm

    for graph in (False, True):
        same(torch.autograd.grad([y, r], inputs, [dy, dr], create_graph=graph, retain_graph=True))
    batched = torch.autograd.grad([y, r], inputs, [torch.stack([t, 2 * t]) for t in (dy, dr)], is_grads_batched=True)
    same([g[0] for g in batched])
    same([g[1] for g in batched], 2.0)


def test_layer_norm_beside_the_other_transforms(sp):
    from paper_2309_12578_amd.sublayer import _Norm
    norm, plain = _Norm(128, device="cuda"), torch.nn.LayerNorm(128, device="cuda")
    x = torch.randn((4, 8, 128), device="cuda", requires_grad=True)
    ad = torch.autograd.forward_ad

    def tangent(f):
        with ad.dual_level():
            return ad.unpack_dual(f(ad.make_dual(x.detach(), x.detach()))).tangent

    def second(f):
        g, = torch.autograd.grad(f(x).pow(3).sum(), x, create_graph=True)
        return torch.autograd.grad(g.square().sum(), x)[0]

    def cast(f):
        with torch.autocast("cuda", dtype=torch.float16):
            return f(x)

    for call in (tangent, second, cast, lambda f: torch.func.vmap(f)(x), lambda f: torch.func.grad(lambda t: f(t).pow(2).sum())(x),
                 lambda f: f(x.detach()), lambda f: f(x.transpose(0, 1))):
        a, b = call(norm), call(plain)
        assert a.dtype == b.dtype and torch.allclose(a, b, rtol=1e-4, atol=1e-4 * b.abs().max().item())


@pytest.mark.parametrize("needs_grad", [False, True])
def test_trace_replays_on_other_inputs(sp, needs_grad):
    """torch.jit.trace records the attention as an operator, also inside the sub-layer: another input, another output."""
    pat, q, k, v, do = _small_attention(sp)
    first, other = [[t.clone().requires_grad_(needs_grad) for t in s] for s in ((q, k, v), (v, q, k))]
    traced = torch.jit.trace(lambda a, b, c: sp.sparse_attention(a, b, c, pat), first, check_trace=False)
    got, want = traced(*other), sp.sparse_attention(*other, pat)
    assert torch.equal(got, want)
    if needs_grad:
        for a, b in zip(torch.autograd.grad(got, other, do), torch.autograd.grad(want, other, do)):
            assert torch.equal(a, b)

    class Layer(torch.nn.Module):
        def __init__(self):
            super().__init__()
            self.mha = sp.SparseMHA(128, 2, device="cuda")

        def forward(self, x):
            return self.mha(x, pat)

    layer = Layer().requires_grad_(needs_grad)
    E, E2 = [t.transpose(1, 2).reshape(1, -1, 128) for t in (q, k)]
    traced = torch.jit.trace(layer, E, check_trace=False)
    got, want = traced(E2), layer(E2)
    # LayerNorm and the products are torch's under a trace: fp32 sums of 128 values in another order
    assert torch.allclose(got, want, rtol=1e-5, atol=1e-5)
    if needs_grad:
        for a, b in zip(*[torch.autograd.grad(t.square().sum(), list(layer.parameters())) for t in (got, want)]):
            assert (a - b).norm() <= 1e-5 * b.norm()


@pytest.mark.parametrize("node", ["projection", "norm"])
def test_incoming_gradients_that_are_not_plain(sp, node):
    """A tangent or a batch that only the incoming gradient has (the loss is differentiated forward, or over a batch of
    losses): the nodes of the sub-layer hand it on as torch's operators do."""
    from paper_2309_12578_amd.sublayer import _Norm, _Projection
    kw = dict(device="cuda", dtype=torch.bfloat16)
    ours, plain = (_Projection(64, 192, **kw), torch.nn.Linear(64, 192, **kw)) if node == "projection" else (_Norm(64, **kw), torch.nn.LayerNorm(64, **kw))
    plain.load_state_dict(ours.state_dict())
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((4, 32, 64), generator=gen, device="cuda").to(torch.bfloat16).requires_grad_(True)
    dy = torch.randn((3, 4, 32, plain(x).shape[-1]), generator=gen, device="cuda").to(torch.bfloat16)
    ad = torch.autograd.forward_ad
    result = []
    for layer in (ours, plain):
        wrt = [x, *layer.parameters()]
        with ad.dual_level():
            duals = [ad.unpack_dual(g) for g in torch.autograd.grad(layer(x), wrt, ad.make_dual(dy[0], dy[1]))]
            assert all(d.tangent is not None for d in duals)
            result.append([t.float() for d in duals for t in d] +
                          [t.float() for t in torch.autograd.grad(layer(x), wrt, dy, is_grads_batched=True)])
    for a, b in zip(*result):   # sums in fp32, one rounding to bf16 each
        assert a.shape == b.shape and (a - b).norm() <= 2.0 ** -7 * b.norm()


# Scores far below 0 under Algorithm 6's denominator, 29 log2 units lower in the first half of the keys (where every
# wave, and every row whose diagonal lies there, starts) than in the second: the waves' sums are scaled down by 2^-154 altogether.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("block,nb,heads", [(16, 40, 1), (32, 16, 1), (64, 8, 1), (16, 40, 256), (32, 16, 512), (64, 8, 512)])
def test_paper_denominator_far_below_zero(sp, dtype, block, nb, heads):
    from test_gpu_parity import _pattern_from_mask
    L, d = nb * block, 64
    rng = np.random.default_rng(block)
    Q, K, V = [np.zeros((1, L, d), dtype=np.float32) for _ in range(3)]
    Q[:, :, 0] = 8.0                                        # scores 8 * K[..., 0] / 8
    K[:, :L // 2, 0], K[:, L // 2:, 0] = -107.0, -87.0
    V[:] = si.round_to_dtype(rng.standard_normal((1, L, d), dtype=np.float32), dtype) * 2.0 ** 24
    fl = np.ones((nb, nb), dtype=np.uint8)
    q, k, v = [torch.from_numpy(t).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32).expand(heads, L, d)[None].contiguous()
               for t in (Q, K, V)]
    # nothing masked: nothing to add to the denominator, however small the kept probabilities' exponentials
    pat = _pattern_from_mask(sp, fl, block)
    for a, b in zip(sp.attn_fwd(q, k, v, pat, flags=sp.SPION_ATTN_PAPER_DENOM), sp.attn_fwd(q, k, v, pat)):
        assert torch.equal(a, b) and a.abs().min() > 0
    low = k.clone()
    low[..., 0] *= 4
    for a, b in zip(sp.attn_fwd(q, low, v, pat, flags=sp.SPION_ATTN_PAPER_DENOM), sp.attn_fwd(q, low, v, pat)):
        assert torch.equal(a, b) and a.abs().min() > 0
    # one block masked: O is of the order of 2^-126 * V / block
    fl[:, nb // 2 + 1] = 0
    fl[nb // 2 + 1, nb // 2 + 1] = 1
    O, LSE = sp.attn_fwd(q, k, v, _pattern_from_mask(sp, fl, block), flags=sp.SPION_ATTN_PAPER_DENOM)
    rO, rLSE = oracle.attn_fwd(Q, K, V, oracle.upsample(fl, block), flags=oracle.ATTN_PAPER_DENOM)
    for h in (0, heads - 1):
        x, lse = O[0, h].double().cpu().numpy(), LSE[0, h].cpu().numpy()
        # fp32: an exponential of 126 +- 2^-17 log2 units; bf16: P and O rounded to 2^-9 of each value
        assert np.linalg.norm(x - rO[0]) <= (2.0 ** -15 if dtype == "f32" else 2.0 ** -7) * np.linalg.norm(rO[0])
        assert np.abs(lse - rLSE[0]).max() <= 1e-5 * np.abs(rLSE[0]).max()


def test_buffers_larger_than_needed(sp):
    """attn_fwd and attn_bwd write the first elements of a buffer that has room for more, and refuse smaller ones."""
    pat, q, k, v, do = _small_attention(sp)
    o, lse = sp.attn_fwd(q, k, v, pat)
    want = sp.attn_bwd(q, k, v, o, do, lse, pat)

    def room(t):
        return torch.full((t.numel() + 100,), 7.0, dtype=t.dtype, device="cuda")

    O, LSE = sp.attn_fwd(q, k, v, pat, O=room(o), LSE=room(lse))
    grads = sp.attn_bwd(q, k, v, O, do, LSE, pat, dQ=room(q), dK=room(q), dV=room(q))
    for a, b in zip((O, LSE, *grads), (o, lse, *want)):
        assert torch.equal(a[:b.numel()], b.flatten()) and (a[b.numel():] == 7.0).all()
    small = torch.empty(q.numel() - 1, device="cuda")
    for kw in (dict(O=small), dict(LSE=small[:lse.numel() - 1]), dict(O=torch.empty_like(q, dtype=torch.bfloat16))):
        with pytest.raises(ValueError):
            sp.attn_fwd(q, k, v, pat, **kw)
    for name in ("dQ", "dK", "dV"):
        with pytest.raises(ValueError):
            sp.attn_bwd(q, k, v, o, do, lse, pat, **{name: small})
    for args in ((q, small, v), (q, k, small)):
        with pytest.raises(ValueError):
            sp.attn_fwd(*args, pat)


# Sorted rows (more workgroups than run at once: 1024 of block 64, 2048 of block 32) at head counts that do not divide
# over the 8 XCDs, workgroup counts that do and do not, and no long row, one, and many.  A row's result does not depend
# on where it runs: the same bits as one head at a time, which is not sorted.
@pytest.mark.parametrize("BH,nb,block,long_rows", [(9, 130, 64, 0), (9, 130, 64, 1), (12, 96, 64, 3), (5, 206, 64, 20), (20, 130, 32, 7),
                                                   (13, 161, 32, 1), (16, 130, 32, 5), (1030, 1, 64, 0), (1033, 2, 32, 1)])
def test_forward_sorted_rows_at_odd_head_counts(sp, BH, nb, block, long_rows):
    from test_gpu_parity import _pattern_from_mask
    rng = np.random.default_rng(nb + BH)
    fl = np.eye(nb, dtype=np.uint8)
    fl[rng.integers(0, nb, nb), rng.integers(0, nb, nb)] = 1
    fl[rng.choice(nb, long_rows, replace=False)] = 1
    pat = _pattern_from_mask(sp, fl, block)
    gen = torch.Generator(device="cuda").manual_seed(BH)
    q, k, v = [torch.randn((1, BH, nb * block, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    O = torch.full_like(q, float("nan"))
    LSE = torch.full(q.shape[:3], float("nan"), device="cuda")
    sp.attn_fwd(q, k, v, pat, O=O, LSE=LSE)
    for h in range(0, BH, max(1, BH // 24)):
        o, lse = sp.attn_fwd(*[t[:, h:h + 1].contiguous() for t in (q, k, v)], pat)
        assert torch.equal(O[:, h:h + 1], o) and torch.equal(LSE[:, h:h + 1], lse), h
    assert not O.isnan().any() and not LSE.isnan().any()


# Heads that do not divide over the XCDs (and some that do), block rows that are no multiple of 8: every row and column of every head once.  Rows as they lie,
# dealt and by length; the backward dealt from 513 workgroups on
@pytest.mark.parametrize("BH,nb,block,mean", [(5, 20, 64, 3), (3, 86, 64, 7), (9, 61, 64, 3), (13, 64, 32, 3), (23, 35, 32, 4), (65, 13, 32, 3), (63, 17, 64, 3),
                                              (7, 100, 64, 1), (7, 150, 64, 8), (31, 70, 32, 7), (127, 9, 64, 2), (24, 27, 64, 3), (1, 600, 32, 3)])
def test_heads_dealt_over_the_xcds(sp, BH, nb, block, mean):
    from test_gpu_parity import _pattern_from_mask
    rng = np.random.default_rng(nb)
    fl = np.eye(nb, dtype=np.uint8)
    if mean > 1:
        fl |= (rng.random((nb, nb)) < (mean - 1) / nb).astype(np.uint8)
        fl[:, 2] = 1
        fl[3, 3] = 0
    pat = _pattern_from_mask(sp, fl, block)
    gen = torch.Generator(device="cuda").manual_seed(BH)
    one = [torch.randn((1, 1, nb * block, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4)]
    # heads told apart by powers of two, so that their results are the first one's, multiplied, to the bit
    h = torch.arange(BH, device="cuda").view(1, BH, 1, 1)
    sq, sv, sdo = [(2.0 ** (h % n)).to(torch.bfloat16) for n in (3, 7, 5)]
    q, k, v, do = [t * f for t, f in zip(one, (sq, 1 / sq, sv, sdo))]
    nan = lambda: torch.full_like(q, float("nan"))
    o, lse = sp.attn_fwd(q, k, v, pat, O=nan(), LSE=torch.full(q.shape[:3], float("nan"), device="cuda"))
    grads = sp.attn_bwd(q, k, v, o, do, lse, pat, dQ=nan(), dK=nan(), dV=nan())
    for x, f in zip((o, lse.unsqueeze(3), *grads), (sv, torch.ones_like(lse).unsqueeze(3), sv * sdo / sq, sv * sdo * sq, sdo)):
        assert torch.equal(x, x[:, :1] * f)   # (a NaN would not be equal)
    want, want_lse = sp.attn_fwd(*one[:3], pat)
    for x, w in zip((o, *grads), (want, *sp.attn_bwd(*one[:3], want, one[3], want_lse, pat))):   # other cuts of rows and columns: sums in another order, rounded to bf16
        assert torch.linalg.vector_norm(x[:, :1].float() - w.float()) <= 1e-2 * torch.linalg.vector_norm(w.float())


# Whole heads on every XCD: rows by length, of one, two, four and more groups of 64 block rows, the last group full and not
@pytest.mark.parametrize("BH,nb,block", [(24, 64, 64), (24, 65, 64), (24, 128, 32), (8, 129, 64), (8, 256, 64), (8, 257, 32), (8, 512, 32), (8, 513, 32), (8, 1000, 32), (8, 1024, 32)])
def test_forward_rows_by_length(sp, BH, nb, block):
    from test_gpu_parity import _pattern_from_mask
    rng = np.random.default_rng(nb)
    fl = (rng.random((nb, nb)) < rng.random((nb, 1)) * 12 / nb).astype(np.uint8)   # 0 to about 20 blocks a row
    fl[rng.choice(nb, 3, replace=False)] = rng.random((3, nb)) < 60 / nb
    fl[5] = 0
    pat = _pattern_from_mask(sp, fl, block)
    gen = torch.Generator(device="cuda").manual_seed(BH)
    q, k, v = [torch.randn((1, BH, nb * block, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    O = torch.full_like(q, float("nan"))
    LSE = torch.full(q.shape[:3], float("nan"), device="cuda")
    index = (pat.row_ptr, pat.col_idx, pat.nnzb)
    shape = (nb * block, 64, block, sp.SPION_BF16)
    sp.spion_attn_fwd(q, k, v, O, LSE, *index, 1, BH, *shape)   # without room for pieces: no row is cut
    for h in (0, BH // 2, BH - 1):
        args = [t[:, h:h + 1].contiguous() for t in (q, k, v, O, LSE)]
        args[3].zero_(), args[4].zero_()
        sp.spion_attn_fwd(*args, *index, 1, 1, *shape)
        assert torch.equal(O[:, h:h + 1], args[3]) and torch.equal(LSE[:, h:h + 1], args[4]), h
    assert not O.isnan().any() and not LSE.isnan().any()


@pytest.mark.parametrize("block,H", [(32, 190000), (64, 90000)])
def test_heads_beside_each_other_whose_rows_are_far_apart(sp, block, H):
    """In the projections' output of so many heads the last rows of a tile lie more than 2^31 bytes from its first."""
    import ctypes
    from test_gpu_parity import TOL, _pattern_from_mask
    L = block
    pat = _pattern_from_mask(sp, np.ones((L // block, L // block), dtype=np.uint8), block)
    qkv = torch.randn((1, L, 3, H, 64), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda", dtype=torch.bfloat16)
    dS = torch.randn((1, L, H, 64), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda", dtype=torch.bfloat16)
    S, dqkv, LSE = torch.zeros_like(dS), torch.zeros_like(qkv), torch.zeros((1, H, L), device="cuda")
    lib, p = sp.load(), sp.binding._AttnParams(1, H, L, 64, block, sp.SPION_BF16, 0.0, 0)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib.spion_heads_attn_fwd(ptr(qkv), ptr(S), ptr(LSE), ptr(pat.row_ptr), ptr(pat.col_idx), pat.nnzb, ctypes.byref(p), None,
                                    ctypes.c_size_t(0), stream) == 0
    ws = torch.zeros(sp.spion_attn_workspace_bytes(1, H, L, 64, block, sp.SPION_BF16, pat.nnzb, True), dtype=torch.uint8, device="cuda")
    assert lib.spion_heads_attn_bwd(ptr(qkv), ptr(S), ptr(dS), ptr(LSE), ptr(dqkv), ptr(pat.row_ptr), ptr(pat.col_idx), ptr(pat.col_ptr),
                                    ptr(pat.row_idx), pat.nnzb, ctypes.byref(p), ptr(ws), ctypes.c_size_t(ws.numel()), stream) == 0
    for h in (0, H // 2, H - 1):
        q, k, v = [qkv[0, :, i, h] for i in range(3)]
        want = _dense_reference(q, k, v, dS[0, :, h], np.ones((L // block, L // block), dtype=np.uint8), block)
        for name, got, w in zip(("O", "dQ", "dK", "dV"), (S[0, :, h], *(dqkv[0, :, i, h] for i in range(3))), want):
            error = torch.linalg.vector_norm(got - w) / torch.linalg.vector_norm(w)
            assert error <= TOL["bf16"], (name, h, float(error))
