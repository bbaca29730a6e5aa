"""The work a user of this package has it do, as named cases with inputs, one pass and its outputs.

Four kinds of case, after the way SPION trains a Transformer:
  attn       block-sparse attention of one layer on a fixed pattern: a training step (forward and
             backward, through autograd or through the two calls) or a forward pass alone
  mha        a training step of the whole sparse multi-head-attention sub-layer (`SparseMHA`)
  pattern    one layer's pattern from its averaged score map (`generate_pattern`)
  producers  what comes before it: the mean of a layer's score maps and the transition test's distance

Sizes are those of the five configurations of `spion_inputs.py`, of the tests, and of longer sequences
in between; `draw` spreads over the same ranges.
"""
import math

import numpy as np
import torch

import paper_2309_12578_amd as sp

HEAD_DIM = 64
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _attn(name, dtype, B, H, L, block, density, via="calls", backward=True, paper_denom=False):
    return dict(name=name, kind="attn", dtype=dtype, B=B, H=H, L=L, block=block, density=density, via=via,
                backward=backward, paper_denom=paper_denom)


def _pattern(name, L, block, filt, mode, value, no_fill=False):
    return dict(name=name, kind="pattern", L=L, block=block, filt=filt, mode=mode, value=value, no_fill=no_fill)


def listed():
    return [
        # configuration 1: one small fp32 head through autograd; nothing but call overhead and launches
        _attn("tiny_f32_step", "f32", 1, 1, 256, 16, 0.074, via="autograd"),
        # configuration 2: many short sequences, block 32
        _attn("cfg2_step", "bf16", 16, 4, 1024, 32, 0.15),
        # configuration 4, the one the benchmark quotes
        _attn("cfg4_step", "bf16", 4, 4, 4096, 64, 0.08),
        # configuration 5, the densest of its four layers
        _attn("cfg5_dense_step", "bf16", 4, 8, 4096, 64, 0.208),
        # full-precision training at the shape of configuration 3
        _attn("f32_step", "f32", 2, 4, 2048, 32, 0.10, via="autograd"),
        # fine blocks, odd batch, head and block counts, the literal denominator of Algorithm 6
        _attn("ragged_b16_step", "bf16", 3, 3, 1936, 16, 0.08, paper_denom=True),
        # inference on long documents: forward only, 255 block rows
        _attn("long_fwd", "bf16", 2, 8, 16320, 64, 0.05, backward=False),
        # the sub-layer a model is built of, at the shape of configuration 3: LayerNorm, projections, heads
        dict(name="mha_step", kind="mha", dtype="bf16", B=8, H=4, L=2048, block=32, density=0.10),
        # pattern generation: the tiny map with its mean + 1 std threshold, the benchmark's map, and a
        # long sequence pooled finely (512 x 512 cells)
        _pattern("pattern_cfg1", 256, 16, 5, "mean_kstd", 1.0),
        _pattern("pattern_cfg4", 4096, 64, 31, "quantile", 0.88),
        _pattern("pattern_grid512", 8192, 16, 15, "quantile", 0.93),
        # the end of an epoch of the dense phase: 16 per-head maps averaged, distance to the map before
        dict(name="producers_cfg4", kind="producers", dtype="bf16", maps=16, L=4096),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_shape(rng, dtype, blocks, B_max, H_max, flops_max, tokens_max):
    """B, H, L, block, density with bounded cost; rejection keeps the spread of each size as it is."""
    while True:
        block = rng.choice(blocks)
        nb = int(round(_log_uniform(rng, 4, 256)))
        B = int(round(_log_uniform(rng, 1, B_max)))
        H = rng.randint(1, H_max)
        density = round(max(_log_uniform(rng, 0.03, 0.30), 1.0 / nb), 4)
        flops = 12 * HEAD_DIM * block * block * density * nb * nb * B * H
        if flops <= flops_max and B * H * nb * block <= tokens_max:
            return dict(B=B, H=H, L=nb * block, block=block, density=density)


def draw(rng):
    kind = rng.choices(("attn", "fwd", "mha", "pattern", "producers"), (9, 3, 2, 5, 1))[0]
    if kind in ("attn", "fwd"):
        dtype = rng.choices(("bf16", "f32"), (3, 1))[0]
        block = rng.choices((16, 32, 64), (1, 2, 3))[0]
        tuned = dtype == "bf16" and block > 16
        shape = _draw_shape(rng, dtype, (block,), 16, 8, 8.5e10 if tuned else 2e9, 2 ** 18)
        return dict(kind="attn", dtype=dtype, via=rng.choice(("calls", "autograd")), backward=kind == "attn",
                    paper_denom=rng.random() < 0.2, **shape)
    if kind == "mha":
        dtype = rng.choices(("bf16", "f32"), (3, 1))[0]
        return dict(kind="mha", dtype=dtype,
                    **_draw_shape(rng, dtype, (32, 64), 8, 8, 2e10 if dtype == "bf16" else 1e9, 2 ** 15))
    if kind == "pattern":
        block = rng.choice((16, 32, 64))
        mode = rng.choices(("quantile", "mean_kstd"), (3, 1))[0]
        nb = int(round(_log_uniform(rng, 8, min(512, 8192 // block) if mode == "quantile" else 64)))
        value = round(rng.uniform(0.5, 0.98), 3) if mode == "quantile" else round(rng.uniform(0.5, 2.0), 2)
        filt = rng.choice([f for f in (1, 5, 15, 31, 63) if (f - 1) // 2 < block])
        return dict(kind="pattern", L=nb * block, block=block, filt=filt, mode=mode, value=value,
                    no_fill=rng.random() < 0.15)
    maps = int(round(_log_uniform(rng, 2, 16)))
    return dict(kind="producers", dtype=rng.choice(("bf16", "f32")), maps=maps,
                L=8 * int(round(_log_uniform(rng, 32, 512 if maps <= 8 else 362))))


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _kept(case):
    nb = case["L"] // case["block"]
    return min(nb * nb, max(nb, int(round(case["density"] * nb * nb))))


def _block_mask(nb, kept, seed):
    """A layer's block pattern with exactly `kept` blocks, of the make the generator's patterns have:
    the diagonal, part of a narrow band beside it, some columns kept over long runs of rows (vertical
    stripes), a row or two far longer than the rest, and a little that is scattered."""
    rng = np.random.default_rng(seed)
    score = rng.random((nb, nb)) * 0.5
    i = np.arange(nb)
    for off in (-1, 1):
        j = i + off
        ok = (j >= 0) & (j < nb)
        score[i[ok], j[ok]] += rng.choice((0.4, 1.2), size=int(ok.sum()))
    spare = kept - nb
    n_cols = max(1, int(round(spare / (0.7 * nb))))
    for c in rng.choice(nb, min(n_cols, nb), replace=False):
        run = max(1, int(nb * rng.uniform(0.35, 1.0)))
        r0 = int(rng.integers(0, nb - run + 1))
        score[r0:r0 + run, c] += 1.0
    if spare > 5 * nb:
        for r in rng.choice(nb, 2, replace=False):
            run = max(1, int(nb * rng.uniform(0.3, 0.6)))
            c0 = int(rng.integers(0, nb - run + 1))
            score[r, c0:c0 + run] += 1.0
    score[i, i] = 10.0
    flat = score.reshape(-1)
    mask = np.zeros(nb * nb, dtype=np.int64)
    mask[np.argpartition(-flat, kept - 1)[:kept]] = 1
    return mask.reshape(nb, nb)


def _index_buffers(L, block, pool):
    """The arrays of one layer's pattern, as a program that makes its patterns anew keeps them (zeroed
    once: of the index arrays only the first nnzb entries are ever written)."""
    nb = L // block
    i32 = dict(dtype=torch.int32, device="cuda")
    return sp.Pattern(L, block, torch.zeros((nb, nb), dtype=torch.uint8, device="cuda"), torch.zeros(nb + 1, **i32),
                      torch.zeros(nb * nb, **i32), torch.zeros(nb + 1, **i32), torch.zeros(nb * nb, **i32),
                      torch.zeros(nb * nb, **i32), torch.zeros(1, **i32), pool)


def _layer_pattern(case, seed):
    """The layer's pattern as spion_pattern leaves it, made from pooled sums that are the mask itself."""
    L, block = case["L"], case["block"]
    nb = L // block
    pool = torch.from_numpy(_block_mask(nb, _kept(case), seed) << 40).cuda()
    pat = _index_buffers(L, block, pool)
    ws = torch.empty(sp.spion_pattern_workspace_bytes(L, block), dtype=torch.uint8, device="cuda")
    sp.spion_pattern(None, L, block, 1, sp.SPION_T_ABS, 0.0, pat.fl_out, pat.row_ptr, pat.col_idx, pat.col_ptr,
                     pat.row_idx, pat.bsr_pos, pat.nnzb_dev, pool, ws,
                     flags=sp.SPION_PATTERN_FROM_POOL | sp.SPION_PATTERN_NO_FILL)
    pat.nnzb = int(pat.nnzb_dev.item())
    return pat


def _score_maps(gen, n, L, filt_band):
    """n maps of row-softmax scores with a diagonal band and vertical stripes, fp32 [n, L, L]."""
    i = torch.arange(L, device="cuda")
    bias = ((i[:, None] - i[None, :]).abs() <= filt_band).to(torch.float32)
    width = max(4, L // 256)
    starts = torch.randint(0, L - width + 1, (max(3, min(16, L // 256)),), generator=gen, device="cuda")
    stripe = ((i[None, :] >= starts[:, None]) & (i[None, :] < starts[:, None] + width)).any(0)
    bias = (bias.bool() | stripe[None, :]).to(torch.float32).mul_(4.0)
    maps = torch.empty((n, L, L), dtype=torch.float32, device="cuda")
    for m in range(n):
        logits = torch.randn((L, L), generator=gen, device="cuda").mul_(0.3 if n == 1 else 1.0).add_(bias)
        torch.softmax(logits, dim=1, out=maps[m])
    return maps


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(DTYPES[case["dtype"]])

    kind = case["kind"]
    if kind == "attn":
        shape = (case["B"], case["H"], case["L"], HEAD_DIM)
        q, k, v = [randn(*shape) for _ in range(3)]
        if case["backward"] and case["via"] == "autograd":
            for t in (q, k, v):
                t.requires_grad_(True)
        return dict(case=case, pat=_layer_pattern(case, seed), q=q, k=k, v=v,
                    do=randn(*shape) if case["backward"] else None,
                    flags=sp.SPION_ATTN_PAPER_DENOM if case["paper_denom"] else 0)
    if kind == "mha":
        D = HEAD_DIM * case["H"]
        mha = sp.SparseMHA(D, case["H"], dropout=0.0, device="cuda", dtype=DTYPES[case["dtype"]])
        with torch.no_grad():
            for p in mha.parameters():
                p.copy_(randn(*p.shape) * (D ** -0.5) if p.dim() == 2 else 1.0 + 0.1 * randn(*p.shape))
        E = randn(case["B"], case["L"], D).requires_grad_(True)
        return dict(case=case, pat=_layer_pattern(case, seed), mha=mha, E=E, dout=randn(case["B"], case["L"], D))
    if kind == "pattern":
        nb = case["L"] // case["block"]
        return dict(case=case, A=_score_maps(gen, 1, case["L"], max(4, case["L"] // 64))[0],
                    pat=_index_buffers(case["L"], case["block"], torch.zeros((nb, nb), dtype=torch.int64, device="cuda")))
    maps = _score_maps(gen, case["maps"], case["L"], max(4, case["L"] // 64)).to(DTYPES[case["dtype"]])
    prev = _score_maps(gen, 1, case["L"], max(4, case["L"] // 32))[0]
    return dict(case=case, maps=maps, prev=prev)


# ------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------
def _run_attn(s):
    case, pat, q, k, v = s["case"], s["pat"], s["q"], s["k"], s["v"]
    if case["via"] == "autograd":
        q.grad = k.grad = v.grad = None
        o = sp.sparse_attention(q, k, v, pat, flags=s["flags"])
        if not case["backward"]:
            return {"O": o}
        o.backward(s["do"])
        return {"O": o.detach(), "dQ": q.grad, "dK": k.grad, "dV": v.grad}
    o, lse = sp.attn_fwd(q, k, v, pat, flags=s["flags"])
    if not case["backward"]:
        return {"O": o, "LSE": lse}
    dq, dk, dv = sp.attn_bwd(q, k, v, o, s["do"], lse, pat, flags=s["flags"])
    return {"O": o, "LSE": lse, "dQ": dq, "dK": dk, "dV": dv}


def run(s):
    case = s["case"]
    if case["kind"] == "attn":
        return _run_attn(s)
    if case["kind"] == "mha":
        mha, E = s["mha"], s["E"]
        E.grad = None
        mha.zero_grad(set_to_none=True)
        out = mha(E, s["pat"])
        out.backward(s["dout"])
        return [out.detach(), E.grad] + [p.grad for p in mha.parameters()]
    if case["kind"] == "pattern":
        mode = sp.SPION_T_QUANTILE if case["mode"] == "quantile" else sp.SPION_T_MEAN_KSTD
        p = sp.generate_pattern(s["A"], case["block"], case["filt"], mode, case["value"],
                                flags=sp.SPION_PATTERN_NO_FILL if case["no_fill"] else 0, out=s["pat"])
        return {"fl_out": p.fl_out, "row_ptr": p.row_ptr, "col_idx": p.col_idx, "col_ptr": p.col_ptr,
                "row_idx": p.row_idx, "bsr_pos": p.bsr_pos, "pool_sum": p.pool_sum, "nnzb": p.nnzb}
    A = sp.score_mean(s["maps"])
    return {"A": A, "distance": sp.frobenius_distance(s["prev"], A)}


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far another correct implementation may be off
# ------------------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind in ("attn", "mha"):
        esz = 4 if case["dtype"] == "f32" else 2
        BH, L = case["B"] * case["H"], case["L"]
        tile = 2 * case["block"] ** 2 * HEAD_DIM * _kept(case) * BH   # one tile product over all kept blocks
        t = BH * L * HEAD_DIM * esz
        if kind == "attn":
            if not case["backward"]:   # Q, K, V in, O and LSE out
                return {"bytes": 4 * t + 4 * BH * L, "flops": 2 * tile}
            # forward as above; backward: Q, K, V, O, dO, LSE in, dQ, dK, dV out
            return {"bytes": 12 * t + 8 * BH * L, "flops": 6 * tile}
        D, rows = HEAD_DIM * case["H"], case["B"] * L
        # E in and out, dOut in, dE out; weights in, their gradients out; four projections, three products each
        return {"bytes": 4 * rows * D * esz + 2 * 4 * D * D * esz, "flops": 6 * tile + 3 * 2 * 4 * rows * D * D}
    if kind == "pattern":
        nb = case["L"] // case["block"]
        return {"bytes": 4 * case["L"] ** 2 + 9 * nb * nb, "flops": 2 * case["L"] ** 2}
    n = case["L"] ** 2
    esz = 4 if case["dtype"] == "f32" else 2
    # the maps and the previous map in, the mean out (its norm is taken on the way); sums and squares
    return {"bytes": (case["maps"] * esz + 8) * n, "flops": (case["maps"] + 5) * n}


def tolerance(case):
    if case["kind"] == "pattern":
        return "exact"   # masks, indices and fixed-point sums
    if case["kind"] == "producers" or (case["kind"] == "attn" and case["dtype"] == "f32"):
        return {"rel": 1e-5, "max": 1e-4}
    if case["dtype"] == "f32":
        return {"rel": 5e-5, "max": 1e-3}   # the sub-layer: five chained products of 32-bit sums
    return {"rel": 1e-2, "max": 1e-1}
