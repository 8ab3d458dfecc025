"""Edges of the kernels' tiles and of the rules that choose between kernels, one small case each (GPU)."""
import numpy as np
import pytest

from helpers import cfg_desc
from workload import CONFIGS, make_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2502_03805_amd as P
    P.load()
    return P


def magnitudes64(v, w_o, H, norm):
    """Row norms of V^g W_O^h in float64: v [b,Hkv,n,dh], w_o [H*dh, d_model] -> [b,H,n]."""
    b, Hkv, n, dh = v.shape
    out = np.empty((b, H, n))
    for bi in range(b):
        for h in range(H):
            p = v[bi, h * Hkv // H].astype(np.float64) @ w_o[h * dh:(h + 1) * dh].astype(np.float64)
            out[bi, h] = np.abs(p).sum(-1) if norm == 1 else np.sqrt(np.square(p).sum(-1))
    return out


def score(P, desc, q, k, v, w_o, ws_bytes=None):
    import torch
    b, H, Hkv, n = desc.batch, desc.n_q_heads, desc.n_kv_heads, desc.n_ctx
    ws = torch.empty(P.workspace_bytes(desc, 1) if ws_bytes is None else ws_bytes, dtype=torch.uint8, device="cuda")
    attn = torch.empty((b, Hkv, n), dtype=torch.float32, device="cuda")
    crit, vnorm = torch.empty_like(attn), torch.empty((b, H, n), dtype=torch.float32, device="cuda")
    P.criticalkv_score(desc, q, k, v, w_o, attn, crit, vnorm, workspace=ws)
    torch.cuda.synchronize()
    return attn.cpu().numpy(), crit.cpu().numpy(), vnorm.cpu().numpy()


# ---- fp32 magnitudes on the matrix cores (every operand as two f16 parts) ---------------------------------------
# n around one and several workgroups of either row-block count, d_model of one tile and of an odd number of tiles
@pytest.mark.parametrize("norm", [1, 2])
@pytest.mark.parametrize("wo_out_in", [False, True])
@pytest.mark.parametrize("dh,H,Hkv,n,dm", [(128, 2, 1, 63, 32), (128, 8, 2, 65, 96), (128, 32, 8, 1217, 64),
                                           (64, 3, 3, 64, 32), (64, 8, 2, 257, 160), (64, 40, 8, 961, 96)])
def test_fp32_magnitudes_against_float64(P, dh, H, Hkv, n, dm, wo_out_in, norm):
    """The split's error is 9e-8 of a product (rms, random in sign); the sums are fp32 (d_h terms, then d_model / 16
    magnitudes per accumulator): 2e-6 covers both, and the vector kernel's error is the yardstick."""
    import torch
    cfg = CONFIGS["tiny"].with_(head_dim=dh, n_q_heads=H, n_kv_heads=Hkv, n_ctx=n, d_model=dm, window=8, batch=2)
    t = make_layer(cfg)
    ref = magnitudes64(t["v"], t["w_o"], H, norm)
    dev = {name: torch.from_numpy(a).cuda() for name, a in t.items()}
    w = dev["w_o"].t().contiguous() if wo_out_in else dev["w_o"]
    v = torch.zeros((2, n, Hkv, dh + 4), device="cuda")[..., :dh].permute(0, 2, 1, 3)  # a strided cache: [b, n, Hkv, dh+4]
    v.copy_(dev["v"])
    flags = P.CKV_WO_OUT_IN if wo_out_in else 0
    err = {}
    for name, extra in (("split", 0), ("vector", P.CKV_NO_MFMA)):
        desc = cfg_desc(P, cfg, flags=flags | extra, norm=norm, v_stride=v.stride()[:3])
        got = score(P, desc, dev["q_win"], dev["k"], v, w)[2]
        err[name] = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        assert np.abs(got - ref).max() <= 2e-6 * np.abs(ref).max()
    assert err["split"] <= max(1.05 * err["vector"], 2e-7), err


@pytest.mark.parametrize("v_scale,w_scale", [(1e30, 1e-30), (1e-25, 1e25), (3.0e38, 1e-20), (1e-30, 1e-3), (1e-35, 1.0), (1e-37, 1.0),
                                             (1.0, 1e-36), (1e-37, 1e30), (2.0 ** -59, 2.0 ** -56), (2.0 ** 59, 2.0 ** 55)])
def test_fp32_magnitudes_over_the_exponent_range(P, v_scale, w_scale):
    """Entries from the last half step below FLT_MAX (whose nearest bf16 is infinite) down to where a third bf16 part would
    be subnormal, and around the ends of the range that the split takes."""
    import torch
    cfg = CONFIGS["tiny"].with_(n_ctx=130, d_model=64)
    t = make_layer(cfg)
    v = np.clip(t["v"] / np.abs(t["v"]).max(), -1, 1).astype(np.float32) * np.float32(v_scale)
    if v_scale > 1e38:
        v[0, 0, 5, 3], v[0, 1, 7, 0] = np.finfo(np.float32).max, -np.finfo(np.float32).max
    w = (t["w_o"] * np.float32(w_scale)).astype(np.float32)
    ref = magnitudes64(v, w, cfg.n_q_heads, 1)
    dev = [torch.from_numpy(a).cuda() for a in (t["q_win"], t["k"], v, w)]
    err = []
    for flags in (0, P.CKV_NO_MFMA):
        got = score(P, cfg_desc(P, cfg, flags=flags), *dev)[2]
        assert np.isfinite(got).all()
        # fp32 sums: 2e-6; where they are subnormal each of the d_h * d_model steps rounds by up to 2^-150 in either kernel
        assert (np.abs(got - ref) <= 2e-6 * ref + cfg.head_dim * cfg.d_model * 2.0 ** -150).all()
        err.append(np.abs(got / ref - 1).max())
    assert err[0] <= 1.2 * err[1] + 1.2e-7, err # a few ulp beyond the vector kernel's at most


@pytest.mark.parametrize("norm", [1, 2])
@pytest.mark.parametrize("dh", [64, 128])
def test_fp32_magnitudes_of_rows_their_largest_entry_does_not_reach(P, dh, norm):
    """A row's largest entry meets nothing (a zero row of W_O, or two opposite equal ones), so that the result comes from
    entries 2^4 .. 2^60 smaller, and a column's entries are that much smaller than their tile's largest: the parts alone
    would lose them.  What is lost of an entry is up to 2^-23 of it and 2^-40 of its row's largest; rows where that could show are
    taken in fp32: 2e-6 as everywhere."""
    import torch
    n, dm = 160, 96
    r = np.random.Generator(np.random.PCG64(dh + norm))
    v, w = (r.standard_normal(s).astype(np.float32) for s in ((1, 2, n, dh), (2 * dh, dm)))
    w = np.sign(w) * np.clip(np.abs(w), 1e-3, None)
    w[5], w[dh + 7], w[dh + 9] = 0.0, w[dh + 8], np.ldexp(w[dh + 9], -45)
    w[:, 40] = np.ldexp(w[:, 40], -33)
    for i in range(n):
        v[0, 0, i, 5] = np.ldexp(1.0, 4 + i % 57)
        if i % 3:
            v[0, 1, i, 7], v[0, 1, i, 8] = np.ldexp(1.0, i % 41), -np.ldexp(1.0, i % 41)
    ref = magnitudes64(v, w, 2, norm)
    cfg = CONFIGS["tiny"].with_(head_dim=dh, n_q_heads=2, n_kv_heads=2, n_ctx=n, d_model=dm, window=8)
    q, k = torch.randn((1, 2, 8, dh), device="cuda"), torch.randn((1, 2, n, dh), device="cuda")
    got = score(P, cfg_desc(P, cfg, norm=norm), q, k, torch.from_numpy(v).cuda(), torch.from_numpy(w).cuda())[2]
    assert (np.abs(got[0, 0] - ref[0, 0]) <= 2e-6 * ref[0, 0]).all()
    # (the opposite pair cancels in exact products; an fp32 chain rounds each of its d_h sums by up to 2^-24 of the pair)
    pair = np.abs(v[0, 1, :, 7]) * (np.abs(w[dh + 8]).sum() if norm == 1 else np.linalg.norm(w[dh + 8]))
    assert (np.abs(got[0, 1] - ref[0, 1]) <= 2e-6 * ref[0, 1] + dh * 2.0 ** -24 * pair * (np.arange(n) % 3 > 0)).all()


@pytest.mark.parametrize("norm", [1, 2])
@pytest.mark.parametrize("wo_out_in", [False, True])
@pytest.mark.parametrize("dh,H,Hkv,n,dm", [(64, 4, 2, 130, 96), (128, 4, 1, 515, 32), (128, 32, 8, 1217, 64)])
def test_fp32_magnitudes_with_infinities(P, dh, H, Hkv, n, dm, wo_out_in, norm):
    """An infinite entry of V or W_O gives the infinite magnitude that the fp32 products give (the entry ranks first), and a
    NaN only where a product is one; every other row is as without it."""
    import torch
    cfg = CONFIGS["tiny"].with_(head_dim=dh, n_q_heads=H, n_kv_heads=Hkv, n_ctx=n, d_model=dm)
    t = make_layer(cfg)
    v, w = t["v"], t["w_o"]
    v[0, 0, 0, 1], v[0, 0, 17, dh - 1], v[0, -1, n - 1, 3] = np.inf, -np.inf, np.inf
    v[0, 0, 40, :2] = np.inf, -np.inf          # both signs in one row: NaN where their products differ in sign
    v[0, 0, 41, 5], v[0, 0, 63, 0] = np.nan, 0.0
    w[0] = np.abs(w[0]) + 1e-3                 # (one sign: the first entry's row has no cancelling infinities)
    w[(H - 1) * dh + 2, dm - 1] = -np.inf      # the last head's rows are all infinite
    with np.errstate(invalid="ignore"):
        ref = magnitudes64(v, w, H, norm)
    dev = [torch.from_numpy(a).cuda() for a in (t["q_win"], t["k"], v, np.ascontiguousarray(w.T) if wo_out_in else w)]
    for extra in (P.CKV_NO_MFMA, 0):
        got = score(P, cfg_desc(P, cfg, flags=(P.CKV_WO_OUT_IN if wo_out_in else 0) | extra, norm=norm), *dev)[2]
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref)), extra
        fin = np.isfinite(ref)
        assert np.abs(got[fin] - ref[fin]).max() <= 2e-6 * np.abs(ref[fin]).max()
    assert np.isinf(ref[0, H - 1]).sum() > n // 2 and np.isinf(ref[0, 0, 0]) and np.isinf(ref[0, 0, 17])


def test_fp32_score_accepts_a_workspace_without_room_for_the_split(P):
    """A workspace that ends before the split's scratch is accepted and gives the vector kernel's magnitudes,
    bit by bit."""
    import torch
    cfg = CONFIGS["tiny"].with_(n_ctx=300)
    t = make_layer(cfg)
    dev = [torch.from_numpy(t[name]).cuda() for name in ("q_win", "k", "v", "w_o")]
    desc = cfg_desc(P, cfg)
    split_bytes = cfg.n_q_heads * cfg.head_dim * cfg.d_model * 6
    small = score(P, desc, *dev, ws_bytes=P.workspace_bytes(desc, 0) - split_bytes + 256)
    vector = score(P, cfg_desc(P, cfg, flags=P.CKV_NO_MFMA), *dev)
    assert np.array_equal(small[2], vector[2])


# ---- layout change of W_O and the Gram constant -----------------------------------------------------------------------
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,dh,dm", [(1, 64, 32), (3, 64, 96), (2, 128, 160), (5, 128, 544), (32, 128, 4096)])
def test_layout_change_is_exact(P, H, dh, dm, dtype):
    """Rows and columns around the blocks a lane and a wave turn."""
    import torch
    cfg = CONFIGS["tiny"].with_(n_q_heads=H, n_kv_heads=H, head_dim=dh, d_model=dm, dtype=dtype)
    w = torch.randn(H * dh, dm, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    out = torch.full((dm, H * dh), float("nan"), dtype=w.dtype, device="cuda")
    P.criticalkv_prepare_wo(cfg_desc(P, cfg), w, out)
    assert torch.equal(out, w.t())


@pytest.mark.parametrize("wo_out_in", [False, True])
@pytest.mark.parametrize("H,dm", [(1, 512), (3, 1024), (8, 4608)])
def test_gram_constant_against_float64(P, H, dm, wo_out_in):
    """hi + lo of the folded Gram matrices: fp32 sums of exact products over d_model (relative to the diagonal, whose terms
    do not cancel), split with a relative error of 2^-17."""
    import torch
    cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=H, d_model=dm, n_ctx=64)
    w = (0.02 * torch.randn(H * 128, dm, device="cuda")).to(torch.bfloat16)
    desc = cfg_desc(P, cfg, flags=P.CKV_WO_OUT_IN if wo_out_in else 0)
    gram = torch.empty(P.gram_bytes(desc), dtype=torch.uint8, device="cuda")
    ws = torch.empty(P.workspace_bytes(desc, 1), dtype=torch.uint8, device="cuda")
    P.criticalkv_prepare_gram(desc, w.t().contiguous() if wo_out_in else w, gram, workspace=ws)
    got = gram.view(torch.bfloat16).view(H, 2, 128, 128).double().sum(1).cpu().numpy()
    wh = w.double().cpu().numpy().reshape(H, 128, dm)
    ref = wh @ wh.transpose(0, 2, 1)
    block = np.arange(128) // 32
    fold = np.where(block[:, None] > block[None, :], 2.0, np.where(block[:, None] == block[None, :], 1.0, 0.0))
    diag = np.sqrt(np.einsum("hii->hi", ref))
    scale = diag[:, :, None] * diag[:, None, :]
    assert (np.abs(got - ref * fold) <= 2.0 ** -16 * np.abs(ref * fold) + 2e-6 * scale).all()


# ---- row blocks per wave of the projection ----------------------------------------------------------------------------
def row_blocks(dtype, dh, heads, n):
    """Row blocks per wave as the launcher chooses them: the cheapest rounds of workgroups."""
    choices, c2, c1 = {("bf16", 128): ((7, 6, 5, 4, 3, 2), 1.07, 0.90), ("bf16", 64): ((10, 8, 6, 4, 3, 2), 1.84, 1.83),
                       ("f32", 128): ((4, 3, 2, 1), 0.40, 0.38), ("f32", 64): ((6, 5, 4, 3, 2, 1), 0.55, 0.55)}[dtype, dh]

    def cost(rb):
        wgs = (heads * -(-n // (64 * rb)) + 7) // 8
        rest = wgs % 64
        return wgs // 64 * (rb + c2) + (rb + c2 if rest > 32 else 0.48 * rb + c1 if rest else 0.0)

    return min(choices, key=cost), set(choices)


@pytest.mark.parametrize("dtype,dh,H,Hkv,dm,ns", [
    ("bf16", 128, 32, 8, 128, (511, 1025, 1537, 2049, 3073, 4097, 6145, 8193)),
    ("bf16", 64, 32, 8, 256, (511, 1025, 1600, 2048, 2816, 3073, 4097, 8193, 10241)),
    ("f32", 128, 16, 4, 32, (1000, 1025, 2049, 6145)),
    ("f32", 64, 16, 4, 32, (900, 1025, 2049, 3073, 4099, 5128, 8193, 9300)),
])
def test_magnitudes_with_every_row_block_count(P, dtype, dh, H, Hkv, dm, ns):
    """fp32 sums of exact products (bf16: d_h of them, then d_model magnitudes): 2e-6 of the result.  The lengths make the
    launcher take every number of row blocks it has."""
    import torch
    picked, choices = {row_blocks(dtype, dh, H, n)[0] for n in ns}, row_blocks(dtype, dh, H, ns[0])[1]
    assert picked == choices
    for n in ns:
        cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, head_dim=dh, d_model=dm, n_ctx=n, dtype=dtype, window=8)
        g = torch.Generator(device="cuda").manual_seed(n)
        dt = torch.bfloat16 if dtype == "bf16" else torch.float32
        q, k, v = (torch.randn(s, generator=g, device="cuda").to(dt) for s in ((1, H, 8, dh), (1, Hkv, n, dh), (1, Hkv, n, dh)))
        w = torch.randn((H * dh, dm), generator=g, device="cuda").to(dt)
        got = score(P, cfg_desc(P, cfg), q, k, v, w)[2]
        for h in (0, H - 1):
            ref = (v[0, h * Hkv // H].double() @ w[h * dh:(h + 1) * dh].double()).abs().sum(-1).cpu().numpy()
            assert np.abs(got[0, h] / ref - 1).max() <= 2e-6, (n, h)


# ---- selection and allocation: rows one workgroup takes, and the sliced kernels behind them ------------------------------
def tied_scores(n, heads, distinct):
    r = np.random.Generator(np.random.PCG64(n + distinct))
    attn = r.integers(0, distinct, (1, heads, n)).astype(np.float32) / 8
    crit = r.integers(0, distinct + 3, (1, heads, n)).astype(np.float32) - 2
    return attn, crit


@pytest.mark.parametrize("n", [2, 6, 8, 4095, 4096, 4097, 4100, 8191, 8192, 8193, 8196, 16383, 16384, 16385, 16388,
                               24572, 24575, 24576, 24577, 24580])
def test_select_at_the_row_lengths_where_the_kernel_changes(P, n):
    from test_gpu_parity import assert_select_exact, run_select
    r = np.random.Generator(np.random.PCG64(n))
    attn, crit = r.standard_normal((1, 3, n)).astype(np.float32), r.lognormal(0, 2, (1, 3, n)).astype(np.float32)
    for alpha in (0.0, 0.5, 1.0):
        assert_select_exact(P, attn, crit, r.integers(0, n + 1, (1, 3)), alpha, max_budget=n)
    for distinct in (1, 3):  # thresholds inside tie groups that cross every quad and wave
        attn, crit = tied_scores(n, 2, distinct)
        for B in sorted({1, n // 3, n - 1, n}):
            if B > 0:
                assert_select_exact(P, attn, crit, B, 0.5)


@pytest.mark.parametrize("n", [130, 4097, 24576, 24579])
def test_select_with_a_kept_window_at_the_row_lengths_where_the_kernel_changes(P, n):
    from oracle import cpu_oracle as O
    from test_gpu_parity import run_select
    attn, crit = tied_scores(n, 2, 40)
    for W, B in ((1, 1), (33, 20), (33, n // 2), (100, n)):
        idx, count, budget = run_select(P, attn, crit, B, 0.5, flags=P.CKV_PROTECT_WINDOW, window=W)
        ref_idx, ref_count, _ = O.select(attn.astype(np.float64), crit.astype(np.float64), budget, np.float32(0.5),
                                         max_budget=idx.shape[-1], protect_last=W)
        assert np.array_equal(idx, ref_idx) and np.array_equal(count, ref_count)


@pytest.mark.parametrize("Hkv,n", [(1, 24576), (1, 24577), (3, 1365), (3, 1366), (24, 1024), (25, 1024), (2000, 3), (30000, 1),
                                   (3000, 11), (7, 5000)])
def test_allocate_at_the_row_lengths_where_the_kernel_changes(P, Hkv, n):
    """Rows of Hkv * n keys around one workgroup's most; slices inside one head, over a few and over thousands of heads."""
    from oracle import cpu_oracle as O
    from test_gpu_parity import run_allocate
    r = np.random.Generator(np.random.PCG64(Hkv + n))
    for attn in (r.random((2, Hkv, n)).astype(np.float32), tied_scores(n, Hkv, 3)[0]):
        for total in sorted({1, Hkv, (Hkv * n) // 3, Hkv * n}):
            for floor_frac in (0.0, 0.3):
                got = run_allocate(P, attn, total, floor_frac)
                assert np.array_equal(got, O.allocate(attn.astype(np.float64), total, np.float32(floor_frac))), (total, floor_frac)


@pytest.mark.parametrize("b,Hkv,n", [(5, 3000, 11), (3, 700, 36), (4, 900, 31), (2, 820, 30), (2, 30000, 1), (33, 8, 3100)])
def test_allocate_counts_of_every_wave_arrive(P, b, Hkv, n):
    """Slices over 64 heads and more (every wave of a workgroup adds counts of its own) and launches of many rows: whole
    numbers, each call on a workspace that an earlier one has filled."""
    import torch
    from oracle import cpu_oracle as O
    cfg = CONFIGS["tiny"].with_(n_q_heads=Hkv, n_kv_heads=Hkv, n_ctx=n, window=1, batch=b)
    desc = cfg_desc(P, cfg)
    r = np.random.Generator(np.random.PCG64(Hkv * n))
    attn = np.concatenate([r.random((b - 1, Hkv, n)).astype(np.float32), tied_scores(n, Hkv, 3)[0]])
    dev, budget = torch.from_numpy(attn).cuda(), torch.empty((b, Hkv), dtype=torch.int32, device="cuda")
    ws = torch.full((P.workspace_bytes(desc, n),), 255, dtype=torch.uint8, device="cuda")
    for total in (Hkv * n // 3, Hkv * n // 2, Hkv * n // 3):
        P.criticalkv_allocate(desc, dev, total, 0.2, budget, workspace=ws)
        assert np.array_equal(budget.cpu().numpy(), O.allocate(attn.astype(np.float64), total, np.float32(0.2)))


# ---- fp32 window attention on the matrix cores -----------------------------------------------------------------------------
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dh,H,Hkv,n,W", [(64, 4, 4, 33, 1), (64, 3, 1, 32, 32), (128, 8, 2, 31, 31), (128, 8, 8, 2049, 33),
                                          (64, 10, 2, 4127, 100), (128, 4, 1, 300, 300), (128, 2, 1, 70, 64),
                                          # over 64 ranges, merged by a launch of their own: 66, 94, 115 and 313 of them
                                          (64, 1, 1, 2081, 8), (64, 4, 2, 9000, 33), (64, 8, 8, 33000, 5), (128, 1, 1, 20000, 40),
                                          # windows that the vector kernel takes, and one entry below
                                          (64, 5, 1, 6600, 1), (128, 2, 2, 33000, 2), (64, 4, 1, 4096, 1)])
def test_fp32_window_attention_against_float64(P, dh, H, Hkv, n, W, causal):
    """One key block and several per range, several row blocks, strided keys.  fp32 logits of d_h products: the error of a
    weight is that of its logit's distance from the row maximum, 2e-6 here; the vector kernel is the yardstick."""
    import torch
    from oracle import cpu_oracle as O
    cfg = CONFIGS["tiny"].with_(head_dim=dh, n_q_heads=H, n_kv_heads=Hkv, n_ctx=n, d_model=32, window=W, batch=2, pool_kernel=1)
    t = make_layer(cfg)
    G = H // Hkv
    s = np.einsum("bhwd,bhnd->bhwn", t["q_win"].astype(np.float64), np.repeat(t["k"], G, axis=1).astype(np.float64)) / np.sqrt(dh)
    if causal:
        s = np.where(np.arange(n)[None, :] > n - W + np.arange(W)[:, None], -np.inf, s)
    p = np.exp(s - s.max(-1, keepdims=True))
    ref = (p / p.sum(-1, keepdims=True)).mean(2).reshape(2, Hkv, G, n).mean(2)
    dev = {name: torch.from_numpy(a).cuda() for name, a in t.items()}
    k = torch.zeros((2, n, Hkv, dh + 8), device="cuda")[..., :dh].permute(0, 2, 1, 3)
    k.copy_(dev["k"])
    err = {}
    for name, extra in (("matrix", 0), ("vector", P.CKV_NO_MFMA)):
        desc = cfg_desc(P, cfg, flags=extra | (P.CKV_CAUSAL_TAIL if causal else 0), k_stride=k.stride()[:3])
        got = score(P, desc, dev["q_win"], k, dev["v"], dev["w_o"])[0]
        err[name] = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        assert np.abs(got - ref).max() <= 4e-6 * ref.max()
    assert err["matrix"] <= max(1.2 * err["vector"], 3e-7), err


@pytest.mark.parametrize("dh,H,Hkv,n,W", [(64, 4, 4, 512, 8), (64, 4, 4, 4096, 8), (128, 16, 4, 1500, 32)])
def test_fp32_window_attention_loses_no_precision(P, dh, H, Hkv, n, W):
    """Scores with heavy entries, over several layers: no further from 64 bits than the vector kernel's.  A logit's error is
    the rounding of its chain over d_h; two chains of half each take a third or more off (0.57 - 0.61 of the vector kernel's
    measured)."""
    import torch
    err = {0: 0.0, P.CKV_NO_MFMA: 0.0}
    for seed in range(8):
        cfg = CONFIGS["tiny"].with_(head_dim=dh, n_q_heads=H, n_kv_heads=Hkv, n_ctx=n, d_model=32, window=W, pool_kernel=1)
        t = make_layer(cfg, seed_offset=seed)
        dev = [torch.from_numpy(t[name]).cuda() for name in ("q_win", "k", "v", "w_o")]
        s = dev[0].double().view(1, Hkv, H // Hkv, W, dh) @ dev[1].double()[:, :, None].transpose(-1, -2).contiguous() / dh ** 0.5
        ref = torch.softmax(s, -1).mean((2, 3)).cpu().numpy()
        for flags in err:
            got = score(P, cfg_desc(P, cfg, flags=flags), *dev)[0]
            err[flags] += np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert err[0] <= 0.8 * err[P.CKV_NO_MFMA], err


# ---- wave-private attention sweeps: heads and keys per wave ----------------------------------------------------------------------
@pytest.mark.parametrize("dh,H,Hkv,W,b,ns", [
    (64, 32, 8, 32, 1, (127, 129, 1000, 3000, 8193)), (64, 32, 8, 32, 4, (3001, 32768)), (128, 40, 8, 64, 1, (65, 2000, 8192, 20000)),
    (64, 3, 3, 100, 3, (129, 2600)), (128, 14, 2, 33, 2, (511, 4100)),
])
def test_wave_sweeps_over_the_choices_of_heads_and_keys_per_wave(P, dh, H, Hkv, W, b, ns):
    """fp32 logits of exact products and fp32 sums over the window: 4e-6 of the largest score."""
    import torch
    for n in ns:
        g = torch.Generator(device="cuda").manual_seed(n)
        q, k = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((b, H, W, dh), (b, Hkv, n, dh)))
        cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, head_dim=dh, d_model=32, window=W, n_ctx=n, batch=b, pool_kernel=1)
        desc = cfg_desc(P, cfg, flags=P.CKV_ATTN_ONLY)
        attn = torch.empty((b, Hkv, n), dtype=torch.float32, device="cuda")
        crit = torch.empty_like(attn)
        ws = torch.empty(P.workspace_bytes(desc, 1), dtype=torch.uint8, device="cuda")
        P.criticalkv_score(desc, q, k, None, None, attn, crit, None, workspace=ws)
        for bi, gi in ((0, 0), (b - 1, Hkv - 1)):
            ref = 0
            for h in range(gi * H // Hkv, (gi + 1) * H // Hkv):
                ref = ref + torch.softmax(q[bi, h].double() @ k[bi, gi].double().t() / dh ** 0.5, -1).mean(0) * Hkv / H
            assert (attn[bi, gi].double() - ref).abs().max() <= 4e-6 * ref.max(), (n, bi, gi)


def wave_heads(dh, G, kv_heads, W, n):
    """Query heads per wave as the launcher chooses them (the cheapest launch; kv_heads over the whole batch)."""
    blocks = (W + 31) // 32

    def cost(h):
        groups, least = -(-G // h), []
        for kpw in (1024, 768, 512, 384, 256, 192, 128):
            chunks = (-(-n // kpw) + 3) // 4
            rounds = (groups * ((kv_heads * chunks + 7) // 8) + 31) // 32
            least.append({1: 1.35, 2: 2.2, 3: 3.1}.get(rounds, rounds) * (kpw + (35 if dh == 128 else 20) * (1 + h * blocks)))
        return min(least) * (h * blocks + (2 if dh == 128 else 0.7)) * (1.04 if h > 1 and h * blocks == 4 else 1)

    return min(range(1, min(G, 4 // blocks) + 1), key=cost)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dh,G,W,b,n,heads", [
    # every number of heads a wave takes, with a last group of fewer heads where one is possible, and heads of two row blocks
    (64, 4, 32, 8, 4101, 2), (64, 7, 32, 8, 2049, 2), (64, 6, 32, 8, 4101, 3), (64, 5, 20, 16, 4101, 3), (64, 7, 32, 8, 16390, 4),
    (64, 8, 33, 16, 4101, 2), (128, 7, 32, 4, 4101, 2), (128, 6, 32, 8, 2049, 3), (128, 5, 7, 8, 4101, 3), (128, 8, 32, 16, 4101, 4),
    (128, 7, 32, 16, 4101, 4), (128, 8, 64, 8, 2049, 2), (128, 7, 33, 8, 2049, 2)])
def test_wave_sweeps_with_several_heads_per_wave(P, dh, G, W, b, n, heads, causal):
    """fp32 logits of exact products and fp32 sums over the window: 4e-6 of the largest score."""
    import torch
    Hkv, H = 8, 8 * G
    assert wave_heads(dh, G, b * Hkv, W, n) == heads
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k = (torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) for s in ((b, H, W, dh), (b, Hkv, n, dh)))
    cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, head_dim=dh, d_model=32, window=W, n_ctx=n, batch=b, pool_kernel=1)
    desc = cfg_desc(P, cfg, flags=P.CKV_ATTN_ONLY | (P.CKV_CAUSAL_TAIL if causal else 0))
    attn = torch.empty((b, Hkv, n), dtype=torch.float32, device="cuda")
    ws = torch.empty(P.workspace_bytes(desc, 1), dtype=torch.uint8, device="cuda")
    P.criticalkv_score(desc, q, k, None, None, attn, torch.empty_like(attn), None, workspace=ws)
    hidden = torch.arange(n, device="cuda")[None, :] > n - W + torch.arange(W, device="cuda")[:, None]
    for bi, gi in ((0, 0), (b // 2, 3), (b - 1, Hkv - 1)):
        ref = 0
        for h in range(gi * G, (gi + 1) * G):
            s = q[bi, h].double() @ k[bi, gi].double().t().contiguous() / dh ** 0.5
            ref = ref + torch.softmax(s.masked_fill(hidden, -torch.inf) if causal else s, -1).mean(0) / G
        assert (attn[bi, gi].double() - ref).abs().max() <= 4e-6 * ref.max(), (bi, gi)


# ---- work dealt to the XCDs: head counts that eight does not divide ---------------------------------------------------------
@pytest.mark.parametrize("dtype,dh,H,Hkv,dm,b,n", [
    ("bf16", 128, 28, 4, 128, 1, 1500), ("bf16", 128, 1, 1, 256, 1, 700), ("bf16", 128, 12, 2, 5120, 1, 450),
    ("bf16", 64, 7, 7, 256, 3, 900), ("f32", 128, 20, 4, 64, 1, 600), ("f32", 64, 5, 1, 32, 1, 5000),
])
def test_magnitudes_over_head_counts(P, dtype, dh, H, Hkv, dm, b, n):
    """L1 magnitudes of every head and row; fp32 sums: 2e-6 of the result."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(H * n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, head_dim=dh, d_model=dm, n_ctx=n, dtype=dtype, window=8, batch=b)
    q, k, v = (torch.randn(s, generator=g, device="cuda").to(dt) for s in ((b, H, 8, dh), (b, Hkv, n, dh), (b, Hkv, n, dh)))
    w = torch.randn((H * dh, dm), generator=g, device="cuda").to(dt)
    got = torch.from_numpy(score(P, cfg_desc(P, cfg), q, k, v, w)[2]).cuda()
    for bi in range(b):
        for h in range(H):
            ref = (v[bi, h * Hkv // H].double() @ w[h * dh:(h + 1) * dh].double()).abs().sum(-1)
            assert (got[bi, h].double() / ref - 1).abs().max() <= 2e-6, (bi, h)


@pytest.mark.parametrize("H,Hkv,b,n", [(28, 4, 1, 3000), (2, 1, 1, 70), (12, 2, 3, 1111), (5, 5, 2, 9000)])
def test_l2_magnitudes_over_head_counts(P, H, Hkv, b, n):
    """The Gram form's split constant has a relative error of 2^-17 per entry: 2e-5 of a row's norm."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(H + n)
    cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, d_model=512, n_ctx=n, window=8, batch=b)
    q, k, v = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((b, H, 8, 128), (b, Hkv, n, 128), (b, Hkv, n, 128)))
    w = (0.02 * torch.randn((H * 128, 512), generator=g, device="cuda")).to(torch.bfloat16)
    got = torch.from_numpy(score(P, cfg_desc(P, cfg, norm=2), q, k, v, w)[2]).cuda()
    for bi in range(b):
        for h in range(H):
            ref = (v[bi, h * Hkv // H].double() @ w[h * 128:(h + 1) * 128].double()).square().sum(-1).sqrt()
            assert (got[bi, h].double() / ref - 1).abs().max() <= 2e-5, (bi, h)


@pytest.mark.parametrize("heads,n", [(1, 1), (1, 2), (1, 3), (3, 1), (2, 2), (5, 1), (1, 5), (3, 3)])
def test_select_and_allocate_on_a_few_keys_in_all(P, heads, n):
    """Arrays with no whole 16-byte piece, and with one that crosses rows."""
    from oracle import cpu_oracle as O
    from test_gpu_parity import assert_select_exact, run_allocate
    r = np.random.Generator(np.random.PCG64(10 * heads + n))
    attn, crit = r.random((1, heads, n)).astype(np.float32), r.random((1, heads, n)).astype(np.float32)
    for B in range(1, n + 1):
        assert_select_exact(P, attn, crit, B, 0.5)
    for total in range(0, heads * n + 1):
        assert np.array_equal(run_allocate(P, attn, total, 0.25), O.allocate(attn.astype(np.float64), total, np.float32(0.25)))


# ---- the gather with new rows behind the kept ones -------------------------------------------------------------------
@pytest.mark.parametrize("dtype,dh", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("n,mb,n_new", [(1, 1, 1), (40, 17, 3), (300, 300, 129)])
def test_compact_append_is_a_gather_and_a_concatenation(P, dtype, dh, n, mb, n_new):
    """Counts below max_budget leave their rows alone; new rows with strides of their own."""
    import torch
    b, Hkv = 2, 3
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = CONFIGS["tiny"].with_(n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=dh, n_ctx=n, window=1, batch=b, dtype=dtype)
    k, v = (torch.randn((b, Hkv, n, dh), device="cuda").to(dt) for _ in range(2))
    k_new = torch.randn((b, n_new, Hkv, dh + 8), device="cuda").to(dt)[..., :dh].permute(0, 2, 1, 3)
    v_new = torch.randn((b, Hkv, n_new + 2, dh), device="cuda").to(dt)[:, :, 1:-1]
    count = torch.tensor([[0, 1, mb]] * b, dtype=torch.int32, device="cuda").clamp(max=mb)
    idx = torch.stack([torch.randperm(n)[:mb].sort().values for _ in range(b * Hkv)]).view(b, Hkv, mb).int().cuda()
    k_out = torch.full((b, Hkv, mb + n_new, dh), 7.0, device="cuda", dtype=dt)
    v_out = torch.full_like(k_out, 7.0)
    P.criticalkv_compact_append(cfg_desc(P, cfg), k, v, idx, count, mb, k_new, v_new, k_out, v_out)
    for src, new, out in ((k, k_new, k_out), (v, v_new, v_out)):
        rows = torch.gather(src, 2, idx.long()[..., None].expand(-1, -1, -1, dh))
        rows = torch.where((torch.arange(mb, device="cuda") < count[..., None])[..., None], rows, torch.full_like(rows, 7.0))
        assert torch.equal(out, torch.cat([rows, new], dim=2))


def test_chunked_prefill_with_chunks_the_gather_cannot_append(P):
    """Chunks that fit the budget, an empty one, and rows that begin off a 16-byte boundary: the same as contiguous ones."""
    import torch
    from paper_2502_03805_amd.chunked import chunked_prefill_evict
    cfg = CONFIGS["llama32k"].with_(n_q_heads=4, n_kv_heads=2, d_model=128, window=16)
    mk = lambda n: cfg_desc(P, cfg.with_(n_ctx=n), flags=P.CKV_CAUSAL_TAIL | P.CKV_PROTECT_WINDOW)
    lengths = (60, 30, 0, 200, 77, 0, 50)
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    w, qs = rnd(512, 128), [rnd(1, 4, 16, 128) for _ in lengths]
    ks, vs = ([rnd(1, 2, n, 128) for n in lengths] for _ in range(2))
    odd = lambda t: torch.cat([t, t[..., :1]], dim=-1)[..., :128] # row stride 129
    first = lambda i, t: t if i == 0 else odd(t)
    a = chunked_prefill_evict(mk, qs, ks, vs, w, 100, 0.5)
    c = chunked_prefill_evict(mk, iter(qs), [first(i, t) for i, t in enumerate(ks)], iter(vs), w, 100, 0.5)
    assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1]) and a[0].shape == (1, 2, 100, 128) and a[0].is_contiguous()
    assert [x is None for x in a[2]] == [True, True, True, False, False, True, False]
    assert all((x is None) == (y is None) and (x is None or torch.equal(x, y)) for x, y in zip(a[2], c[2]))


# ---- short contexts: rows merged by the second sweep, and that sweep beside the projection ---------------------------
@pytest.mark.parametrize("G,Hkv,W,b,norm,ns", [
    (4, 8, 32, 1, 1, (100, 511, 600, 1025, 1601, 2100, 3072, 3500, 3700)), # every row-block count; two workgroups per CU
    (1, 2, 7, 2, 1, (40, 257, 4100)), (3, 2, 20, 1, 1, (1, 300, 2049)), (2, 1, 33, 1, 1, (300,)), (4, 1, 32, 1, 2, (500,)),
    (4, 2, 32, 1, None, (16383, 16384, 16385)), (2, 2, 64, 1, None, (5000,)), # 64 and 65 chunks
    # ranges of 64, 128 and 256 keys, either side of each line; ranges that rows of the window do not see at all
    (4, 8, 32, 1, None, (64, 65, 129, 2048, 2049, 4096, 4097)), (1, 1, 96, 1, None, (97, 160, 192, 1000)), (2, 4, 64, 2, 1, (66, 2049)),
    (4, 1, 32, 1, 1, (4096, 4097, 16384, 16385, 32768, 32769)), (4, 1, 32, 1, None, (4096, 4097, 16384, 16385, 32768, 32769)),
])
def test_short_contexts_against_float64(P, G, Hkv, W, b, norm, ns):
    """fp32 softmax sums of bf16 products (d_h exact terms) and exponentials of an ulp each: 4e-6 of the result by the 2-norm;
    the stage by stage call is the same computation in other launches."""
    import ctypes
    import torch
    H = G * Hkv
    for n in ns:
        W_n = min(W, n)
        cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, d_model=512, n_ctx=n, window=W_n, batch=b, pool_kernel=1)
        g = torch.Generator(device="cuda").manual_seed(n)
        q, k, v = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in
                   ((b, H, W_n, 128), (b, Hkv, n, 128), (b, Hkv, n, 128)))
        w = (0.02 * torch.randn((H * 128, 512), generator=g, device="cuda")).to(torch.bfloat16)
        for causal in (0, P.CKV_CAUSAL_TAIL):
            desc = cfg_desc(P, cfg, norm=norm or 1, flags=causal | (0 if norm else P.CKV_ATTN_ONLY))
            ws = torch.empty(P.workspace_bytes(desc, 1), dtype=torch.uint8, device="cuda")
            attn, crit = (torch.full((b, Hkv, n), float("nan"), device="cuda") for _ in range(2))
            vnorm = torch.full((b, H, n), float("nan"), device="cuda") if norm else None
            P.criticalkv_score(desc, q, k, v, w, attn, crit, vnorm, workspace=ws)
            s = torch.einsum("bgrwd,bgnd->bgrwn", q.double().view(b, Hkv, G, W_n, 128), k.double()) / 128 ** 0.5
            if causal:
                s.masked_fill_(torch.arange(n, device="cuda") > n - W_n + torch.arange(W_n, device="cuda")[:, None], -np.inf)
            ref = s.softmax(-1).mean((2, 3))
            assert (attn.double() - ref).norm() <= 4e-6 * ref.norm(), (n, causal)
            if norm:
                p = torch.einsum("bgnd,grdc->bgrnc", v.double(), w.double().view(Hkv, G, 128, 512)).reshape(b, H, n, 512)
                ref = p.abs().sum(-1) if norm == 1 else p.square().sum(-1).sqrt()
                assert ((vnorm.double() / ref - 1).abs() <= (2e-6 if norm == 1 else 2e-5)).all(), (n, causal)
            again = [torch.empty_like(t) if t is not None else None for t in (attn, crit, vnorm)]
            P.criticalkv_score_profiled(desc, q, k, v, w, *again, workspace=ws, stage_events=(ctypes.c_void_p * 10)())
            assert all(x is None or torch.equal(x, y) for x, y in zip(again, (attn, crit, vnorm))), (n, causal)


@pytest.mark.parametrize("dh,H,Hkv,W,b,wo_out_in,ns", [
    (64, 4, 4, 8, 1, True, (8, 33, 1024, 2049, 2080)),   # 65 ranges and more: the pairs are merged by a launch between
    (64, 16, 4, 40, 1, False, (512, 1025, 2049, 3073, 4099, 5121, 6145)),
    (128, 16, 4, 32, 1, True, (512, 1100, 2100, 3100, 4097)), (128, 2, 1, 33, 3, False, (100,)),
])
def test_short_fp32_contexts_against_float64(P, dh, H, Hkv, W, b, wo_out_in, ns):
    """The sweeps beside the split and the project kernel (every row-block count, and the first lengths past them): fp32 chains
    of d_h products and exponentials of an ulp each, 2e-6 by the 2-norm, as for the launches by themselves."""
    import torch
    G = H // Hkv
    for n in ns:
        cfg = CONFIGS["tiny"].with_(n_q_heads=H, n_kv_heads=Hkv, head_dim=dh, d_model=96, n_ctx=n, window=W, batch=b, pool_kernel=1)
        g = torch.Generator(device="cuda").manual_seed(n)
        q, k, v = (torch.randn(s, generator=g, device="cuda") for s in ((b, H, W, dh), (b, Hkv, n, dh), (b, Hkv, n, dh)))
        w = torch.randn((H * dh, 96), generator=g, device="cuda")
        for causal in (0, P.CKV_CAUSAL_TAIL):
            desc = cfg_desc(P, cfg, flags=causal | (P.CKV_WO_OUT_IN if wo_out_in else 0))
            attn, _, vnorm = score(P, desc, q, k, v, w.t().contiguous() if wo_out_in else w)
            s = torch.einsum("bgrwd,bgnd->bgrwn", q.double().view(b, Hkv, G, W, dh), k.double()) / dh ** 0.5
            if causal:
                s.masked_fill_(torch.arange(n, device="cuda") > n - W + torch.arange(W, device="cuda")[:, None], -np.inf)
            ref = s.softmax(-1).mean((2, 3)).cpu().numpy()
            assert np.linalg.norm(attn - ref) <= 2e-6 * np.linalg.norm(ref), (n, causal)
            p = torch.einsum("bgnd,grdc->bgrnc", v.double(), w.double().view(Hkv, G, dh, 96)).reshape(b, H, n, 96).abs().sum(-1)
            assert np.abs(vnorm / p.cpu().numpy() - 1).max() <= 2e-6, (n, causal)


@pytest.mark.parametrize("n", [7, 4093, 9001, 20011])
def test_select_of_rows_with_signed_zeros_and_infinities(P, n):
    """Keys at the ends of the order: -0 and +0 are one key, -inf competes (it is not a position outside the row), +inf is first."""
    from test_gpu_parity import assert_select_exact
    r = np.random.Generator(np.random.PCG64(n))
    pool = np.array([-np.inf, -1.0, -1e-45, -0.0, 0.0, 1e-45, 2.0, np.inf], np.float32)
    attn, crit = pool[r.integers(0, 8, (1, 3, n))], pool[r.integers(0, 8, (1, 3, n))]
    attn[0, 2], crit[0, 2] = -np.inf, pool[r.integers(0, 3, n)]
    for B in sorted({1, n // 3, n // 2 + 1, n - 1, n}):
        for alpha in (0.0, 0.5, 1.0):
            assert_select_exact(P, attn, crit, B, alpha, max_budget=n)


def test_calls_go_to_the_current_stream(P):
    import torch
    from paper_2502_03805_amd import binding as B
    assert B._stream(None) == (torch.cuda.current_stream().cuda_stream or None)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert B._stream(None) == side.cuda_stream != 0
    assert B._stream(side) == side.cuda_stream and B._stream(None) == (torch.cuda.current_stream().cuda_stream or None)


@pytest.mark.parametrize("n", [1984, 1985, 2111, 4097])
def test_l2_magnitudes_of_long_ranges(P, n):
    """One range per head pair: 31 blocks of rows per workgroup (the kernel for short ranges) and 32 and more, which its eight
    waves take as they ask; ragged last blocks.  2e-5 as for the other lengths, and the same bits on every call."""
    import torch
    b, H, Hkv = 8, 64, 32
    g = torch.Generator(device="cuda").manual_seed(n)
    cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, d_model=512, n_ctx=n, window=8, batch=b)
    q, k, v = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((b, H, 8, 128), (b, Hkv, n, 128), (b, Hkv, n, 128)))
    w = (0.02 * torch.randn((H * 128, 512), generator=g, device="cuda")).to(torch.bfloat16)
    got = torch.from_numpy(score(P, cfg_desc(P, cfg, norm=2), q, k, v, w)[2]).cuda()
    for bi, h in ((0, 0), (0, 1), (3, 31), (7, 62), (7, 63)):
        ref = (v[bi, h * Hkv // H].double() @ w[h * 128:(h + 1) * 128].double()).square().sum(-1).sqrt()
        assert (got[bi, h].double() / ref - 1).abs().max() <= 2e-5, (bi, h)
    for _ in range(3):
        assert torch.equal(torch.from_numpy(score(P, cfg_desc(P, cfg, norm=2), q, k, v, w)[2]).cuda(), got)


@pytest.mark.parametrize("b,Hkv,n", [(1, 30, 1023), (2, 30, 1024), (1, 64, 1025), (1, 65, 1025), (3, 13, 2047), (2, 13, 2048), (1, 13, 2049),
                                     (2, 3, 20011)])
def test_allocate_where_slices_belong_to_heads(P, b, Hkv, n):
    """Around the lengths and head counts from which the histogram kernels keep the heads' counts; rows that start off a
    16-byte boundary, ties across heads and slices, a head that gets everything, pools of one slot and of all."""
    from oracle import cpu_oracle as O
    from test_gpu_parity import run_allocate
    r = np.random.Generator(np.random.PCG64(n + Hkv))
    tied = r.integers(0, 3, (b, Hkv, n)).astype(np.float32)
    one = r.random((b, Hkv, n)).astype(np.float32)
    one[:, Hkv // 2] += 2
    for attn in (tied, one, r.lognormal(0, 2, (b, Hkv, n)).astype(np.float32)):
        for total, floor_frac in ((1, 0.0), (n, 0.0), (Hkv * n // 3, 0.25), (Hkv * n - 1, 0.0), (Hkv * n, 0.5)):
            got = run_allocate(P, attn, total, floor_frac)
            assert np.array_equal(got, O.allocate(attn.astype(np.float64), total, np.float32(floor_frac))), (total, floor_frac)


@pytest.mark.parametrize("dh,H,Hkv,W,b,ns", [
    (64, 32, 8, 32, 1, (33, 1024, 3000, 4096, 4097, 4500)), (64, 6, 2, 40, 2, (100, 2000)), (128, 40, 8, 64, 1, (1024, 4096, 4200, 8192)),
    (128, 6, 1, 128, 1, (700,)), (64, 3, 3, 5, 1, (9000,)),
])
def test_short_contexts_of_the_wave_private_sweeps_against_float64(P, dh, H, Hkv, W, b, ns):
    """Around 32 ranges of keys, several heads per wave and windows of several row blocks among them: 4e-6 by the 2-norm, as for
    the shared-tile sweeps."""
    import torch
    G = H // Hkv
    for n in ns:
        W_n = min(W, n)
        cfg = CONFIGS["llama32k"].with_(n_q_heads=H, n_kv_heads=Hkv, head_dim=dh, d_model=512, n_ctx=n, window=W_n, batch=b, pool_kernel=1)
        g = torch.Generator(device="cuda").manual_seed(n)
        q, k = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((b, H, W_n, dh), (b, Hkv, n, dh)))
        for causal in (0, P.CKV_CAUSAL_TAIL):
            desc = cfg_desc(P, cfg, flags=causal | P.CKV_ATTN_ONLY)
            ws = torch.empty(P.workspace_bytes(desc, 1), dtype=torch.uint8, device="cuda")
            attn, crit = (torch.full((b, Hkv, n), float("nan"), device="cuda") for _ in range(2))
            P.criticalkv_score(desc, q, k, None, None, attn, crit, None, workspace=ws)
            s = torch.einsum("bgrwd,bgnd->bgrwn", q.double().view(b, Hkv, G, W_n, dh), k.double()) / dh ** 0.5
            if causal:
                s.masked_fill_(torch.arange(n, device="cuda") > n - W_n + torch.arange(W_n, device="cuda")[:, None], -np.inf)
            ref = s.softmax(-1).mean((2, 3))
            assert (attn.double() - ref).norm() <= 4e-6 * ref.norm(), (n, causal)
