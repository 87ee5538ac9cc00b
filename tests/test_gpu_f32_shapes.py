"""The fp32 kernels at the shapes where their tiling, vector loads and padding change: head widths on both sides of a multiple
of 32, widths and weight pointers that rule out 16-byte loads, row statistics with and without registers, launches large
enough for the big projection tile.  Against the fp64 oracle on hot inputs, at the bar of the fp32 path."""
import numpy as np
import pytest

import oracle
from paper_2509_22681_amd import workloads as W
from tests.test_gpu_parity import TOL_HOT, score_err

pytestmark = pytest.mark.gpu

CASES = {
    "one_chunk_16": dict(L=[70, 3, 0], M=[9, 33, 2], d=16, H=1),        # a single chunk of 32 k: W is waited for with no second chunk behind it
    "one_chunk_20": dict(L=[70, 3, 0], M=[9, 33, 2], d=20, H=2),
    "one_chunk_32": dict(L=[70, 3, 0], M=[9, 33, 2], d=32, H=2),
    "head_10_no_vector_loads": dict(L=[70, 3, 0], M=[9, 33, 2], d=30, H=3),
    "head_24": dict(L=[65, 31], M=[1, 40], d=48, H=2),
    "head_48": dict(L=[64, 129], M=[64, 7], d=96, H=2),
    "head_96": dict(L=[33, 200], M=[65, 3], d=192, H=2),
    "head_160": dict(L=[40, 70], M=[5, 66], d=160, H=1),
    "head_256": dict(L=[97], M=[35], d=256, H=1),
    "wide_512": dict(L=[130], M=[70], d=512, H=8),
    "wide_640": dict(L=[66], M=[12], d=640, H=10),
    "wide_520_head_65": dict(L=[40, 33], M=[3, 34], d=520, H=8),
    "big_projection_tile": dict(L=[130] * 32 + [64], M=[10] * 32 + [0], d=256, H=4),
    "wide_output_tile_256": dict(L=[1, 33] * 64, M=[2, 64] * 64, d=256, H=4),            # 256 row blocks: the first of the 64 x 128 tiles
    "narrow_output_tile_256": dict(L=[1, 33] * 63 + [5], M=[2, 64] * 63 + [0], d=256, H=4),
    "wide_output_tile_124": dict(L=[1, 33] * 128, M=[2, 64] * 128, d=124, H=2),         # 512, the last columns of a tile empty
}


@pytest.mark.parametrize("kind", ["silu", "softmax"])
@pytest.mark.parametrize("unaligned", [False, True])
@pytest.mark.parametrize("case", list(CASES))
def test_f32_shape(case, unaligned, kind):
    import torch
    from paper_2509_22681_amd import binding as B
    c = CASES[case]
    wl = W.make_custom(c["L"], c["M"], d=c["d"], H=c["H"], n_layers=2, n_buckets=16, max_rel_dist=128, dtype="f32", seed=5,
                       emb_std=1.0, rab_std=1.0, bias_amp=0.1, affine_random=True, attn_kind=kind, name=case)
    want = oracle.forward(wl.cfg.to_dict(), wl.weights, wl.history_emb, wl.history_offsets, wl.cand_emb, wl.cand_offsets)
    dw, hist, cand = B.to_device(wl)

    def shifted(t):     # the same values one float past a 16-byte boundary
        flat = torch.empty(t.numel() + 1, device=t.device, dtype=t.dtype)[1:]
        return flat.copy_(t.reshape(-1)).view(t.shape)

    if unaligned:
        dw = {k: shifted(v) if torch.is_tensor(v) else v for k, v in dw.items()}
        hist, cand = shifted(hist), shifted(cand)
    h = B.flame_gr_create(B.config_for(wl))
    try:
        out = torch.full((int(wl.cand_offsets[-1]),), float("nan"), device="cuda:0")
        B.flame_gr_forward(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, out)
        torch.cuda.synchronize()
        g = out.cpu().numpy()
    finally:
        B.flame_gr_destroy(h)
    assert np.isfinite(g).all()
    worst = score_err(g, want)
    print(f"{case} unaligned={unaligned} {kind}: {worst:.2e}")
    assert worst <= TOL_HOT["f32"], worst


def test_f32_more_items_than_one_grid_dimension_holds():
    """70 000 requests of one history row are more attention items than a launch may have along y; each scores as it does alone."""
    import torch
    from paper_2509_22681_amd import binding as B
    n = 70_000
    wl = W.make_custom([1] * n, [1] * n, d=32, H=1, n_layers=2, n_buckets=16, max_rel_dist=16, dtype="f32", seed=5, name="many_items")

    def scores(w):
        h = B.flame_gr_create(B.config_for(w))
        try:
            dw, hist, cand = B.to_device(w)
            out = torch.full((int(w.cand_offsets[-1]),), float("nan"), device="cuda:0")
            B.flame_gr_forward(h, dw, hist, w.history_offsets, cand, w.cand_offsets, out)
            torch.cuda.synchronize()
            return out.cpu().numpy()
        finally:
            B.flame_gr_destroy(h)

    whole = scores(wl)
    assert np.isfinite(whole).all()
    idx = [0, 32_767, 32_768, 65_535, 65_536, n - 1]
    assert np.array_equal(scores(wl.subset(idx)), whole[idx])


@pytest.mark.parametrize("d,H", [(64, 2), (96, 2), (100, 2), (90, 2), (256, 4)])
def test_f32_products_do_not_depend_on_the_tile(d, H):
    """The projection and output products split their operands into three bf16 parts, exactly, and add up in one order: large and small tiles, the packed weights
    and those that the kernels split themselves (the static workspace, where there is no room for the packed copy) give the same bits."""
    import ctypes
    import torch
    from paper_2509_22681_amd import binding as B
    need, size = ctypes.c_int64(), 64 << 20
    split = 5 * 2 * ((d + 31) // 32 * 32) ** 2 * 6
    L, M = [], []
    cfg = B.config_for(W.make_custom([1], [1], d=d, H=H, n_layers=2, n_buckets=16, max_rel_dist=1024, dtype="f32", seed=7, name="tiles"))
    while True:                                    # as many rows as leave no room for the packed weights
        rows = sum(-(-a // 64) + -(-b // 64) for a, b in zip(L, M)) * 64
        assert B._lib.flame_gr_static_scratch_bytes(ctypes.byref(cfg), ctypes.c_int64(rows + 128), ctypes.byref(need)) == 0
        if need.value > size:
            break
        L.append([64, 23][len(L) % 2])
        M.append([17, 64][len(M) % 2])
    assert B._lib.flame_gr_static_scratch_bytes(ctypes.byref(cfg), ctypes.c_int64(rows), ctypes.byref(need)) == 0
    assert need.value <= size < need.value + split
    wl = W.make_custom(L, M, d=d, H=H, n_layers=2, n_buckets=16, max_rel_dist=1024, dtype="f32", seed=7, emb_std=1.0, rab_std=1.0, bias_amp=0.1,
                       affine_random=True, name="tiles")
    dw, hist, cand = B.to_device(wl)

    def forward(first, last):
        ho, co = wl.history_offsets[first:last + 1], wl.cand_offsets[first:last + 1]
        out = torch.full((int(co[-1] - co[0]),), float("nan"), device="cuda:0")
        args = (dw, hist[ho[0]:ho[-1]].contiguous(), ho - ho[0], cand[co[0]:co[-1]].contiguous(), co - co[0], out)
        return args, out

    h = B.flame_gr_create(B.config_for(wl))
    try:
        args, whole = forward(0, len(L))
        B.flame_gr_forward(h, *args)
        parts = []
        for r in (0, 1, len(L) - 1):
            args, out = forward(r, r + 1)
            B.flame_gr_forward(h, *args)
            parts.append((r, out))
    finally:
        torch.cuda.synchronize()
        B.flame_gr_destroy(h)
    args, static = forward(0, len(L))
    c = B.config_for(wl)
    c.max_requests = c.max_total_tokens = 0
    B.flame_gr_forward_static(c, *args)
    torch.cuda.synchronize()
    assert torch.isfinite(whole).all()
    assert torch.equal(whole, static)
    for r, out in parts:
        assert torch.equal(out, whole[wl.cand_offsets[r]:wl.cand_offsets[r + 1]]), r


def planes_of_layer(wl, keys=("U", "V", "Q", "K", "O")):
    """The planes of a one-layer fp32 model by capture, rows in merged token order."""
    import torch
    from paper_2509_22681_amd import binding as B
    dw, hist, cand = B.to_device(wl)
    h = B.flame_gr_create(B.config_for(wl))
    try:
        B.flame_gr_debug_capture(h, 0)
        out = torch.empty((int(wl.cand_offsets[-1]),), device="cuda:0")
        B.flame_gr_forward(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, out)
        torch.cuda.synchronize()
        n = int(wl.history_offsets[-1] + wl.cand_offsets[-1])
        return {k: B.flame_gr_debug_stage(h, "UVQKO".index(k), n, wl.cfg.d_model) for k in keys}
    finally:
        B.flame_gr_destroy(h)


@pytest.mark.parametrize("d,H", [(64, 2), (48, 1)])       # heads that are staged through LDS, and that are not
def test_f32_silu_over_the_whole_range(d, H):
    """silu as the quotient x / (1 + exp(-x)) has it over the range of fp32: 0 far below zero, whatever the magnitude, in projections and attention weights."""
    wl = W.make_custom([70, 3], [5, 33], d=d, H=H, n_layers=1, n_buckets=16, max_rel_dist=128, dtype="f32", seed=5, emb_std=1.0, name="ends")
    x = np.array([0.0, 1e-30, -1e-30, 1.0, -1.0, -20.0, -50.0, -86.0, -87.2, -87.5, -88.5, -88.8, -90.0, -150.0, -1e4, -1e30, -3.4e38, 20.0, 86.0, 90.0, 1e4, 1e30, 3.4e38],
                 np.float32)
    wl.weights["w1"][:] = 0.0
    wl.weights["b1"][0, :d] = np.resize(np.concatenate([x, np.array([-np.inf, np.nan, np.inf], np.float32)]), d)       # U = silu(b1)
    got = planes_of_layer(wl, ("U",))["U"]
    assert (got == got[0])[:, ~np.isnan(got[0])].all()
    x64 = x.astype(np.float64)
    want = x64 * np.exp(-np.logaddexp(0.0, -x64))
    # exp of an argument of up to 87 in fp32: the argument's rounding (87 ulps of 2^-24 and the scaling to base 2) and a few ulps; below -87, where 1e-36 may be flushed, absolute
    err = np.abs(got[0, :len(x)] - want)
    assert (err <= np.maximum(2e-5 * np.abs(want), 1.5e-36)).all(), list(zip(x, got[0], want))
    assert np.isnan(got[0, len(x):len(x) + 2]).all() and got[0, len(x) + 2] == np.inf
    # attention weights: logits of -1e36 weigh nothing (and their values add nothing), the self term's likewise
    wl = W.make_custom([70, 3], [5, 33], d=d, H=H, n_layers=1, n_buckets=16, max_rel_dist=128, dtype="f32", seed=5, emb_std=1.0, name="ends")
    wl.weights["rab"][:] = -1e36
    got = planes_of_layer(wl, ("V", "O"))
    assert np.abs(got["V"]).max() > 0.1 and np.abs(got["O"]).max() < 1e-30


@pytest.mark.parametrize("d,H", [(32, 1), (90, 2), (256, 4)])
def test_f32_products_at_the_ends_of_the_range(d, H):
    """Operands that round past bf16's largest value, and infinities: the finite and infinite products that fp32 arithmetic has."""
    big, tiny = np.finfo(np.float32).max, np.float32(2.0 ** -122)
    M = 9
    wl = W.make_custom([70], [M], d=d, H=H, n_layers=1, n_buckets=16, max_rel_dist=128, dtype="f32", seed=5, emb_std=1.0, name="range")
    w1 = wl.weights["w1"][0]
    # meets the large embeddings.  (One bf16 part each: the lower parts of anything else below 2^-110 are under the range of normal numbers and lost, up to 2^-125, which
    # a factor of 2^128 would show as 8.)
    w1[:, 1] = tiny * np.resize(np.array([1.0, -1.0, 0.25, -0.5, 3.0, 1.25], np.float32), 4 * d)
    x = wl.cand_emb
    x[:, 1] = [big, -big, 3.4e38, 3.396e38, 3.39e38, -3.3953e38, np.inf, -np.inf, 1.0]
    wl.history_emb[:, 1] = 1.0
    x[:, 2] = tiny * np.resize(np.array([1.0, -0.75], np.float32), M)                                     # meets the large weights
    wl.history_emb[:, 2] = tiny
    w1[:, 2] = 0.0
    w1[:9, 2] = [big, -big, 3.4e38, 3.396e38, 3.39e38, -3.3953e38, np.inf, -np.inf, 1.0]
    w1[d:d + 6, 2] = big
    got = planes_of_layer(wl, ("U", "V", "Q", "K"))
    rows = np.concatenate([wl.history_emb, wl.cand_emb]).astype(np.float64)
    with np.errstate(invalid="ignore"):
        z = (rows[:, None, :] * w1.astype(np.float64)[None]).sum(-1)
        want = z * np.exp(-np.logaddexp(0.0, -z))                 # NaN at -inf, as -inf / (1 + inf)
    assert np.isfinite(want).sum() > 0.9 * want.size * 70 / 79 and np.isinf(want).any() and np.isnan(want).any()
    for p, name in enumerate("UVQK"):
        g, t = got[name].astype(np.float64), want[:, p * d:(p + 1) * d]
        assert np.array_equal(np.isnan(g), np.isnan(t)), name
        assert np.array_equal(np.isposinf(g), np.isposinf(t)), name
        ok = np.isfinite(t)
        assert (np.abs(g[ok] - t[ok]) <= 2e-5 * (1.0 + np.abs(t[ok]))).all(), name    # sums of up to 256 terms of size 1 (256 x 2^-24) and two terms of up to 200
