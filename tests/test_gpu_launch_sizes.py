"""K1, K2 and K3 choose their tiles and their cache policy by the size of a launch and change none of an output's arithmetic with it: a
request has the same bits scored alone and in a batch on either side of every limit of its width.  The limits are read from the
sources that dispatch on them.  (Accuracy against the oracle: the parity tests.)"""
import re
from pathlib import Path

import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W

pytestmark = pytest.mark.gpu

CSRC = Path(W.__file__).parent / "csrc"


def _constant(text, name):
    m = re.search(rf"\b{name} = (\d+)(?: << (\d+))?[,;]", text)
    return int(m.group(1)) << int(m.group(2) or 0)


def limits(d):
    """Launch sizes, in 64-row blocks, after which one of the kernels of width d changes: the largest before each change."""
    common, k1 = (CSRC / "kernels.h").read_text(), (CSRC / "gemm_mfma.hip").read_text()
    row_block = 64 * d * 2                                                          # bytes of a plane's row block
    stream = _constant(common, "kStreamBytes") // row_block                         # K1's large tile and K3
    out = {stream, stream // 2}                                                     # K2 counts 128 rows per tile; a batch of the test fills half of each
    out |= {_constant(common, n) for n in ("kK3CutInFour", "kK3CutInTwo", "kK3HalfBlocks")}
    cases = re.search(r"static int small_tile_blocks.*?\n}", k1, re.S).group(0)
    small = re.search(rf"case {d}:.*?return (.*?);", cases)
    small = eval(small.group(1)) if small else 0
    if 0 < small < 1 << 20:
        out.add(small)
    small_stream = _constant(k1, "kSmallStreamBytes") // row_block                  # from here on, not past it
    if small > small_stream:
        out.add(-(-_constant(k1, "kSmallStreamBytes") // row_block) - 1)
    return sorted(out)


MODELS = {64: 2, 128: 2, 192: 3, 256: 4, 384: 6, 512: 8, 320: 5, 448: 7}
UNITS = 12                                                                          # distinct requests of 64 + 64 rows: two row blocks each
RAGGED = ([65, 1, 130, 0], [3, 70, 0, 5])                                           # ten row blocks together


@pytest.mark.parametrize("d", list(MODELS))
def test_same_bits_at_every_launch_size(d):
    import torch
    from paper_2509_22681_amd import binding as B
    wl = W.make_custom([64] * UNITS + RAGGED[0], [64] * UNITS + RAGGED[1], d=d, H=MODELS[d], n_layers=2, n_buckets=16, max_rel_dist=128, dtype="bf16", seed=3,
                       emb_std=1.0, rab_std=1.0, bias_amp=0.1, affine_random=True, name=f"sizes{d}")
    dw, hist, cand = B.to_device(wl)
    ho, co = wl.history_offsets.astype(np.int64), wl.cand_offsets.astype(np.int64)

    def scores(idx):
        """The requests idx, any number of times each, as one batch."""
        idx = np.asarray(idx)

        def take(rows, off):
            n = np.diff(off)[idx]
            start = np.concatenate([[0], np.cumsum(n)])
            src = np.arange(start[-1]) - np.repeat(start[:-1], n) + np.repeat(off[idx], n)
            return rows[torch.as_tensor(src, device="cuda:0")].contiguous(), start.astype(np.int32)

        h, nho = take(hist, ho)
        c, nco = take(cand, co)
        cfg = B.make_config(wl.cfg.n_layers, d, MODELS[d], wl.cfg.n_buckets, wl.cfg.max_rel_dist, "bf16", ln_eps=wl.cfg.ln_eps, attn_scale=wl.cfg.attn_scale,
                            max_requests=len(idx), max_total_tokens=int(nho[-1]) + int(nco[-1]))
        handle = B.flame_gr_create(cfg)
        try:
            out = torch.full((int(nco[-1]),), float("nan"), device="cuda:0")
            B.flame_gr_forward(handle, dw, h, nho, c, nco, out)
            torch.cuda.synchronize()
            return out, nco
        finally:
            B.flame_gr_destroy(handle)

    alone = [scores([i])[0] for i in range(wl.n_requests)]
    assert all(bool(torch.isfinite(a).all()) for a in alone)
    ragged = list(range(UNITS, wl.n_requests))
    for limit in limits(d):
        # blocks of a whole batch of units: the largest even number up to the limit, the next one past it, and past it with ragged requests among
        # them; the last layer's launches are over half as many
        n = limit // 2
        for idx in (np.arange(n) % UNITS, np.arange(n + 1) % UNITS, np.concatenate([np.arange(max(0, n - 4)) % UNITS, ragged])):
            got, nco = scores(idx)
            want = torch.cat([alone[i] for i in idx])
            same = got.view(torch.int32) == want.view(torch.int32)
            assert bool(same.all()), (d, limit, len(idx), int((~same).sum()))


@pytest.mark.parametrize("d,H", [(64, 2), (192, 3), (320, 5)])
def test_hidden_rows_at_any_alignment(d, H):
    """The gather of the candidates' rows stores 16 bytes at a time where the caller's array allows it."""
    import torch
    from paper_2509_22681_amd import binding as B
    wl = W.make_custom([70, 0, 33], [65, 3, 16], d=d, H=H, n_layers=2, n_buckets=16, max_rel_dist=128, dtype="bf16", seed=5, name=f"hidden{d}")
    n = int(wl.cand_offsets[-1]) * d
    h = B.flame_gr_create(B.config_for(wl))
    try:
        dw, hist, cand = B.to_device(wl)
        rows = []
        for shift in (0, 1, 2, 4):
            buf = torch.full((n + 8,), float("nan"), device="cuda:0")
            B.flame_gr_forward_hidden(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, buf[shift:shift + n].view(-1, d))
            torch.cuda.synchronize()
            got = buf.cpu().numpy()
            assert np.isnan(got[:shift]).all() and np.isnan(got[shift + n:]).all()
            rows.append(got[shift:shift + n])
    finally:
        B.flame_gr_destroy(h)
    assert np.isfinite(rows[0]).all()
    for r in rows[1:]:
        assert np.array_equal(r, rows[0])
