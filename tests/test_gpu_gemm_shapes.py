"""Every GEMM tile shape through its fused epilogues (RoPE, residual, SwiGLU) at
ragged row counts, and K-slices of uneven depth.  All tiles add the same products
in the same order, so a bf16 forward forced onto any of them gives the same bits;
in fp16 the compiler may fuse RoPE's last multiply-add with its rounding to 16 bits
(one rounding instead of two), which moves a few q and k values by one ulp."""
import numpy as np
import pytest
import torch

import wino_inputs as wi
from oracle import model as M
from helpers import batch_tokens, rowwise_rel_err, tile_table, to_cpu

pytestmark = pytest.mark.gpu


def forward(P, cfg, wd, act, p, g, lb, B, n_sub):
    model = P.WinoModel(cfg, wd, B, p + g + lb, act_precision=act)
    tok = batch_tokens(cfg, B, p, g, seed=3, fill=[(0, lb, 0.5)])
    bstart = [(lb * b) % g for b in range(B)]
    out = torch.empty(B, p + g + lb, cfg.d_model, dtype=torch.float32, device="cuda")
    P.wino_debug_forward(model.ctx, P.make_params(B, p, g, lb, cfg.mask_id),
                         torch.tensor(tok, dtype=torch.int32, device="cuda"),
                         torch.tensor(bstart, dtype=torch.int32, device="cuda"), n_sub, out)
    torch.cuda.synchronize()
    model.close()
    return out.cpu().numpy(), tok, bstart


def oracle(wd, cfg, tok, bstart, p, g, lb, n_sub):
    w = to_cpu(wd)
    rows = []
    for b in range(len(tok)):
        ext, pos, allowed, _ = M.extended_inputs(tok[b], p, g, lb, bstart[b], cfg.mask_id)
        rows.append(M.forward_residual(w, cfg, ext, pos, allowed, n_sublayers=n_sub))
    return np.stack(rows)


# T = 40 (a wave's rows span several sequences), 109 (odd), 200 and 592 (whole
# 8-row runs; 592 rows cross every tile height); ff = 704 and 1088 leave the 256-wide
# tiles out of the gate/up product, 768 and 1152 do not
@pytest.mark.parametrize("hd,d,ff,p,g,lb,B,f16", [
    (64, 256, 704, 12, 24, 4, 5, False), (64, 256, 768, 77, 24, 8, 3, False), (64, 256, 768, 560, 24, 8, 1, True),
    (128, 512, 1152, 12, 24, 4, 5, True), (128, 512, 1088, 77, 24, 8, 3, False), (128, 512, 1152, 168, 24, 8, 2, False),
])
def test_tiles_give_the_same_bits(hd, d, ff, p, g, lb, B, f16, monkeypatch):
    import paper_2605_16941_amd as P
    cfg = wi.preset("tiny", d_model=d, n_heads=d // hd, head_dim=hd, n_layers=1, d_ff=ff, vocab=512, mask_id=511)
    wd = wi.model_weights(cfg, seed=d, device="cuda", gain_std=0.1)
    act = P.ACT_FP16 if f16 else P.ACT_BF16
    monkeypatch.setenv("WINO_GEMM_TAIL", "0")  # whole-K tiles
    first = None
    for tile in range(len(tile_table())):
        monkeypatch.setenv("WINO_GEMM_TILE", str(tile))
        got, tok, bstart = forward(P, cfg, wd, act, p, g, lb, B, 2)
        if first is None:
            first = got
            # 16-bit activations: 2^-9 per rounding, a few roundings deep
            assert rowwise_rel_err(got, oracle(wd, cfg, tok, bstart, p, g, lb, 2)) < 1e-2
        if f16:
            assert rowwise_rel_err(got, first) < 2.0 ** -10, tile  # an fp16 ulp
        else:
            assert np.array_equal(got, first), tile


# A width of each row-kernel shape (64, 128 and 256 threads of one 8-element chunk,
# 256 of two).  The down projection's K = 2368 is 37 steps of 64: uneven in every split.
@pytest.mark.parametrize("d,f16", [(512, False), (1024, True), (2048, False), (4096, True)])
@pytest.mark.parametrize("split", [2, 3, 4, 6, 8])
def test_uneven_k_slices(d, f16, split, monkeypatch):
    """The down projection in K-slices, against whole K: the fp32 partials added to
    the stream by the reduce kernel (two sublayers, at fp32 accuracy) and by the
    next layer's norm (three sublayers)."""
    import paper_2605_16941_amd as P
    ff, p, g, lb, B = 2368, 77, 24, 8, 3
    T, M = p + g + lb, B * (p + g + lb)
    cfg = wi.preset("tiny", d_model=d, n_heads=d // 64, n_layers=2, d_ff=ff, vocab=512, mask_id=511)
    wd = wi.model_weights(cfg, seed=9, device="cuda", gain_std=0.1)
    model = P.WinoModel(cfg, wd, B, T, act_precision=P.ACT_FP16 if f16 else P.ACT_BF16)
    prm = P.make_params(B, p, g, lb, cfg.mask_id)
    tok = torch.tensor(batch_tokens(cfg, B, p, g, seed=3, fill=[(0, lb, 0.5)]), dtype=torch.int32, device="cuda")
    bs = torch.tensor([0, 8, 16], dtype=torch.int32, device="cuda")

    def run(n_sub, tail, tile):
        monkeypatch.setenv("WINO_GEMM_TAIL", str(tail))
        monkeypatch.setenv("WINO_GEMM_TILE", str(tile))
        out = torch.empty(M, d, device="cuda")
        P.wino_debug_forward(model.ctx, prm, tok, bs, n_sub, out)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    monkeypatch.setenv("WINO_GEMM_SPLIT", str(split))
    want = {n: run(n, 0, 0) for n in (2, 3)}
    x = np.abs(want[2]).max(-1, keepdims=True)
    table = tile_table()
    # a two-, three-, four- and six-stage tile, a third W stage, three-block waves
    for bm, kind in ((128, (2, 2, 0)), (64, (3, 2, 0)), (128, (4, 1, 0)), (64, (6, 1, 0)), (128, (2, 1, 1)), (192, (2, 1, 1))):
        (tile,) = [i for i, t in enumerate(table) if t[0] == bm and t[2:4] != (4, 1) and t[4] == 64 and t[5:] == kind]
        assert d % table[tile][1] == 0
        for tail in (1, 99):  # the last row tile or all of them
            got = run(2, tail, tile)
            first = 0 if tail == 99 else (M - 1) // bm * bm
            if d == 512 and split > 2:  # (the O projection's 8 steps are too few for these slices)
                assert np.array_equal(got[:first], want[2][:first])
            assert not np.array_equal(got[first:], want[2][first:]), "no split ran"
            # K fp32 additions in another order: at most K * 2^-24 of the terms'
            # absolute sum, itself about sqrt(K) times the result (one step missing
            # or doubled moves the result by sqrt(1 / 37)); where the O projection is
            # split too, a few of the normed rows' roundings flip, 2^-9 each
            assert (np.abs(got - want[2]) / x).max() < 2368 ** 1.5 * 2.0 ** -24, (tile, tail)
            # (the next layer's normed rows round likewise)
            assert rowwise_rel_err(run(3, tail, tile), want[3]) < 1e-2, (tile, tail)
    model.close()
