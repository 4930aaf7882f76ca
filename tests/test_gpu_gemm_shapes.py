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
from helpers import batch_tokens, rowwise_rel_err, to_cpu

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
# 8-row runs; 592 rows cross every tile height)
@pytest.mark.parametrize("hd,d,ff,p,g,lb,B,f16", [
    (64, 256, 704, 12, 24, 4, 5, False), (64, 256, 704, 77, 24, 8, 3, False), (64, 256, 704, 560, 24, 8, 1, True),
    (128, 512, 1088, 12, 24, 4, 5, True), (128, 512, 1088, 77, 24, 8, 3, False), (128, 512, 1088, 168, 24, 8, 2, False),
])
def test_tiles_give_the_same_bits(hd, d, ff, p, g, lb, B, f16, monkeypatch):
    import paper_2605_16941_amd as P
    cfg = wi.preset("tiny", d_model=d, n_heads=d // hd, head_dim=hd, n_layers=1, d_ff=ff, vocab=512, mask_id=511)
    wd = wi.model_weights(cfg, seed=d, device="cuda", gain_std=0.1)
    act = P.ACT_FP16 if f16 else P.ACT_BF16
    monkeypatch.setenv("WINO_GEMM_TAIL", "0")  # whole-K tiles
    first = None
    for tile in range(17):
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


@pytest.mark.parametrize("split", [2, 3, 6, 8])
@pytest.mark.parametrize("tail", [1, 99])
def test_uneven_k_slices(split, tail, monkeypatch):
    """The O projection over K = 1408 (22 steps of 64) in slices: the fp32 sums in
    another order."""
    import paper_2605_16941_amd as P
    cfg = wi.preset("tiny", d_model=1408, n_heads=22, n_layers=1, d_ff=256, vocab=512, mask_id=511)
    wd = wi.model_weights(cfg, seed=9, device="cuda", gain_std=0.1)
    args = (P, cfg, wd, P.ACT_BF16, 77, 24, 8, 2, 1)
    monkeypatch.setenv("WINO_GEMM_TAIL", "0")
    want, _, _ = forward(*args)
    monkeypatch.setenv("WINO_GEMM_TAIL", str(tail))
    monkeypatch.setenv("WINO_GEMM_SPLIT", str(split))
    for tile in (5, 8, 12, 14):  # two and six stages, a third W stage, three-block waves
        monkeypatch.setenv("WINO_GEMM_TILE", str(tile))
        got, _, _ = forward(*args)
        # K fp32 additions in another order: at most K * 2^-24 of the terms'
        # absolute sum, itself about sqrt(K) times the result
        assert rowwise_rel_err(got, want) < 1408 ** 1.5 * 2.0 ** -24
