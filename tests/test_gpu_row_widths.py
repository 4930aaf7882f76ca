"""The row kernels (embedding + norm, norm with split-K partials, final norm) at
the edges of their workgroup shapes: d = 512 | 1024 | 2048 | 4096 are the widest
rows of one shape, the next multiple of 64 the narrowest of the next."""
import numpy as np
import pytest
import torch

import wino_inputs as wi
from oracle import model as M
from helpers import LOGIT_TOL, batch_tokens, rowwise_rel_err, to_cpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 512, 640, 1024, 1152, 2048, 2176, 4096])
def test_forward_at_row_widths(d):
    import paper_2605_16941_amd as P
    cfg = wi.preset("tiny", d_model=d, n_heads=d // 64, n_layers=2, d_ff=256, vocab=512, mask_id=511)
    wd = wi.model_weights(cfg, seed=d, device="cuda", gain_std=0.1)
    p, g, lb, B = 9, 16, 8, 2
    T = p + g + lb
    tok = batch_tokens(cfg, B, p, g, seed=3, fill=[(0, 8, 0.5)])
    bstart = [0, 8]
    model = P.WinoModel(cfg, wd, B, T)
    prm = P.make_params(B, p, g, lb, cfg.mask_id)
    args = (model.ctx, prm, torch.tensor(tok, dtype=torch.int32, device="cuda"),
            torch.tensor(bstart, dtype=torch.int32, device="cuda"))
    # a buffer at a 16-byte boundary and one 4 bytes past it (copied out at the end)
    room = torch.full((B * T * d + 4,), 7.0, dtype=torch.float32, device="cuda")
    aligned = torch.empty(B * T * d, dtype=torch.float32, device="cuda")
    P.wino_debug_forward(*args, 4, aligned)
    P.wino_debug_forward(*args, 4, room[1:1 + B * T * d])
    logits = torch.empty(B, 2 * lb, cfg.vocab, dtype=torch.float32, device="cuda")
    P.wino_debug_logits(*args, logits)
    torch.cuda.synchronize()
    model.close()
    assert torch.equal(room[1:1 + B * T * d], aligned)
    assert room[0] == 7.0 and bool((room[1 + B * T * d:] == 7.0).all())
    w = to_cpu(wd)
    got, gl = aligned.view(B, T, d).cpu().numpy(), logits.cpu().numpy()
    for b in range(B):
        ext, pos, allowed, c0 = M.extended_inputs(tok[b], p, g, lb, bstart[b], cfg.mask_id)
        x = M.forward_residual(w, cfg, ext, pos, allowed)
        # bf16 activations: 2^-9 per rounding, a few roundings deep
        assert rowwise_rel_err(got[b], x) < 1e-2
        h = M.rmsnorm(x, M.f64(w["final_norm"]), cfg.rms_eps)
        sel = np.concatenate([h[c0:c0 + lb], h[T - lb:]])
        assert rowwise_rel_err(gl[b], M.lm_logits(w, sel)) < LOGIT_TOL
