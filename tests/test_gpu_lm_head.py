"""The LM head's fused statistics on each tile that serves them (32, 128 and 256
rows), at row counts around the tiles' edges: exact ties (every id k < V/2 has
a twin k + V/2 with the same weights and bias), a mask id inside the vocabulary
that often holds the maximum, and targets in both halves."""
import numpy as np
import pytest
import torch

import wino_inputs as wi
from oracle import model as M
from helpers import tile_table

pytestmark = pytest.mark.gpu
V, MASK = 1024, 100


# (the last: more response rows than the step's decision rows, B * (max_seq / 2 + 1),
# that the workspace's partials are sized by)
@pytest.mark.parametrize("B,G,lb", [(1, 1, 1), (3, 11, 11), (2, 64, 64), (3, 43, 43), (4, 64, 64), (3, 86, 86), (4, 64, 8)])
def test_tiles_agree_and_match_oracle(B, G, lb, monkeypatch):
    import paper_2605_16941_amd as P
    cfg = wi.preset("tiny", n_layers=1, vocab=V, mask_id=MASK)
    w = wi.model_weights(cfg, seed=5, lm_head_std=wi.wide_lm_head_std(cfg), gain_std=0.1)
    w["lm_bias"] = w["lm_bias"].clone()
    w["lm_bias"][MASK] = float(w["lm_bias"].max()) + 1.0
    for k in ("lm_head", "lm_bias"):
        w[k][V // 2:] = w[k][:V // 2]
    wd = {k: (v.cuda() if isinstance(v, torch.Tensor) else v) for k, v in w.items() if k != "layers"}
    wd["layers"] = [{k: v.cuda() for k, v in lw.items()} for lw in w["layers"]]
    p = 5
    rng = np.random.default_rng(B * G)
    tok = rng.integers(0, V, (B, p + G))
    tgt = rng.integers(0, V, (B, G))
    prm = P.make_params(B, p, G, lb, MASK)
    tok_d, tgt_d = (torch.tensor(a, dtype=torch.int32, device="cuda") for a in (tok, tgt))
    got = {}
    tiles = [i for i, t in enumerate(tile_table()) if t[:4] in ((32, 256, 1, 4), (128, 256, 2, 4)) or t[4] == 32]
    assert len(tiles) == 3
    for tile in (None, *tiles):
        if tile is not None:
            monkeypatch.setenv("WINO_GEMM_TILE", str(tile))
        model = P.WinoModel(cfg, wd, B, p + G + lb)
        out = torch.full((B * G, 4), float("nan"), device="cuda")
        P.wino_row_losses(model.ctx, prm, tok_d, tgt_d, out)
        torch.cuda.synchronize()
        model.close()
        got[tile] = out.cpu().numpy()
    ids = {t: o.view(np.int32)[:, 3] for t, o in got.items()}
    ent, nll, conf, best = [], [], [], []
    for b in range(B):
        n = p + G
        h = M.forward_hidden(w, cfg, tok[b], np.arange(n), np.ones((n, n), dtype=bool))[p:]
        z = M.lm_logits(w, h)
        lse = np.log(np.exp(z - z.max(-1, keepdims=True)).sum(-1)) + z.max(-1)
        lp = z - lse[:, None]
        ent.append(-(np.exp(lp) * lp).sum(-1))
        nll.append(-lp[np.arange(G), tgt[b]])
        zz = lp.copy()
        zz[:, MASK] = -np.inf
        conf.append(np.exp(zz.max(-1)))
        # lowest id among ties, the mask excluded; -1 where two distinct values are close
        top = np.argmax(zz, -1)
        srt = np.sort(np.where(np.arange(V) < V // 2, np.maximum(zz, np.roll(zz, V // 2, axis=-1)), -np.inf), -1)
        best.append(np.where(srt[:, -1] - srt[:, -2] > 0.1, top, -1))
    ent, nll, conf, best = (np.concatenate(a) for a in (ent, nll, conf, best))
    assert (best >= 0).any() and (B * G < 100 or (best == MASK + V // 2).any())
    for t in got:
        o = got[t]
        # bf16 activations move a logit by about 1e-2 here
        assert np.abs(o[:, 0] - ent).max() < 0.1 and np.abs(o[:, 1] - nll).max() < 0.1
        assert np.abs(o[:, 2] - conf).max() < 0.03
        assert np.array_equal(ids[t][best >= 0], best[best >= 0])
        assert ((ids[t] < V // 2) | (ids[t] == MASK + V // 2)).all() and (ids[t] != MASK).all()
        # the tiles compute the same logits; only the sums' orders differ
        assert np.array_equal(ids[t], ids[tiles[0]])
        np.testing.assert_allclose(o[:, :3], got[tiles[0]][:, :3], rtol=2e-5, atol=2e-5)
