"""Draws that exclude tokens (u = 0) from passes of more than 16 LM-head rows:
a row with fewer than k tokens left lists those and then ids -1 with NaN
probabilities."""
import numpy as np
import pytest

from fe_synth import configs as C
from fe_synth import make_inputs, make_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [6, 45])  # 18 rows; 135, which take the 256-row tile
def test_excluded_tokens_are_not_listed(batch):
    import torch
    from paper_2509_20416_amd import Drafter
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg, k = C.SMALL_GQA_BF16.with_(batch=batch), 5
    N, V = cfg.n_layers, cfg.draft_vocab
    inp = make_inputs(cfg, 0, np.arange(batch, dtype=np.int32) % 7)
    rng = np.random.default_rng(4)
    u = np.zeros((batch * N, V), np.float32)
    left = []
    for r in range(batch * N):
        ids = rng.choice(V if r % 2 else 64, r % 4, replace=False)  # spread over tiles, or in one
        u[r, ids] = rng.uniform(0.1, 0.9, len(ids))
        left.append(set(ids.tolist()))
    dr = Drafter(cfg, make_weights(cfg, 0), max_batch=batch, max_prefix=6, max_topk=k)
    out = dr.forward(dr.upload_inputs(inp), k, temperature=1.0,
                     uniforms=torch.from_numpy(u.reshape(batch, N, V)).to(dr.device))
    ids, probs = (out[n].cpu().numpy().reshape(batch * N, k) for n in ("topk_draft", "topk_probs"))
    dr.close()
    for r, want in enumerate(left):
        n = len(want)
        assert set(ids[r, :n].tolist()) == want and (ids[r, n:] == -1).all(), (r, want, ids[r])
        assert (probs[r, :n] > 0).all() and np.isnan(probs[r, n:]).all(), (r, probs[r])
