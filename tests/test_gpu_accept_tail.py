"""The final draw of the sampling acceptance at the very end of the line: a
last uniform of 1 asks for the whole remaining mass, which the walk's running
sum may or may not reach in fp32; either way the token is the last unmapped
target id with mass."""
import numpy as np
import pytest

from fe_synth import configs as C
from tests.test_gpu_accept_sample import _cycle, _weights_with_layers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,sampled", [(1, True), (3, True), (3, False)])
def test_last_uniform_takes_the_last_token(B, sampled):
    import torch
    from paper_2509_20416_amd import Drafter
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    k, cfg = 5, C.SMALL_GQA_BF16.with_(batch=B, topk=5)
    cy = _cycle(cfg, B, k, 1.0, sampled, seed=31)
    last = max(set(range(cfg.target_vocab)) - set(cy["d2t"].tolist()))
    cy["tp"][..., last + 1:] = 0.0
    cy["tp"][..., last] = 0.3
    cy["u"][:, -1] = 1.0
    dr = Drafter(cfg, _weights_with_layers(cy["w"], cfg.n_layers), max_batch=B, max_prefix=0, max_topk=k)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dr.device)
    got = dr.accept_sample({n: t(a) for n, a in cy["tree"].items()}, t(cy["cand"]), t(cy["z"]),
                           t(cy["tp"]), t(cy["u"]), temperature=1.0,
                           draft_uniforms=t(cy["ud"]) if sampled else None, topk=k)
    n, acc = got["accept_len"].cpu().numpy(), got["accepted"].cpu().numpy()
    dr.close()
    assert (acc[np.arange(B), n] == last).all()
