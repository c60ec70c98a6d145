"""Sampling acceptance when one draft id holds nearly all of q: once it is
rejected, the remaining children are tested against what is left of q, whose
share (1e-7 and less) fp32 cannot get from 1 - q(x), and the residual is still
(p - q)^+."""
import numpy as np
import pytest

from fe_synth import configs as C
from fe_synth import make_uniforms
from tests.test_gpu_accept_sample import _weights_with_layers, make_weights

pytestmark = pytest.mark.gpu


def _cycle(cfg, B, k, gap, seed):
    """Level logits with one id `gap` above the others, which the target gives
    no mass; the target agrees with the draft on the others, up to 64 random ids."""
    from oracle import feo
    rng = np.random.default_rng(seed)
    N, V, Vt = cfg.n_layers, cfg.draft_vocab, cfg.target_vocab
    w = make_weights(cfg.with_(n_layers=1), 0)
    z = (rng.standard_normal((B, N, V)) * 2.5).astype(np.float32)
    rest = np.exp(z - z.max(-1, keepdims=True))
    top = rng.integers(0, V, (B, N))
    np.put_along_axis(rest, top[..., None], 0.0, -1)
    rest /= rest.sum(-1, keepdims=True)
    np.put_along_axis(z, top[..., None], z.max(-1, keepdims=True) + np.float32(gap), -1)
    ud = make_uniforms((B, N, V), seed=seed + 1)
    keys = z - np.log(-np.log(ud.astype(np.float64)))
    cand = np.argsort(-keys, axis=-1, kind="stable")[..., :k]
    zc = np.take_along_axis(z, cand, -1)
    cand = np.take_along_axis(cand, np.argsort(-zc, axis=-1, kind="stable"), -1).astype(np.int32)
    assert (cand[..., 0] == top).all()
    tree = feo.build_tree(N, k, rng.integers(0, Vt, B).astype(np.int32), w.d2t[cand],
                          np.zeros(B, np.int32))
    T = 1 + N * k
    tp = np.zeros((B, T, Vt), np.float32)
    for b in range(B):
        for n in range(T):
            lvl = min(tree["depth"][b, n], N - 1)   # the level drafted after this node
            ids = rng.choice(Vt, 64, replace=False)
            tp[b, n, ids] = 0.5 * rng.dirichlet(np.ones(64))
            tp[b, n, w.d2t] += 0.5 * rest[b, lvl]
            tp[b, n, w.d2t[top[b, lvl]]] = 0.0
    return dict(z=z, ud=ud, cand=cand, tree=tree, tp=tp, u=make_uniforms((B, N * k + 1), seed=seed + 2),
                top=w.d2t[top], w=w)


def _gpu(cfg, B, k, cy):
    import torch
    from paper_2509_20416_amd import Drafter
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dr = Drafter(cfg, _weights_with_layers(cy["w"], cfg.n_layers), max_batch=B, max_prefix=0, max_topk=k)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dr.device)
    got = dr.accept_sample({n: t(a) for n, a in cy["tree"].items()}, t(cy["cand"]), t(cy["z"]),
                           t(cy["tp"]), t(cy["u"]), draft_uniforms=t(cy["ud"]), topk=k)
    got = {n: a.cpu().numpy() for n, a in got.items()}
    dr.close()
    return got


VOCABS = {"some_mapped": C.SMALL_GQA_BF16, "all_mapped": C.TINY_F32_B1.with_(n_layers=3)}


@pytest.mark.parametrize("B", [1, 16])           # one sequence: with the row pre-pass
@pytest.mark.parametrize("gap", [12, 18, 25])
@pytest.mark.parametrize("vocab", list(VOCABS))
def test_peaked_draft_matches_oracle(vocab, gap, B):
    from oracle import feo
    k, same = 4, 0
    cfg = VOCABS[vocab].with_(batch=B, topk=4)
    for seed in range(41, 41 + 16 // B):
        cy = _cycle(cfg, B, k, gap, seed)
        got = _gpu(cfg, B, k, cy)
        ref = feo.accept_sample(cfg.n_layers, k, cy["tree"]["tokens"], cy["tree"]["retrieve"], cy["cand"],
                                cy["z"], 1.0, cy["w"].d2t, cy["tp"], cy["u"], draft_uniforms=cy["ud"])
        for b in np.flatnonzero(ref["margin"] > 1e-4):
            same += 1
            for n in ("accept_len", "accept_path", "accepted"):
                np.testing.assert_array_equal(got[n][b], ref[n][b], err_msg=f"seed {seed} seq {b} {n}")
    assert same >= 8


@pytest.mark.parametrize("B", [1, 16])
@pytest.mark.parametrize("vocab", list(VOCABS))
def test_nothing_left_of_the_draft(vocab, B):
    """A gap beyond the range of exp: only the top id has weight.  The draw is
    then from the target without it."""
    k = 4
    cfg = VOCABS[vocab].with_(batch=B, topk=k)
    cy = _cycle(cfg, B, k, 200, 40)
    got = _gpu(cfg, B, k, cy)
    assert (got["accept_len"] == 0).all()
    tok = got["accepted"][:, 0]
    assert (tok >= 0).all() and (tok != cy["top"][:, 0]).all()
    assert (cy["tp"][np.arange(B), 0, tok] > 0).all()
