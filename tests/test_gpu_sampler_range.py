"""The accept rule on rows whose logits are large against their differences: the float32 spacing at
the largest logit exceeds every range the kernels clamp to, so a clamp formed in float32 there is the
largest logit itself. Forced tokens (one logit of 1e9 .. the largest float32) and rows of masked tokens
(the lowest float32, -inf), against the oracle; few sequences and many (the two ways to the
decisions), aligned and unaligned rows, one and several chunks, with and without q."""
import numpy as np
import pytest
import torch

from oracle import sampler as osamp

pytestmark = pytest.mark.gpu
BIG = float(np.finfo(np.float32).max)


def _rows(g, B, kp1, V, top, equal):
    """Logits whose largest is `top` at one place (with `equal`: at two) and the places of the first."""
    if top > 0:
        l = g.uniform(-1, 1, (B, kp1, V)).astype(np.float32)
    else:
        l = np.full((B, kp1, V), -BIG, np.float32)
        l[..., ::3] = -np.inf
    at = g.integers(0, V - 1, (B, kp1))
    np.put_along_axis(l, at[..., None], np.float32(top), 2)
    if equal:
        np.put_along_axis(l, at[..., None] + 1, np.float32(top), 2)
    return l, at


def _run(lib, logits, drafts, u, q):
    t = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    toks, n, lp = lib.spec_accept(t(logits), t(drafts), t(u), t(q))
    return toks.cpu().numpy(), n.cpu().numpy(), lp.cpu().numpy()


@pytest.mark.parametrize("top", [1.0737e9, 1.1e9, 4e9, 1e10, 1e30, BIG, -1.1e9, -1e10, -1e30])
@pytest.mark.parametrize("B,k,V,with_q", [(3, 0, 1000, False), (3, 2, 20003, False), (200, 2, 8200, False)])
def test_draw(lib, top, B, k, V, with_q):
    """Drafts that p rules out: the draw alone decides."""
    print(f"case top={top} B={B} k={k} V={V} q={with_q}", flush=True)
    g = np.random.Generator(np.random.Philox(V + k))
    for equal in (False, True):
        logits, at = _rows(g, B, k + 1, V, top, equal)
        drafts = ((at[:, :k] + 7) % V).astype(np.int32)
        q = None
        if with_q:
            q = g.random((B, k, V), dtype=np.float32)
            q /= q.sum(-1, keepdims=True)
        u = g.random((B, k + 1), dtype=np.float32)
        toks, n, _ = _run(lib, logits, drafts, u, q)
        o = osamp.spec_accept(logits, drafts, u, q)
        ok = o["draw_margin"] > 2e-8
        assert ok.mean() > 0.95
        assert (n == o["n_accepted"]).all()
        assert (toks[ok] == o["tokens"][ok]).all()


@pytest.mark.parametrize("top", [1.0737e9, 4.2e9, 4.4e9, 1e10, 1e30, BIG, -4.4e9, -1e10, -1e30, -BIG])
@pytest.mark.parametrize("B,k,V,with_q", [(3, 2, 20003, True), (2, 0, 1000, False), (200, 2, 8200, False),
                                          (200, 1, 1001, True)])
def test_row_sums(lib, top, B, k, V, with_q):
    """Forced drafts and log-probs: the row's sum is the number of its largest logits."""
    print(f"case top={top} B={B} k={k} V={V} q={with_q}", flush=True)
    g = np.random.Generator(np.random.Philox(V + k))
    for equal in (False, True):
        logits, at = _rows(g, B, k + 1, V, top, equal)
        if top == -BIG:          # the lowest float32 is the largest: beside it only -inf
            logits = np.where(logits == -BIG, -np.inf, logits).astype(np.float32)
            np.put_along_axis(logits, at[..., None], np.float32(top), 2)
            if equal:
                np.put_along_axis(logits, at[..., None] + 1, np.float32(top), 2)
        drafts = at[:, :k].astype(np.int32)
        drafts[::4] = (drafts[::4] + 7) % V
        q = None
        if with_q:
            q = g.random((B, k, V), dtype=np.float32)
            q /= q.sum(-1, keepdims=True)
        u = g.random((B, k + 1), dtype=np.float32)
        toks, n, lp = _run(lib, logits, drafts, u, q)
        o = osamp.spec_accept(logits, drafts, u, q)
        ok = o["draw_margin"] > 2e-8
        if k:
            ok &= np.nan_to_num(o["accept_margin"], nan=np.inf).min(1) > 1e-6
        assert ok.mean() > 0.9
        assert (n[ok] == o["n_accepted"][ok]).all()
        assert (toks[ok] == o["tokens"][ok]).all()
        np.testing.assert_allclose(lp[ok], o["logprobs"][ok], rtol=1e-6, atol=1e-6, equal_nan=True)
