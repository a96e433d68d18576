"""The row kernels (log-softmax / argmax / top-k of logit rows, and the rows of
speculative sampling) where they can go wrong: rows that start at every
alignment (odd vocabularies), fewer ids than threads, vocabularies beyond the
register groups and segments, equal values at group and thread borders, -inf
and NaN entries.  References: float64 numpy, ids exact (the kernels compare the
same fp32 values)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _order(row, k):
    """The k best ids: value descending, id ascending, NaN never."""
    ids = np.flatnonzero(~np.isnan(row))
    return ids[np.lexsort((ids, -row[ids]))][:k]


@pytest.mark.parametrize("M,V", [(3, 5), (9, 64), (6, 1023), (5, 4097), (4, 8193), (3, 16387), (400, 8200), (2, 70001),
                                 (2, 150001), (1, 300007)])
@pytest.mark.parametrize("kk", [0, 1, 5, 16])
def test_logit_rows_alignment_ties_and_infinities(M, V, kk):
    from paper_2412_10418_amd.binding import cdsl_op_logit_rows
    kk = min(kk, V)
    rng = np.random.default_rng([M, V, kk])
    z = (rng.standard_normal((M, V)) * 2).astype(np.float32)
    z[0] = np.round(z[0])                          # many equal values
    if M > 1:
        z[1, rng.random(V) < 0.7] = -np.inf        # most entries ruled out
    if M > 2:
        z[2] = -np.inf                             # fewer finite entries than places
        z[2, V // 2] = 1.0
    if M > 3:
        z[3, V // 3] = np.nan
    g = rng.integers(0, V, M).astype(np.int32)
    lp, amax, tk, tl = (t.cpu().numpy() for t in
                        cdsl_op_logit_rows(torch.from_numpy(z).cuda(), torch.from_numpy(g).cuda(), kk))
    for m in range(M):
        want = _order(z[m], max(kk, 1))
        assert amax[m] == want[0]
        assert list(tk[m][:len(want)]) == list(want[:kk])
        if np.isnan(z[m]).any():
            continue
        x = z[m].astype(np.float64)
        lse = x.max() + np.log(np.sum(np.exp(x - x.max())))
        ref = x[g[m]] - lse
        # fp32 logsumexp: rounding of max + log(sum) and of the sum, with room
        assert lp[m] == ref or abs(lp[m] - ref) < 2e-5
        for u in range(kk):
            r = x[want[u]] - lse
            assert tl[m, u] == r or abs(tl[m, u] - r) < 2e-5


@pytest.mark.parametrize("G,d,V,skew", [(2, 3, 5, 0), (3, 2, 1023, 0), (2, 2, 4099, 0), (2, 2, 9001, 1), (1, 3, 40003, 0),
                                        (1, 2, 131077, 0), (1, 2, 600011, 0)])
def test_soft_rows_alignment_and_segments(G, d, V, skew):
    """Draws against the float64 inverse CDF, for uniforms in the middle of an
    interval that is wide beside fp32 rounding (1e-5 of the mass)."""
    from paper_2412_10418_amd.binding import cdsl_op_soft_rows
    M = G * d
    gen = torch.Generator(device="cuda").manual_seed(V)
    p = torch.randn((M, V), generator=gen, device="cuda") * 3
    flat = torch.empty(M * V + 4, device="cuda")      # q may start at another alignment than p
    q = flat[skew:skew + M * V].view(M, V)
    q.copy_(torch.randn((M, V), generator=gen, device="cuda") * 3)
    q[0, V // 2:] = -float("inf")
    if M > 3:
        q[3] = p[3]                                   # no mass left: argmax p
    look = torch.randint(0, V, (G, d + 1), generator=gen, device="cuda", dtype=torch.int32)
    lp, lq = p.double().log_softmax(-1), q.double().log_softmax(-1)
    w = (lp.exp() - lq.exp()).clamp_min(0)
    cum = w.cumsum(-1)
    wide = torch.where(w >= 1e-5 * cum[:, -1:].clamp_min(1e-30), w, torch.zeros_like(w)).cumsum(-1)
    u = torch.rand((M, 1), generator=gen, device="cuda", dtype=torch.float64) * wide[:, -1:]
    at = torch.searchsorted(wide, u, right=True).clamp_max(V - 1)
    v = ((cum - 0.5 * w).gather(-1, at) / cum[:, -1:].clamp_min(1e-30)).clamp(0, 0.9999999).float().view(-1).contiguous()
    dlp, rid, rlp = cdsl_op_soft_rows(p, q, d, look, v)
    want = torch.searchsorted(cum, v.double()[:, None] * cum[:, -1:], right=True).clamp_max(V - 1)[:, 0]
    want = torch.where(cum[:, -1] > 0, want, p.argmax(-1))
    assert rid.long().tolist() == want.tolist()
    tok = look[:, 1:].reshape(-1, 1).long()
    ref = lq.gather(-1, tok)[:, 0]
    assert bool(((dlp.double() == ref) | ((dlp.double() - ref).abs() < 2e-5)).all())
    assert float((rlp.double() - lp.gather(-1, want[:, None])[:, 0]).abs().max()) < 2e-5
