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


def _us(f, n=8, runs=9):
    """The median over runs of n calls' GPU time per call, enqueued behind a busy stream."""
    ts = []
    f()
    for _ in range(runs):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda._sleep(2000000)
        a.record()
        for _ in range(n):
            f()
        b.record()
        torch.cuda.synchronize()
        ts.append(a.elapsed_time(b) * 1e3 / n)
    return sorted(ts)[runs // 2]


@pytest.mark.parametrize("M,V,K", [(1, 128256, 1024), (24, 128256, 1024), (16, 50257, 2048)])
def test_head_places_cost_little_beside_the_product(M, V, K):
    """Eight places of the top-k are one round over the tiles' lists, not eight: at these few rows the head with them
    takes at most 1.8 times the head without (8 rounds that read every list again took 2.8 times)."""
    from paper_2412_10418_amd.binding import cdsl_op_lm_head_rows
    g = torch.Generator(device="cuda").manual_seed(V)
    a = torch.randn((M, K), generator=g, device="cuda")
    w = torch.empty((V, K), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    ids = torch.zeros(M, dtype=torch.int32, device="cuda")
    assert _us(lambda: cdsl_op_lm_head_rows(a, w, ids, 8)) < 1.8 * _us(lambda: cdsl_op_lm_head_rows(a, w, ids, 0))


@pytest.mark.parametrize("kk", [1, 7, 16])
@pytest.mark.parametrize("every", [1, 16, 786])
def test_head_places_with_the_best_entries_in_few_tiles(kk, every):
    """The columns of every every-th tile of 64 are raised far above the rest: the best entries lie in all tiles, in
    those of one sixteenth of the merge's threads (more than its list holds at kk = 16), or in one."""
    from paper_2412_10418_amd.binding import cdsl_op_lm_head_rows
    M, V, K = 5, 50257, 256
    g = torch.Generator(device="cuda").manual_seed(kk)
    a = 1.0 + 0.1 * torch.randn((M, K), generator=g, device="cuda")
    w = torch.empty((V, K), device="cuda").normal_(0.0, 0.02, generator=g)
    w[(torch.arange(V, device="cuda") // 64) % every == 3 % every] += 0.25
    w = w.bfloat16()
    lp, amax, ids, tlp = cdsl_op_lm_head_rows(a, w, torch.zeros(M, dtype=torch.int32, device="cuda"), kk)
    lsm = torch.matmul(a.double(), w.double().t()).log_softmax(-1)
    ref = lsm.topk(kk, -1).values
    assert float((tlp.double() - ref).abs().max()) < 1e-4
    assert float((lsm.gather(-1, ids.long()) - ref).abs().max()) < 1e-4
    assert all(len(set(r)) == kk for r in ids.tolist())
    assert torch.equal(amax, ids[:, 0])


def _order(row, k):
    """The k best ids: value descending, id ascending, NaN never."""
    ids = np.flatnonzero(~np.isnan(row))
    return ids[np.lexsort((ids, -row[ids]))][:k]


@pytest.mark.parametrize("M,V", [(3, 5), (9, 64), (6, 1023), (5, 4097), (4, 8193), (3, 16387), (400, 8200), (2, 70001),
                                 (2, 150001), (1, 300007), (7, 2041), (600, 20001)])
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


@pytest.mark.parametrize("V", [1, 2, 3, 5, 63, 1023, 4098, 20001])
@pytest.mark.parametrize("kk", [0, 1, 2, 16])
def test_logit_rows_without_a_finite_entry(V, kk):
    """Rows at each alignment (they begin and end inside a 16-byte slot) whose entries are all -inf, or NaN up to a
    place and -inf from there: the lowest ids of the -inf entries, in order."""
    from paper_2412_10418_amd.binding import cdsl_op_logit_rows
    z = np.full((8, V), -np.inf, np.float32)
    for m in range(4, 8):
        z[m, :min(m - 3, V - 1)] = np.nan
    kk = min(kk, V)
    _, amax, tk, _ = (t.cpu().numpy() for t in
                      cdsl_op_logit_rows(torch.from_numpy(z).cuda(), torch.zeros(8, dtype=torch.int32).cuda(), kk))
    for m in range(8):
        want = _order(z[m], max(kk, 1))
        assert amax[m] == want[0]
        assert list(tk[m][:min(kk, len(want))]) == list(want[:kk])


@pytest.mark.parametrize("V", [20001, 128256])
def test_logit_rows_with_the_best_entries_in_few_threads(V):
    """Every entry of one slot of four in 32 (the slots of one group of threads) lies above all others: more entries
    reach the bound than a workgroup lists."""
    from paper_2412_10418_amd.binding import cdsl_op_logit_rows
    rng = np.random.default_rng(V)
    z = rng.standard_normal((6, V)).astype(np.float32)
    z[:, np.arange(V) // 4 % 32 == 5] += 100.0
    z[5] = np.round(z[5])
    _, amax, tk, _ = (t.cpu().numpy() for t in
                      cdsl_op_logit_rows(torch.from_numpy(z).cuda(), torch.zeros(6, dtype=torch.int32).cuda(), 16))
    for m in range(6):
        assert list(tk[m]) == list(_order(z[m], 16)) and amax[m] == tk[m, 0]


@pytest.mark.parametrize("M,V", [(384, 128256), (900, 32000), (100, 1000)])
def test_logit_rows_time_depends_on_neither_places_nor_values(M, V):
    """Sixteen places are one round, not sixteen (which took 3.5 to 10 times as long as one place, now 1.9 to 2.6), and rows of one
    value or with all but three entries at -inf cost no more than others (up to 2.3 times before)."""
    from paper_2412_10418_amd.binding import cdsl_op_logit_rows
    g = torch.Generator(device="cuda").manual_seed(V)
    z = torch.randn((M, V), generator=g, device="cuda") * 3
    masked = torch.full((M, V), -float("inf"), device="cuda")
    masked[:, V // 2:V // 2 + 3] = 1.0
    ids = torch.zeros(M, dtype=torch.int32, device="cuda")
    us = {n: _us(lambda: cdsl_op_logit_rows(x, ids, kk))
          for n, x, kk in [("one", z, 1), ("5", z, 5), ("16", z, 16), ("const", torch.ones_like(z), 5), ("masked", masked, 5)]}
    print(us, flush=True)
    assert us["16"] < 3.3 * us["one"] and us["const"] < 1.5 * us["5"] and us["masked"] < 1.5 * us["5"]


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
