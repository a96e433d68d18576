"""The bf16 projection kernel at the edges of its tiles: row counts around the
tile heights (16, 32, 48, 64, 128, 160, 256), ragged columns, K of whole and
half stages, K splits, both ends of the row range, weights that are not
16-byte aligned, and the static scratch's limited split.  Reference: float64.

Tolerance: A = hi + lo to 2^-17 per element, so a K-term sum is off by at most
2^-17 sum |a||w| (random signs: about 2^-17 sqrt(K) |a||w|), plus fp32
accumulation; relative to the largest output both are below 5e-6."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 64, 64), (1, 8200, 1056), (15, 1000, 96), (16, 16384, 1024), (17, 3072, 1024), (31, 130, 4096), (33, 2048, 2048),
    (47, 777, 160), (48, 12288, 1024), (49, 2048, 8192), (64, 11264, 2048), (65, 515, 224), (80, 2048, 2080),
    (81, 16384, 512), (97, 6144, 1024), (127, 255, 64), (128, 22016, 1024), (129, 257, 1056), (159, 3000, 2048),
    (160, 256, 32), (161, 4096, 4096), (255, 6144, 992), (257, 1025, 2048), (320, 16384, 512), (500, 2111, 1088),
    (800, 4096, 2048), (1023, 2050, 544), (2049, 4100, 288),
]


def _operands(M, N, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn((M, K), generator=g, device="cuda")
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.02).bfloat16()
    return a, w


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_projection_at_tile_edges(M, N, K):
    from paper_2412_10418_amd.binding import cdsl_op_gemm
    a, w = _operands(M, N, K, M * 7 + N * 3 + K)
    # rows and columns past the product's edge must not be written
    buf = torch.full((M * N + 4096,), 7.0, device="cuda")
    got = cdsl_op_gemm(a, w, buf[:M * N].view(M, N))
    ref = torch.matmul(a.double(), w.double().t())
    assert float((got.double() - ref).abs().max() / ref.abs().max()) < 5e-6
    assert bool((buf[M * N:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [(1, 200, 64), (20, 1000, 96), (80, 2048, 1024), (300, 1030, 576)])
@pytest.mark.parametrize("skew", [1, 2, 4])
def test_projection_with_unaligned_weights(M, N, K, skew):
    """Weights at an address that is a multiple of 2, 4 or 8 bytes only: the
    same product, bit for bit."""
    from paper_2412_10418_amd.binding import cdsl_op_gemm
    a, w = _operands(M, N, K, 5)
    flat = torch.zeros(N * K + 8, dtype=torch.bfloat16, device="cuda")
    flat[skew:skew + N * K] = w.reshape(-1)
    moved = flat[skew:skew + N * K].view(N, K)
    assert moved.data_ptr() % 16 != 0
    assert torch.equal(cdsl_op_gemm(a, moved), cdsl_op_gemm(a, w))


@pytest.mark.parametrize("M,N,K", [(1, 64, 1 << 25), (33, 64, (1 << 24) + 32), (64, 3, 1 << 25)])
def test_projection_over_tiles_beyond_two_gib(M, N, K):
    """Rows so long that a tile of either operand spans 2 GiB or more.  Tolerance: a split sums at most K / 32 MFMA
    steps per plane in fp32, each off by 2^-24 of the running sum: 2^-24 sqrt(2 K / 32), below 1e-4, in units of
    the outputs' size."""
    from paper_2412_10418_amd.binding import cdsl_op_gemm
    g = torch.Generator(device="cuda").manual_seed(K + M)
    a = torch.empty((M, K), device="cuda").normal_(0.0, 1.0, generator=g)
    w = torch.empty((N, K), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    ref = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    for k in range(0, K, 1 << 22):
        ref += torch.matmul(a[:, k:k + (1 << 22)].double(), w[:, k:k + (1 << 22)].double().t())
    got = cdsl_op_gemm(a, w)
    assert float((got.double() - ref).abs().max() / ref.abs().max()) < 1e-4


@pytest.mark.parametrize("M,V,K,kk", [(1, 1000, 64, 16), (16, 32000, 1024, 5), (48, 4099, 96, 3), (80, 32000, 512, 0),
                                      (128, 1030, 256, 8), (161, 2000, 1024, 5), (300, 50257, 160, 2)])
def test_head_rows_over_the_tile_shapes(M, V, K, kk):
    """Row statistics of each tile shape against float64 logits; every weight
    row appears twice, so every place of the top-k is a tie by columns."""
    from paper_2412_10418_amd.binding import cdsl_op_lm_head_rows
    a, w = _operands(M, V, K, 11)
    w = w[torch.arange(V, device="cuda") // 2 * 2 % V].contiguous()
    gather = torch.randint(0, V, (M,), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda",
                           dtype=torch.int32)
    lp, amax, ids, tlp = cdsl_op_lm_head_rows(a, w, gather, kk)
    z = torch.matmul(a.double(), w.double().t())
    lsm = z.log_softmax(-1)
    assert float((lp.double() - lsm.gather(-1, gather.long()[:, None])[:, 0]).abs().max()) < 1e-4
    top = z.max(-1)
    gap = z.topk(3, -1).values
    clear = gap[:, 0] - gap[:, 2] > 1e-3     # the two equal columns of the maximum stand clear of the third
    assert bool((amax.long() == top.indices)[clear].all() | (z.gather(-1, amax.long()[:, None])[:, 0] == top.values)[clear].all())
    assert bool((amax % 2 == 0)[clear].all())   # the lower of the two equal columns
    if kk:
        ref = lsm.topk(kk, -1).values
        assert float((tlp.double() - ref).abs().max()) < 1e-4
        picked = lsm.gather(-1, ids.long())
        assert float((picked - ref).abs().max()) < 1e-4
        assert all(len(set(r)) == kk for r in ids.tolist())


def test_static_scratch_takes_a_smaller_split_than_the_plan():
    """A shape that the static scratch takes although the plan's own split
    needs more than it holds: a smaller split runs, with the same accuracy."""
    from paper_2412_10418_amd import binding as bd
    M, N, K = STATIC_SHAPE
    assert bd.lib().cdsl_op_gemm_workspace(M, N, K, bd.CDSL_BF16) > (64 << 20)
    a, w = _operands(M, N, K, 17)
    c = torch.empty((M, N), device="cuda")
    rc = bd.lib().cdsl_op_gemm_static(a.data_ptr(), w.data_ptr(), c.data_ptr(), M, N, K, bd.CDSL_BF16,
                                      bd.CDSL_EPI_STORE, torch.cuda.current_stream().cuda_stream)
    assert rc == bd.CDSL_OK
    ref = torch.matmul(a.double(), w.double().t())
    assert float((c.double() - ref).abs().max() / ref.abs().max()) < 5e-6


STATIC_SHAPE = (716, 2830, 12000)


@pytest.mark.parametrize("M,N,K", [(1, 33, 16), (15, 384, 48), (17, 65, 80), (16, 2048, 256), (33, 1000, 128), (130, 777, 640),
                                   (512, 2047, 1024), (500, 1030, 336)])
def test_fp32_projection_at_tile_edges(M, N, K):
    """fp32 weights: fp32 sums (K terms: below 2^-24 sqrt(K) of the row times
    column norms, far inside 2e-6 of the largest output), operands at any
    4-byte alignment, and every row the same bits whatever the batch."""
    from paper_2412_10418_amd.binding import cdsl_op_gemm
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    flat = torch.randn(M * K + N * K + 8, generator=g, device="cuda")
    a, w = flat[1:1 + M * K].view(M, K), flat[3 + M * K:3 + M * K + N * K].view(N, K)
    buf = torch.full((M * N + 4096,), 7.0, device="cuda")
    got = cdsl_op_gemm(a, w, buf[:M * N].view(M, N))
    ref = torch.matmul(a.double(), w.double().t())
    assert float((got.double() - ref).abs().max() / ref.abs().max()) < 2e-6
    assert bool((buf[M * N:] == 7.0).all())
    for r in (0, M // 2, M - 1):
        assert torch.equal(cdsl_op_gemm(a[r:r + 1].clone(), w), got[r:r + 1])
