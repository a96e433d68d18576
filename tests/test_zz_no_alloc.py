"""cdsl_op_gemm_static (the projection for callers that cannot allocate)
through the C ABI: calls in a row, with and without a K split, each equal to
cdsl_op_gemm with a caller workspace (the same kernels, so bitwise) and
within fp32 accuracy of float64; shapes whose workspace fits are taken, one
whose planes of A alone exceed the static scratch is refused."""
import ctypes

import numpy as np
import pytest
import torch

import cdsl_inputs as ci

pytestmark = pytest.mark.gpu


def _operands(M, N, K, seed):
    rng = np.random.default_rng([seed, M, N, K])
    a = rng.uniform(-1, 1, (M, K)).astype(np.float32)
    b = ci.round_to_bf16(rng.uniform(-1, 1, (N, K)).astype(np.float32))
    tb = torch.from_numpy(ci.f32_to_bf16_bits(b).view(np.int16)).cuda().view(torch.bfloat16)
    return a, b, torch.from_numpy(a).cuda(), tb


def _static(ta, tb, M, N, K):
    from paper_2412_10418_amd import binding as bd
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    rc = bd.lib().cdsl_op_gemm_static(ta.data_ptr(), tb.data_ptr(), C.data_ptr(), M, N, K, bd.CDSL_BF16,
                                      bd.CDSL_EPI_STORE, torch.cuda.current_stream().cuda_stream)
    return rc, C


def test_static_scratch_gemm_matches_the_workspace_entry_point():
    from paper_2412_10418_amd import binding as bd
    # an unsplit call, one whose K is split over several planes (42 MB of
    # workspace), then smaller ones on the same scratch, split and not
    for M, N, K, split in [(800, 4096, 4096, False), (400, 4096, 11008, True), (80, 2048, 8192, True),
                           (80, 3072, 2048, False)]:
        print(f"static-scratch gemm {M}x{N}x{K}", flush=True)
        need = bd.lib().cdsl_op_gemm_workspace(M, N, K, bd.CDSL_BF16)
        assert need <= (64 << 20)
        if split:   # the hi / lo planes of A and at least two planes of the product
            assert need >= 4 * M * K + 8 * M * N
        a, b, ta, tb = _operands(M, N, K, 31)
        ref = bd.cdsl_op_gemm(ta, tb)
        rc, got = _static(ta, tb, M, N, K)
        assert rc == bd.CDSL_OK, bd.lib().cdsl_last_error(None)
        torch.cuda.synchronize()
        assert torch.equal(got, ref)
        exact = a.astype(np.float64) @ b.astype(np.float64).T
        err = np.max(np.abs(got.cpu().numpy() - exact)) / max(1.0, np.max(np.abs(exact)))
        assert err < 5e-6, err


@pytest.mark.parametrize("M,N,K", [(426, 12288, 4096), (500, 22016, 4096), (833, 4096, 11008)])
def test_static_scratch_takes_every_shape_whose_planes_fit(M, N, K):
    """The first two need no K split, so their workspace is far below the scratch's size; the third's planes of A leave
    room for a small split only.  Bitwise cdsl_op_gemm's result where its workspace fits, else as accurate (the
    tolerance of the calls above)."""
    from paper_2412_10418_amd import binding as bd
    g = torch.Generator(device="cuda").manual_seed(M)
    ta = torch.randn((M, K), generator=g, device="cuda")
    tb = (torch.randn((N, K), generator=g, device="cuda") * 0.02).bfloat16()
    rc, got = _static(ta, tb, M, N, K)
    assert rc == bd.CDSL_OK, bd.lib().cdsl_last_error(None)
    if bd.lib().cdsl_op_gemm_workspace(M, N, K, bd.CDSL_BF16) <= (64 << 20):
        assert torch.equal(got, bd.cdsl_op_gemm(ta, tb))
    ref = torch.matmul(ta.double(), tb.double().t())
    assert float((got.double() - ref).abs().max() / ref.abs().max()) < 5e-6


def test_static_scratch_refuses_a_shape_beyond_its_size():
    from paper_2412_10418_amd import binding as bd
    M, N, K = 4160, 4096, 4096        # 65 MiB of hi / lo planes alone
    assert bd.lib().cdsl_op_gemm_workspace(M, N, K, bd.CDSL_BF16) > (64 << 20)
    a, b, ta, tb = _operands(M, N, K, 32)
    rc, got = _static(ta, tb, M, N, K)
    assert rc == bd.CDSL_ERANGE
    assert b"static scratch" in bd.lib().cdsl_last_error(None)
    assert torch.isnan(got).all()
