"""Automatic split counts stay within the library's static scratch (128 MiB) for FP64 and FP32 outputs of any size
whose K is below the limit of an accumulation chain: the contraction without allocations takes what the
allocating one takes.  Outputs of 342 to 511 tiles of 128 x 128 are the largest that are cut (three chunks of them
are 135 to 200 MB in FP64).  Against float64, at 1e-13 and 2e-6 of the norm as for the other contractions.
"""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(2560, 2560, 1024), (2816, 2944, 2000), (2368, 2400, 4000), (511, 65408, 130)])
def test_gpu_noalloc_takes_the_automatic_choice(prec, shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding as B

    M, N, K = shape
    dt = torch.float64 if prec == "fp64" else torch.float32
    g = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    A = torch.randn(M, K, generator=g, device="cuda:0", dtype=dt)
    Bm = torch.randn(N, K, generator=g, device="cuda:0", dtype=dt)
    print(f"[gpu] noalloc choice {prec} {shape}", flush=True)
    C = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda:0")
    B.dtrg_contract(prec, A, Bm, C, noalloc=True)
    D = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda:0")
    B.dtrg_contract(prec, A, Bm, D)
    assert torch.equal(C, D)
    ref = A.cpu().double()[:64] @ Bm.cpu().double().T
    assert float((C[:64].cpu() - ref).norm() / ref.norm()) < (1e-13 if prec == "fp64" else 2e-6)
