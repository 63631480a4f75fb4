"""FP32 contractions whose output fills the chip by itself (512 tiles of 128 x 128 or more) and whose K is below the
limit of an accumulation chain run in one chunk: the automatic choice gives the bits of the run with one, in every
layout.  (In several chunks the sums associate differently, and a partial buffer and a pass over it come on top.)
"""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4096, 4096, 2048), (8192, 2048, 1536), (4096, 2048, 4096), (4000, 3000, 1100)])
def test_gpu_fp32_large_output_in_one_chunk(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding as B

    M, N, K = shape
    g = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    A = torch.randn(M, K, generator=g, device="cuda:0")
    Bm = torch.randn(N, K, generator=g, device="cuda:0")
    for akm in (False, True):
        for bkm in (False, True):
            print(f"[gpu] fp32 one chunk {shape} {akm} {bkm}", flush=True)
            a = A.T.contiguous() if akm else A
            b = Bm.T.contiguous() if bkm else Bm
            auto = B.dtrg_contract("fp32", a, b, torch.empty(M, N, device="cuda:0"), a_kmajor=akm, b_kmajor=bkm)
            one = [B.dtrg_contract("fp32", a, b, torch.empty(M, N, device="cuda:0"), a_kmajor=akm, b_kmajor=bkm,
                                   tile=t, splits=1) for t in (1, 2)]
            assert any(torch.equal(auto, c) for c in one)
