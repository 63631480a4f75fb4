"""The products between two Rayleigh-Ritz solves of a block-locked eigensolve apply the whole Chebyshev polynomial,
its first zero (in the block built from the solve) included.  On the eigenvalues that the block leaves out it is
the smallest of all polynomials of that degree with the same value at a wanted pair, so that four products shared by a
solve never gain less than four with a solve each ((G + 2^-45 I) V: the power of the same degree); on chains
whose solves take many products there are fewer of them, where a cycle without that zero takes more.
"""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# MPO, chi, steps
CASES = {"random_chi100": ("random", 100, 3), "xy_chi128": ("xy", 128, 8), "xy_chi96": ("xy_slow", 96, 18)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_gpu_locked_products(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding as B
    from paper_1912_02780_amd import inputs as I

    kind, chi, n = CASES[name]
    M = I.random_mpo(4, 3, 2) if kind == "random" else I.xy_trotter_mpo(0.05 if kind == "xy" else 12.8 / 2 ** 18)
    M = torch.from_numpy(M).to("cuda:0")
    products = {}
    for skip in (0, 3):
        print(f"[gpu] locked products {name} rr_skip {skip}", flush=True)
        plan, _ = B.dtrg_chain_forward(M, chi, n, B.default_options(max_subspace_iters=600, rr_skip=skip))
        info = [plan.step_info(k) for k in range(1, n + 1)]
        assert all(s["resid"] <= 1e-12 for s in info)
        products[skip] = sum(max(0, s["iters"]) for s in info)
    print(f"    products {products}", flush=True)
    assert products[3] < products[0]
