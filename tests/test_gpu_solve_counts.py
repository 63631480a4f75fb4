"""How many Rayleigh-Ritz solves the products of the subspace iteration share (dtrg_plan_step_solves): the schedule
really runs where rr_skip asks for it, on one block and block by block, from cold and warm starts, and with
rr_skip = 0 there is a solve after every product.  A solve follows every product up to the one that takes the
stride up and at most every (rr_skip + 1)-th after it, so that products <= (rr_skip + 1) solves, and where the
sharing has begun there are fewer solves than products.
"""

import ctypes

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# scheme (b), random MPO: chi, steps, block size (24: block by block); scheme (a): Ising at beta_c, chi = 32
CHAINS = {"one_block": (24, 5, 0), "one_block_odd": (13, 5, 0), "blocks": (24, 5, 24), "blocks_chi100": (100, 3, 0)}


def _counts(plan, n):
    c = [plan.step_solves(k) for k in range(1, n + 1)]
    for k, (products, solves) in enumerate(c, start=1):
        assert products == max(0, plan.step_info(k)["iters"])
        assert (solves == 0) == (products == 0) and solves <= products
    return sum(p for p, _ in c), sum(s for _, s in c)


@pytest.mark.parametrize("skip", [0, 1, 3])
@pytest.mark.parametrize("name", sorted(CHAINS))
def test_gpu_chain_solve_counts(name, skip):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding as B
    from paper_1912_02780_amd import inputs as I

    chi, n, block = CHAINS[name]
    print(f"[gpu] solve counts {name} rr_skip {skip}", flush=True)
    M = torch.from_numpy(I.random_mpo(4, 3, 2)).to("cuda:0")
    plan, _ = B.dtrg_chain_forward(M, chi, n, B.default_options(block_size=block, max_subspace_iters=600, rr_skip=skip))
    products, solves = _counts(plan, n)
    print(f"    {products} products, {solves} solves", flush=True)
    assert products <= (skip + 1) * solves
    assert solves == products if skip == 0 else solves < products


def test_gpu_ising_solve_counts_at_criticality():
    """The counts behind the figures of the default schedule: less than half the solves of one per product."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding as B
    from paper_1912_02780_amd import inputs as I

    T0 = torch.from_numpy(I.ising_T0(0.4406868)).to("cuda:0")
    solves = {}
    for skip in (0, 3):
        plan, _ = B.dtrg_hotrg_forward(T0, 32, 30, B.default_options(rr_skip=skip))
        products, solves[skip] = _counts(plan, 30)
        print(f"[gpu] solve counts ising rr_skip {skip}: {products} products, {solves[skip]} solves", flush=True)
        assert products == solves[skip] if skip == 0 else products <= 4 * solves[skip]
    assert solves[3] < 0.5 * solves[0]


def test_gpu_solve_counts_of_steps_that_do_not_iterate():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding as B
    from paper_1912_02780_amd import inputs as I

    T0 = torch.from_numpy(I.ising_T0(0.44)).to("cuda:0")
    plan, _ = B.dtrg_hotrg_forward(T0, 8, 4, B.default_options())
    assert [plan.step_solves(k) for k in range(1, 5)] == [(0, 0)] * 4   # whole spectra
    p, s = ctypes.c_int(), ctypes.c_int()
    for k in (0, 5):
        assert B.lib.dtrg_plan_step_solves(plan._h, k, ctypes.byref(p), ctypes.byref(s)) == B.DTRG_EINVAL
    assert B.lib.dtrg_plan_step_solves(plan._h, 1, None, ctypes.byref(s)) == B.DTRG_EINVAL
