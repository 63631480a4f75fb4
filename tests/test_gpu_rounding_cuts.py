"""Results that rounding decides, held to how much rounding moves them.

Where a cut goes through a pair or multiplet of (nearly) equal eigenvalues, or the kept spectrum has gaps far below the
square root of the broadening, T0bar is not determined by the input: any change of how a kernel rounds (an
order of summation, the shift of the one-sided Jacobi solve) takes it elsewhere within a range that the FP64 oracle has
too.  Fixed bounds on such values say which of the outcomes a build happens to have; here the bound is ten times
the largest movement of the oracle under noise at the path's rounding level: 2^-22 of every step's output for the
mixed formats (their products are good to 2^-22 to 2^-24), 2^-52 of the Gram in FP64.  What is determined stays at
fixed bounds: ln Z, and the part of the gradient with the model's symmetries.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SEEDS = range(6)


def _elem(a, b, floor=1e-6):
    a, b = np.asarray(a), np.asarray(b)
    return float(np.max(np.abs(a - b) / (np.abs(b) + floor * np.abs(b).max())))


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / np.linalg.norm(b))


def _moved(eps, what, f, dist):
    """Largest dist(f() under noise, f()) over the seeds; what: 'project' (a step's output) or 'gram'."""
    from oracle import hotrg as O
    ref, exact, worst = f(), getattr(O, what), 0.0
    for seed in SEEDS:
        rng = np.random.default_rng(seed)

        def project(T, w):
            P, Q, Tn = exact(T, w)
            return P, Q, Tn * (1.0 + eps * rng.standard_normal(Tn.shape))

        def gram(A, B):
            G = exact(A, B)
            N = rng.standard_normal(G.shape)
            return G * (1.0 + eps * (N + N.T))
        setattr(O, what, project if what == "project" else gram)
        try:
            worst = max(worst, dist(f(), ref))
        finally:
            setattr(O, what, exact)
    return worst


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding
    return binding


@pytest.mark.parametrize("beta", [0.48, 0.50, 0.55])
def test_gpu_split_pairs_in_the_ordered_phase(B, beta):
    from oracle import hotrg as O
    from paper_1912_02780_amd import inputs as I
    T0 = I.ising_T0(beta)
    Lo, go, _ = O.lnZ_and_grad(T0, 12, 14)
    moved = _moved(2.0 ** -22, "project", lambda: O.lnZ_and_grad(T0, 12, 14)[1], _elem)

    def symmetric(g):
        images = I.square_group_images(np.asarray(g))
        images = images + [np.flip(x, axis=(0, 1, 2, 3)) for x in images]
        return sum(images) / len(images)
    for prec in ("fp32", "bf16x6"):
        print(f"[gpu] split pairs beta {beta} {prec}", flush=True)
        plan, L = B.dtrg_hotrg_forward(torch.from_numpy(T0).to("cuda:0"), 12, 14, B.default_options(contract=prec))
        g = B.dtrg_hotrg_backward(plan, 1.0)[0].cpu().numpy()
        print(f"    elem {_elem(g, go):.1e} (oracle moves {moved:.1e})  symmetric {_elem(symmetric(g), symmetric(go)):.1e}  "
              f"lnZ {abs(L / Lo - 1):.1e}", flush=True)
        assert abs(L / Lo - 1) < 1e-6
        assert _elem(symmetric(g), symmetric(go)) < 1e-5
        assert _elem(g, go) < 10 * moved


def test_gpu_kept_multiplets_of_the_chain(B):
    from oracle import xtrg as C
    from paper_1912_02780_amd import inputs as I
    M = I.xy_trotter_mpo(0.05)
    fwd = C.chain_forward(M, 25, 7)
    go = C.chain_backward(fwd)
    moved = _moved(2.0 ** -22, "project", lambda: C.chain_backward(C.chain_forward(M, 25, 7)), _rel)
    print("[gpu] kept multiplets chi 25 bf16x6", flush=True)
    plan, L = B.dtrg_chain_forward(torch.from_numpy(M).to("cuda:0"), 25, 7, B.default_options(contract="bf16x6"))
    g = B.dtrg_hotrg_backward(plan, 1.0)[0].cpu().numpy()
    print(f"    rel {_rel(g, go):.1e} (oracle moves {moved:.1e})  lnZ {abs(L / fwd.lnZ_per_tensor - 1):.1e}", flush=True)
    assert abs(L / fwd.lnZ_per_tensor - 1) < 1e-6
    assert _rel(g, go) < 10 * moved


def test_gpu_small_gaps_at_criticality(B):
    from oracle import hotrg as O
    from paper_1912_02780_amd import inputs as I
    T0 = I.ising_T0(0.4406868)
    Lo, go, _ = O.lnZ_and_grad(T0, 16, 20)
    moved = _moved(2.0 ** -52, "gram", lambda: O.lnZ_and_grad(T0, 16, 20)[1], _rel)
    print("[gpu] small gaps at criticality chi 16", flush=True)
    plan, L = B.dtrg_hotrg_forward(torch.from_numpy(T0).to("cuda:0"), 16, 20, B.default_options())
    g = B.dtrg_hotrg_backward(plan, 1.0)[0].cpu().numpy()
    print(f"    rel {_rel(g, go):.1e} (oracle moves {moved:.1e})  lnZ {abs(L / Lo - 1):.1e}", flush=True)
    assert abs(L / Lo - 1) < 1e-12
    assert _rel(g, go) < 10 * moved


@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_gpu_sides_of_mirror_symmetric_inputs(B, seed):
    """Equal sides: their truncated weights differ by rounding (each is one minus a sum of chi' eigenvalues, good to
    2^-53 chi', amplified by the steps), and whichever is taken, ln Z is the plain rule's."""
    from paper_1912_02780_amd import inputs as I
    T0 = torch.from_numpy(I.random_d4_T0(seed, 4)).to("cuda:0")
    print(f"[gpu] sides of mirror symmetric input {seed}", flush=True)
    p0, L0 = B.dtrg_hotrg_forward(T0, 16, 10, B.default_options())
    p1, L1 = B.dtrg_hotrg_forward(T0, 16, 10, B.default_options(side_rule=1))
    info = [p1.step_info(k) for k in range(1, 11)]
    diff = max(abs(s["trunc_weight_left"] - s["trunc_weight_right"]) for s in info)
    print(f"    weights differ by {diff:.1e}, sides {[s['side'] for s in info]}, ln Z {abs(L1 / L0 - 1):.1e}", flush=True)
    assert diff < 1e-10
    assert abs(L1 / L0 - 1) < 1e-12
