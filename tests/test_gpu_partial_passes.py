"""The isometry optimisation's partial passes, forward from the layer that changes and backward down to it, with the
forward intermediates kept, kept for some steps, or recomputed from the steps' checkpoints (which partial passes
leave in place): the trajectories are bit-identical, and so are a gradient taken afterwards and a plan's second
optimisation of another input.  Scheme (a) at chi = 12 and 24 with two and three layers, the side rule (whole forward
passes), scheme (b).

The isometries that the optimisation leaves also stand for themselves: fixed in a plan of their own, a whole forward
pass gives the last ln Z of the trajectory to 1e-12 (the steps above them start their eigensolves elsewhere).
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# kind, chi, steps, layers, options
CASES = {"ising_chi12": ("ising", 12, 12, 2, {}), "ising_chi24": ("ising", 24, 10, 3, {}),
         "ising_side_rule": ("ising", 12, 10, 2, {"side_rule": 1}), "xy_chi12": ("xy", 12, 7, 2, {})}


def _plan(B, kind, chi, n, gib, opt):
    o = B.default_options(checkpoint_gib=gib, max_subspace_iters=200, **opt)
    return B.dtrg_chain_plan_create(4, 4, chi, n, o) if kind == "xy" else B.dtrg_plan_create(2, chi, n, o)


@pytest.mark.parametrize("name", sorted(CASES))
def test_gpu_partial_passes(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_02780_amd import binding as B
    from paper_1912_02780_amd import inputs as I

    kind, chi, n, layers, opt = CASES[name]
    ins = [I.xy_trotter_mpo(0.05), I.xy_trotter_mpo(0.06)] if kind == "xy" else [I.ising_T0(0.43), I.ising_T0(0.425)]
    ins = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in ins]
    out = {}
    for gib in (64.0, 0.002, 0.0):
        print(f"[gpu] partial passes {name} checkpoint budget {gib} GiB", flush=True)
        plan = _plan(B, kind, chi, n, gib, opt)
        runs = []
        for T in ins:
            l0, l1, hist = B.dtrg_isometry_optimize(plan, T, layers, 2, 2)
            g, _ = B.dtrg_hotrg_backward(plan, 1.0)
            assert len(hist) == 4 * layers and hist[-1] == l1
            runs.append((l0, tuple(hist), g.cpu().numpy()))
        out[gib] = runs
    for gib in (0.002, 0.0):
        for a, b in zip(out[64.0], out[gib]):
            assert a[0] == b[0] and a[1] == b[1], gib
            assert np.array_equal(a[2], b[2]), gib
    fixed = [k for k in range(1, n + 1) if plan.step_info(k)["iters"] == -1 and plan.step_info(k)["chi_kept"] < plan.step_info(k)["X"] ** 2]
    assert len(fixed) == layers
    fresh = _plan(B, kind, chi, n, 64.0, opt)
    for k in fixed:
        B.dtrg_plan_fix_isometry(fresh, k, B.dtrg_plan_isometry(plan, k))
    L = B.dtrg_plan_forward(fresh, ins[1])
    print(f"    whole pass on the optimised isometries: {abs(L / out[0.0][1][1][-1] - 1):.1e}", flush=True)
    assert abs(L / out[0.0][1][1][-1] - 1) < 1e-12
