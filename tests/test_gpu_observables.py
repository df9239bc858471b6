"""GPU parity of U(t, t0) and the averaged probabilities from given eigenpairs,
single and batched, at the sizes where their kernels change form: D^2 below and
above 64, 128 and 256 (elements per group of threads), D T around 128 and 256,
orders around the column chunks.  Against the oracle on the oracle's own
eigenpairs; tolerance M eps times 100 (sums of M terms of modulus at most one)."""
import numpy as np
import pytest

import oracle
from workloads import Problem, random_problem
from gpu_util import require_gpu, to_dev_cm, log

pytestmark = pytest.mark.gpu


def _problem(D, N, seed):
    if D > 1:
        return random_problem(D, N, seed=seed)
    return Problem(E=np.array([[0.4]]), omega=[1.3] * len(N), N=N, axis=[0], harm=[1], V=[np.array([[0.2 + 0.1j]])])


@pytest.mark.parametrize("D,N,T", [(1, (20,), 3), (2, (64,), 7), (2, (127, 0), 1), (3, (5, 4), 33), (8, (8, 8), 5),
                                   (11, (3, 3), 4), (12, (3, 3), 4), (16, (16,), 3), (17, (15,), 3), (64, (2,), 2)])
def test_evolve_and_avg_prob_forms(D, N, T):
    torch, mmf = require_gpu()
    p = _problem(D, N, seed=D)
    H = oracle.build_floquet(p)
    w, Phi = oracle.eigh(H)
    M = H.shape[0]
    log(f"observables D={D} M={M} T={T}")
    ts = np.linspace(0.3, 5.0, T)
    dp = mmf.DeviceProblem(p)
    Pt, wg = to_dev_cm(torch, Phi), torch.from_numpy(w).cuda()
    U = mmf.evolve(dp, Pt, wg, 0.1, torch.from_numpy(ts).cuda())
    P, _ = mmf.avg_prob(dp, Pt, wg)
    torch.cuda.synchronize()
    tol = 100 * M * np.finfo(float).eps
    assert np.abs(U.cpu().numpy() - oracle.evolve(p, Phi, w, 0.1, ts)).max() <= tol
    assert np.abs(P.cpu().numpy() - oracle.avg_prob(p, Phi)).max() <= tol


@pytest.mark.parametrize("Ds,T", [((2, 3, 8), 16), ((1, 2, 2), 64), ((2, 9, 16), 8), ((4, 17, 33), 5), ((64, 2, 5), 32)])
def test_batched_observables_forms(Ds, T):
    """Mixed D in one batch (the largest D picks the kernels' form) against the
    oracle's U and P on the eigenpairs the batch returns."""
    torch, mmf = require_gpu()
    from paper_2005_03426_amd.batch import BatchPlan
    ps = [_problem(D, (3 + k, 2) if D < 20 else (1,), seed=50 + D) for k, D in enumerate(Ds)]
    ts = np.linspace(0.0, 4.0, T)
    log(f"batched observables D={Ds} T={T}")
    plan = BatchPlan(ps, ts, t0=0.2, graph=False)
    plan.run()
    plan.synchronize()
    for p, r in zip(ps, plan.results()):
        assert int(r["info"].item()) == 0
        w, Phi = r["w"].cpu().numpy(), r["Pt"].T.cpu().numpy()
        tol = 100 * len(w) * np.finfo(float).eps
        assert np.abs(r["U"].cpu().numpy() - oracle.evolve(p, Phi, w, 0.2, ts)).max() <= tol
        assert np.abs(r["P"].cpu().numpy() - oracle.avg_prob(p, Phi)).max() <= tol
