"""Roots of matrices of at most 128 x 128 (the whole iteration in one
workgroup) at the edges of its 32 x 32 blocks, for every kind of product
program (powers of two, odd, mixed bits), both start scalings and both kinds
of damping, against the oracle; a zero-iteration start, a NOT_PD matrix and an
escalated one; and a mixed call, whose small matrices must come out bit for
bit as in a call of their own.

Tolerance (relative, Frobenius), u = 2^-24: M0 = z (A + eps I) rounded to fp32 is
a perturbation of u that the root amplifies by kappa / p (or by that of the first
update, if larger: 66000 at p = 16, where it takes eigenvalues of 8.5 to 3e-4); X
is rounded at each of the iters products; and the last residual r (per element, so at most n r in norm)
is not followed by another update of X, which leaves n r / p:
  err <= 2 (kappa / p + iters) u + n r / p,
the factor 2 for the affine terms and z^(1/p).  A product without the third plane
or without the three products of order 2^-16 is further off
(emulated in numpy, p = 4, kappa 40: 4.6e-6 to 7.2e-6 against a limit of 2.0e-6).
"""
import numpy as np
import pytest

import oracle.shampoo_oracle as O
from tests.gpu_util import gpu_env, host, rel, say, spd, to_dev
from tests.test_gpu_warm import drift_case, warm_roots

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, B, dev = gpu_env()
    h = B.shampoo_create(0)
    yield torch, B, dev, h
    B.shampoo_destroy(h)


def _roots(env, mats, **params):
    torch, B, dev, h = env
    As = [to_dev(torch, a.astype(np.float32), dev) for a in mats]
    Xs = [torch.full_like(a, float("nan")) for a in As]
    prm = B.shampoo_root_params_default(**params)
    ws = torch.empty(B.shampoo_inv_root_workspace_bytes([a.shape[0] for a in mats], prm.precision),
                     dtype=torch.uint8, device=dev)
    info = torch.zeros(8 * len(mats), dtype=torch.int32, device=dev)
    B.shampoo_inv_root_batched(h, As, Xs, prm, ws, info)
    torch.cuda.synchronize()
    return [host(x) for x in Xs], B.decode_root_info(info)


def bound(kappa, p, n, info):
    # the first update takes a largest eigenvalue of (p + 1) / 2 down to `low`
    # in a product of matrices of norm (1 + 1/p)^p and (p + 1) / 2
    low = ((p + 1) / (2 * p)) ** p * (p + 1) / 2
    kappa = max(kappa, (1 + 1 / p) ** p * (p + 1) / 2 / low)
    return 2 * (kappa / p + info["iters"]) * 2.0 ** -24 + n * info["resid"] / p


SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128]
KAPPA = 40.0


@pytest.mark.parametrize("p", [1, 2, 3, 4, 6, 7, 8, 16])
@pytest.mark.parametrize("scaling", [0, 1])
def test_sizes_and_orders(env, p, scaling):
    torch, B, dev, h = env
    mats = [spd(n, KAPPA, 100 + n) for n in SIZES]
    say(f"small roots p={p} scaling={scaling}")
    xs, info = _roots(env, mats, p=p, scaling=scaling, precision=B.PRECISION_FP32)
    for a, x, i in zip(mats, xs, info):
        n = a.shape[0]
        assert i["status"] == B.ROOT_CONVERGED, (n, i)
        assert np.array_equal(x, x.T)
        err = rel(x, O.inv_root(a.astype(np.float64), p, 1e-6)[0])
        assert err <= bound(KAPPA, p, n, i), (n, err, i)


@pytest.mark.parametrize("p", [4, 7])
def test_launch_shapes_same_bits(env, p):
    """A matrix alone (a launch shaped for its blocks) and beside larger ones."""
    torch, B, dev, h = env
    mats = [spd(n, KAPPA, 100 + n) for n in SIZES]
    say(f"small roots launch shapes p={p}")
    xs, info = _roots(env, mats, p=p)
    for a, x, i in zip(mats, xs, info):
        (y,), (k,) = _roots(env, [a], p=p)
        assert np.array_equal(x, y) and i == k, a.shape
    for k in (3, 6, 9):  # the largest of 32, 64 and 96 rows and those below it
        ys, _ = _roots(env, mats[:k + 1][::-1] * 3, p=p)
        for j, y in enumerate(ys):
            assert np.array_equal(y, xs[k - j % (k + 1)]), (k, j)


@pytest.mark.parametrize("n", [16, 32, 64])
@pytest.mark.parametrize("p", [6, 8])
def test_rounding_does_not_accumulate_near_identity(env, n, p):
    """Root mean square error over 24 well-conditioned matrices (kappa 9): the
    roundings of M0 (amplified by kappa / p), of X in each iteration and of the
    result, taken as independent and half a unit each.  Products of iterates
    near I that lose their small terms add the same error to every eigenvalue
    (5 to 7 units here)."""
    say(f"small roots rms n={n} p={p}")
    mats = [spd(n, 9.0, 1000 + k) for k in range(24)]
    torch, B, dev, h = env
    xs, info = _roots(env, mats, p=p, precision=B.PRECISION_FP32)
    e = np.array([rel(x, O.inv_root(a.astype(np.float64), p, 1e-6)[0]) for a, x in zip(mats, xs)])
    limit = 0.5 * (9.0 / p + np.sqrt(max(i["iters"] for i in info)) + 1) * 2.0 ** -24
    assert np.sqrt((e ** 2).mean()) <= limit, (float(np.sqrt((e ** 2).mean())), limit)


def test_relative_damping_asymmetric_input(env):
    """The root of the symmetric part, scaled damping, odd sizes."""
    torch, B, dev, h = env
    r = np.random.default_rng(5)
    mats = [spd(n, KAPPA, n) + 1e-3 * r.standard_normal((n, n)) for n in (5, 40, 101)]
    say("small roots relative damping")
    xs, info = _roots(env, mats, p=4, eps=1e-2, eps_relative=1, precision=B.PRECISION_FP32)
    for a, x, i in zip(mats, xs, info):
        a = a.astype(np.float32).astype(np.float64)
        s = 0.5 * (a + a.T)
        lam = np.linalg.eigvalsh(s)[-1]
        assert abs(i["lambda_max"] / lam - 1) < 0.05
        w = O.inv_root(s, 4, i["eps_eff"])[0]
        assert rel(x, w) <= bound(KAPPA, 4, len(a), i), (len(a), rel(x, w), i)


def test_outcomes_and_mixed_call(env):
    torch, B, dev, h = env
    n = 70
    ill = spd(n, 1e7, 3)
    bad = spd(n, 10.0, 4)
    bad[3, 3] = -1.0
    nan = spd(n, 10.0, 4)
    nan[1, 2] = np.nan
    # z A = I: p = 1 and a 1 x 1 matrix start converged
    small = [np.array([[2.0]], np.float32), spd(n, 20.0, 6), ill, bad, nan, spd(128, 30.0, 7), spd(33, 5.0, 8)]
    big = [spd(200, 30.0, 9), spd(300, 1e7, 10)]
    say("small roots outcomes")
    alone, ia = _roots(env, small, p=4)
    mixed, im = _roots(env, big[:1] + small[:4] + big[1:] + small[4:], p=4)
    order = [1, 2, 3, 4, 6, 7, 8]
    for k, (x, i) in enumerate(zip(alone, ia)):
        m, j = mixed[order[k]], im[order[k]]
        assert i == j or (np.isnan(i["resid"]) and np.isnan(j["resid"])), (k, i, j)
        if k not in (3, 4):
            assert np.array_equal(x, m), k
    assert ia[2]["precision"] == 64 and rel(alone[2], O.inv_root(ill.astype(np.float64), 4, 1e-6)[0]) <= 5e-3
    assert ia[3]["status"] == B.ROOT_NOT_PD and ia[4]["status"] == B.ROOT_NOT_PD
    for k in (0, 1, 5, 6):
        a = small[k].astype(np.float64)
        assert ia[k]["precision"] == 32
        assert rel(alone[k], O.inv_root(a, 4, 1e-6)[0]) <= bound(30, 4, len(a), ia[k]), k
    assert rel(mixed[0], O.inv_root(big[0].astype(np.float64), 4, 1e-6)[0]) <= 1e-4
    # zero iterations: 1 x 1, p = 1, Frobenius scaling: z A = 1 exactly
    x, i = _roots(env, [np.array([[4.0]], np.float32)], p=1, eps=0.0, scaling=0, precision=B.PRECISION_FP32)
    assert i[0]["iters"] == 0 and float(x[0][0, 0]) == 0.25


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,p,tol,iters", [(96, 4, 1e-3, 1), (33, 2, 1e-3, 1), (128, 3, 1e-3, 1), (96, 4, 1e-6, 2)])
def test_warm_call_of_small_matrices(env, prec, n, p, tol, iters):
    """A warm call whose matrices are all small returns the kept warm result,
    in whichever buffer its last iterate is.  The residuals (oracle: 3e-3 to
    1.4e-2 before, at most 3.4e-4 after one iteration) are far from tol 1e-3.
    Bounds as in the warm tests at larger sizes; the start X0 is 1.8e-3 or
    more from the limit, so X0 itself would fail the second."""
    say(f"small warm roots n={n} p={p} tol={tol} prec={prec}")
    A, X0 = drift_case(n, 1e2, 3e-3, p, 7 * n + p)
    (X,), (i,), (w,) = warm_roots(env, [A], [X0], p=p, eps=1e-6, tol=tol, precision=prec)
    ref = O.coupled_newton_warm(A, p, X0, eps=1e-6, tol=tol)
    assert not ref["warm_aborted"] and ref["warm_iters"] == iters
    assert w[0] == 1 and i["status"] in (0, 1), (w, i)
    assert w[1] == iters if iters == 1 else abs(int(w[1]) - iters) <= 1, w
    e = rel(X, ref["X"])
    assert e <= 1e-3 and e < 0.2 * rel(ref["X"], X0), (e, w)


@pytest.mark.parametrize("count", [1, 40])
@pytest.mark.parametrize("n", [33, 128, 200])
@pytest.mark.parametrize("scaling", [0, 1])
def test_inverses_of_huge_statistics(env, n, count, scaling):
    """p = 1 and eigenvalues of 2^118 to 2^121: X is around 2^-120 and its
    iterate must not lose bits for that.  Same accuracy as for eigenvalues of 1
    to 8 (within a half and 2^-21 for the other rounding of the scaled input);
    one matrix and 40 (every launch form), and a warm call that keeps X0."""
    torch, B, dev, h = env
    say(f"inverses of huge statistics n={n} count={count} scaling={scaling}")
    errs = []
    for sc in (1.0, 2.0 ** 118):
        A = (spd(n, 8.0, n).astype(np.float64) * sc).astype(np.float32)
        xs, info = _roots(env, [A] * count, p=1, scaling=scaling, eps=0.0, precision=B.PRECISION_FP32)
        assert all(i["status"] in (B.ROOT_CONVERGED, B.ROOT_STAGNATED) for i in info)
        want = np.linalg.inv(A.astype(np.float64))
        errs.append(max(rel(x, want) for x in (xs[0], xs[-1])))
    assert errs[1] <= 1.5 * errs[0] + 2.0 ** -21, errs
    (X,), (i,), (w,) = warm_roots(env, [A], [want.astype(np.float32)], p=1, eps=0.0, tol=1e-6, precision=1)
    assert w[0] == 1 and rel(X, want) <= 1.5 * errs[0] + 2.0 ** -21, (w, i, rel(X, want))
