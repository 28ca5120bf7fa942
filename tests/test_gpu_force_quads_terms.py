"""Every term of the FP32 sums on the matrix cores, for the force in both radial bases and for
the jerk, at the edges of their layout: odd and even nmax (pairs of orders), every lmax bucket
with lmax at and below it (one or two coefficient registers per pair), partly filled
wavefronts.

The coefficients are not those of a model, whose high orders vanish in the sum: each is scaled
so that its own term has a root mean square of about 1 over the points, with random signs.  A
term that is left out, doubled or multiplied by another order changes the result by about 1 (in
root mean square); the FP32 rounding of up to 4725 terms of size 1 at a relative error of about
3e-6 each (a recurrence over 20 orders, one over 14 rows) is 3e-6 sqrt(4725) = 2e-4, and a few
times that for derivatives.  The bound between them is 0.02 for the force and 0.05 for the jerk."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CUTOFFS = [(0, 0), (1, 0), (1, 1), (2, 2), (3, 3), (4, 5), (1, 7), (6, 8), (9, 9), (2, 11), (11, 12), (19, 13),
           (20, 14)]
MIXED = 1
NS = (1, 63, 65, 257)


def points(n=257, seed=17):
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    return d * rng.uniform(0.3, 3.0, (n, 1)), rng.normal(size=(n, 3)) * 0.4


def term_sizes(orc, X, nmax, lmax, basis):
    """Root mean squares over the points of every (n, lm) term's potential and, about, of its
    gradient: [2][nmax+1, lm] of the cosine terms; the sine terms' are alike."""
    from oracle import jerk as J
    r = np.linalg.norm(X, axis=1)
    phi, dphi = (np.stack(v) for v in zip(*[orc.phi_nl(nmax, lmax, float(ri), basis) for ri in r]))
    phi, dphi = phi.reshape(len(r), nmax + 1, lmax + 1), dphi.reshape(len(r), nmax + 1, lmax + 1)
    ls = np.array([l for l in range(lmax + 1) for _ in range(l + 1)])
    ct = X[:, 2] / r
    Y = J._ylm(torch.from_numpy(ct), torch.from_numpy(np.sqrt(1 - ct * ct)), lmax).numpy()
    p, dp = phi[:, :, ls] * Y[:, None], dphi[:, :, ls] * Y[:, None]
    g = np.sqrt(dp * dp + (ls * p / r[:, None, None]) ** 2)
    return np.sqrt((p * p).mean(0)), np.sqrt((g * g).mean(0))


def coefficients(size, lmax, seed):
    rng = np.random.default_rng(seed)
    m = np.array([m for l in range(lmax + 1) for m in range(l + 1)])
    A = rng.choice([-1.0, 1.0], size.shape) / size
    B = rng.choice([-1.0, 1.0], size.shape) / size * (m > 0)
    return A.ravel(), B.ravel()


def dev(*arrs):
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in arrs]


def rms(d):
    return float(np.sqrt((d * d).sum(-1).mean()))


@pytest.mark.parametrize("basis", [0, 1])
@pytest.mark.parametrize("nmax,lmax", CUTOFFS)
def test_force_terms(orc, nmax, lmax, basis):
    from paper_1406_4254_amd import etics as E
    X, _ = points()
    x, y, z = X.T
    sizes = term_sizes(orc, X, nmax, lmax, basis)
    for outputs in (1, 2):
        A, B = coefficients(sizes[outputs - 1], lmax, 3)
        ref = orc.scf_force(x, y, z, nmax, lmax, A, B, basis=basis)
        ref = np.stack(ref[:1] if outputs == 1 else ref[1:], 1)
        for n in NS:
            got = E.etics_scf_force_basis(*dev(x[:n], y[:n], z[:n]), nmax, lmax, *dev(A, B), MIXED, basis, outputs)
            got = torch.stack([t for t in got if t is not None], 1).cpu().numpy()
            e = rms(got - ref[:n])
            print(f"force terms ({nmax},{lmax}) basis {basis} outputs {outputs} n {n}: {e:.2e}", flush=True)
            assert e < 0.02


@pytest.mark.parametrize("nmax,lmax", CUTOFFS)
def test_jerk_terms(orc, nmax, lmax):
    """The coefficients' time derivatives alone (whose jerk is the force of those), the
    coefficients alone (the force's change along the motion), and both."""
    from oracle import jerk as J
    from paper_1406_4254_amd import etics as E
    X, V = points()
    P, Q = torch.from_numpy(X), torch.from_numpy(V)
    g = term_sizes(orc, X, nmax, lmax, 0)[1]
    # a gradient's change along the motion: about |v| (n + l + 1) / r of it
    n, l = np.arange(nmax + 1)[:, None], np.array([l for l in range(lmax + 1) for _ in range(l + 1)])[None, :]
    A, B = coefficients(g * (0.4 * (n + l + 1)), lmax, 4)
    dA, dB = coefficients(g, lmax, 5)
    shape = (nmax + 1, (lmax + 1) * (lmax + 2) // 2)
    for fa, fd in ((0.0, 1.0), (1.0, 0.0), (1.0, 1.0)):
        c = [f * v for f, v in ((fa, A), (fa, B), (fd, dA), (fd, dB))]
        tA, tB, tdA, tdB = (torch.from_numpy(v.reshape(shape)) for v in c)

        def acc_t(t):
            return J.acceleration(P + Q * t, tA + tdA * t, tB + tdB * t, nmax, lmax)
        a_ref, j_ref = torch.func.jvp(acc_t, (torch.zeros((), dtype=torch.float64),),
                                      (torch.ones((), dtype=torch.float64),))
        for k in NS:
            out = E.etics_scf_jerk(*dev(*X[:k].T), *dev(*V[:k].T), nmax, lmax, *dev(*c), MIXED)
            a, j = (torch.stack(out[i:i + 3], 1).cpu().numpy() for i in (0, 3))
            ea, ej = rms(a - a_ref.numpy()[:k]), rms(j - j_ref.numpy()[:k])
            print(f"jerk terms ({nmax},{lmax}) A {fa:.0f} dA {fd:.0f} n {k}: {ea:.2e} {ej:.2e}", flush=True)
            assert ea < 0.02 and ej < 0.05
