"""Rounding of the clover term: against 80-bit arithmetic its error is no larger
than that of the definition's own evaluation in FP64, four leaves per plane, each
a product of two products.  (GPU)

The FP64 evaluation is modelled on the CPU with the multiply-adds of the device
(one rounding for a * b + c, taken in 80 bits and rounded to FP64)."""
import numpy as np
import pytest

from paper_2407_00041_amd import clover_term, synth

from util import need_gpu, to_dev

pytestmark = pytest.mark.gpu
LD = np.longdouble


def mul(x, y, rnd):
    """x y of [V, 3, 3, 2] matrices (re, im), each multiply-add rounded by rnd."""
    s = np.zeros_like(x)
    for k in range(3):
        a, b = x[:, :, k:k + 1], y[:, k:k + 1, :]
        ar, ai, br, bi = (np.broadcast_to(q, s.shape[:-1]) for q in (a[..., 0], a[..., 1], b[..., 0], b[..., 1]))
        s[..., 0] = rnd(ar * br + s[..., 0])
        s[..., 0] = rnd(-ai * bi + s[..., 0])
        s[..., 1] = rnd(ar * bi + s[..., 1])
        s[..., 1] = rnd(ai * br + s[..., 1])
    return s


def dag(x):
    t = x.transpose(0, 2, 1, 3).copy()
    t[..., 1] = -t[..., 1]
    return t


def clover_model(dims, U, rnd):
    """Packed unit term [V, 42] (complex long double) from the four leaves of each plane, Eqs. (1.11)-(1.12)."""
    V = int(np.prod(dims))
    idx = np.arange(V).reshape(dims)
    L = np.stack([U.real, U.imag], -1).astype(LD)

    def sh(*steps):
        i = idx
        for mu, n in steps:
            i = np.roll(i, -n, axis=mu)
        return i.ravel()

    B = [np.eye(2, dtype=complex), np.diag([-1j, 1j]), np.array([[0, -1], [1, 0]], complex),
         np.array([[0, -1j], [-1j, 0]])]
    blk = np.zeros((2, V, 6, 6, 2), dtype=LD)
    for mu in range(4):
        for nu in range(mu + 1, 4):
            u = lambda s, d: L[s, d]
            x, pm, pn, mm, mn = sh(), sh((mu, 1)), sh((nu, 1)), sh((mu, -1)), sh((nu, -1))
            mmpn, mmmn, mnpm = sh((mu, -1), (nu, 1)), sh((mu, -1), (nu, -1)), sh((nu, -1), (mu, 1))
            m = lambda a, b: mul(a, b, rnd)
            q = m(m(u(x, mu), u(pm, nu)), m(dag(u(pn, mu)), dag(u(x, nu))))
            q = rnd(q + m(m(u(x, nu), dag(u(mmpn, mu))), m(dag(u(mm, nu)), u(mm, mu))))
            q = rnd(q + m(m(dag(u(mm, mu)), dag(u(mmmn, nu))), m(u(mmmn, mu), u(mn, nu))))
            q = rnd(q + m(m(dag(u(mn, nu)), u(mn, mu)), m(u(mnpm, nu), dag(u(x, mu)))))
            F = rnd(q - dag(q))
            for b, P in enumerate((B[mu] @ B[nu].conj().T, B[mu].conj().T @ B[nu])):
                for i in range(2):
                    for j in range(2):
                        f = -P[i, j] / 16
                        s = blk[b][:, 3 * i:3 * i + 3, 3 * j:3 * j + 3]
                        if f.real:
                            s[...] = rnd(s + LD(f.real) * F)
                        if f.imag:  # i F = (-Im F, Re F)
                            s[...] = rnd(s + LD(f.imag) * np.stack([-F[..., 1], F[..., 0]], -1))
    out = np.zeros((V, 42, 2), dtype=LD)
    iu = np.triu_indices(6, 1)
    for b in range(2):
        for i in range(6):
            out[:, 21 * b + i] = blk[b][:, i, i]
        out[:, 21 * b + 6:21 * b + 21] = blk[b][:, iu[0], iu[1]]
    return out


@pytest.mark.parametrize("eps", [0.05, 0.3])
def test_clover_term_error(eps):
    need_gpu()
    dims = (8, 8, 8, 10)
    U = synth.smooth_links(dims, 17, eps).numpy()
    want = clover_model(dims, U, lambda x: x)
    norm = np.sqrt((want ** 2).sum())
    err = lambda a: float(np.sqrt(((a - want) ** 2).sum()) / norm)
    four_leaves = err(clover_model(dims, U, lambda x: x.astype(np.float64).astype(LD)))
    got = clover_term(dims, to_dev(U)).cpu().numpy()
    e = err(np.stack([got.real, got.imag], -1).astype(LD))
    # 5120 sites x 30 independent complex entries: the two sample errors scatter by well under 1 %
    assert e <= 1.01 * four_leaves, (e, four_leaves)
