"""The in-range square root and reciprocal of the step loop against IEEE.

The RK4 loop runs the square roots and the reciprocal without operand
rescaling, and certifies each interval by the size of D = D1 D2 and by the
last residual of its reciprocal. States therefore equal the oracle's bit for
bit, also where the certificate fails: next to a primary and far out, where D
leaves the range, and at a D whose mantissa is all ones, where the
reciprocal's last step would round to the wrong neighbour."""
from fractions import Fraction

import numpy as np
import pytest

import oracle
import paper_2207_13175_amd as iod

pytestmark = pytest.mark.gpu


def first_step(mu, xs):
    """State after one step of 1e-3 TU from each of xs [n, 6], by the library."""
    import torch
    h = iod.iod_create(mu, [0.9, 0.1, 0, 0, 0.2, 0], [1e-3], np.zeros((1, 2)), 1e-5, h=1e-3)
    ld = (len(xs) + 63) // 64 * 64
    x = torch.zeros((6, ld), dtype=torch.float64, device="cuda")
    x[:, :len(xs)] = torch.from_numpy(np.ascontiguousarray(xs.T)).cuda()
    out = torch.zeros((1, 6, ld), dtype=torch.float64, device="cuda")
    iod.iod_propagate(h, x, len(xs), out)
    torch.cuda.synchronize()
    return out[0, :, :len(xs)].cpu().numpy().T


def reference(mu, xs):
    return np.stack([oracle.propagate(mu, 1e-3, x, [1e-3])[0] for x in xs])


def all_ones_state():
    """A position whose D1 D2 is 2 - 2^-52, with mu = 0.5: pairs of radicands
    near r2^2 = 1 whose product of r^2 fl(sqrt(r^2)) rounds there, then x and y
    searched by single units so that both come out exactly."""
    top = 2.0 - 2.0 ** -52
    j = np.arange(-400, 401)
    for r2 in 1.0 + np.arange(1, 400) * 2.0 ** -52:
        D2 = r2 * np.sqrt(r2)
        r1 = 2.0 ** (2 / 3) + j * 2.0 ** -52
        for t1 in r1[(r1 * np.sqrt(r1)) * D2 == top]:
            d1 = (t1 - r2 + 1.0) / 2
            y0 = np.sqrt(t1 - d1 * d1)
            for i in range(-12, 13):
                x = d1 - 0.5 + i * 2.0 ** -54
                a, b = Fraction(x + 0.5) ** 2, Fraction(x - 0.5) ** 2
                for k in range(-12, 13):
                    y = y0 + k * np.spacing(y0)
                    q = Fraction(y * y)
                    if float(a + q) == t1 and float(b + q) == r2:
                        return np.array([x, y, 0.0]), t1, r2
    raise AssertionError("no such state found")


def test_states_at_the_edges_of_the_certificate():
    rng = np.random.default_rng(5)
    xs = []
    for e in (-1, -60, -126, -127, -200, -253, -254, -300, -340, 30, 110, 166, 167, 168, 250, 300, 340):
        # next to the second primary (1 - mu = 0.75 exactly) and far from both
        s = rng.normal(0, 1, 6)
        s[:3] *= 2.0 ** e
        s[3:] *= 0.1
        if e < 0:
            s[0] += 0.75
        xs.append(s)
    xs = np.array(xs)
    for x in xs:   # one at a time: each decides its own wave's path
        a, b = first_step(0.25, x[None]), reference(0.25, x[None])
        assert np.array_equal(a, b, equal_nan=True), (x, a, b)
    a, b = first_step(0.25, xs), reference(0.25, xs)
    assert np.array_equal(a, b, equal_nan=True)


def test_mantissa_of_all_ones():
    p, r1, r2 = all_ones_state()
    assert (r1 * np.sqrt(r1)) * (r2 * np.sqrt(r2)) == 2.0 - 2.0 ** -52
    xs = np.concatenate([p, [0.0, 0.1, 0.0]])[None]
    assert np.array_equal(first_step(0.5, xs), reference(0.5, xs))


@pytest.mark.parametrize("partial", [False, True])
@pytest.mark.parametrize("m", [1, 20000, 40000])
def test_last_stage_next_to_a_primary(m, partial):
    """A step whose fourth stage alone comes within 2^-345 to 2^-350 of the second
    primary (a tiny mass: x and y are chosen such that the stage lands on its x
    and y exactly), where 1 / (D1 D2) is infinite. The position after the step is
    a number and the velocity along z an infinity, not NaN, with one, two or
    four lanes per particle; also where it is the partial step to an off-grid
    observation, of a grid step twice as long."""
    import torch
    t, mu = 2.0 ** -10, 1e-300
    h = 2 * t if partial else t
    xs = np.array([[1.000739122972962, 0.0009516530515198243, 2.0 ** e, -0.7559108123501284,
                    -0.9752318481629676, 0.0] for e in (-350, -345, -341, -330)])
    want = np.stack([oracle.propagate(mu, h, x, [t])[0] for x in xs])
    assert np.array_equal(want[:, 5] == -np.inf, [True, True, False, False])
    assert np.all(np.isfinite(want[:, :3]))
    hd = iod.iod_create(mu, [0.9, 0.1, 0, 0, 0.2, 0], [t], np.zeros((1, 2)), 1e-5, h=h)
    for x, w in zip(xs, want):
        d = torch.from_numpy(np.tile(x[:, None], (1, m))).cuda()
        out = torch.zeros((1, 6, m), dtype=torch.float64, device="cuda")
        iod.iod_propagate(hd, d, m, out)
        torch.cuda.synchronize()
        assert np.array_equal(out[0].cpu().numpy(), np.tile(w[:, None], (1, m)), equal_nan=True), (x, w)


@pytest.mark.parametrize("mu", [0.0, 0.25, 0.5])
def test_tangent_of_many_particles_at_the_edges_of_the_certificate(mu):
    """The one-thread tangent sweep (many particles) takes its reciprocals from
    the hardware's seed and is certified by their residuals alone. States next to
    the second primary and far out (mu = 0: next to where it would be, with no
    attraction, so that a tiny D goes with finite results) and the D with a
    mantissa of all ones, one to a wave, against the pipelined sweep."""
    import torch
    rng = np.random.default_rng(9)
    xs = []
    for e in (-1, -60, -126, -200, -253, -254, -255, -300, -333, -334, -340, -341, -342, -350, -384, -400,
              30, 110, 166, 167, 168, 169, 170, 171, 172, 250, 340):
        s = rng.normal(0, 1, 6)
        s[:3] *= 2.0 ** e
        s[3:] *= 0.1
        if e < 0:
            s[0] += 1.0 - mu
            if e < -60:   # (the offset in x is lost)
                s[0] = 1.0 - mu
        xs.append(s)
    xs.append(np.array([1.0 - mu, 0.0, 0.0, 0.0, 0.1, 0.0]))
    if mu == 0.5:
        xs.append(np.concatenate([all_ones_state()[0], [0.0, 0.1, 0.0]]))
    n, many = len(xs), 24640
    x = np.tile(np.array([0.9, 0.12, 0.01, 0.0, 0.1, 0.0]), (many, 1))
    x[:64 * n:64] = xs
    t = np.array([0.0, 1e-3, 2.4e-3, 4e-3])
    h = iod.iod_create(mu, [0.9, 0.1, 0, 0, 0.2, 0], t, np.zeros((len(t), 2)), 1e-5, h=1e-3, cost_mode=1)

    def normal(x):
        m = len(x)
        kw = dict(dtype=torch.float64, device="cuda")
        out = [torch.zeros((k, m), **kw) for k in (1, 21, 6)]
        iod.iod_normal_eq(h, torch.from_numpy(np.ascontiguousarray(x.T)).cuda(), m, out[0][0], out[1], out[2])
        torch.cuda.synchronize()
        return [o.cpu().numpy() for o in out]

    got = [o[:, :64 * n:64] for o in normal(x)]
    for i, s in enumerate(xs):   # one at a time: each decides its own wave's path
        for a, b in zip(got, normal(s[None])):
            assert np.array_equal(a[:, i], b[:, 0], equal_nan=True), (i, s)
