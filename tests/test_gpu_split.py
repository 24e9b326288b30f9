"""Several lanes to a particle, and one: the same bits.

Launches that would leave SIMDs idle give each particle two or four lanes.
A particle's result does not depend on how many others it is launched with,
so every size is compared, bit for bit, with the same particles inside a
launch of one lane per particle. Intervals of 1 to 9 steps between the
observations, off-grid times, and particles that leave the certified range
(their waves redo the interval on the IEEE path) are among them."""
import numpy as np
import pytest

import paper_2207_13175_amd as iod
from paper_2207_13175_amd import workloads as W

pytestmark = pytest.mark.gpu

FULL = 65536


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = W.tiny(3)
    steps = np.cumsum([1, 2, 3, 4, 5, 6, 7, 8, 9, 4])
    t = steps * 1e-3
    t[3] += 0.0004
    t[7] += 0.0007
    rng = np.random.default_rng(11)
    h = iod.iod_create_ranged(wl.mu, wl.chief, t, rng.normal(0, 0.3, (len(t), 2)),
                              rng.uniform(1e-3, 2e-3, len(t)), 1e-5, 1e-7, h=1e-3)
    x = torch.from_numpy(np.ascontiguousarray(W.random_swarm(7, FULL, wl.lo, wl.hi).T)).cuda()
    # scattered particles on a primary, next to it, far away and not finite
    x[:3, 70] = torch.tensor([1 - wl.mu, 0.0, 0.0], dtype=torch.float64, device="cuda")
    x[:3, 5000] = torch.tensor([1 - wl.mu + 1e-80, 0.0, 0.0], dtype=torch.float64, device="cuda")
    x[0, 16383] = 1e120
    x[4, 31] = float("nan")

    def run(m):
        kw = dict(dtype=torch.float64, device="cuda")
        K, xm = len(t), x[:, :m].contiguous()
        out = [torch.full((K, 6, m), 7.0, **kw), torch.full((K, 2, m), 7.0, **kw),
               torch.full((K, m), 7.0, **kw), torch.full((m,), 7.0, **kw)]
        iod.iod_propagate(h, xm, m, out[0])
        iod.iod_predict(h, xm, m, out[1])
        iod.iod_predict_ranges(h, xm, m, out[2])
        iod.iod_eval_swarm(h, xm, m, out[3])
        torch.cuda.synchronize()
        return [o.cpu().numpy() for o in out]
    return run, run(FULL)


@pytest.mark.parametrize("m", [1, 16, 63, 64, 65, 129, 1000, 16383, 16384, 16385, 32767, 32768, 32769])
def test_any_lane_count_gives_the_same_bits(setup, m):
    run, full = setup
    for got, want in zip(run(m), full):
        assert np.array_equal(got, want[..., :m], equal_nan=True)


@pytest.mark.parametrize("m", [200, 20000])
def test_swarm_of_split_particles_in_a_batch(m):
    """A problem alone (several lanes per particle) and inside a batch large
    enough for one lane per particle: the same global bests."""
    wl = W.tiny(4, K=4, T=0.02)
    rng = np.random.default_rng(3)
    ang = rng.normal(0, 0.3, (wl.K, 2))
    p = iod.pso_params(0.7, 1.5, 1.5, 5, wl.lo, wl.hi, problem=0)
    h = iod.iod_create(wl.mu, wl.chief, wl.t, ang, wl.sigma, h=wl.h)
    g, J, hist = iod.iod_solve(h, p, m, 3)
    n = 1 + 90000 // m
    b = iod.iod_create_batch([wl.mu] * n, [wl.chief] * n, [wl.t] * n, [ang] * n, [wl.sigma] * n, h=wl.h)
    gs, Js, hists = iod.iod_batch_solve(b, [p] * n, np.full(n, m), 3)
    assert all(np.array_equal(gs[q], g) and Js[q] == J and np.array_equal(hists[q], hist)
               for q in range(n))


@pytest.mark.parametrize("steps", [1, 15, 16, 17, 32, 50])
@pytest.mark.parametrize("tau", [0.0, 0.0003])
def test_chief_tables_of_the_offset_formulation(steps, tau):
    """The chief's own state has offset zero, so its FP32 propagation returns
    the chief states of the tables: the FP64 ones, bit for bit. A particle near
    it, which reads every stage row, stays within the offset formulation's
    rounding (2^-24 of an offset of 1e-3 per step, times the growth of a
    deviation over so short an arc, below 2)."""
    import torch
    wl = W.tiny(5)
    t = np.unique([1e-3, max(1, steps // 2) * 1e-3 + tau, steps * 1e-3 + tau])
    h = iod.iod_create(wl.mu, wl.chief, t, np.zeros((len(t), 2)), 1e-5, h=1e-3)
    x = torch.zeros((6, 64), dtype=torch.float64, device="cuda")
    x[:] = torch.from_numpy(wl.chief).cuda()[:, None]
    x[:, 1] += 1e-3
    a, b = (torch.zeros((len(t), 6, 64), dtype=torch.float64, device="cuda") for _ in range(2))
    iod.iod_propagate(h, x, 2, a)
    iod.iod_propagate_f32(h, x, 2, b)
    torch.cuda.synchronize()
    a, b = a.cpu().numpy(), b.cpu().numpy()
    assert np.array_equal(a[:, :, 0], b[:, :, 0])
    assert np.max(np.abs(a[:, :, 1] - b[:, :, 1])) <= 2 * steps * 2.0 ** -24 * 1e-3


@pytest.mark.parametrize("lanes_one", [False, True])
def test_first_mixed_iteration_keeps_the_initial_record(lanes_one):
    """The first iteration only moves the swarm: the record and the history
    entry of the initial evaluation stay (few problems: four lanes to a
    candidate; 1,100: one)."""
    n = 1100 if lanes_one else 3
    wls = [W.tiny(s % 3, K=2, T=0.01) for s in range(n)]
    b = iod.iod_create_batch([w.mu for w in wls], [w.chief for w in wls], [w.t for w in wls],
                             [np.zeros((w.K, 2)) for w in wls], [w.sigma for w in wls], h=wls[0].h)
    params = [iod.pso_params(0.7, 1.5, 1.5, 3, w.lo, w.hi, problem=i) for i, w in enumerate(wls)]
    m = np.full(n, 64)
    out = [iod.iod_batch_solve_mixed(b, params, m, k, top_k=8) for k in (0, 1, 3)]
    for a, c in zip(out[0][:2], out[1][:2]):
        assert np.array_equal(a, c)
    assert np.array_equal(out[1][2], out[2][2][:, :2])
    assert np.array_equal(out[1][2][:, 0], out[1][2][:, 1])


@pytest.mark.parametrize("block", [64, 128, 256])
@pytest.mark.parametrize("top", [40, 700, 6000])
def test_uneven_batches_do_not_depend_on_their_neighbours(block, top):
    """Batches whose workgroups the SIMDs take in one or two rounds run one wave
    to a SIMD, with one, two or four lanes to a particle: every problem's
    result is that of the problem in a batch of its own."""
    rng = np.random.default_rng([block, top])
    n = 24
    wls = [W.tiny(s % 4, K=3, T=float(rng.uniform(0.01, 0.06))) for s in range(n)]
    m = np.exp(rng.uniform(np.log(20), np.log(top), n)).astype(int)
    m[0], m[1] = top, 1
    obs = [rng.normal(0, 0.3, (w.K, 2)) for w in wls]
    par = [iod.pso_params(0.7, 1.5, 1.5, 3, w.lo, w.hi, problem=i) for i, w in enumerate(wls)]

    def solve(idx):
        b = iod.iod_create_batch([wls[i].mu for i in idx], [wls[i].chief for i in idx], [wls[i].t for i in idx],
                                 [obs[i] for i in idx], [wls[i].sigma for i in idx], h=wls[0].h)
        iod.iod_batch_set_config(b, block=block)
        return iod.iod_batch_solve(b, [par[i] for i in idx], m[idx], 3)

    whole = solve(np.arange(n))
    for i in range(n):
        for a, w in zip(solve(np.array([i])), whole):
            assert np.array_equal(a[0], w[i]), i


@pytest.mark.parametrize("m,lanes", [(200, 4), (20000, 2), (40000, 1)])
@pytest.mark.parametrize("other", [1, 2, 4])
def test_swarm_goes_on_with_the_lanes_it_was_initialised_with(m, lanes, other):
    """The slots of a swarm's work buffer follow its lanes per particle, and a
    device with other compute units would choose others. A swarm whose buffer is
    laid out for `other` lanes, as such a device leaves it, goes on from there:
    states, personal bests, history and global best of the one left alone."""
    import torch
    wl = W.tiny(4, K=4, T=0.02)
    ang = np.random.default_rng(3).normal(0, 0.3, (wl.K, 2))
    h = iod.iod_create(wl.mu, wl.chief, wl.t, ang, wl.sigma, h=wl.h)
    p = iod.pso_params(0.7, 1.5, 1.5, 5, wl.lo, wl.hi)

    def start():
        w = iod.Swarm(m, hist_len=8)
        iod.iod_swarm_init(h, w, p)
        iod.iod_step(h, w, p, 3)
        return w

    ref = start()
    assert ref.s.reserved == lanes and ref.s.block == 256
    moved = start()
    # the records and the stop flag, and the slots of iteration 3, for other lanes
    per = 256 // other
    n0, n = -(-m // (256 // lanes)), -(-m // per)
    old, new = moved.work.clone(), torch.full_like(moved.work, float("nan"))
    new[2 * n * 8:2 * n * 8 + 17] = old[2 * n0 * 8:2 * n0 * 8 + 17]
    key = torch.nan_to_num(moved.jp[:m], nan=float("inf"))
    for s in range(n):
        i = s * per + int(torch.argmin(key[s * per:(s + 1) * per]))
        row = torch.cat([key[i:i + 1], torch.tensor([float(i)], dtype=torch.float64, device="cuda"), moved.p[:, i]])
        new[(n + s) * 8:(n + s + 1) * 8] = row
    moved.work.copy_(new)
    moved.s.reserved = other
    for w in (ref, moved):
        iod.iod_step(h, w, p, 4)
    a, b = (iod.iod_swarm_best(h, w) for w in (ref, moved))
    assert np.array_equal(a[0], b[0]) and a[1:] == b[1:]
    for f in ("x", "v", "p", "jp", "cost", "hist"):
        assert torch.equal(getattr(ref, f), getattr(moved, f)), f
