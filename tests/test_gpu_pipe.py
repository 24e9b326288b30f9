"""The pipelined sensitivity sweeps against the one-thread-per-particle ones.

Few particles take the pipelined form, many the other; a particle's result
does not depend on how many others it is launched with, so each size is
compared, bit for bit, with the same particles inside a launch too large to be
pipelined. Step counts sit at the edges of the hand-over chunks and the reverse
blocks (8 steps each), the checkpoints' segments and the largest evaluation that is
pipelined (4,096 steps), with off-grid times, two observations in one step, an
epoch observation, ranges, and particles whose waves leave the certified
range."""
import numpy as np
import pytest

import oracle
import paper_2207_13175_amd as iod
from paper_2207_13175_amd import workloads as W

pytestmark = pytest.mark.gpu

FULL = 24640   # more than either sweep is pipelined for


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def times(steps, kind):
    if steps == 0:
        return np.array([0.0])
    if kind == "end":
        return np.array([steps * 1e-3])
    n = min(steps, 7)
    j = np.unique(np.linspace(0, steps, n + 1).astype(int))
    t = j * 1e-3
    if kind == "offgrid" and steps > 1:
        t = np.unique(np.concatenate([t, [0.0003, (steps - 1) * 1e-3 + 0.0002, (steps - 1) * 1e-3 + 0.0006]]))
    return t


def sweeps(torch, h, x, m):
    kw = dict(dtype=torch.float64, device="cuda")
    xm = x[:, :m].contiguous()
    out = [torch.full(s, 7.0, **kw) for s in ((m,), (21, m), (6, m), (m,), (6, m))]
    iod.iod_normal_eq(h, xm, m, out[0], out[1], out[2])
    iod.iod_grad(h, xm, m, out[3], out[4])
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("steps,kind", [(0, "end"), (1, "end"), (3, "offgrid"), (4, "grid"), (5, "offgrid"),
                                        (8, "end"), (9, "grid"), (64, "offgrid"), (65, "end"),
                                        (257, "offgrid"), (1000, "grid"), (4096, "offgrid"), (4097, "end")])
@pytest.mark.parametrize("mode", [0, 1])
def test_pipelined_sweeps_give_the_same_bits(torch_dev, steps, kind, mode):
    torch = torch_dev
    wl = W.tiny(3)
    t = times(steps, kind)
    rng = np.random.default_rng([steps, mode])
    args = (wl.mu, wl.chief, t, rng.normal(0, 0.3, (len(t), 2)))
    if mode:
        h = iod.iod_create_ranged(*args, rng.uniform(1e-3, 2e-3, len(t)), 1e-5, 1e-7, h=1e-3, cost_mode=1)
    else:
        h = iod.iod_create(*args, 1e-5, h=1e-3)
    x = torch.from_numpy(np.ascontiguousarray(W.random_swarm(7, FULL, wl.lo, wl.hi).T)).cuda()
    x[:3, 20] = torch.tensor([1 - wl.mu + 1e-80, 0.0, 0.0], dtype=torch.float64, device="cuda")
    x[0, 40] = 1e120
    full = sweeps(torch, h, x, FULL)
    for m in (1, 15, 16, 17, 300):
        for got, want in zip(sweeps(torch, h, x, m), full):
            assert np.array_equal(got, want[..., :m], equal_nan=True), m


@pytest.mark.parametrize("kind", ["grid", "offgrid"])
@pytest.mark.parametrize("steps", [7, 15, 16, 17, 23, 24, 25, 592, 593, 1376, 1377, 2472, 2473])
def test_pipelined_sweeps_at_the_edges_of_blocks_and_segments(torch_dev, steps, kind):
    """Blocks of 8 steps; checkpoints every 8, 16, 24 and 32 steps (up to 592,
    1,376, 2,472 and 4,096 steps)."""
    test_pipelined_sweeps_give_the_same_bits(torch_dev, steps, kind, 1)


def test_refinement_of_few_and_many_problems_agrees(torch_dev):
    """A problem refined in a small batch (pipelined throughout) and inside a
    batch of 900 (which switches as problems retire): the same bits."""
    wls = [W.tiny(s, K=6, T=0.12) for s in range(5)]
    obs = []
    for wl in wls:
        P = oracle.Problem(wl.mu, wl.h, wl.sigma, wl.chief, wl.t, np.zeros((wl.K, 2)))
        obs.append(oracle.predict(P, wl.truth) + wl.noise)

    def refine(idx):
        b = iod.iod_create_batch([wls[i].mu for i in idx], [wls[i].chief for i in idx],
                                 [wls[i].t for i in idx], [obs[i] for i in idx],
                                 [wls[i].sigma for i in idx], h=wls[0].h)
        params = [iod.pso_params(0.7, 1.5, 1.5, 3, wls[i].lo, wls[i].hi, problem=int(i)) for i in idx]
        return iod.iod_batch_solve_polished(b, params, np.full(len(idx), 64), 2, top_k=16, n_cand=8, n_gn=12)
    few = refine(np.arange(5))
    many_idx = np.arange(900) % 5
    many = refine(many_idx)
    for f, m in zip(few, many):
        assert np.array_equal(f[many_idx], m)


@pytest.mark.parametrize("n_cand", [1, 7, 16, 20, 64])
@pytest.mark.parametrize("kind", ["grid", "offgrid"])
def test_refinement_does_not_depend_on_the_batch(torch_dev, n_cand, kind):
    """The refinement's launches divide the work by the number of problems
    still active: pipelined sweeps from the trials' checkpoints or packed ones,
    four, two or one lanes to a trial. Problems whose evaluations end at the
    edges of the checkpoints' segments (8 steps), with off-grid and epoch
    observations, get the same bits in batches of every share."""
    wl = W.tiny(3)
    steps = [8, 9, 15, 16, 121, 1]
    rng = np.random.default_rng([n_cand, len(kind)])
    t = [times(s, kind) for s in steps] + [np.array([0.0, 1e-3])]
    obs = []
    for tk in t:
        P = oracle.Problem(wl.mu, wl.h, wl.sigma, wl.chief, tk, np.zeros((len(tk), 2)))
        obs.append(oracle.predict(P, wl.truth) + rng.normal(0, wl.sigma, (len(tk), 2)))

    def refine(idx):
        n = len(idx)
        b = iod.iod_create_batch([wl.mu] * n, [wl.chief] * n, [t[i] for i in idx], [obs[i] for i in idx],
                                 [wl.sigma] * n, h=wl.h)
        params = [iod.pso_params(0.7, 1.5, 1.5, 3, wl.lo, wl.hi, problem=int(i)) for i in idx]
        return iod.iod_batch_solve_polished(b, params, np.full(n, 64), 2, top_k=64, n_cand=n_cand, n_gn=6)

    each = len(t)
    alone = refine(np.arange(each))
    for n in (1, 300, 600, 1300):
        idx = np.arange(n) % each
        for a, b in zip(alone, refine(idx)):
            assert np.array_equal(a[idx], b, equal_nan=True), n


@pytest.mark.parametrize("steps", [(2000, 4097), (1377, 3000, 4097, 4096), (4097,), (2473, 5000, 8)])
def test_refinement_with_a_problem_beyond_the_pipelined_sweeps(torch_dev, steps):
    """One problem of more than 4,096 steps: its batch refines without the
    trials' checkpoints, whatever segments the other problems' own sweeps would
    take, and every problem gets the bits that it gets in a batch of its own."""
    wl = W.tiny(5)
    rng = np.random.default_rng(list(steps))
    t = [times(s, "grid")[1:] for s in steps]
    obs = []
    for tk in t:
        P = oracle.Problem(wl.mu, wl.h, wl.sigma, wl.chief, tk, np.zeros((len(tk), 2)))
        obs.append(oracle.predict(P, wl.truth) + rng.normal(0, wl.sigma, (len(tk), 2)))

    def refine(idx):
        n = len(idx)
        b = iod.iod_create_batch([wl.mu] * n, [wl.chief] * n, [t[i] for i in idx], [obs[i] for i in idx],
                                 [wl.sigma] * n, h=wl.h)
        params = [iod.pso_params(0.7, 1.5, 1.5, 3, wl.lo, wl.hi, problem=int(i)) for i in idx]
        return iod.iod_batch_solve_polished(b, params, np.full(n, 64), 2, top_k=16, n_cand=4, n_gn=3)

    together = refine(range(len(steps)))
    for i in range(len(steps)):
        for a, b in zip(together, refine([i])):
            assert np.array_equal(a[i], b[0], equal_nan=True), steps[i]


@pytest.mark.parametrize("problems", [2048, 4096])
def test_refinement_with_longer_checkpoint_segments(torch_dev, problems):
    """Checkpoints every 8 steps would take more than 2 GiB: the trials leave them
    every 16 (2,048 problems of up to 3,000 steps) or 32 steps (4,096). The
    packed sweeps begin, and as the short problems retire, those from the
    checkpoints take over; each problem's bits are those of a small batch."""
    wl = W.tiny(5)
    rng = np.random.default_rng(problems)
    steps = [3000, 2993, 120, 121, 122, 123, 124, 125, 126, 127, 128, 129]
    t = [times(s, "grid")[1:] for s in steps]
    obs = []
    for tk in t:
        P = oracle.Problem(wl.mu, wl.h, wl.sigma, wl.chief, tk, np.zeros((len(tk), 2)))
        obs.append(oracle.predict(P, wl.truth) + rng.normal(0, wl.sigma, (len(tk), 2)))

    def refine(idx):
        n = len(idx)
        b = iod.iod_create_batch([wl.mu] * n, [wl.chief] * n, [t[i] for i in idx], [obs[i] for i in idx],
                                 [wl.sigma] * n, h=wl.h)
        params = [iod.pso_params(0.7, 1.5, 1.5, 3, wl.lo, wl.hi, problem=int(i)) for i in idx]
        return iod.iod_batch_solve_polished(b, params, np.full(n, 64), 2, top_k=16, n_cand=2, n_gn=30)

    few = refine(range(len(steps)))
    idx = np.concatenate([np.arange(problems - 64) % 10 + 2, np.arange(64) % len(steps)])
    for a, b in zip(few, refine(idx)):
        assert np.array_equal(a[idx], b)
