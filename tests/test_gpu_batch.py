"""Batched execution (many chains, one launch per colour phase): every chain
must follow exactly the trajectory it follows alone, and small ones the
oracle's, whatever the launch shape (rows per wavefront) or graph replay."""
import hashlib
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def cvf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05919_amd import cvf as mod
    mod.lib()
    return mod


def params(cvf, L, T, P, seed, **kw):
    return cvf.cvf_params_from_si(T, P, L=L, seed=seed, **kw)


def digest(ch):
    return hashlib.sha256(ch.sigma.cpu().numpy().tobytes()).hexdigest()


def mixed_jobs(n, seed=3):
    rng = np.random.default_rng(seed)
    Ls = [int(2 * round(np.exp(rng.uniform(np.log(6), np.log(300))) / 2)) for _ in range(n)]
    Ls[:4] = [2, 4, 66, 128]                      # degenerate, quad, byte-lane and quad layouts
    return [(L, 270.0 + 60.0 * rng.random(), 50.0 * rng.random(), 500 + k) for k, L in enumerate(Ls)]


@pytest.mark.parametrize("rows,graph", [(0, 0), (2, 0), (8, 0), (32, 5), (4, 3)])
def test_batch_equals_alone(cvf, rows, graph):
    jobs = mixed_jobs(24)
    say(f"case batch rows={rows} graph={graph} Ls={[j[0] for j in jobs]}")
    alone = []
    for L, T, P, s in jobs:
        ch = cvf.Chain(params(cvf, L, T, P, s), cvf.CVF_ALGO_METROPOLIS)
        ch.metropolis(7)
        alone.append((digest(ch), ch.obs()))
        ch.close()
    chains = [cvf.Chain(params(cvf, L, T, P, s), cvf.CVF_ALGO_METROPOLIS) for L, T, P, s in jobs]
    b = cvf.Batch(chains)
    if rows:
        b.set_rows(rows)
    b.metropolis(7, graph_block=graph)
    for k, ch in enumerate(chains):
        o = ch.obs()
        assert digest(ch) == alone[k][0], (k, jobs[k])
        assert o == alone[k][1], (k, jobs[k])
        assert o["consistent"] == 1
    b.close()
    for ch in chains:
        ch.close()


def test_batch_vs_oracle_and_mixed_calls(cvf, oracle_mod):
    """Batched sweeps interleaved with single-chain Metropolis and SW calls
    on the same chains, against the oracle doing the same sequence."""
    jobs = [(2, 300.0, 0.1, 11), (6, 280.0, 10.0, 12), (40, 320.0, 40.0, 13), (64, 300.0, 0.1, 14)]
    chains, orcs = [], []
    for L, T, P, s in jobs:
        op = oracle_mod.params_from_si(T, P, L=L, seed=s)
        p = cvf.cvf_params()
        for k, v in op.as_dict().items():
            setattr(p, k, v)
        chains.append(cvf.Chain(p))
        orcs.append(oracle_mod.Chain(op))
    b = cvf.Batch(chains)
    b.metropolis(3)
    chains[1].sw(2)
    chains[2].metropolis(1)
    b.metropolis(4, graph_block=2)
    for o in orcs:
        o.metropolis(3)
    orcs[1].sw(2)
    orcs[2].metropolis(1)
    for o in orcs:
        o.metropolis(4)
    for ch, oc in zip(chains, orcs):
        assert np.array_equal(ch.sigma.cpu().numpy(), oc.sigma())
        og, oo = ch.obs(), oc.obs()
        for k in ("step", "n_hb_raw", "n_coop", "met_accepted", "vol_accepted", "count"):
            assert og[k] == oo[k], k
        assert og["v"] == pytest.approx(oo["v"], rel=1e-12)
    b.close()
    for ch in chains:
        ch.close()


def test_batch_autotune_and_graph_replays(cvf):
    jobs = mixed_jobs(16, seed=9)
    chains = [cvf.Chain(params(cvf, L, T, P, s), cvf.CVF_ALGO_METROPOLIS) for L, T, P, s in jobs]
    b = cvf.Batch(chains)
    rows = b.autotune(2)
    assert rows in (2, 4, 8, 16, 32)
    b.metropolis(9, graph_block=4)        # two replays + one plain sweep
    b.metropolis(8, graph_block=4)        # two more replays of the same graph
    got = [digest(ch) for ch in chains]
    b.close()
    for ch in chains:
        ch.close()
    for k, (L, T, P, s) in enumerate(jobs):
        ch = cvf.Chain(params(cvf, L, T, P, s), cvf.CVF_ALGO_METROPOLIS)
        ch.metropolis(11 * 2 + 17)       # the autotuner's 11 blocks of 2 sweeps, then 17
        assert digest(ch) == got[k], k
        ch.close()


def test_batch_rejects_mixed_q(cvf):
    a = cvf.Chain(params(cvf, 8, 300.0, 0.1, 1), cvf.CVF_ALGO_METROPOLIS)
    b = cvf.Chain(params(cvf, 8, 300.0, 0.1, 2, q=4), cvf.CVF_ALGO_METROPOLIS)
    with pytest.raises(cvf.CvfError):
        cvf.Batch([a, b])
    a.close()
    b.close()


def test_batch_sw_equals_alone(cvf):
    jobs = mixed_jobs(20, seed=5)
    say(f"case batch sw Ls={[j[0] for j in jobs]}")
    alone = []
    for L, T, P, s in jobs:
        ch = cvf.Chain(params(cvf, L, T, P, s))
        ch.sw(4).metropolis(2).sw(3)
        alone.append((digest(ch), ch.obs(), ch.labels().cpu().numpy().copy()))
        ch.close()
    chains = [cvf.Chain(params(cvf, L, T, P, s)) for L, T, P, s in jobs]
    b = cvf.Batch(chains)
    b.sw(4).metropolis(2).sw(3)
    for k, ch in enumerate(chains):
        assert digest(ch) == alone[k][0], (k, jobs[k])
        assert ch.obs() == alone[k][1], (k, jobs[k])
        assert np.array_equal(ch.labels().cpu().numpy(), alone[k][2]), (k, jobs[k])
    b.close()
    for ch in chains:
        ch.close()


def test_batch_of_many_chains(cvf):
    """More chains than one round of the workgroups' chain search covers
    (256 prefix-sum entries per round), Metropolis and SW batches."""
    rng = np.random.default_rng(17)
    jobs = [(int(2 * rng.integers(1, 20)), 270.0 + 60.0 * rng.random(), 50.0 * rng.random(), 900 + k)
            for k in range(300)]
    say(f"case batch of {len(jobs)} chains, L {min(j[0] for j in jobs)}..{max(j[0] for j in jobs)}")
    alone = []
    for L, T, P, s in jobs:
        ch = cvf.Chain(params(cvf, L, T, P, s))
        ch.metropolis(3).sw(2)
        alone.append((digest(ch), ch.obs()))
        ch.close()
    chains = [cvf.Chain(params(cvf, L, T, P, s)) for L, T, P, s in jobs]
    b = cvf.Batch(chains)
    b.metropolis(3).sw(2)
    for k, ch in enumerate(chains):
        assert digest(ch) == alone[k][0], (k, jobs[k])
        assert ch.obs() == alone[k][1], (k, jobs[k])
    b.close()
    for ch in chains:
        ch.close()


def test_batch_sw_vs_oracle(cvf, oracle_mod):
    jobs = [(2, 300.0, 0.1, 31), (10, 270.0, 50.0, 32), (34, 330.0, 3000.0, 33)]
    chains, orcs = [], []
    for L, T, P, s in jobs:
        op = oracle_mod.params_from_si(T, P, L=L, seed=s)
        p = cvf.cvf_params()
        for k, v in op.as_dict().items():
            setattr(p, k, v)
        chains.append(cvf.Chain(p))
        orcs.append(oracle_mod.Chain(op))
    b = cvf.Batch(chains)
    b.sw(6)
    for ch, oc in zip(chains, orcs):
        oc.sw(6)
        assert np.array_equal(ch.sigma.cpu().numpy(), oc.sigma())
        assert np.array_equal(ch.labels().cpu().numpy().view(np.uint32), oc.labels())
        og, oo = ch.obs(), oc.obs()
        for k in ("step", "n_hb_raw", "n_coop", "vol_accepted", "count"):
            assert og[k] == oo[k], k
    b.close()
    for ch in chains:
        ch.close()


def test_batch_sw_needs_workspace(cvf):
    a = cvf.Chain(params(cvf, 8, 300.0, 0.1, 1), cvf.CVF_ALGO_METROPOLIS)
    b = cvf.Batch([a])
    with pytest.raises(cvf.CvfError) as e:
        b.sw(1)
    assert e.value.code == cvf.CVF_ENOMEM
    b.close()
    a.close()


def test_step_limit(cvf):
    """cvf_set_stop: a batch runs more steps than some chains need; each chain
    ends exactly where its own run of `stop` steps ends, whatever follows."""
    jobs = mixed_jobs(12, seed=13)
    stops = [3 + (k % 5) for k in range(len(jobs))]
    chains = [cvf.Chain(params(cvf, L, T, P, s)) for L, T, P, s in jobs]
    for ch, st in zip(chains, stops):
        ch.set_stop(st)
    b = cvf.Batch(chains)
    b.metropolis(4).sw(2).metropolis(3)
    chains[0].metropolis(5)                     # single-chain calls respect the limit too
    for k, ((L, T, P, s), ch) in enumerate(zip(jobs, chains)):
        ref = cvf.Chain(params(cvf, L, T, P, s))
        n = stops[k]
        m1 = min(n, 4)
        m2 = min(n - m1, 2)
        m3 = min(n - m1 - m2, 3)
        ref.metropolis(m1).sw(m2).metropolis(m3)
        assert digest(ch) == digest(ref), k
        assert ch.obs() == ref.obs(), k
        ref.close()
    b.close()
    for ch in chains:
        ch.close()


def test_batch_create_async_and_observables_async(cvf):
    """The no-wait variants give the same results: a batch created from pinned
    staging (behind earlier work on its stream) sweeps exactly as one created
    with the waiting upload, and the observables record copied to pinned host
    memory without synchronising equals cvf_observables."""
    import ctypes
    import torch
    jobs = mixed_jobs(12, seed=21)
    s = torch.cuda.Stream()
    a = [cvf.Chain(params(cvf, L, T, P, sd), cvf.CVF_ALGO_METROPOLIS | cvf.CVF_ALGO_SW, stream=s)
         for L, T, P, sd in jobs]
    b = [cvf.Chain(params(cvf, L, T, P, sd), cvf.CVF_ALGO_METROPOLIS | cvf.CVF_ALGO_SW) for L, T, P, sd in jobs]
    ba = cvf.Batch(a, stream=s, nowait=True)
    bb = cvf.Batch(b)
    ba.metropolis(7)
    bb.metropolis(7)
    ba.sw(3)
    bb.sw(3)
    ba2 = cvf.Batch(a[::2], stream=s, nowait=True)       # rebuilt while the sweeps may still run
    ba2.metropolis(4)
    bb2 = cvf.Batch(b[::2])
    bb2.metropolis(4)
    n = ctypes.sizeof(cvf.cvf_obs)
    bufs = []
    for ch in a:
        buf = torch.empty(n, dtype=torch.uint8, pin_memory=True)
        cvf.cvf_observables_async(ch.h, buf.data_ptr(), s)
        bufs.append(buf)
    s.synchronize()
    torch.cuda.synchronize()
    for k, (ca, cb) in enumerate(zip(a, b)):
        assert digest(ca) == digest(cb), k
        got = cvf.cvf_obs.from_buffer_copy(bufs[k].numpy().tobytes()).as_dict()
        assert got == cb.obs(), k
    with pytest.raises(cvf.CvfError):
        cvf.cvf_observables_async(a[0].h, bufs[0].data_ptr() + 4, s)   # misaligned
    for x in (ba, bb, ba2, bb2):
        x.close()
    for ch in a + b:
        ch.close()


@pytest.mark.parametrize("algo", ["met", "sw"])
def test_batch_across_the_liquid_limit(cvf, algo):
    """Batched steps are opened beside the step before them; chains that cross
    v = 2 again and again follow the trajectory they have alone, one call per
    step (where every step is opened with N_HB_raw known), also from a graph."""
    Ls = [4, 6, 34, 64, 66, 130]
    def mk(L):
        p = cvf.cvf_params_from_si(300.0, 0.1, L=L, seed=60 + L, v_init=1.98, dv_max=0.3)
        p.beta, p.J, p.P, p.vHB = 1.0 / (L * L), 2.0, 0.5, 0.3
        return cvf.Chain(p)

    alone, chains = [mk(L) for L in Ls], [mk(L) for L in Ls]
    for ch in alone:
        for _ in range(41):
            getattr(ch, "metropolis" if algo == "met" else "sw")(1)
    b = cvf.Batch(chains)
    if algo == "met":
        b.metropolis(5, 0).metropolis(36, 9)
    else:
        b.sw(5).sw(36)
    for L, x, y in zip(Ls, alone, chains):
        assert digest(x) == digest(y), L
        assert x.obs() == y.obs(), L
    b.close()


@pytest.mark.parametrize("count", [4, 5])
def test_batch_sw_either_side_of_the_cache_limit(cvf, count):
    """What the tile kernel writes through L2 follows from the cells of the
    whole batch: four chains of L = 1024 stay below the limit, five do not."""
    mk = lambda k: cvf.Chain(cvf.cvf_params_from_si(290.0, 0.1, L=1024 if k else 1022, seed=80 + k))
    alone, chains = [mk(k) for k in range(count)], [mk(k) for k in range(count)]
    for ch in alone:
        ch.sw(3)
    b = cvf.Batch(chains).sw(3)
    for x, y in zip(alone, chains):
        assert digest(x) == digest(y)
        assert x.obs() == y.obs()
        assert (x.labels() == y.labels()).all()
    b.close()


@pytest.mark.parametrize("Ls", [[4096, 4094], [4096, 4096, 66]])
def test_batch_default_rows_either_side_of_the_limit(cvf, Ls):
    """The default rows per lane follow from the cells of the whole batch (up
    to 2^25 and more): the trajectories are those of the chains alone."""
    mk = lambda L: cvf.Chain(cvf.cvf_params_from_si(290.0, 0.1, L=L, seed=90 + L), cvf.CVF_ALGO_METROPOLIS)
    alone, chains = [mk(L) for L in Ls], [mk(L) for L in Ls]
    for ch in alone:
        ch.metropolis(3)
    b = cvf.Batch(chains).metropolis(3)
    for x, y in zip(alone, chains):
        assert digest(x) == digest(y)
        assert x.obs() == y.obs()
    b.close()
