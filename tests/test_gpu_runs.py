"""Runs of many commits in one launch against the oracle, bit for bit.  A vector
of up to 8 blocks of 64 elements a compute unit goes to the short-vector kernel
(with at most 128 workers in a launch), a longer one to the run kernel: a size
written "+x" is x elements past that limit, and is compared at the vector's ends
and about its tiles' edges.  Covered: sizes at the edges of chunks, blocks and
tiles; worker counts at the edges of the run kernel's LDS slots (5, 6 and 10
chunks, 10, 13 and 20 with the shared moment); lengths at the edges of a launch
(993 commits, 495 with adaptive staleness) and of the short-vector kernel's
phases; every rule in both kernels; the cache policies; and the same schedule
in calls of one pass, which run the pass kernels."""
import numpy as np
import pytest

import oracle as O
from gpu_util import assert_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_08469_amd import gem
    return gem


def _hp(G, **kw):
    hp = G.gem_hyperparams_default()
    for k, v in kw.items():
        setattr(hp, k, v)
    return hp


def _size(P):
    """A size, or "+x": x elements past the short-vector kernel's limit."""
    import torch
    if isinstance(P, int):
        return P
    return 64 * 8 * torch.cuda.get_device_properties(0).multi_processor_count + int(P)


def _sample(P):
    """Every element of a short vector; of a longer one the first block's and the
    last ones, and some on both sides of the first tile's edge."""
    if P <= 20_000:
        return np.arange(P)
    return np.unique(np.concatenate([np.arange(0, 1100), np.arange(8100, 8300), np.arange(P - 1100, P)]))


def _oracle(G, hp, P, n, worker, tau, h, ts, bf16, idx):
    ohp = O.Hyper(lr=0.01, sigma=0.1, momentum=hp.momentum, eps=hp.eps, kappa=hp.kappa,
                  pi_mode=hp.pi_mode, kappa_mode=hp.kappa_mode, pull_mode=hp.pull_mode,
                  rule=hp.rule, bf16=bf16, proxy=hp.proxy_mode, seed=77)
    st = O.State.initial(n, idx.size)
    O.run(ohp, P, st, idx, h[idx], ts[idx], worker, tau)
    return st


def _case(G, P, n, T, K, hp, bf16=False, policy=0, law=0, p0=0.0, p1=0.0, chunks=(0,)):
    """chunks: lengths of the gem_sim_run calls (0: one call of T commits)."""
    from paper_1805_08469_amd.workloads import make_problem
    P = _size(P)
    idx = _sample(P)
    print(f"[run] P={P} n={n} T={T} K={K} bf16={bf16} policy={policy} chunks={chunks}", flush=True)
    h, ts = make_problem(P, 1e-3, 1.0, 3)
    worker, tau = G.gem_schedule_make(n, T, law, p0, p1, seed=n + T, pull_mode=hp.pull_mode)
    st = _oracle(G, hp, P, n, worker, tau, h, ts, bf16, idx)
    for c in chunks:
        with G.Gem(P, n, hp) as g:
            g.set_cache_policy(policy)
            g.set_quadratic(h, ts, 0.01, 0.1, 77, bf16=bf16)
            for j in range(0, T, c or T):
                g.sim_run(worker[j:j + (c or T)], tau[j:j + (c or T)], K)
            assert g.clock == st.t and np.array_equal(g.pull_clocks(), st.pc)
            theta, S, M = (g.theta(), g.S(), g.M()) if idx.size == P else g.gather(idx)
            assert_parity(f"theta (calls of {c})", theta, st.theta)
            assert_parity(f"S (calls of {c})", S, st.S)
            assert_parity(f"M (calls of {c})", M, st.M)
            s = g.stats()
            assert s.commits == T
            if c == 0:
                assert s.passes == -(-T // K)


@pytest.mark.parametrize("P", [1, 4, 63, 1025, "+1", "+63", "+1027", "+8193"])
def test_sizes(G, P):
    _case(G, P, 7, 150, 16, _hp(G))


@pytest.mark.parametrize("proxy", [0, 1])
@pytest.mark.parametrize("n", [1, 5, 6, 7, 10, 11, 13, 14, 20, 21, 101, 260])
def test_worker_counts(G, n, proxy):
    _case(G, "+1100", n, 600, 8, _hp(G, proxy_mode=proxy))


@pytest.mark.parametrize("P", [300, "+300"])
@pytest.mark.parametrize("T", [2, 3, 4, 993, 994, 2 * 993 + 1])
def test_launch_lengths(G, T, P):
    _case(G, P, 20, T, 1, _hp(G))


MODES = {
    "kappa": dict(kappa=2.0), "sqrt_kappa": dict(kappa=3.0, kappa_mode=1), "pre_pull": dict(pull_mode=1),
    "downpour": dict(rule=1, momentum=0.0), "adaptive": dict(rule=2), "tiny_eps": dict(eps=1e-30),
    "shared_kappa": dict(proxy_mode=1, kappa=2.0), "shared_tiny_eps": dict(proxy_mode=1, eps=1e-25),
    "shared_pre_pull": dict(proxy_mode=1, pull_mode=1), "big_eps": dict(eps=1e-3),
    "literal_big_eps": dict(pi_mode=1, eps=0.5),   # (an eps that keeps its values finite)
}


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("P,bf16", [(2050, False), (66, True), ("+2050", False), ("+66", True)])
def test_modes(G, mode, P, bf16):
    """One call (a run), and calls of one pass (the pass kernels)."""
    _case(G, P, 9, 520, 16, _hp(G, **MODES[mode]), bf16=bf16, chunks=(0, 16))


@pytest.mark.parametrize("P", [200, "+200"])
@pytest.mark.parametrize("T", [494, 495, 496, 991])
def test_adaptive_launch_lengths(G, T, P):
    _case(G, P, 12, T, 4, _hp(G, rule=G.GEM_RULE_ADAPTIVE))


@pytest.mark.parametrize("T", [23, 24, 25, 48, 49])
@pytest.mark.parametrize("n,P", [(1, 64), (2, 65), (5, 129)])
def test_short_vector_phases(G, T, n, P):
    """The short-vector kernel at the edges of its phases of 24 commits and of its
    blocks of 64 elements, with workers that commit twice in a row."""
    _case(G, P, n, T, 1, _hp(G), bf16=(T == 25))


@pytest.mark.parametrize("n", [127, 128, 129])
def test_short_vector_worker_limit(G, n):
    """128 workers' rows are held in LDS; a launch of more takes the other kernel."""
    from paper_1805_08469_amd.workloads import make_problem
    P, T = 700, 1500
    h, ts = make_problem(P, 1e-3, 1.0, 3)
    worker = np.arange(T, dtype=np.int32) * 7 % n
    hp = _hp(G)
    st = _oracle(G, hp, P, n, worker, None, h, ts, False, np.arange(P))
    with G.Gem(P, n, hp) as g:
        g.set_quadratic(h, ts, 0.01, 0.1, 77)
        g.sim_run(worker, None, 8)
        assert_parity("theta", g.theta(), st.theta)
        assert_parity("S", g.S(), st.S)
        assert_parity("M", g.M(), st.M)


LONG = [("kappa", 9, 520, False), ("adaptive", 9, 991, True), ("adaptive", 5, 496, False),
        ("downpour", 9, 130, True), ("pre_pull", 9, 520, False), ("tiny_eps", 9, 130, True),
        ("shared_kappa", 14, 300, False), ("shared_pre_pull", 9, 300, True),
        ("shared_tiny_eps", 9, 300, False), ("default", 1, 40, False), ("default", 5, 600, True),
        ("default", 7, 993, False), ("default", 11, 994, False), ("default", 101, 600, True),
        ("shared", 10, 600, False), ("shared", 11, 600, True), ("default", 20, 3, False)]


@pytest.mark.parametrize("policy", [0, 1, 2])
@pytest.mark.parametrize("mode,n,T,bf16", LONG)
def test_long_vectors(G, mode, n, T, bf16, policy):
    """The run kernel under each cache policy, a pass of one commit each."""
    from paper_1805_08469_amd.workloads import make_problem
    P = _size("+1029")
    hp = _hp(G, **{**MODES, "default": {}, "shared": dict(proxy_mode=1)}[mode])
    h, ts = make_problem(P, 1e-3, 1.0, 3)
    worker, tau = G.gem_schedule_make(n, T, 0, 0.0, 0.0, seed=n + T, pull_mode=hp.pull_mode)
    idx = _sample(P)
    st = _oracle(G, hp, P, n, worker, tau, h, ts, bf16, idx)
    print(f"[long] {mode} n={n} T={T} bf16={bf16} policy={policy} P={P}", flush=True)
    with G.Gem(P, n, hp) as g:
        g.set_cache_policy(policy)
        g.set_quadratic(h, ts, 0.01, 0.1, 77, bf16=bf16)
        g.sim_run(worker, tau, 1)
        theta, S, M = g.gather(idx)
        assert_parity("theta", theta, st.theta)
        assert_parity("S", S, st.S)
        assert_parity("M", M, st.M)


@pytest.mark.parametrize("policy", [1, 2])
@pytest.mark.parametrize("proxy", [0, 1])
def test_policies_and_heavy_tails(G, policy, proxy):
    """Both cache policies, a Pareto schedule (runs of one worker), in the run
    kernel and in the pass kernels of every depth (calls of 1, 8 and 32 commits)."""
    _case(G, "+3000", 30, 320, 32, _hp(G, proxy_mode=proxy), bf16=True, policy=policy, law=3, p0=1.5,
          p1=1 / 3, chunks=(0, 1, 8, 32))


@pytest.mark.parametrize("P", [1030, "+1030"])
def test_literal_pi_with_nan(G, P):
    """The literal rule diverges to infinities and NaN: the same ones."""
    n, T = 6, 400
    hp = _hp(G, pi_mode=G.GEM_PI_LITERAL)
    _case(G, P, n, T, 8, hp, chunks=(0, 8))


@pytest.mark.parametrize("P", [1, 3, 4, 5, 8191, 8192, 8195, 24_581])
def test_read_state_into_any_alignment(G, P):
    """Rows read to device addresses 0 to 3 elements past a 16-byte boundary,
    and one byte off: the same elements, and nothing beside them."""
    import torch
    n = 3
    theta = np.random.default_rng(P).standard_normal(P).astype(np.float32)
    with G.Gem(P, n) as g:
        G.gem_set_theta(g.h, theta)
        raw = torch.zeros(4 * P + 64, dtype=torch.uint8, device="cuda")
        for off in (0, 4, 8, 12, 1):
            raw.fill_(0xAB)
            rc = G.lib().gem_read_state(g.h, 2, G.GEM_SNAPSHOT, raw.data_ptr() + 16 + off, 1)
            assert rc == G.GEM_OK
            got = raw.cpu().numpy()
            assert np.array_equal(got[16 + off:16 + off + 4 * P], theta.view(np.uint8)), off
            assert (got[:16 + off] == 0xAB).all() and (got[16 + off + 4 * P:] == 0xAB).all(), off
