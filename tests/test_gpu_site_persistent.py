"""The persistent kernels on the site-operator form (one workgroup up to 2^10
rows, a team of workgroups up to 2^14) against the CPU oracle, at every
launch shape: fewer rows than a wavefront, one row per thread, two (2^10 rows),
teams of 8 to 32 blocks with one row per thread.

Bars: propagation 1e-10 and the oracle's number of H applications; gradient as
in the gradient tests (1e-8 of its largest entry).
"""
import numpy as np
import pytest

from oracle import adjoint as A
from oracle import cfet as O
from paper_1102_5071_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1102_5071_amd.binding")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    B.load()
    yield
    torch.cuda.synchronize()


def dev(v):
    return torch.from_numpy(np.ascontiguousarray(v, dtype=np.complex128)).to("cuda")


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def chain(model, L, seed):
    rng = np.random.default_rng(seed)
    if model == "spins":                       # two drives, complex values
        H0, Hk, drives = I.noninteracting_spins(L, 0.3, 0.7, 1.1)
    elif model == "y":                         # one drive with complex values
        H0, Hk = I.heisenberg_chain(L, 1.0, rng.uniform(-1, 1, L)), [I.sigma_y_sum(L)]
        drives = [{"kind": "cos", "A": 0.8, "omega": 2.0, "phi": 0.3}]
    elif model == "driven_diag":               # the diagonal is the driven term
        H0 = I.sigma_x_sum(L, rng.uniform(0.5, 1.5, L))
        Hk = [I.ising_chain(L, 1.0, rng.uniform(-1, 1, L))]
        drives = [{"kind": "cos", "A": 0.8, "omega": 2.0, "phi": 0.3}]
    else:
        H0 = (I.heisenberg_chain if model == "heisenberg" else I.ising_chain)(
            L, 1.0, rng.uniform(-1, 1, L))
        Hk = [I.sigma_x_sum(L)]
        drives = [{"kind": "cos", "A": 0.8, "omega": 2.0, "phi": 0.3}]
    return H0, Hk, drives, I.random_state(1 << L, rng)


@pytest.mark.parametrize("L", list(range(1, 17)))
@pytest.mark.parametrize("model", ["ising", "heisenberg", "spins", "y", "driven_diag"])
def test_propagate_matches_oracle(model, L):
    if model == "heisenberg" and L == 1:
        pytest.skip("a chain of one site has no bond")
    H0, Hk, drives, psi0 = chain(model, L, 10 * L)
    steps, m = (3, 12) if L < 14 else (1, 10)
    scheme = "CF6:5Opt" if L < 12 else "CF4:2"
    stats = {}
    ref = O.propagate(H0, Hk, drives, psi0, 0.1, 0.04, steps, scheme, m=m, stats=stats)
    with B.Propagator(H0, Hk, drives) as P:
        psi = dev(psi0)
        P.propagate(psi, 0.1, 0.04, steps, scheme, m)
        st = P.stats()
        out = psi.cpu().numpy()
        again = dev(psi0)
        P.propagate(again, 0.1, 0.04, steps, scheme, m)
        assert torch.equal(again, psi)          # fixed order of every sum
    assert st["status"] == 0
    assert B.PATH_NAMES[st["path"]] == ("single" if L <= 10 else "coop" if L <= 15 else "multi")
    assert st["matvecs"] == stats["n_matvec"]
    assert abs(st["last_norm"] - 1.0) < 1e-10
    assert rel(out, ref) <= 1e-10


@pytest.mark.parametrize("L,m", [(4, 64), (9, 64), (12, 1), (12, 2), (13, 40), (5, 3)])
def test_krylov_sizes(L, m):
    H0, Hk, drives, psi0 = chain("heisenberg", L, L + m)
    dt = 0.02 if m > 3 else 1e-4
    ref = O.propagate(H0, Hk, drives, psi0, 0.0, dt, 2, "CF4:2", m=m)
    with B.Propagator(H0, Hk, drives) as P:
        psi = dev(psi0)
        P.propagate(psi, 0.0, dt, 2, "CF4:2", m)
        assert P.stats()["status"] == 0
        assert rel(psi.cpu().numpy(), ref) <= 1e-10


@pytest.mark.parametrize("L", [7, 13])
def test_early_stop_zero_state_and_faults(L):
    n = 1 << L
    H0 = I.diagonal(np.full(n, 0.7))
    plus = np.full(n, 2.0 ** (-L / 2), dtype=complex)
    with B.Propagator(H0, [I.sigma_x_sum(L)],
                      [{"kind": "cos", "A": 0.5, "omega": 0.0, "phi": 0.0}]) as P:
        psi = dev(plus)
        P.propagate(psi, 0.0, 0.2, 2, "CF4:2", 10)
        st = P.stats()
        out = psi.cpu().numpy()
        assert st["status"] == 0 and st["matvecs"] == 4 and st["breakdowns"] == 4
        assert rel(out, plus * np.exp(-0.4j * (0.7 + 0.5 * L))) < 1e-13
        zero = dev(np.zeros(n))
        P.propagate(zero, 0.0, 0.2, 2, "CF4:2", 10)
        st = P.stats()
        assert st["status"] == 0 and st["min_m_eff"] == 0 and not torch.any(zero != 0)
        bad = dev(plus)
        bad[n // 2] = float("nan")
        P.propagate(bad, 0.0, 0.2, 1, "CF4:2", 10)
        assert P.stats()["status"] != 0
        psi = dev(plus)
        P.propagate(psi, 0.0, 0.2, 2, "CF4:2", 10)
        assert P.stats()["status"] == 0 and np.array_equal(psi.cpu().numpy(), out)


@pytest.mark.parametrize("model,L", [("ising", 6), ("ising", 11), ("heisenberg", 12),
                                     ("driven_diag", 12), ("y", 12), ("heisenberg", 15)])
def test_gradient_matches_oracle(model, L):
    H0, Hk, _, psi0 = chain(model, L, 3 * L)
    rng = np.random.default_rng(L)
    K, steps, dt = 3, (6 if L < 15 else 3), 0.05
    u = rng.uniform(-1, 1, K)
    drives = [{"kind": "pwc", "t_edges": np.linspace(0.0, steps * dt, K + 1), "u": u}]
    target = I.random_state(1 << L, rng)
    F, g = A.fidelity_gradient(H0, Hk, drives, psi0, target, 0.0, dt, steps, "CF4:2", 14)[:2]
    with B.Propagator(H0, Hk, drives) as P:
        Fg, gg = P.gradient(dev(psi0), dev(target), 0.0, dt, steps, "CF4:2", 14)
    assert abs(Fg - F) <= 1e-10 * max(F, 1e-3)
    assert np.max(np.abs(gg - g)) <= 1e-8 * np.max(np.abs(g))


@pytest.mark.parametrize("L,N,scheme,m", [
    (6, 40, "CF4:2", 40),         # the whole pass kept, more than one wavefront of scalars
    (12, 45, "CF6:5Opt", 20),     # kept, the backward exponentials in two launches
    (14, 27, "CF6:5Opt", 64),     # recomputed by segments of two launches, the last shorter
    (9, 3, "CF8:11", 1),          # one vector per basis
])
def test_gradient_batches_match_one_exponential_at_a_time(L, N, scheme, m):
    H0, Hk, _, psi0 = chain("ising", L, L)
    rng = np.random.default_rng(L)
    u, dt = rng.uniform(-1, 1, 4), 0.01 if m > 1 else 1e-4
    drives = [{"kind": "pwc", "t_edges": np.linspace(0.0, N * dt, 5), "u": u}]
    target = I.random_state(1 << L, rng)
    got = []
    for path in (None, "multi"):
        with B.Propagator(H0, Hk, drives, path=path) as P:
            got.append(P.gradient(dev(psi0), dev(target), 0.0, dt, N, scheme, m))
            assert P.stats()["status"] == 0
    (F, g), (Fo, go) = got
    assert abs(F - Fo) <= 1e-10 * max(Fo, 1e-3)
    assert np.max(np.abs(g - go)) <= 1e-8 * np.max(np.abs(go))


@pytest.mark.parametrize("L", [8, 12])
def test_short_and_long_calls_agree(L):
    # weights in the launch's arguments (short calls) and in a device table
    H0, Hk, drives, psi0 = chain("spins", L, L)
    with B.Propagator(H0, Hk, drives) as P:
        a, b = dev(psi0), dev(psi0)
        P.propagate(a, 0.0, 0.0625, 8, "CF4:2", 12)       # 48 weights
        count = P.stats()["matvecs"]                      # (the state spans few vectors)
        assert count > 0
        for q in range(8):                                # 6 weights a call
            P.propagate(b, q * 0.0625, 0.0625, 1, "CF4:2", 12)
        assert P.stats()["matvecs"] == 2 * count
        torch.cuda.synchronize()
        assert torch.equal(a, b)


@pytest.mark.parametrize("L", [11, 12, 13, 14])
@pytest.mark.parametrize("sites", [[0], [2, -1], [-3, -2, -1]])
def test_few_driven_sites(L, sites):
    # fewer terms that leave a workgroup's rows than the kernel has places for
    X, k = I.sigma_x_sum(L), len(sites)
    Hk = type(X)(X.n, np.arange(X.n + 1, dtype=X.row_ptr.dtype) * k,
                 X.col.reshape(-1, L)[:, sites].ravel(), X.val.reshape(-1, L)[:, sites].ravel())
    H0, _, drives, psi0 = chain("ising", L, L)
    ref = O.propagate(H0, [Hk], drives, psi0, 0.0, 0.05, 2, "CF4:2", m=12)
    with B.Propagator(H0, [Hk], drives) as P:
        psi = dev(psi0)
        P.propagate(psi, 0.0, 0.05, 2, "CF4:2", 12)
        assert P.stats()["status"] == 0
        assert rel(psi.cpu().numpy(), ref) <= 1e-10


def test_two_streams_and_two_contexts():
    # two contexts in flight on two streams, teams of 32 and 16 blocks
    jobs = []
    for L in (13, 12):
        H0, Hk, drives, psi0 = chain("heisenberg", L, L)
        P = B.Propagator(H0, Hk, drives)
        ref = dev(psi0)
        P.propagate(ref, 0.0, 0.05, 4, "CF6:5Opt", 16)
        jobs.append((P, psi0, ref, torch.cuda.Stream()))
    torch.cuda.synchronize()
    outs = []
    for P, psi0, ref, s in jobs:
        psi = dev(psi0)
        torch.cuda.synchronize()
        outs.append(psi)
    for (P, psi0, ref, s), psi in zip(jobs, outs):
        for _ in range(1):
            P.propagate(psi, 0.0, 0.05, 4, "CF6:5Opt", 16, stream=s)
    torch.cuda.synchronize()
    for (P, psi0, ref, s), psi in zip(jobs, outs):
        assert P.stats()["status"] == 0 and torch.equal(psi, ref)
        P.close()


def test_a_team_that_does_not_form_is_reported():
    H0, Hk, drives, psi0 = chain("ising", 12, 5)
    with B.Propagator(H0, Hk, drives, test="no_team") as P:
        psi = dev(psi0)
        P.propagate(psi, 0.0, 0.05, 2, "CF4:2", 12)
        torch.cuda.synchronize()
        assert np.array_equal(psi.cpu().numpy(), psi0)
        with pytest.raises(B.CfetError) as e:       # the next call reports it
            P.propagate(psi, 0.0, 0.05, 2, "CF4:2", 12)
        assert B.ERRORS[e.value.code] == "CFET_EDEVICE"
        with pytest.raises(B.CfetError) as e:       # and so does a run that waits
            P.select_dt(psi, 0.0, 0.1, 2, "CF4:2", 12, 1.0, 1e-6)
        assert B.ERRORS[e.value.code] == "CFET_EDEVICE"
        assert P.stats()["status"] == e.value.code


@pytest.mark.parametrize("model,L", [("ising", 11), ("heisenberg", 12), ("spins", 12),
                                     ("y", 13), ("driven_diag", 13), ("ising", 14)])
def test_a_team_spread_over_the_xcds_gives_the_same_bits(model, L):
    # the exchange with device-scope stores, taken where no XCD holds a team
    H0, Hk, drives, psi0 = chain(model, L, 7 * L)
    rng = np.random.default_rng(L)
    n, N, dt = 1 << L, 6, 0.04
    pwc = [{"kind": "pwc", "t_edges": np.linspace(0.0, N * dt, 4), "u": rng.uniform(-1, 1, 3)}]
    target = I.random_state(n, rng)
    plus = np.full(n, 2.0 ** (-L / 2), dtype=complex)
    got = []
    for test in (None, "spread_team"):
        with B.Propagator(H0, Hk, drives, test=test) as P:
            psi = dev(psi0)
            P.propagate(psi, 0.1, dt, N, "CF6:5Opt", 14)
            zero = dev(np.zeros(n))
            P.propagate(zero, 0.1, dt, 1, "CF4:2", 14)
            st = P.stats()
            assert st["status"] == 0 and B.PATH_NAMES[st["path"]] == "coop"
            got.append([psi.cpu().numpy(), zero.cpu().numpy(), st["matvecs"], st["last_norm"]])
        # a recurrence that stops early
        with B.Propagator(I.diagonal(np.full(n, 0.7)), [I.sigma_x_sum(L)],
                          [dict(drives[0], omega=0.0)], test=test) as P:
            psi = dev(plus)
            P.propagate(psi, 0.0, 0.2, 2, "CF4:2", 10)
            st = P.stats()
            assert st["status"] == 0 and st["breakdowns"] == 4
            got[-1].append(psi.cpu().numpy())
        if len(Hk) == 1:
            with B.Propagator(H0, Hk, pwc, test=test) as P:
                got[-1] += P.gradient(dev(psi0), dev(target), 0.0, dt, N, "CF4:2", 14)
                assert P.stats()["status"] == 0
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("model,L", [("heisenberg", 8), ("spins", 9), ("ising", 10), ("ising", 12),
                                     ("heisenberg", 13)])
@pytest.mark.parametrize("power", [-513, 505])
def test_very_small_and_large_norms(model, L, power):
    # ||psi||^2 = 2^-1026: its reciprocal overflows, its root's does not.  Squares of
    # the elements round to multiples of 2^-1074, a part 2^(L - 49) of the sum at
    # most; a dozen vectors leave 1e-9 of that.
    H0, Hk, drives, psi0 = chain(model, L, L)
    with B.Propagator(H0, Hk, drives) as P:
        a, b = dev(psi0), dev(psi0 * 2.0 ** power)
        P.propagate(a, 0.0, 0.04, 2, "CF4:2", 12)
        P.propagate(b, 0.0, 0.04, 2, "CF4:2", 12)
        assert P.stats()["status"] == 0
    assert rel(b.cpu().numpy() * 2.0 ** -power, a.cpu().numpy()) < 1e-9


def test_gradient_in_little_free_memory():
    # 4100 small exponentials: their batches would take over 400 MiB; with less left
    # on the device they come in shorter ones
    L, N, dt = 2, 820, 0.01
    H0, Hk, _, psi0 = chain("ising", L, 1)
    rng = np.random.default_rng(2)
    drives = [{"kind": "pwc", "t_edges": np.linspace(0.0, N * dt, 5), "u": rng.uniform(-1, 1, 4)}]
    psi, target = dev(psi0), dev(I.random_state(1 << L, rng))
    with B.Propagator(H0, Hk, drives) as P:
        F, g = P.gradient(psi, target, 0.0, dt, N, "CF6:5Opt", 4)
        torch.cuda.empty_cache()
        hold = []
        for _ in range(3):
            spare = torch.cuda.mem_get_info()[0] - (200 << 20)
            if spare > 0:
                hold.append(torch.empty(spare, dtype=torch.uint8, device="cuda"))
        assert torch.cuda.mem_get_info()[0] <= 210 << 20
        Fs, gs = P.gradient(psi, target, 0.0, dt, N, "CF6:5Opt", 4)
        assert P.stats()["status"] == 0
        del hold
        torch.cuda.empty_cache()
    assert abs(Fs - F) <= 1e-12 and np.max(np.abs(gs - g)) <= 1e-10 * np.max(np.abs(g))


@pytest.mark.parametrize("sites,form", [(1, "merged"), (3, "merged"), (4, "site_persistent")])
def test_short_rows_of_two_sets_at_2_to_the_10(sites, form):
    # bonds and a few driven sites: rows of up to 13 entries stay on the CSR kernel
    L, rng = 10, np.random.default_rng(sites)
    X = I.sigma_x_sum(L)
    Hk = I.CSR(X.n, np.arange(X.n + 1, dtype=np.int64) * sites,
               X.col.reshape(-1, L)[:, :sites].ravel(), X.val.reshape(-1, L)[:, :sites].ravel())
    H0, _, drives, psi0 = chain("heisenberg", L, L)
    ref = O.propagate(H0, [Hk], drives, psi0, 0.0, 0.05, 2, "CF4:2", m=12)
    with B.Propagator(H0, [Hk], drives) as P:
        assert P.form() == form
        psi = dev(psi0)
        P.propagate(psi, 0.0, 0.05, 2, "CF4:2", 12)
        st = P.stats()
        assert st["status"] == 0 and B.PATH_NAMES[st["path"]] == "single"
        assert rel(psi.cpu().numpy(), ref) <= 1e-10
