"""GPU parity of the batched path (cfet_batch_*) against the CPU FP64 oracle.

Each instance of a batch is an independent trajectory; the oracle propagates
them one after another (oracle.cfet.propagate_batch).  Bar: relative 2-norm
1e-10 per instance for the same scheme, Krylov bound and tolerance, and the
same number of H applications per instance (the adaptive Krylov dimension is
an integer decided in FP64 on both sides).
"""
import numpy as np
import pytest

from oracle import cfet as O
from paper_1102_5071_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1102_5071_amd.binding")

TOL = 1e-10


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    B.load()
    yield
    torch.cuda.synchronize()


def rel(a, b):
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / (nb if nb > 0 else 1.0)


def mixed_batch(seed=0):
    """Ragged batch exercising every layout case: shared driven operators,
    per-instance diagonal H0, per-instance off-diagonal H0, an H0 shared by two
    instances, two driven terms, a dimension below m, and a zero state."""
    rng = np.random.default_rng(seed)
    ops, insts = [], []
    sx = {}

    def sxop(L):
        if L not in sx:
            sx[L] = len(ops)
            ops.append(I.sigma_x_sum(L))
        return sx[L]

    for L in (3, 5, 4, 5, 6, 3, 7, 5):
        h = rng.uniform(-1, 1, L)
        ops.append(I.ising_chain(L, 1.0, h))
        insts.append({"h0": len(ops) - 1, "hk": [sxop(L)],
                      "drives": [{"kind": "cos", "A": float(rng.uniform(0.2, 1.5)),
                                  "omega": float(rng.uniform(0.5, 3.0)), "phi": 0.3}],
                      "psi0": I.random_state(1 << L, rng)})
    # off-diagonal H0 (Heisenberg), per instance
    for L in (4, 5):
        ops.append(I.heisenberg_chain(L, 1.0, rng.uniform(-1, 1, L)))
        insts.append({"h0": len(ops) - 1, "hk": [sxop(L)],
                      "drives": [{"kind": "sin2cos", "A": 0.7, "omega": 1.1, "phi": 0.0,
                                  "Tp": 5.0}],
                      "psi0": I.random_product_state(L, rng)})
    # one H0 shared by two instances (then it is read once for both)
    ops.append(I.heisenberg_chain(4, 0.8, rng.uniform(-1, 1, 4)))
    shared = len(ops) - 1
    for A in (0.4, 1.3):
        insts.append({"h0": shared, "hk": [sxop(4)],
                      "drives": [{"kind": "cos", "A": A, "omega": 2.0, "phi": 0.0}],
                      "psi0": I.random_state(16, rng)})
    # two driven terms (circular drive) on a chain of 3
    ops.append(I.sigma_y_sum(3))
    sy3 = len(ops) - 1
    ops.append(I.ising_chain(3, 1.0, rng.uniform(-1, 1, 3)))
    insts.append({"h0": len(ops) - 1, "hk": [sxop(3), sy3],
                  "drives": [{"kind": "cos", "A": 0.9, "omega": 1.5, "phi": 0.0},
                             {"kind": "cos", "A": 0.9, "omega": 1.5, "phi": -np.pi / 2}],
                  "psi0": I.random_state(8, rng)})
    # dimension 4 < m, and a zero state
    ops.append(I.ising_chain(2, 1.0, rng.uniform(-1, 1, 2)))
    insts.append({"h0": len(ops) - 1, "hk": [sxop(2)],
                  "drives": [{"kind": "cos", "A": 1.0, "omega": 1.0, "phi": 0.0}],
                  "psi0": I.random_state(4, rng)})
    ops.append(I.ising_chain(4, 1.0, rng.uniform(-1, 1, 4)))
    insts.append({"h0": len(ops) - 1, "hk": [sxop(4)],
                  "drives": [{"kind": "cos", "A": 1.0, "omega": 1.0, "phi": 0.0}],
                  "psi0": np.zeros(16, complex)})
    return ops, insts


def oracle_run(ops, insts, t0, dt, nsteps, scheme, m, tol):
    resolved = [{"H0": ops[i["h0"]], "Hk": [ops[k] for k in i["hk"]], "drives": i["drives"],
                 "psi0": i["psi0"]} for i in insts]
    stats = []
    outs = O.propagate_batch(resolved, t0, dt, nsteps, scheme, m, tol, stats=stats)
    return outs, [s["n_matvec"] for s in stats]


def gpu_run(ops, insts, t0, dt, nsteps, scheme, m, tol, **kw):
    with B.BatchPropagator(ops, insts, **kw) as P:
        psi = torch.from_numpy(np.concatenate([i["psi0"] for i in insts])).to("cuda")
        P.propagate(psi, t0, dt, nsteps, scheme, m, tol)
        st = P.stats()
        mv = P.instance_matvecs()
        out = [x.cpu().numpy() for x in P.split(psi)]
    assert st["status"] == 0, st
    return out, mv, st


@pytest.mark.parametrize("tol", [0.0, 1e-10])
@pytest.mark.parametrize("scheme", ["CF4:2", "CF6:5Opt"])
def test_mixed_batch_matches_oracle(tol, scheme):
    ops, insts = mixed_batch(1)
    dt, nsteps, m = 0.05, 12, 12
    ref, ref_mv = oracle_run(ops, insts, 0.2, dt, nsteps, scheme, m, tol)
    out, mv, st = gpu_run(ops, insts, 0.2, dt, nsteps, scheme, m, tol)
    for t, (a, b) in enumerate(zip(out, ref)):
        assert rel(a, b) <= TOL, (t, rel(a, b))
    assert list(mv) == list(ref_mv)
    assert st["ninst"] == len(insts)
    assert st["graph"] == 1
    if tol > 0:
        assert st["early_stops"] > 0
        assert st["max_m_eff"] <= m


def test_graph_and_direct_launches_agree_exactly():
    ops, insts = mixed_batch(2)
    a, mva, _ = gpu_run(ops, insts, 0.0, 0.04, 6, "CF4:2", 10, 1e-10, autotune=False)
    b, mvb, st = gpu_run(ops, insts, 0.0, 0.04, 6, "CF4:2", 10, 1e-10, graph=False,
                         autotune=False)
    assert st["graph"] == 0
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    assert list(mva) == list(mvb)


def test_split_calls_equal_one_call():
    ops, insts = mixed_batch(3)
    with B.BatchPropagator(ops, insts) as P:
        psi = torch.from_numpy(np.concatenate([i["psi0"] for i in insts])).to("cuda")
        ref = psi.clone()
        P.propagate(ref, 0.1, 0.03, 10, "CF4:2", 12, 1e-10)
        P.propagate(psi, 0.1, 0.03, 4, "CF4:2", 12, 1e-10)
        P.propagate(psi, 0.1 + 4 * 0.03, 0.03, 6, "CF4:2", 12, 1e-10)
        a = psi.cpu().numpy()
        b = ref.cpu().numpy()
    assert rel(a, b) < 1e-12


def test_more_instances_than_one_group():
    # 70 instances sharing sum sx of L = 3: split into groups of at most 64 instances
    rng = np.random.default_rng(7)
    ops = [I.sigma_x_sum(3)]
    insts = []
    for t in range(70):
        ops.append(I.ising_chain(3, 1.0, rng.uniform(-1, 1, 3)))
        insts.append({"h0": len(ops) - 1, "hk": [0],
                      "drives": [{"kind": "cos", "A": float(rng.uniform(0.2, 1.5)),
                                  "omega": float(rng.uniform(0.5, 3)), "phi": 0.0}],
                      "psi0": I.random_state(8, rng)})
    ref, ref_mv = oracle_run(ops, insts, 0.0, 0.05, 5, "CF4:2", 8, 1e-10)
    out, mv, st = gpu_run(ops, insts, 0.0, 0.05, 5, "CF4:2", 8, 1e-10)
    assert st["ngroups"] == 3          # power-of-two groups: 64 + 4 + 2
    for a, b in zip(out, ref):
        assert rel(a, b) <= TOL
    assert list(mv) == list(ref_mv)


def test_batched_ising_config_reduced():
    # the many-trajectory workload at reduced size: 12 chains, L = 8..12
    Bt = I.config_batched(n_traj=12, L_min=8, L_max=12, seed=5, nsteps=20)
    insts = Bt.instances
    ref, ref_mv = oracle_run(Bt.ops, insts, 0.0, Bt.dt, 20, Bt.scheme, Bt.m, Bt.tol)
    out, mv, st = gpu_run(Bt.ops, insts, 0.0, Bt.dt, 20, Bt.scheme, Bt.m, Bt.tol)
    for a, b in zip(out, ref):
        assert rel(a, b) <= TOL
        assert abs(np.linalg.norm(a) - 1.0) < 1e-10
    assert list(mv) == list(ref_mv)
    assert st["max_m_eff"] < Bt.m


def test_batch_argument_errors():
    ops, insts = mixed_batch(4)
    with B.BatchPropagator(ops, insts) as P:
        with pytest.raises(ValueError):
            P.propagate(torch.zeros(P.total - 1, dtype=torch.complex128, device="cuda"),
                        0.0, 0.1, 1, "CF4:2", 8)
        psi = torch.zeros(P.total, dtype=torch.complex128, device="cuda")
        for bad in [dict(m=0), dict(m=65), dict(tol=-1.0), dict(nsteps=-1),
                    dict(scheme=99)]:
            kw = dict(t0=0.0, dt=0.1, nsteps=1, scheme="CF4:2", m=8, tol=0.0)
            kw.update(bad)
            with pytest.raises(B.CfetError) as ei:
                P.propagate(psi, **kw)
            assert ei.value.code == 1
        P.propagate(psi, 0.0, 0.1, 0, "CF4:2", 8)  # nsteps = 0 is a no-op
        assert not psi.any()


def layout_batch():
    """The mixed batch plus two longer chains, so that in every launch layout
    some group spans several blocks (block partials summed across blocks)."""
    ops, insts = mixed_batch(4)
    rng = np.random.default_rng(44)
    for L in (11, 12):
        ops.append(I.sigma_x_sum(L))
        sx = len(ops) - 1
        ops.append(I.ising_chain(L, 1.0, rng.uniform(-1, 1, L)))
        insts.append({"h0": len(ops) - 1, "hk": [sx],
                      "drives": [{"kind": "cos", "A": 0.8, "omega": 1.7, "phi": 0.1}],
                      "psi0": I.random_state(1 << L, rng)})
    return ops, insts


@pytest.fixture(scope="module")
def layout_case():
    ops, insts = layout_batch()
    ref, ref_mv = oracle_run(ops, insts, 0.1, 0.04, 4, "CF4:2", 12, 1e-10)
    return ops, insts, ref, ref_mv


@pytest.mark.parametrize("threads", [128, 256, 512])
def test_every_launch_layout_matches_oracle(layout_case, threads):
    # the create-time tuner may keep any of the twelve layouts: each one,
    # fixed with cfet_batch_set_layout, against the oracle (graph replays,
    # re-recorded after each change of layout)
    ops, insts, ref, ref_mv = layout_case
    psi0 = np.concatenate([i["psi0"] for i in insts])
    with B.BatchPropagator(ops, insts, autotune=False) as P:
        before = P.instance_matvecs()
        for rows in (2, 4, 8, 16):
            P.set_layout(threads, rows)
            psi = torch.from_numpy(psi0).to("cuda")
            P.propagate(psi, 0.1, 0.04, 4, "CF4:2", 12, 1e-10)
            st = P.stats()
            assert st["status"] == 0 and st["graph"] == 1, st
            assert (st["block_threads"], st["unroll"]) == (threads, rows)
            mv = P.instance_matvecs()
            assert list(mv - before) == list(ref_mv), (threads, rows)
            before = mv
            for t, (a, b) in enumerate(zip(P.split(psi), ref)):
                r = rel(a.cpu().numpy(), b)
                assert r <= TOL, (threads, rows, t, r)


def test_autotune_keeps_the_documented_layout(layout_case):
    # of the twelve timed layouts, the kept one is within 3 % of the fastest,
    # covers the most rows per block among those, and of equals has the
    # fewest threads per block; the batch then matches the oracle
    ops, insts, ref, ref_mv = layout_case
    with B.BatchPropagator(ops, insts) as P:
        st = P.stats()
        t = st["tune_us"]
        assert len(t) == 12 and all(x > 0 for x in t), t
        fastest = min(t)
        cands = [(threads, rows) for threads in (128, 256, 512) for rows in (2, 4, 8, 16)]
        ok = [c for c, x in zip(cands, t) if x <= fastest * 1.03]
        most = max(th * r for th, r in ok)
        want = min((c for c in ok if c[0] * c[1] == most), key=lambda c: c[0])
        assert (st["block_threads"], st["unroll"]) == want, (st, t)
        psi = torch.from_numpy(np.concatenate([i["psi0"] for i in insts])).to("cuda")
        P.propagate(psi, 0.1, 0.04, 4, "CF4:2", 12, 1e-10)
        assert P.stats()["status"] == 0
        for k, (a, b) in enumerate(zip(P.split(psi), ref)):
            r = rel(a.cpu().numpy(), b)
            assert r <= TOL, (want, k, r)


def test_set_layout_rejects_other_values():
    ops, insts = mixed_batch(5)
    with B.BatchPropagator(ops, insts, autotune=False) as P:
        for bad in ((64, 8), (1024, 8), (256, 3), (256, 32), (256, 0)):
            with pytest.raises(B.CfetError):
                P.set_layout(*bad)
        P.set_layout(512, 2)
        assert (P.stats()["block_threads"], P.stats()["unroll"]) == (512, 2)


def test_status_starts_clear_without_autotune():
    # the latched device status must read CFET_OK on a batch created without
    # the layout timing, also when its device memory was used before
    # (regression: it was left as allocated)
    ops, insts = layout_batch()
    psi0 = np.concatenate([i["psi0"] for i in insts])
    for _ in range(3):
        with B.BatchPropagator(ops, insts, autotune=False) as P:
            psi = torch.from_numpy(psi0).to("cuda")
            P.propagate(psi, 0.0, 0.04, 2, "CF4:2", 12, 1e-10)
            assert P.stats()["status"] == 0
    with B.BatchPropagator(ops, insts, autotune=False) as P:
        assert P.stats()["status"] == 0


@pytest.mark.parametrize("sizes", [
    [(1, 3), (2, 1), (3, 2), (6, 64), (9, 9)],     # within one tile
    [(11, 2), (12, 1), (12, 2), (13, 1), (10, 7)],  # a full tile, the first flip above it
    [(15, 1), (13, 8), (14, 3)],                    # flips above the tile gathered
    [(16, 1), (13, 12), (12, 65)],                  # the second sweep, fewest and many instances
    [(16, 32), (17, 2)],                            # the largest groups it serves
    [(16, 64), (18, 9)],                            # more instances than such a group holds
], ids=str)
def test_flip_sweeps_match_oracle(sizes):
    rng = np.random.default_rng(7)
    ops, insts = [], []
    for L, count in sizes + [(17, 8)]:              # (the sweeps start at 2^20 elements)
        ops.append(I.sigma_x_sum(L, rng.uniform(0.5, 1.5, L)))
        hk = len(ops) - 1
        for j in range(count):
            ops.append(I.ising_chain(L, 1.0, rng.uniform(-1, 1, L)))
            psi0 = I.random_state(1 << L, rng)
            insts.append({"h0": len(ops) - 1, "hk": [hk],
                          "drives": [{"kind": "cos", "A": float(rng.uniform(0.2, 1.5)),
                                      "omega": float(rng.uniform(0.5, 3.0)), "phi": 0.3}],
                          "psi0": 0 * psi0 if L < 13 and j == 1 else psi0})
    args = (0.1, 0.03, 1, "CF4:2", 24, 1e-10)
    refs, rmv = oracle_run(ops, insts, *args)
    outs, mv, _ = gpu_run(ops, insts, *args)
    assert list(mv) == list(rmv)
    for r, o in zip(refs, outs):
        assert rel(o, r) <= 1e-11


@pytest.mark.parametrize("sites,groups", [(6, 1), (7, 2)])
def test_few_flips_per_row_keep_the_gathering_product(sites, groups):
    # 64 chains of 2^16 rows: one group, unless the flip sweeps take groups of 2^21
    # elements; they do from seven flips a row
    L, rng = 16, np.random.default_rng(sites)
    X = I.sigma_x_sum(L)
    at = np.arange(sites) * L // sites
    ops = [I.CSR(X.n, np.arange(X.n + 1, dtype=np.int64) * sites,
                 X.col.reshape(-1, L)[:, at].ravel(), X.val.reshape(-1, L)[:, at].ravel())]
    insts = []
    for j in range(64):
        ops.append(I.ising_chain(L, 1.0, rng.uniform(-1, 1, L)))
        insts.append({"h0": len(ops) - 1, "hk": [0],
                      "drives": [{"kind": "cos", "A": float(rng.uniform(0.2, 1.5)),
                                  "omega": float(rng.uniform(0.5, 3.0)), "phi": 0.3}],
                      "psi0": I.random_state(1 << L, rng)})
    with B.BatchPropagator(ops, insts) as P:
        psi = torch.from_numpy(np.concatenate([i["psi0"] for i in insts])).to("cuda")
        P.propagate(psi, 0.1, 0.03, 1, "CF4:2", 24, 1e-10)
        st, mv = P.stats(), P.instance_matvecs()
        outs = [v.cpu().numpy() for v in P.split(psi)]
    assert st["status"] == 0 and st["ngroups"] == groups
    pick = [0, 31, 32, 63]
    resolved = [{"H0": ops[insts[j]["h0"]], "Hk": [ops[0]], "drives": insts[j]["drives"],
                 "psi0": insts[j]["psi0"]} for j in pick]
    stats = []
    refs = O.propagate_batch(resolved, 0.1, 0.03, 1, "CF4:2", 24, 1e-10, stats=stats)
    for j, r, s in zip(pick, refs, stats):
        assert rel(outs[j], r) <= 1e-11 and mv[j] == s["n_matvec"]
