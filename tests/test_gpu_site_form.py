"""The sweeps on the site-operator form (operators on 2^b rows whose entries
depend on one parity of the row's bits: sums of Pauli strings) against the
general sparse product and the CPU oracle.

The sizes take every tile of the sweeps (2^9 rows at 2^16, 2^10 at 2^17 and
2^18, 2^11 at 2^19 to 2^22, 2^12 in the second sweep of 2^21 and from 2^23), for
products with and without terms that a tile cannot hold; the recurrence and the
Chebyshev series are compared with the oracle up to 2^18 rows and with the
multi-kernel CSR path at 2^20 to 2^22, where the rows per thread differ.  Bars as elsewhere: apply 1e-14, propagation 1e-10, Chebyshev its
tolerance; H applications equal the oracle's.
"""
import numpy as np
import pytest

from oracle import cfet as O
from oracle import chebyshev as C
from paper_1102_5071_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1102_5071_amd.binding")

COS = [{"kind": "cos", "A": 0.7, "omega": 1.3, "phi": 0.2},
       {"kind": "cos", "A": 0.4, "omega": 0.9, "phi": -0.5}]


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


def from_columns(n, cols, vals, keep):
    """CSR of the entries (row, cols[j][row]) = vals[j][row] where keep[j][row]."""
    keep = np.stack(keep, axis=1)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(keep.sum(axis=1))
    return I.CSR(n, rp, np.stack(cols, axis=1)[keep].astype(np.int32),
                 np.stack(vals, axis=1)[keep].astype(complex))


def parity(x):
    x = x.copy()
    for s in (16, 8, 4, 2, 1):
        x ^= x >> s
    return x & 1


def strings(L, offs, rng, complex_values, sparse, diag):
    """A sum of terms with flips offs: v0 or v1 by the parity of a random mask
    (sparse: 0 on one parity, so half the rows store nothing)."""
    n = 1 << L
    r = np.arange(n)
    cols, vals, keep = [], [], []
    if diag:
        cols.append(r)
        vals.append(rng.uniform(-1, 1, n).astype(complex))
        keep.append(np.ones(n, bool))
    for j, off in enumerate(offs):
        kind = j % 3
        v = rng.standard_normal(2)
        if kind == 0:                               # one value everywhere
            val = np.full(n, v[0] + 0j)
            k = np.ones(n, bool)
        else:
            # Hermitian needs the parity over the flipped bits to be even for
            # real values and odd for imaginary ones of either sign
            mask = int(rng.integers(1, n)) | off
            odd = bin(mask & off).count("1") & 1
            if complex_values and kind == 2:
                mask = mask if odd else mask & ~(off & -off)
                val = 1j * v[0] * (1 - 2 * parity(r & mask))
                k = np.ones(n, bool)
            else:
                mask = mask & ~(off & -off) if odd else mask
                p = parity(r & mask)
                val = np.where(p == 1, v[0], 0.0 if sparse else v[1]).astype(complex)
                k = val != 0
        cols.append(r ^ off)
        vals.append(val)
        keep.append(k)
    return from_columns(n, cols, vals, keep)


def flips(L, rng, far):
    """Flips of single bits, neighbouring pairs and a few wider sets; with
    far, a set across the tile of the second sweep and the high bits."""
    offs = [1 << b for b in range(0, L, 2)] + [3 << b for b in range(0, L - 1, 3)]
    offs += [0b1011, 1 << (L - 1) | 1 << (L - 3), 0b11 << (L - 2) | 1]
    if far:
        offs += [1 << (L - 1) | 1 << 6]
    return sorted(set(offs))


@pytest.mark.parametrize("L", [16, 17, 18, 19, 21])
@pytest.mark.parametrize("complex_values", [False, True])
def test_apply_random_strings(L, complex_values):
    rng = np.random.default_rng(100 * L + complex_values)
    offs = flips(L, rng, far=L != 17)
    H0 = strings(L, offs[::2] if L > 19 else offs, rng, complex_values, sparse=True, diag=L != 18)
    Hk = [strings(L, offs[1::2], rng, complex_values, sparse=False, diag=False),
          strings(L, offs[:5], rng, complex_values, sparse=True, diag=False)]
    x = I.random_state(1 << L, rng)
    with B.Propagator(H0, Hk, COS, validate_hermitian=L == 16) as P:
        y = P.apply(dev(x), -0.37, [0.81, -1.3]).cpu().numpy()
        # the compact form's operator is one value per row and the terms
        assert P.stats()["matrix_bytes"] < 16 * (1 << L)
    ref = -0.37 * (H0.to_scipy() @ x) + 0.81 * (Hk[0].to_scipy() @ x) - 1.3 * (Hk[1].to_scipy() @ x)
    assert rel(y, ref) < 1e-14


def broken(H, how):
    """One entry of a spin operator changed: no parity describes it any more."""
    H = I.CSR(H.n, H.row_ptr.copy(), H.col.copy(), H.val.copy())
    if how == "value":          # a third value of one flip
        e = np.flatnonzero(H.col[H.row_ptr[77]:H.row_ptr[78]] != 77)[0] + H.row_ptr[77]
        H.val[e] *= 1.5
    elif how == "missing":      # stored as zero in one row
        e = np.flatnonzero(H.col[H.row_ptr[77]:H.row_ptr[78]] != 77)[0] + H.row_ptr[77]
        H.val[e] = 0.0
    return H


@pytest.mark.parametrize("how", ["value", "missing", "rows"])
def test_operators_off_the_form_keep_the_general_path(how):
    rng = np.random.default_rng(3)
    L = 16
    H0 = I.heisenberg_chain(L, 1.0, rng.uniform(-1, 1, L))
    H1 = I.sigma_x_sum(L)
    if how == "rows":           # 2^16 - 3 rows: a principal block
        n = H0.n - 3

        def cut(H):
            M = H.to_scipy()[:n, :n].tocsr()
            return I.CSR(n, M.indptr.astype(np.int64), M.indices.astype(np.int32),
                         M.data.astype(complex))
        H0, H1 = cut(H0), cut(H1)
    else:
        H1 = broken(H1, how)
    x = I.random_state(H0.n, rng)
    with B.Propagator(H0, [H1], COS[:1]) as P:
        y = P.apply(dev(x), 0.9, [-0.4]).cpu().numpy()
        assert P.stats()["matrix_bytes"] >= 20 * (H0.nnz + H1.nnz)
    assert rel(y, 0.9 * (H0.to_scipy() @ x) - 0.4 * (H1.to_scipy() @ x)) < 1e-14


@pytest.mark.parametrize("model,L,m", [("heisenberg", 16, 18), ("ising", 17, 12), ("spins", 16, 14),
                                       ("heisenberg", 18, 1), ("heisenberg", 16, 2)])
def test_propagate_matches_oracle(model, L, m):
    rng = np.random.default_rng(L + m)
    if model == "spins":
        H0, Hk, drives = I.noninteracting_spins(L, 0.3, 0.7, 1.1)
    else:
        h = rng.uniform(-1, 1, L)
        H0 = (I.heisenberg_chain if model == "heisenberg" else I.ising_chain)(L, 1.0, h)
        Hk, drives = [I.sigma_x_sum(L)], COS[:1]
    psi0 = I.random_product_state(L, rng)
    dt = 0.05 if m > 2 else 0.001
    with B.Propagator(H0, Hk, drives) as P:
        psi = dev(psi0)
        P.propagate(psi, 0.1, dt, 2, "CF4:2", m)
        st = P.stats()
        out = psi.cpu().numpy()
    ref = O.propagate(H0, Hk, drives, psi0, 0.1, dt, 2, "CF4:2", m=m)
    assert st["status"] == 0 and B.PATH_NAMES[st["path"]] == "multi"
    assert st["matvecs"] == 4 * m and abs(st["last_norm"] - np.linalg.norm(ref)) < 1e-10
    assert rel(out, ref) <= 1e-10


def test_early_stop_and_zero_state():
    # an eigenvector of the whole operator: the recurrence stops after one product
    L = 16
    H0 = I.diagonal(np.full(1 << L, 0.7))
    H1 = I.sigma_x_sum(L)
    plus = np.full(1 << L, 2.0 ** (-L / 2), dtype=complex)
    with B.Propagator(H0, [H1], [{"kind": "cos", "A": 0.5, "omega": 0.0, "phi": 0.0}]) as P:
        psi = dev(plus)
        P.propagate(psi, 0.0, 0.2, 1, "CF4:2", 10)
        st = P.stats()
        out = psi.cpu().numpy()
        assert st["status"] == 0 and st["matvecs"] == 2 and st["breakdowns"] == 2
        assert rel(out, plus * np.exp(-0.2j * (0.7 + 0.5 * L))) < 1e-13
        zero = dev(np.zeros(1 << L))
        P.propagate(zero, 0.0, 0.2, 1, "CF4:2", 10)
        assert P.stats()["status"] == 0 and not torch.any(zero != 0)
        # the context is clean again for the next state
        psi = dev(plus)
        P.propagate(psi, 0.0, 0.2, 1, "CF4:2", 10)
        assert np.array_equal(psi.cpu().numpy(), out)
        # not-a-number states are reported
        bad = dev(plus)
        bad[5] = float("nan")
        P.propagate(bad, 0.0, 0.2, 1, "CF4:2", 10)
        assert P.stats()["status"] != 0


@pytest.mark.parametrize("L", [16, 18])
def test_chebyshev_matches_oracle(L):
    p = I.config_heisenberg(L=L)
    with B.Propagator(p.H0, p.Hk, p.drives) as P:
        psi = dev(p.psi0)
        P.propagate_chebyshev(psi, 0.0, 0.05, 1, "CF4:2", 1e-12)
        st = P.stats()
        out = psi.cpu().numpy()
    ref = C.propagate_chebyshev(p.H0, p.Hk, p.drives, p.psi0, 0.0, 0.05, 1, "CF4:2", 1e-12)
    assert st["status"] == 0 and rel(out, ref) <= 1e-10


@pytest.mark.parametrize("dt", [0.0, 1e-13, 1e-7, 1e-5, 1e-4, 5e-4, 1e-3, 2e-3, 4e-3, 8e-3])
def test_chebyshev_short_series(dt):
    # psi takes three terms at a time: series of zero to a dozen terms
    p = I.config_heisenberg(L=16)
    with B.Propagator(p.H0, p.Hk, p.drives) as P:
        psi = dev(p.psi0)
        P.propagate_chebyshev(psi, 0.0, dt, 1, "CF4:2", 1e-12)
        assert P.stats()["status"] == 0
        out = psi.cpu().numpy()
    ref = C.propagate_chebyshev(p.H0, p.Hk, p.drives, p.psi0, 0.0, dt, 1, "CF4:2", 1e-12)
    assert rel(out, ref) <= 1e-12


def test_static_and_streams_and_repeat():
    # the allocation-free entry point, another stream, and bit-equal repeats
    p = I.config_heisenberg(L=16)
    with B.Propagator(p.H0, p.Hk, p.drives) as P:
        a = dev(p.psi0)
        P.propagate(a, 0.0, 0.05, 1, "CF4:2", 12)
        b = dev(p.psi0)
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        P.propagate(b, 0.0, 0.05, 1, "CF4:2", 12, stream=s)
        s.synchronize()
        c = dev(p.psi0)
        P.propagate_static(c, 0.0, 0.05, 1, "CF4:2", 12)
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(a, c)


def driven_sites(L, k):
    """sigma^x on the k highest sites."""
    X = I.sigma_x_sum(L)
    return I.CSR(X.n, np.arange(X.n + 1, dtype=np.int64) * k,
                 X.col.reshape(-1, L)[:, L - k:].ravel(), X.val.reshape(-1, L)[:, L - k:].ravel())


@pytest.mark.parametrize("L,k,route", [
    (16, 2, "coop"), (16, 15, "coop"), (16, 16, "sweeps"),
    (17, 7, "coop"), (17, 8, "coop"), (17, 10, "sweeps"),
    (18, 1, "csr"), (18, 2, "csr"), (18, 3, "sweeps")])
def test_few_driven_sites_keep_the_csr_kernels(L, k, route):
    # 1 + k entries per row: rows that the cooperative kernel holds (16 at 2^16, 8
    # and one more at 2^17), or fewer than 2^20 entries
    rng = np.random.default_rng(L + k)
    H0, H1 = I.ising_chain(L, 1.0, rng.uniform(-1, 1, L)), driven_sites(L, k)
    psi0 = I.random_product_state(L, rng)
    with B.Propagator(H0, [H1], COS[:1]) as P:
        x = dev(psi0)
        y = P.apply(x, 0.9, [-0.4]).cpu().numpy()
        psi, che = x.clone(), x.clone()
        P.propagate(psi, 0.1, 0.02, 1, "CF4:2", 12)
        st = P.stats()
        P.propagate_chebyshev(che, 0.1, 0.02, 1, "CF4:2", 1e-12)
        assert P.stats()["status"] == 0
    assert B.PATH_NAMES[st["path"]] == ("coop" if route == "coop" else "multi")
    assert (st["matrix_bytes"] < 16 << L) == (route == "sweeps")
    ref = O.propagate(H0, [H1], COS[:1], psi0, 0.1, 0.02, 1, "CF4:2", m=12)
    assert rel(y, 0.9 * (H0.to_scipy() @ psi0) - 0.4 * (H1.to_scipy() @ psi0)) < 1e-14
    assert rel(psi.cpu().numpy(), ref) <= 1e-10
    assert rel(che.cpu().numpy(), ref) <= 1e-10


@pytest.mark.parametrize("model,L,form", [("ising", 16, False), ("heisenberg", 16, False),
                                          ("ising", 17, True)])
def test_one_product_of_few_entries_runs_on_the_csr_kernel(model, L, form):
    # below 9 * 2^18 entries: the same bits as on the multi-kernel CSR path
    rng = np.random.default_rng(L)
    h = rng.uniform(-1, 1, L)
    H0 = (I.heisenberg_chain if model == "heisenberg" else I.ising_chain)(L, 1.0, h)
    H1, x = I.sigma_x_sum(L), I.random_state(1 << L, rng)
    got = []
    for path in (None, "multi"):
        with B.Propagator(H0, [H1], COS[:1], path=path, reorder=False) as P:
            got.append(P.apply(dev(x), 0.9, [-0.4]).cpu().numpy())
    assert rel(got[0], got[1]) < 1e-14
    assert np.array_equal(got[0], got[1]) == (not form)


def test_few_entries_where_no_csr_is_kept():
    # 2^23 rows, a diagonal on every sixth of them: the sweeps, whatever the count
    n = 1 << 23
    at = np.arange(0, n, 6)
    rp = np.zeros(n + 1, np.int64)
    rp[at + 1] = 1
    d = np.random.default_rng(2).uniform(-1, 1, at.size)
    H0 = I.CSR(n, np.cumsum(rp), at.astype(np.int32), d.astype(complex))
    H1 = I.CSR(n, np.zeros(n + 1, np.int64), np.zeros(0, np.int32), np.zeros(0, complex))
    x = I.random_state(n, np.random.default_rng(3))
    with B.Propagator(H0, [H1], COS[:1]) as P:
        y = P.apply(dev(x), 1.7, [0.3]).cpu().numpy()
    ref = np.zeros(n, complex)
    ref[at] = 1.7 * d * x[at]
    assert rel(y, ref) < 1e-14


@pytest.mark.parametrize("L", [17, 19, 21])
@pytest.mark.parametrize("complex_values,diag", [(False, False), (True, True)])
def test_nonfinite_elements_reach_the_rows_that_couple_to_them(L, complex_values, diag):
    # an infinity or a NaN meets no entry that the operator does not store
    rng = np.random.default_rng(7 * L + complex_values)
    n = 1 << L
    offs = flips(L, rng, far=True)
    H0 = strings(L, offs if L < 20 else offs[::2], rng, complex_values, sparse=True, diag=diag)
    H1 = strings(L, offs[:9], rng, complex_values, sparse=True, diag=False)
    x = I.random_state(n, rng)
    bad = [5, n // 3, n - 7]
    x[bad[0]] = complex(np.inf, 0.0)
    x[bad[1]] = complex(0.1, np.nan)
    x[bad[2]] = complex(-np.inf, np.nan)
    with B.Propagator(H0, [H1], COS[:1]) as P:
        y = P.apply(dev(x), 0.9, [-0.4]).cpu().numpy()
        assert P.stats()["matrix_bytes"] < 16 * n        # on the sweeps
    hit = np.zeros(n)
    for H in (H0, H1):
        M = H.to_scipy()
        hit += abs(M[:, bad]) @ np.ones(len(bad))
    assert np.array_equal(np.isfinite(y), hit == 0.0)
    ok = hit == 0.0
    assert 0 < np.count_nonzero(~ok) < 150
    clean = np.where(np.isfinite(x), x, 0.0)
    ref = 0.9 * (H0.to_scipy() @ clean) - 0.4 * (H1.to_scipy() @ clean)
    assert rel(y[ok], ref[ok]) < 1e-14


def test_nonfinite_sector_chebyshev():
    # bonds and pair flips keep the parity of a row's bits: a NaN stays in its half
    L = 17
    rng = np.random.default_rng(17)
    n = 1 << L
    H0 = I.heisenberg_chain(L, 1.0, rng.uniform(-1, 1, L))
    H1 = strings(L, [5 << b for b in range(L - 2)], rng, False, sparse=True, diag=False)
    x = I.random_state(n, rng)
    odd = parity(np.arange(n)) == 1
    out = []
    for poison in (False, True):
        z = x.copy()
        if poison:
            z[1] = complex(np.nan, 0.0)
        with B.Propagator(H0, [H1], COS[:1]) as P:
            psi = dev(z)
            P.propagate_chebyshev(psi, 0.0, 0.02, 1, "CF4:2", 1e-10)
            assert P.stats()["matrix_bytes"] < 16 * n
            out.append(psi.cpu().numpy())
    assert np.all(np.isfinite(out[0])) and not np.all(np.isfinite(out[1][odd]))
    assert rel(out[1][~odd], out[0][~odd]) < 1e-13


@pytest.mark.parametrize("L,form", [(12, "site_persistent"), (15, "merged"), (17, "site_sweeps")])
def test_the_form_is_told(L, form):
    p = I.config_heisenberg(L=L)
    with B.Propagator(p.H0, p.Hk, p.drives) as P:
        assert P.form() == form
    with B.Propagator(p.H0, p.Hk, p.drives, path="multi") as P:
        assert P.form() == "merged"


def test_split_layout_at_2_to_the_24_rows():
    # the layout of large operators off the form, by its flag: sampled rows, and
    # the state returns over a step forward and one back
    p = I.config_heisenberg(L=24)
    n, rng = p.dim, np.random.default_rng(24)
    with B.Propagator(p.H0, p.Hk, p.drives, layout="sell_split") as P:
        assert P.form() == "merged" and P.stats()["layout"] == 3
        x = I.random_state(n, rng)
        y = P.apply(dev(x), 0.83, [-1.7]).cpu().numpy()
        rows = np.unique(np.concatenate([[0, 1, 63, 64, n - 64, n - 1],
                                         rng.choice(n, 2000, replace=False)]))
        ref = O.apply_rows(p.H0, p.Hk, 0.83, [-1.7], x, rows)
        assert np.all(np.abs(y[rows] - ref) <= 1e-13 * (1.0 + np.abs(ref)))
        del x, y
        psi = dev(p.psi0)
        P.propagate(psi, 0.0, p.dt, 1, p.scheme, p.m)
        assert abs(torch.linalg.vector_norm(psi).item() - 1.0) < 1e-12
        P.propagate(psi, p.dt, -p.dt, 1, p.scheme, p.m)
        st = P.stats()
        assert st["status"] == 0 and st["matvecs"] == 10 * p.m
        assert rel(psi.cpu().numpy(), p.psi0) < 1e-10


@pytest.mark.parametrize("model,L", [("spins", 19), ("heisenberg", 20), ("heisenberg", 21),
                                     ("spins", 21), ("heisenberg", 22)])
def test_four_and_eight_rows_per_thread_match_the_csr_path(model, L):
    rng = np.random.default_rng(L)
    if model == "spins":
        H0, Hk, drives = I.noninteracting_spins(L, 0.3, 0.7, 1.1)
    else:
        H0, Hk, drives = I.heisenberg_chain(L, 1.0, rng.uniform(-1, 1, L)), [I.sigma_x_sum(L)], COS[:1]
    psi0 = dev(I.random_product_state(L, rng))
    got = []
    for path in (None, "multi"):
        with B.Propagator(H0, Hk, drives, path=path) as P:
            assert (P.form() == "site_sweeps") == (path is None)
            a, b = psi0.clone(), psi0.clone()
            P.propagate(a, 0.1, 0.05, 1, "CF4:2", 18)
            st = P.stats()
            P.propagate_chebyshev(b, 0.1, 0.05, 1, "CF4:2", 1e-12)
            assert P.stats()["status"] == 0
            got.append((a, b, st["matvecs"]))
    (a, b, mv), (ao, bo, mvo) = got
    assert mv == mvo

    def drel(x, y):
        return (torch.linalg.vector_norm(x - y) / torch.linalg.vector_norm(y)).item()
    assert drel(a, ao) <= 1e-10 and drel(b, bo) <= 1e-10


def test_complex_values_on_the_largest_tiles():
    # 2^23 rows: both sweeps on 2^12-row tiles, no CSR; sampled rows, and a step back
    L, rng = 23, np.random.default_rng(23)
    H0 = strings(L, [3, 3 << 11, 3 << 21], rng, False, sparse=True, diag=True)
    H1 = strings(L, [1, 1 << 11, 1 << 12, 1 << 20, 1 << 22, 1 << 17], rng, True, sparse=False,
                 diag=False)
    x = I.random_state(1 << L, rng)
    rows = np.unique(np.concatenate([[0, 1, (1 << L) - 1], rng.choice(1 << L, 3000)]))
    with B.Propagator(H0, [H1], COS[:1]) as P:
        assert P.form() == "site_sweeps" and not np.all(H1.val.imag == 0.0)
        psi = dev(x)
        y = P.apply(psi, 0.83, [-1.7]).cpu().numpy()
        P.propagate(psi, 0.0, 0.05, 1, "CF4:2", 20)
        P.propagate_chebyshev(psi, 0.05, -0.05, 1, "CF4:2", 1e-12)
        assert P.stats()["status"] == 0
        back = psi.cpu().numpy()
    ref = O.apply_rows(H0, [H1], 0.83, [-1.7], x, rows)
    assert np.all(np.abs(y[rows] - ref) <= 1e-13 * (1.0 + np.abs(ref)))
    assert rel(back, x) < 1e-10
