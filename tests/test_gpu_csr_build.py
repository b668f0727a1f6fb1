"""The CSR builder's kernels at the edges of their ranges: rows fewer than a
wave, one and many waves per 64 rows, groups beyond the 64-row kernels' table,
registers beyond its dense prefix table, operators passed as a kernel argument,
through pinned staging and from pageable memory; every entry bit for bit the
oracle's ordered sum."""
import time

import numpy as np
import pytest

from oracle import oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2606_29692_amd as P  # noqa: E402
from paper_2606_29692_amd import binding as B  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = P.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _terms(n, T, masks, real, seed):
    """T terms over `masks` distinct flip masks, in random order, some cancelling."""
    rng = np.random.default_rng(seed)
    pick = rng.choice(1 << n, size=min(masks, 1 << n), replace=False).astype(np.uint64)
    x = rng.choice(pick, size=T)
    z = rng.integers(0, 1 << n, T).astype(np.uint64)
    c = np.round(rng.standard_normal(T), 1) + 0j
    if real:
        c = np.where(np.bitwise_count(x & z) % 2 == 1, 1j * c, c)
    else:
        c = c + 1j * rng.standard_normal(T)
    half = T // 4
    return (np.concatenate([x, x[:half]]), np.concatenate([z, z[:half]]),
            np.concatenate([c, -c[:half]]))


@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("n,T,masks", [
    (1, 3, 2), (3, 9, 8), (5, 40, 32), (6, 50, 20), (7, 7, 7), (7, 70, 63), (8, 90, 64),
    (9, 400, 65), (10, 1500, 300), (11, 3000, 2048), (12, 1, 3000), (12, 60000, 1500),
    (16, 60, 12), (21, 6, 3)])
def test_csr_build_ranges(ctx, n, T, masks, real):
    print(f"csr build n={n} T={T} masks={masks} real={real}", flush=True)
    x, z, c = _terms(n, T, masks, real, 7 * n + T)
    if masks > 2048:      # more groups than the supported row length: each vanishes on half its rows
        x = np.repeat(np.random.default_rng(n).permutation(1 << n)[:masks].astype(np.uint64), 2)
        z = np.where(np.arange(x.size) % 2 == 0, np.uint64(0), (x & np.uint64(1023)) + np.uint64(1))
        c = np.where(np.bitwise_count(x & z) % 2 == 1, 1j, 1.0 + 0j) * (1.0 if real else 1j)
    o = orc.csr_build(n, x, z, c)
    d = B.csr_build_from_pauli(ctx, n, x, z, c)
    torch.cuda.synchronize()
    assert d.real == real and d.nnz == o.nnz
    np.testing.assert_array_equal(d.rowptr.cpu().numpy().astype(np.int64), o.rowptr)
    np.testing.assert_array_equal(d.col.cpu().numpy()[:o.nnz], o.col)
    np.testing.assert_array_equal(d.val.cpu().numpy()[:o.nnz].view(np.uint64), o.val.view(np.uint64))


@pytest.mark.parametrize("n,identity", [(2, False), (7, True), (10, False), (15, False)])
def test_csr_build_shift_keeps_the_diagonal(ctx, n, identity):
    """FP32 storage about a shift: every row stores its diagonal, present or not in the sum."""
    x, z, c = _terms(n, 30, 5, True, n)
    at = x != 0
    x, z, c = x[at], z[at], c[at]
    if identity:
        x, z, c = np.append(x, np.uint64(0)), np.append(z, np.uint64(5)), np.append(c, 0.75)
    d = B.csr_build_from_pauli(ctx, n, x, z, c, dtype="c64", diag_shift=0.5)
    o = orc.csr_build(n, np.append(x, np.uint64(0)), np.append(z, np.uint64(0)), np.append(c, 1e3))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(d.rowptr.cpu().numpy().astype(np.int64), o.rowptr)
    np.testing.assert_array_equal(d.col.cpu().numpy(), o.col)
    want = o.val.copy()
    diag = o.col == np.repeat(np.arange(1 << n), np.diff(o.rowptr))
    sign = 1.0 - 2.0 * (np.bitwise_count(o.col[diag].astype(np.uint64) & np.uint64(5)) % 2)
    want[diag] = (0.75 * sign if identity else 0.0) - 0.5
    np.testing.assert_array_equal(d.val.cpu().numpy(), want.astype(np.complex64))


@pytest.mark.parametrize("n,T,masks", [(9, 511, 200), (9, 512, 200), (11, 1023, 60), (11, 1024, 60),
                                       (11, 40000, 1700), (12, 30000, 4096), (16, 20000, 1900), (23, 600, 2)])
def test_csr_build_term_order(ctx, n, T, masks):
    """Terms given in any order compile as the same terms grouped by flip mask
    beforehand (each group's in the given order), on both sides of the sizes where
    the grouping and the kernels change."""
    print(f"csr build order n={n} T={T} masks={masks}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.choice(rng.choice(1 << n, size=masks, replace=False).astype(np.uint64), size=T)
    z = rng.integers(0, 1 << n, T).astype(np.uint64)
    c = rng.standard_normal(T) + 1j * rng.standard_normal(T)
    at = np.argsort(x, kind="stable")
    if masks > 2048:      # (rows of at most 2048 entries)
        c[x >= np.uint64(2000)] = 0
    a = B.csr_build_from_pauli(ctx, n, x, z, c)
    b = B.csr_build_from_pauli(ctx, n, x[at], z[at], c[at])
    torch.cuda.synchronize()
    assert a.nnz == b.nnz
    assert torch.equal(a.rowptr, b.rowptr) and torch.equal(a.col, b.col)
    assert torch.equal(torch.view_as_real(a.val).view(torch.int64), torch.view_as_real(b.val).view(torch.int64))


def test_csr_build_of_many_terms_costs_no_more_out_of_order(ctx):
    """Grouping 10^5 terms is a small part of compiling them: given out of order
    they took three times as long as grouped when they were sorted by comparison."""
    rng = np.random.default_rng(1)
    n, T = 8, 100000
    x = rng.integers(0, 1 << n, T).astype(np.uint64)
    z = rng.integers(0, 1 << n, T).astype(np.uint64)
    c = rng.standard_normal(T) + 0j
    at = np.argsort(x, kind="stable")

    def best(*terms):
        times = []
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            B.csr_build_from_pauli(ctx, n, *terms)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
        return min(times)
    mixed, grouped = best(x, z, c), best(x[at], z[at], c[at])
    print(f"csr build of {T} terms: out of order {mixed * 1e3:.2f} ms, grouped {grouped * 1e3:.2f} ms", flush=True)
    assert mixed <= 2 * grouped


def test_csr_build_operator_past_2_gib(ctx):
    """108 million complex terms (20 bytes each on the device) compile: some entries
    against their ordered sums, bit for bit."""
    n, G, per = 12, 2048, 52800
    T = G * per
    rng = np.random.default_rng(2)
    xs = np.sort(rng.choice(1 << n, size=G, replace=False).astype(np.uint64))
    x = np.repeat(xs, per)
    z = np.resize(rng.integers(0, 1 << n, 999983).astype(np.uint64), T)
    c = np.resize(rng.standard_normal(1000003) + 1j * rng.standard_normal(1000003), T)
    print(f"csr build T={T}", flush=True)
    d = B.csr_build_from_pauli(ctx, n, x, z, c, drop_tol=0.0)
    torch.cuda.synchronize()
    assert d.nnz == G << n and not d.real
    for g in (0, 1, 1000, G - 1):
        zg, cg = z[g * per:(g + 1) * per], c[g * per:(g + 1) * per]
        k = np.bitwise_count(xs[g] & zg) % 4
        cg = np.select([k == 0, k == 1, k == 2], [cg, -cg.imag + 1j * cg.real, -cg], cg.imag - 1j * cg.real)
        for r in (0, 777, (1 << n) - 1):
            col = r ^ int(xs[g])
            v = np.where(np.bitwise_count(zg & np.uint64(col)) % 2 == 1, -cg, cg)
            lo, hi = (int(i) for i in d.rowptr[r:r + 2].cpu())
            cols, vals = d.col[lo:hi].cpu().numpy(), d.val[lo:hi].cpu().numpy()
            assert vals[np.searchsorted(cols, col)] == np.cumsum(v.real)[-1] + 1j * np.cumsum(v.imag)[-1]
