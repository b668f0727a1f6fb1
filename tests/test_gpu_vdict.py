"""The sliced product with a value dictionary (VQE_SPMV_VDICT) where its rules
meet their edges: masks of one to eight magnitudes, imaginary entries, more
pairs than the table holds, rows with codes only or none, registers smaller
than a slice; whole, halved and quartered row blocks; rebinding.  sigma is
compared with the stored CSR in FP64: half an ulp of FP32 for the result's
rounding, and n eps sum |a||x| for the order of an FP64 sum of n terms."""
import numpy as np
import pytest

import vqe_system as vs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2606_29692_amd as P  # noqa: E402
from paper_2606_29692_amd import batch as PB  # noqa: E402
from paper_2606_29692_amd import binding as B  # noqa: E402
from paper_2606_29692_amd import tune as T  # noqa: E402

VD = B.VQE_SPMV_LDS | B.VQE_SPMV_SLICED | B.VQE_SPMV_XIDX | B.VQE_SPMV_VDICT
SCHEDULES = [3 | VD, 6 | VD, 3 | VD | B.VQE_SPMV_REAL, 6 | VD | B.VQE_SPMV_REAL]


@pytest.fixture(scope="module")
def ctx():
    stream = torch.cuda.Stream()
    c = P.Context(0, stream)
    yield c
    torch.cuda.synchronize()
    c.close()


def _sum(n, masks, terms, real, seed):
    """A Pauli sum with `terms(i)` terms on the i-th of `masks` flip masks: k
    generic terms give 2^(k-1) magnitudes.  Real entries unless real is False,
    when every other mask's are complex."""
    rng = np.random.default_rng(seed)
    xs = rng.permutation(1 << n)[:masks].astype(np.uint64)
    x = np.repeat(xs, [terms(i) for i in range(masks)])
    z = rng.integers(0, 1 << n, x.size).astype(np.uint64)
    c = rng.uniform(0.1, 1.0, x.size) * rng.choice([-1.0, 1.0], x.size) + 0j
    c = np.where(np.bitwise_count(x & z) % 2 == 1, 1j * c, c)
    if not real:
        odd = np.isin(x, xs[::2])
        c = np.where(odd, c * np.exp(0.3j), c)
    return n, x, z, c


CASES = {
    "tiny": lambda: _sum(3, 5, lambda i: 1 + i % 3, True, 1),
    "five": lambda: _sum(5, 32, lambda i: 1 + i % 4, True, 2),
    "codes_only": lambda: _sum(8, 70, lambda i: 1, True, 3),
    "no_codes": lambda: _sum(8, 40, lambda i: 5, True, 4),
    "mixed": lambda: _sum(9, 120, lambda i: 1 + i % 5, True, 5),
    "complex": lambda: _sum(9, 120, lambda i: 1 + i % 4, False, 6),
    "past_the_table": lambda: _sum(11, 600, lambda i: 2 + i % 2, True, 7),
    "widest": lambda: _sum(12, 1024, lambda i: 1, True, 8),
}


def _molecule(n, mapping):
    s = vs.make_system(vs.SystemSpec(n, vs.ELECTRONS[n], mapping, False, 77 + n))
    p = s.hamiltonian
    return n, p.xmask, p.zmask, p.coeff


def _pool(n):
    e = {3: 1, 5: 1}.get(n)
    if e is None:
        even = n - n % 2
        return [vs.PauliPack(n, p.xmask, p.zmask, p.coeff)
                for p in vs.shared_pool(even, vs.ELECTRONS[even], "jw")[:4]]
    # one excitation between modes 0 and 2
    p = vs.shared_pool(4, 2, "jw")[0]
    return [vs.PauliPack(n, p.xmask & np.uint64(7), p.zmask & np.uint64(7), p.coeff)]


def _state(n, kind, seed):
    rng = np.random.default_rng(seed)
    z = rng.standard_normal(1 << n) + 1j * (rng.standard_normal(1 << n) if kind == "complex" else 0.0)
    return torch.from_numpy((z / np.linalg.norm(z)).astype(np.complex64)).cuda()


def _products(ctx, H, pool, psis, sched):
    with torch.cuda.stream(ctx.stream):
        plan = B.BatchPlan(ctx, [(H, pool, p) for p in psis], schedules=[sched] * len(psis))
        plan.step(update=False)
        out = [s.clone() for s in plan.sigma], plan.energies.clone().view(-1, 3)
    torch.cuda.synchronize()
    plan.close()
    return out


def _reference(H, psi):
    rp = H.rowptr.cpu().numpy().astype(np.int64)
    col, val = H.col.cpu().numpy()[:H.nnz], H.val.cpu().numpy()[:H.nnz].astype(np.complex128)
    x = psi.cpu().numpy().astype(np.complex128)
    rows = np.repeat(np.arange(H.dim), np.diff(rp))
    prod = val * x[col]
    out = np.zeros(H.dim, dtype=np.complex128)
    np.add.at(out, rows, prod)
    size = np.bincount(rows, weights=np.abs(prod), minlength=H.dim)
    return out, size * (np.diff(rp) + 2) * 2.0 ** -52


def _check(H, psi, sigma):
    torch.cuda.synchronize()
    want, order = _reference(H, psi)
    got = sigma.cpu().numpy().astype(np.complex128)
    for a, b in ((got.real, want.real), (got.imag, want.imag)):
        assert np.all(np.abs(a - b) <= 2.0 ** -24 * np.abs(b) + order + 2.0 ** -149)


@pytest.mark.parametrize("sched", SCHEDULES)
@pytest.mark.parametrize("name", [*CASES, "jw6", "jw10", "bk12", "jw14"])
def test_vdict_product(ctx, name, sched):
    print(f"vdict {name} schedule {sched:#x}", flush=True)
    n, x, z, c = CASES[name]() if name in CASES else _molecule(int(name[2:]), name[:2])
    with torch.cuda.stream(ctx.stream):
        H = B.csr_build_from_pauli(ctx, n, x, z, c, dtype="c64")
        pool = B.MatrixFreePool(_pool(n), "c64")
    for kind in ("complex", "real"):
        psi = _state(n, kind, n)
        (sigma,), energy = _products(ctx, H, pool, [psi], sched)
        _check(H, psi, sigma)
        # the energy: the same order bound over the states' sum
        s = sigma.cpu().numpy().astype(np.complex128)
        p = psi.cpu().numpy().astype(np.complex128)
        want = np.vdot(p, _reference(H, psi)[0]).real / np.vdot(p, p).real
        slack = 2.0 ** -50 * (np.abs(p) @ np.abs(s)) * H.dim + 1e-12
        assert abs(float(energy[0, 0]) - want) <= slack


@pytest.mark.parametrize("n", [8, 12])
def test_vdict_alone_and_in_batches(ctx, n):
    """Quarter, half and whole blocks per workgroup: the same bits."""
    print(f"vdict batches n={n}", flush=True)
    _, x, z, c = _molecule(n, "jw")
    with torch.cuda.stream(ctx.stream):
        H = B.csr_build_from_pauli(ctx, n, x, z, c, dtype="c64")
        pool = B.MatrixFreePool(_pool(n), "c64")
    cu, _ = ctx.info()
    blocks = max((1 << n) // 2048, 1)
    psi = _state(n, "complex", 3)
    ref = None
    for count in (1, cu // (4 * blocks) + 1, cu // (2 * blocks) + 1, cu // blocks + 1):
        sigma, energy = _products(ctx, H, pool, [psi.clone() for _ in range(count)], 3 | VD)
        if ref is None:
            ref = sigma[0], energy[0]
        for s in (sigma[0], sigma[-1]):
            assert torch.equal(torch.view_as_real(s), torch.view_as_real(ref[0]))
        assert torch.equal(energy, ref[1].expand_as(energy))


def test_vdict_rebind(ctx):
    """A slot bound to other operators, rebuilt and through a layout, smaller and larger."""
    n = 9
    ops = []
    with torch.cuda.stream(ctx.stream):
        for name in ("mixed", "mixed_few", "mixed_many"):
            _, x, z, c = _sum(9, {"mixed": 120, "mixed_few": 20, "mixed_many": 300}[name],
                              lambda i: 1 + i % 5, True, len(name))
            ops.append(B.csr_build_from_pauli(ctx, n, x, z, c, dtype="c64"))
        pool = B.MatrixFreePool(_pool(n), "c64")
        psi = _state(n, "complex", 4)
        plan = B.BatchPlan(ctx, [(ops[0], pool, psi)], schedules=[3 | VD])
        for H in (ops[1], ops[2], ops[0]):
            alone = _products(ctx, H, pool, [psi], 3 | VD)[0][0]
            layout = B.Layout(ctx, H, 3 | VD)
            for lay in (None, layout):
                print(f"vdict rebind nnz={H.nnz} layout={lay is not None}", flush=True)
                plan.rebind(0, H, pool, psi, layout=lay)
                plan.step(update=False)
                _check(H, psi, plan.sigma[0])
                assert torch.equal(torch.view_as_real(plan.sigma[0]), torch.view_as_real(alone))
            plan.rebind(0, H, pool, psi)
            ctx.stream.synchronize()
            layout.close()
        plan.close()


def test_vdict_fp64_storage_takes_the_index_form(ctx):
    _, x, z, c = _molecule(8, "jw")
    with torch.cuda.stream(ctx.stream):
        H = B.csr_build_from_pauli(ctx, 8, x, z, c)
        pool = B.MatrixFreePool(_pool(8), "c128")
    psi = _state(8, "complex", 5).to(torch.complex128)
    a = _products(ctx, H, pool, [psi], 3 | VD)
    b = _products(ctx, H, pool, [psi], (3 | VD) & ~B.VQE_SPMV_VDICT)
    assert torch.equal(torch.view_as_real(a[0][0]), torch.view_as_real(b[0][0]))
    assert torch.equal(a[1], b[1])


def _ragged(n, seed):
    """Rows of 0 to 150 entries in no order, some with codes only, some with none:
    the masks' magnitudes are one, two or (past four) per row and mask their own."""
    rng = np.random.default_rng(seed)
    dim = 1 << n
    xs = rng.choice(dim, size=150, replace=False)
    kinds = rng.integers(0, 3, xs.size)
    rowptr, cols, vals = [0], [], []
    for r in range(dim):
        k = rng.choice(xs.size, size=rng.choice([0, 1, 7, 63, 64, 65, 128, 150]), replace=False)
        c = xs[k] ^ r
        v = np.where(kinds[k] == 0, 0.5 + k, np.where(kinds[k] == 1, rng.choice([0.25, 2.0], k.size),
                                                      rng.uniform(0.1, 1.0, k.size)))
        v = v * rng.choice([-1.0, 1.0], k.size)
        at = np.argsort(c)
        cols.append(c[at])
        vals.append(v[at])
        rowptr.append(rowptr[-1] + k.size)
    rowptr = torch.from_numpy(np.array(rowptr, dtype=np.int32)).cuda()
    col = torch.from_numpy(np.concatenate(cols).astype(np.int32)).cuda()
    val = torch.from_numpy(np.concatenate(vals).astype(np.complex64)).cuda()
    desc = B.vqe_csr()
    desc.n_qubits, desc.dim, desc.nnz, desc.dtype, desc.flags = n, dim, col.numel(), B.VQE_C64, B.VQE_REAL
    desc.rowptr, desc.col, desc.val = rowptr.data_ptr(), col.data_ptr(), val.data_ptr()
    return B.DeviceCSR(desc, rowptr, col, val)


@pytest.mark.parametrize("n", [8, 11])
def test_vdict_rows_one_after_another(ctx, n):
    """The builder's wave takes rows in turn through the same buffers: long ones
    behind short and empty ones, and rows that leave some lanes without an entry."""
    H = _ragged(n, n)
    with torch.cuda.stream(ctx.stream):
        pool = B.MatrixFreePool(_pool(n), "c64")
    for sched in (3 | VD, 6 | VD | B.VQE_SPMV_REAL):
        print(f"vdict ragged n={n} schedule {sched:#x}", flush=True)
        psi = _state(n, "complex", 6)
        (sigma,), _ = _products(ctx, H, pool, [psi], sched)
        _check(H, psi, sigma)


@pytest.mark.parametrize("form", ["any", "complex"])
def test_vdict_more_masks_than_the_index_form(ctx, form):
    """The shipped 12-qubit schedules take operators of more than 1024 flip masks
    (entries as 16-bit columns): real and complex ones, alone and in batches of whole,
    halved and quartered blocks, through plans, layouts and rebinding to and from
    an operator with a dictionary."""
    n = 12
    cu, _ = ctx.info()
    with torch.cuda.stream(ctx.stream):
        pool = B.MatrixFreePool(_pool(n), "c64")
        ops = {"few": _sum(n, 300, lambda i: 1 + i % 5, True, 21), "1100": _sum(n, 1100, lambda i: 1, True, 22),
               "1500": _sum(n, 1500, lambda i: 1 + i % 6, True, 23), "1100c": _sum(n, 1100, lambda i: 1, False, 24)}
        ops = {k: B.csr_build_from_pauli(ctx, *v, dtype="c64") for k, v in ops.items()}
        psi = {k: _state(n, k, 7) for k in ("real", "complex")}

    class Shape:
        n_qubits, dtype, key = n, "c64", (n, 4, "jw")
    sched = T.schedule_for(ctx, Shape, value_form=form)
    for name, H in ops.items():
        for kind in psi:
            ref = None
            for count in (1, cu // 4 + 1, cu // 2 + 1):
                print(f"vdict masks {form} {name} {kind} x{count}", flush=True)
                sigma, energy = _products(ctx, H, pool, [psi[kind].clone() for _ in range(count)], sched)
                if ref is None:
                    ref = sigma[0], energy[0]
                    _check(H, psi[kind], sigma[0])
                assert torch.equal(torch.view_as_real(sigma[-1]), torch.view_as_real(ref[0]))
                assert torch.equal(energy, ref[1].expand_as(energy))
    # a slot of the real schedule takes real operators only, as before
    names = ["few", "1100", "few", "1500"] + (["1100c", "few"] if form == "complex" else [])
    with torch.cuda.stream(ctx.stream):
        plan = B.BatchPlan(ctx, [(ops["few"], pool, psi["complex"])], schedules=[sched])
        for name in names:
            H = ops[name]
            layout = B.Layout(ctx, H, sched)
            alone = _products(ctx, H, pool, [psi["complex"]], sched)[0][0]
            for lay in (layout, None):
                print(f"vdict masks rebind {form} {name} layout={lay is not None}", flush=True)
                plan.rebind(0, H, pool, psi["complex"], layout=lay)
                plan.step(update=False, graph=True)
                ctx.stream.synchronize()
                assert torch.equal(torch.view_as_real(plan.sigma[0]), torch.view_as_real(alone))
            layout.close()
        plan.close()
