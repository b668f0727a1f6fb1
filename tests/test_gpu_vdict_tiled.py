"""The value dictionary (VQE_SPMV_VDICT) on states larger than LDS, where its
rules meet their edges: two to 64 tiles, tiles that no row reaches, more pairs
than a tile's table and more masks than are indexed, imaginary entries, masks of
more than four magnitudes; whole, halved and quartered row blocks; rebinding.
sigma is compared with the stored CSR in FP64: half an ulp of FP32 for the
result's rounding, and n eps sum |a||x| for the order of an FP64 sum of n terms."""
import numpy as np
import pytest

from test_gpu_vdict import VD, B, _molecule, _pool, _products, _state, _sum, ctx, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _low(case):
    """The sum's masks cut to the low 14 bits: every row meets one tile."""
    n, x, z, c = case
    return n, x & np.uint64(0x3fff), z, np.where(np.bitwise_count(x & np.uint64(0x3fff) & z) % 2 == 1, 1j, 1.0) * abs(c)


CASES = {
    "two_tiles": lambda: _sum(15, 60, lambda i: 1 + i % 5, True, 1),
    "one_tile_of_four": lambda: _low(_sum(16, 40, lambda i: 1 + i % 4, True, 2)),
    "codes_only": lambda: _sum(16, 33, lambda i: 1, True, 3),
    "no_codes": lambda: _sum(15, 17, lambda i: 5, True, 4),
    "complex": lambda: _sum(15, 70, lambda i: 1 + i % 4, False, 5),
    "past_the_tables": lambda: _sum(15, 1500, lambda i: 1 + i % 2, True, 6),
    "widest": lambda: _sum(20, 9, lambda i: 1 + i % 3, True, 8),
}


def _check(H, psi, sigma):
    """As the module's oracle on states that fit LDS, summed by torch in FP64."""
    n = torch.diff(H.rowptr).long()
    rows = torch.repeat_interleave(torch.arange(H.dim, device=n.device), n)
    x = psi.to(torch.complex128)
    prod = H.val[:H.nnz].to(torch.complex128) * x[H.col[:H.nnz].long()]
    want, size = torch.zeros_like(x), torch.zeros(H.dim, dtype=torch.float64, device=n.device)
    for part, out in ((prod.real, want.real), (prod.imag, want.imag), (prod.abs(), size)):
        out.copy_(torch.zeros_like(size).index_add_(0, rows, part.contiguous()))
    order = size * (n + 2) * 2.0 ** -52
    got = sigma.to(torch.complex128)
    for a, b in ((got.real, want.real), (got.imag, want.imag)):
        assert bool(((a - b).abs() <= 2.0 ** -24 * b.abs() + order + 2.0 ** -149).all())
    return float(torch.vdot(x, want).real / torch.vdot(x, x).real), float(x.abs() @ want.abs())


def _scattered(n, per_row):
    """per_row random columns in each row, four magnitudes: the masks are all of n bits'."""
    g = torch.Generator().manual_seed(n)
    dim = 1 << n
    step = dim // per_row
    col = torch.arange(per_row) * step + torch.randint(step, (dim, per_row), generator=g)
    val = 0.25 * torch.randint(-4, 4, (dim, per_row), generator=g) + 0.125
    rowptr = torch.arange(dim + 1) * per_row
    rowptr, col, val = rowptr.int().cuda(), col.reshape(-1).int().cuda(), val.reshape(-1).to(torch.complex64).cuda()
    desc = B.vqe_csr()
    desc.n_qubits, desc.dim, desc.nnz, desc.dtype, desc.flags = n, dim, dim * per_row, B.VQE_C64, B.VQE_REAL
    desc.rowptr, desc.col, desc.val = rowptr.data_ptr(), col.data_ptr(), val.data_ptr()
    return B.DeviceCSR(desc, rowptr, col, val)


def _operator(ctx, name):
    """The named operator; "real9" and "complex9" fit LDS."""
    if name in ("real9", "complex9"):
        n, x, z, c = _sum(9, 60, lambda i: 1 + i % 6, name == "real9", 9)
        return n, B.csr_build_from_pauli(ctx, n, x, z, c, dtype="c64"), B.MatrixFreePool(_pool(n), "c64")
    if name == "past_the_masks":
        return 15, _scattered(15, 32), B.MatrixFreePool(_pool(15), "c64")
    n, x, z, c = CASES[name]() if name in CASES else _molecule(int(name[2:]), name[:2])
    return n, B.csr_build_from_pauli(ctx, n, x, z, c, dtype="c64"), B.MatrixFreePool(_pool(n), "c64")


@pytest.mark.parametrize("sched", [3 | VD, 6 | VD | B.VQE_SPMV_REAL])
@pytest.mark.parametrize("name", [*CASES, "past_the_masks", "jw16", "bk16"])
def test_tiled_product(ctx, name, sched):  # noqa: F811
    print(f"vdict tiled {name} schedule {sched:#x}", flush=True)
    with torch.cuda.stream(ctx.stream):
        n, H, pool = _operator(ctx, name)
        for kind in ("complex", "real"):
            psi = _state(n, kind, n)
            (sigma,), energy = _products(ctx, H, pool, [psi], sched)
            e, scale = _check(H, psi, sigma)
            assert abs(float(energy[0, 0]) - e) <= 2.0 ** -50 * scale * H.dim + 1e-12


def test_tiled_alone_and_in_batches(ctx):  # noqa: F811
    """Quarter, half and whole blocks per workgroup: the same bits."""
    with torch.cuda.stream(ctx.stream):
        n, H, pool = _operator(ctx, "two_tiles")
        cu, _ = ctx.info()
        blocks, psi, ref = (1 << n) // 2048, _state(n, "complex", 3), None
        for count in (1, cu // (4 * blocks) + 1, cu // (2 * blocks) + 1, cu // blocks + 1):
            print(f"vdict tiled batch of {count}", flush=True)
            sigma, energy = _products(ctx, H, pool, [psi.clone() for _ in range(count)], 3 | VD)
            if ref is None:
                ref = sigma[0], energy[0]
            for s in (sigma[0], sigma[-1]):
                assert torch.equal(torch.view_as_real(s), torch.view_as_real(ref[0]))
            assert torch.equal(energy, ref[1].expand_as(energy))


@pytest.mark.parametrize("names", [("two_tiles", "no_codes", "complex"), ("real9", "complex9")])
def test_rebind(ctx, names):  # noqa: F811
    """A slot bound to other operators, rebuilt and through a layout: smaller,
    larger, and from real entries to complex ones and back."""
    with torch.cuda.stream(ctx.stream):
        (n, first, pool), *rest = [_operator(ctx, k) for k in names]
        psi = _state(n, "complex", 4)
        plan = B.BatchPlan(ctx, [(first, pool, psi)], schedules=[3 | VD])
        for H in [r[1] for r in rest] + [first]:
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


@pytest.mark.parametrize("call", ["run", "linesearch", "reoptimise"])
def test_plan_calls_after_a_rebind(ctx, call):  # noqa: F811
    """Replayed steps, line search and re-optimisation on a column-tiled dictionary:
    a slot rebound to another operator and back gives the bits of a plan made for it,
    and the energies of the layout without a dictionary (FP32 results of products
    summed in another order: 2^-20 of the operator's bound)."""
    with torch.cuda.stream(ctx.stream):
        (n, A, pool), (_, H, _) = [_operator(ctx, k) for k in ("two_tiles", "complex")]
        start = _state(n, "complex", 11)
        rows = torch.tensor([[0.1], [-0.2]], dtype=torch.float64, device="cuda")
        ks = torch.tensor([[0, 2, 1]], dtype=torch.int32, device="cuda")

        def go(plan, psi):
            th = torch.full((1, 3), 0.05, dtype=torch.float64, device="cuda")
            psi.copy_(start)
            if call == "run":
                plan.run(rows)
            elif call == "linesearch":
                plan.set_line_search(0.5)
                plan.run(None, line_search_steps=2)
            else:
                plan.reoptimize(ks, th, 3, [start], 1, 0.5)
            plan.step(update=False, graph=True)
            ctx.stream.synchronize()
            return psi.clone(), th, plan.theta.clone(), plan.k.clone(), plan.energies.clone()

        def alone(op, sched):
            psi = start.clone()
            plan = B.BatchPlan(ctx, [(op, pool, psi)], schedules=[sched])
            out = go(plan, psi)
            plan.close()
            return out

        psi = start.clone()
        plan = B.BatchPlan(ctx, [(A, pool, psi)], schedules=[3 | VD])
        built = B.Layout(ctx, A, 3 | VD)
        for op, layout in ((A, None), (H, None), (A, built), (H, None), (A, None)):
            print(f"vdict tiled {call} nnz={op.nnz} layout={layout is not None}", flush=True)
            plan.rebind(0, op, pool, psi, layout=layout)
            got = go(plan, psi)
            want = alone(op, 3 | VD)
            assert all(torch.equal(torch.view_as_real(a) if a.is_complex() else a,
                                   torch.view_as_real(b) if b.is_complex() else b) for a, b in zip(got, want))
            plain = alone(op, 2 | B.VQE_SPMV_LDS | B.VQE_SPMV_SLICED)
            bound = float(op.val[:op.nnz].abs().max()) * op.nnz / op.dim
            assert abs(float(got[4][0] - plain[4][0])) <= 2.0 ** -20 * bound
            again = go(plan, psi)
            assert all(torch.equal(torch.view_as_real(a) if a.is_complex() else a,
                                   torch.view_as_real(b) if b.is_complex() else b) for a, b in zip(got, again))
        plan.close()
        built.close()
