"""Single calls and CSR-pool plans on both sides of the sizes where one
workgroup does a whole call (256 rows: energy; 1024: the gradients of one chunk;
2048: update, norm and rescale), odd register sizes among them, against the
stored operators in FP64: n terms of an FP64 sum differ by n eps sum |terms|."""
import numpy as np
import pytest

import vqe_system as vs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2606_29692_amd as P  # noqa: E402
from paper_2606_29692_amd import binding as B  # noqa: E402


def _packs(n):
    """A seeded Hermitian sum and a few excitations on n qubits (odd n: those of n - 1)."""
    even = n - n % 2
    s = vs.make_system(vs.SystemSpec(even, vs.ELECTRONS[even], "jw", False, 31))
    H, pool = s.hamiltonian, s.pool[:2] + s.pool[-2:]
    z_top = np.uint64(1 << (n - 1))
    ham = vs.PauliPack(n, np.append(H.xmask, np.uint64(0)), np.append(H.zmask, z_top),
                       np.append(H.coeff, 0.3))
    return ham, [vs.PauliPack(n, p.xmask, p.zmask, p.coeff) for p in pool]


def _dense(op):
    rp, col, val = (t.cpu().numpy() for t in (op.rowptr, op.col, op.val))
    return np.repeat(np.arange(op.dim), np.diff(rp)), col[:op.nnz], val[:op.nnz].astype(np.complex128)


def _apply(m, x):
    out = np.zeros_like(x)
    np.add.at(out, m[0], m[2] * x[m[1]])
    return out


def _taylor(m, theta, x):
    acc, v, c = x.copy(), x, 1.0
    for k in range(1, 6):
        v, c = _apply(m, v), c * theta / k
        acc = acc + c * v
    return acc


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [4, 7, 8, 9, 10, 11, 12])
def test_single_calls_and_plan(n, dtype):
    print(f"small calls n={n} {dtype}", flush=True)
    eps = 1e-12 if dtype == "c128" else 2.0 ** -24
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = P.Context(0, stream)
        ham, packs = _packs(n)
        H = B.csr_from_pack(ctx, ham, dtype)
        pool = B.pool_from_packs(ctx, packs, dtype)
        rng = np.random.default_rng(n)
        z = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
        psi = torch.from_numpy(z / np.linalg.norm(z)).cuda().to(tdt)
        start = psi.clone()
        x = psi.cpu().numpy().astype(np.complex128)
        mh, mp = _dense(H), [_dense(o) for o in pool.ops]

        sigma = torch.empty_like(psi)
        e = B.energy(ctx, H, psi, sigma).cpu().numpy()
        g = B.pool_gradients(ctx, H, pool, psi, sigma).cpu().numpy()
        sg = _apply(mh, x)
        np.testing.assert_allclose(sigma.cpu().numpy(), sg, rtol=0, atol=eps * np.abs(sg).max() + 1e-13)
        want_e = np.vdot(x, sg).real / np.vdot(x, x).real
        assert abs(e[0] - want_e) <= 1e-11 * max(1.0, abs(want_e))
        s_used = sigma.cpu().numpy().astype(np.complex128)
        want_g = np.array([2.0 * np.vdot(s_used, _apply(m, x)).real for m in mp])
        np.testing.assert_allclose(g, want_g, rtol=0, atol=1e-11 * np.abs(s_used).sum() / s_used.size ** 0.5)

        norm2 = torch.zeros(1, dtype=torch.float64, device="cuda")
        for renorm in (False, True):
            psi.copy_(start)
            B.taylor5_apply(ctx, pool.ops[1], 0.07, psi, renormalize=renorm, norm2_out=norm2)
            raw = _taylor(mp[1], 0.07, x)
            stored = raw if dtype == "c128" else raw.astype(np.complex64).astype(np.complex128)
            n2 = np.vdot(stored, stored).real
            assert abs(float(norm2.cpu()[0]) - n2) <= 1e-11 + (0 if dtype == "c128" else 2.0 ** -22)
            want = raw / np.sqrt(n2) if renorm else raw
            np.testing.assert_allclose(psi.cpu().numpy(), want, rtol=0, atol=2 * eps)

        # a plan on the CSR pool: steps from rows of angles, eager and one graph, one slot off
        rows = torch.from_numpy(rng.uniform(-0.1, 0.1, (3, 2))).cuda()
        results = []
        for graph in (False, True):
            states = [start.clone(), start.clone()]
            plan = B.BatchPlan(ctx, [(H, pool, p) for p in states], with_active=True)
            plan.active[1] = 0
            plan.run(rows, graph=graph)
            stream.synchronize()
            assert torch.equal(states[1], start)
            assert float(plan.theta[0]) == float(rows[2, 0])
            alone = start.clone()
            for i in range(3):
                B.energy(ctx, H, alone, sigma)
                k, _ = B.vqe_select(ctx, B.pool_gradients(ctx, H, pool, alone, sigma))
                B.taylor5_apply(ctx, pool.ops[int(k.cpu()[0])], float(rows[i, 0]), alone)
            stream.synchronize()
            assert torch.equal(states[0], alone)
            results.append(states[0].clone())
            plan.close()
        assert torch.equal(*results)
        ctx.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [4, 9, 11, 12])
def test_updates_without_a_norm(n, dtype):
    """An update that is neither normalised nor measured takes the wider kernel:
    the same bits as one that is measured, alone and in a plan."""
    print(f"small updates n={n} {dtype}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = P.Context(0, stream)
        ham, packs = _packs(n)
        H, pool = B.csr_from_pack(ctx, ham, dtype), B.pool_from_packs(ctx, packs, dtype)
        rng = np.random.default_rng(n)
        z = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
        start = torch.from_numpy(z).cuda().to(torch.complex128 if dtype == "c128" else torch.complex64)
        plain, measured = start.clone(), start.clone()
        B.taylor5_apply(ctx, pool.ops[1], 0.07, plain, renormalize=False)
        B.taylor5_apply(ctx, pool.ops[1], 0.07, measured, renormalize=False,
                        norm2_out=torch.zeros(1, dtype=torch.float64, device="cuda"))
        assert torch.equal(plain, measured)
        rows = torch.full((1, 1), 0.07, dtype=torch.float64, device="cuda")
        for run in (False, True):
            psi = start.clone()
            plan = B.BatchPlan(ctx, [(H, pool, psi)])
            plan.theta.fill_(0.07)
            plan.k.fill_(1)
            if run:
                plan.theta.zero_()
                plan.run(rows, renorm=False, forced=True)
            else:
                plan.step(renorm=False, forced=True)
            stream.synchronize()
            assert torch.equal(psi, plain) and float(plan.theta[0]) == 0.07
            plan.close()
        ctx.close()


@pytest.mark.parametrize("n", [8, 12])
def test_angle_rows_reach_skipped_slots(n):
    """After a run every slot of a CSR-pool plan holds its last angle, a slot that is
    switched off too, whether the update reads the rows itself or they are copied."""
    print(f"angles of skipped slots n={n}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = P.Context(0, stream)
        ham, packs = _packs(n)
        H, pool = B.csr_from_pack(ctx, ham), B.pool_from_packs(ctx, packs)
        states = [torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.complex128, device="cuda") for _ in range(3)]
        plan = B.BatchPlan(ctx, [(H, pool, p) for p in states], with_active=True)
        plan.active[1] = 0
        before = states[1].clone()
        rows = torch.tensor([[0.1, 0.2, 0.3], [0.4, 0.5, 0.6]], dtype=torch.float64, device="cuda")
        for graph in (False, True):
            plan.theta.zero_()
            plan.run(rows, graph=graph)
            stream.synchronize()
            assert torch.equal(plan.theta, rows[1]) and torch.equal(states[1], before)
        plan.close()
        ctx.close()


@pytest.mark.parametrize("masks", [20, 21, 64])
def test_energy_of_few_rows_and_more_entries(masks):
    """256 rows on both sides of the entries that one workgroup takes."""
    print(f"small energy {masks} entries a row", flush=True)
    ctx = P.Context(0)
    rng = np.random.default_rng(masks)
    x = rng.choice(256, size=masks, replace=False).astype(np.uint64)
    H = B.csr_build_from_pauli(ctx, 8, x, rng.integers(0, 256, masks).astype(np.uint64), rng.standard_normal(masks) + 0j)
    assert H.nnz == masks * 256
    z = rng.standard_normal(256) + 1j * rng.standard_normal(256)
    psi = torch.from_numpy(z).cuda()
    sigma = torch.empty_like(psi)
    e = B.energy(ctx, H, psi, sigma).cpu().numpy()
    sg = _apply(_dense(H), z)
    np.testing.assert_allclose(sigma.cpu().numpy(), sg, rtol=0, atol=1e-13 * masks * np.abs(sg).max())
    assert abs(e[0] - np.vdot(z, sg).real / np.vdot(z, z).real) <= 1e-11
    ctx.close()
