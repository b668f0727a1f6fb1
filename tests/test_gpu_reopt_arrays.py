"""Re-optimisation calls in a row on one plan: with the same arrays, with other
angle, index and reference arrays, fewer updates and another range, each equal
to the same call on a plan of its own (the plan uploads its descriptors only
when they differ from the last call's)."""
import numpy as np
import pytest

import vqe_system as vs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2606_29692_amd as P  # noqa: E402
from paper_2606_29692_amd import batch as PB  # noqa: E402


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("states,n", [(1, 4), (3, 8), (2, 10)])
def test_reoptimize_calls_in_a_row(dtype, states, n):
    print(f"reopt arrays n={n} states={states} {dtype}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = P.Context(0, stream)
        pools = PB.PoolCache(ctx, matrix_free=True)
        ds = [PB.device_system(ctx, vs.make_system(vs.SystemSpec(n, vs.ELECTRONS[n], "jw", False, 9 + s)),
                               dtype, pools) for s in range(states)]
        refs = [d.psi.clone() for d in ds]
        other = [torch.roll(r, 3).contiguous() for r in refs]
        rng = np.random.default_rng(n)
        m = ds[0].pool.M

        def arrays(ld):
            ks = torch.from_numpy(rng.integers(0, m, (states, ld)).astype(np.int32)).cuda()
            return ks, torch.from_numpy(rng.uniform(-0.2, 0.2, (states, ld))).cuda()

        a, b = arrays(4), arrays(5)
        calls = [(a, 4, refs, 1.0), (a, 4, refs, 1.0), (a, 2, refs, 1.0), (b, 5, refs, 0.05),
                 (b, 5, other, 0.05), (a, 4, refs, 1.0)]
        plan = PB.make_batch(ctx, ds)
        for (ks, th), count, ref, tm in calls:
            alone_th = th.clone()
            plan.reoptimize(ks, th, count, ref, 1, tm)
            got = [d.psi.clone() for d in ds]
            alone = PB.make_batch(ctx, ds)
            alone.reoptimize(ks, alone_th, count, ref, 1, tm)
            stream.synchronize()
            assert torch.equal(th, alone_th)
            assert all(torch.equal(g, d.psi) for g, d in zip(got, ds))
            alone.close()
        plan.close()
        ctx.close()


def test_reoptimize_from_references_on_the_host():
    """References in host memory, pageable and pinned, give what device ones give."""
    n = 8
    print("reopt host references", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = P.Context(0, stream)
        pools = PB.PoolCache(ctx, matrix_free=True)
        ds = [PB.device_system(ctx, vs.make_system(vs.SystemSpec(n, vs.ELECTRONS[n], "jw", False, 9 + s)),
                               "c64", pools) for s in range(2)]
        refs = [d.psi.clone() for d in ds]
        host = [refs[0].cpu(), refs[1].cpu().pin_memory()]
        ks = torch.tensor([[0, 3, 5], [7, 2, 1]], dtype=torch.int32, device="cuda")
        plan, out = PB.make_batch(ctx, ds), []
        for ref in (refs, host, [refs[0], host[1]]):
            th = torch.full((2, 3), 0.1, dtype=torch.float64, device="cuda")
            plan.reoptimize(ks, th, 3, ref, 1, 1.0)
            stream.synchronize()
            out.append([th] + [d.psi.clone() for d in ds])
        for other in out[1:]:
            assert all(torch.equal(a, b) for a, b in zip(out[0], other))
        plan.close()
        ctx.close()
