"""The work that a user of this library has it do, as cases to be timed.

A case is one call pattern of the public entry points (`paper_2606_29692_amd.binding`
and `batch`) at one size.  The kinds:

  request     one adaptive step of one state through the single calls: energy, pool
              gradients, selection (its index read by the host), Taylor update
  energy      one energy of one state (a Rayleigh quotient of a given operator)
  compile     one Pauli sum compiled to CSR on the device
  pool        a whole pool compiled to CSR, generator by generator
  admit       what a serving loop does when a run arrives: the FP32 operator compiled
              about its reference energy, and its sliced layout
  batch       adaptive steps of many states through a batch plan (one graph launch)
  linesearch  a batched adaptive step whose angles are chosen by line search
  reopt       one sweep that re-optimises every angle of each state's ansatz

Systems are the synthetic ones of `vqe_system` (seeded integrals, Jordan-Wigner or
Bravyi-Kitaev), with the register sizes and electron counts of its configurations.
"""
import math
from functools import lru_cache

import numpy as np
import torch

import vqe_system as vs
from paper_2606_29692_amd import batch as PB
from paper_2606_29692_amd import binding as B
from paper_2606_29692_amd import tune as T

DROP = 1e-12      # entries below DROP * max|c| are not stored
THETA_MAX = 1.0   # range of the line searches


def listed():
    return [
        # the smallest request: one 8-qubit run, one call after another; latency and launches
        {"name": "request_8q", "kind": "request", "qubits": 8, "mapping": "jw", "dtype": "c128"},
        # the same at the size of the published 14-qubit runs, in the other mapping
        {"name": "request_14q", "kind": "request", "qubits": 14, "mapping": "bk", "dtype": "c128"},
        # an energy of a register too large for on-chip memory, untuned
        {"name": "energy_16q", "kind": "energy", "qubits": 16, "mapping": "jw", "dtype": "c128"},
        # a new molecule's operator, the largest single compilation
        {"name": "compile_16q", "kind": "compile", "qubits": 16, "mapping": "bk", "dtype": "c128"},
        # the pool of a 12-qubit run: many small operators
        {"name": "pool_12q", "kind": "pool", "qubits": 12, "mapping": "jw", "dtype": "c128"},
        # a run admitted by the serving loop
        {"name": "admit_14q", "kind": "admit", "qubits": 14, "mapping": "jw", "dtype": "c64"},
        # a few small states in full precision, library defaults, CSR pool
        {"name": "batch_5x10q_fp64", "kind": "batch", "qubits": 10, "states": 5, "steps": 1,
         "mapping": "jw", "dtype": "c128", "start": "reference", "tuned": False},
        # the throughput workload: 64 complex 14-qubit states, several steps a launch
        {"name": "batch_64x14q", "kind": "batch", "qubits": 14, "states": 64, "steps": 3,
         "mapping": "jw", "dtype": "c64", "start": "complex", "tuned": True},
        # registers of 10, 12 and 14 qubits in one launch
        {"name": "batch_mixed_48", "kind": "batch", "qubits": 0, "states": 48, "steps": 1,
         "mapping": "jw", "dtype": "c64", "start": "complex", "tuned": True},
        # large registers: the state does not fit a compute unit's memory
        {"name": "batch_2x18q", "kind": "batch", "qubits": 18, "states": 2, "steps": 1,
         "mapping": "jw", "dtype": "c64", "start": "complex", "tuned": True},
        # adaptive runs from the reference with angles by line search
        {"name": "linesearch_48x12q", "kind": "linesearch", "qubits": 12, "states": 48, "steps": 1,
         "mapping": "jw", "dtype": "c64", "start": "reference", "tuned": True},
        # the ansatz so far re-optimised, angle by angle
        {"name": "reopt_16x14q", "kind": "reopt", "qubits": 14, "states": 16, "steps": 4,
         "mapping": "jw", "dtype": "c64", "start": "reference", "tuned": True},
    ]


def draw(rng):
    while True:
        kind = rng.choice(["request", "energy", "compile", "pool", "admit", "batch", "batch",
                           "batch", "linesearch", "reopt"])
        case = {"kind": kind, "qubits": rng.choice([4, 6, 8, 10, 12, 14, 16]),
                "mapping": rng.choice(["jw", "jw", "bk"]), "dtype": rng.choice(["c128", "c64"])}
        if kind == "pool":
            case["qubits"] = min(case["qubits"], 12)
        if kind == "admit":
            case.update(qubits=max(case["qubits"], 12), mapping="jw", dtype="c64")
        if kind in ("batch", "linesearch", "reopt"):
            case["states"] = int(round(math.exp(rng.uniform(0.0, math.log(64.0)))))
            case["steps"] = rng.randint(1, 4)
            case["start"] = rng.choice(["complex", "reference"]) if kind == "batch" else "reference"
            case["tuned"] = rng.random() < 0.75
            if case["tuned"]:
                case["dtype"] = "c64"
            if kind != "batch":
                # full-precision angles of a flat minimum are not comparable
                case["dtype"] = "c64"
            if case["tuned"] and kind == "batch" and rng.random() < 0.2:
                case.update(qubits=0, mapping="jw", start="complex")
        if _cost(case) <= _cost(LARGEST):
            return case


# ------------------------------------------------------------------ sizes
def _sizes(case):
    """Register size of every state of the case."""
    if "states" not in case:
        return [case["qubits"]]
    return [case["qubits"] or (10, 12, 14)[s % 3] for s in range(case["states"])]


@lru_cache(maxsize=None)
def _counts(n):
    """(entries of H, entries of the pool's generators, generators, terms of H) at n qubits."""
    m, dim, e = n // 2, 1 << n, vs.ELECTRONS[n] // 2
    c2, c4 = math.comb(m, 2), math.comb(m, 4)
    nnz = dim - 1 + dim * c2 + (2 * c4 * 6 * dim) // 16 + (c2 * c2 * dim) // 4
    v = m - e
    singles, doubles = 2 * e * v, 2 * math.comb(e, 2) * math.comb(v, 2) + (e * v) ** 2
    return nnz, singles * dim // 2 + doubles * dim // 8, singles + doubles, n ** 4 // 11


def _cost(case):
    """A size to hold drawn cases below the largest listed one."""
    per = sum(_counts(n)[0] for n in _sizes(case))
    kind = case["kind"]
    if kind in ("compile", "admit"):
        return 40 * per
    if kind == "pool":
        return 40 * _counts(case["qubits"])[1]
    return per * {"linesearch": 3, "reopt": 4}.get(kind, 1) * case.get("steps", 1)


LARGEST = next(c for c in listed() if c["name"] == "batch_64x14q")


def work(case):
    """Bytes and operations of a pass: each input and output once; two multiply-adds for
    each entry of H (real entries, complex amplitudes), six for each pair of a generator."""
    el = 8 if case["dtype"] == "c64" else 16
    kind, nb, fl = case["kind"], 0.0, 0.0
    for n in _sizes(case):
        dim, (nnz, pool, m, terms) = 1 << n, _counts(n)
        csr = 4 * (dim + 1) + nnz * (4 + el)
        if kind == "energy":
            nb, fl = nb + csr + 2 * dim * el, fl + 4 * nnz
        elif kind == "request":
            nb += csr + pool * (4 + el) + 4 * m * (dim + 1) + 3 * dim * el
            fl += 4 * nnz + 6 * pool
        elif kind in ("compile", "admit"):
            nb, fl = nb + 32 * terms + csr, fl + nnz
        elif kind == "pool":
            nb, fl = nb + pool * (4 + el) + 4 * m * (dim + 1), fl + pool
        else:
            # the plan keeps H in a form of its own; the least it can hold is the Pauli sum
            products = {"batch": 1, "linesearch": 3, "reopt": 3}[kind] * case["steps"]
            nb += 32 * terms + 3 * dim * el + 8 * m
            fl += 4 * nnz * products + (6 * pool * case["steps"] if kind != "reopt" else 0)
    return {"bytes": nb, "flops": fl}


# ------------------------------------------------------------------ inputs
@lru_cache(maxsize=None)
def _context():
    """The program's stream and context, made once."""
    stream = torch.cuda.Stream()
    torch.cuda.set_stream(stream)
    return B.Context(0, stream)


def _use():
    ctx = _context()
    torch.cuda.set_stream(ctx.stream)
    return ctx


def _seed(seed, state):
    return int(np.random.SeedSequence([int(seed), int(state)]).generate_state(1)[0])


def _systems(case, seed):
    return [vs.make_system(vs.SystemSpec(n, vs.ELECTRONS[n], case["mapping"], False, _seed(seed, s)))
            for s, n in enumerate(_sizes(case))]


@lru_cache(maxsize=None)
def _sector(n, mapping):
    return vs.sector_indices(vs.make_system(vs.SystemSpec(n, vs.ELECTRONS[n], mapping, False, 0),
                                            with_pool=False))


def _state(system, kind, seed, eps=0.1):
    """A state of the system's particle sector: the reference determinant, or with it a
    Gaussian complex part over the sector."""
    spec = system.spec
    psi = np.zeros(1 << spec.n_qubits, dtype=np.complex128)
    if kind == "complex":
        idx = _sector(spec.n_qubits, spec.mapping)
        rng = np.random.default_rng([int(seed) & 0x7fffffff, 7])
        z = rng.standard_normal(idx.size) + 1j * rng.standard_normal(idx.size)
        psi[idx] = eps * z / np.sqrt(2.0 * idx.size)
    psi[system.reference_index] += 1.0
    return psi / np.linalg.norm(psi)


def _states(case, seed, systems):
    kind = case.get("start", "complex")
    out = [_state(s, kind, _seed(seed, i)) for i, s in enumerate(systems)]
    return [p.astype(np.complex64) for p in out] if case["dtype"] == "c64" else out


def _angles(case, seed):
    rng = np.random.default_rng([int(seed) & 0x7fffffff, 11])
    return rng.uniform(-0.1, 0.1, size=(case.get("steps", 1), case.get("states", 1)))


def _indices(case, seed):
    rng = np.random.default_rng([int(seed) & 0x7fffffff, 13])
    m = [_counts(n)[2] for n in _sizes(case)]
    return np.stack([rng.integers(0, k, size=case["steps"]) for k in m]).astype(np.int32)


def _schedules(ctx, case, ds):
    """The tuned schedule of each register size where the library ships one, else its default."""
    if not case["tuned"]:
        return None
    form = "complex" if case["start"] == "complex" else "any"
    out = []
    for d in ds:
        known = case["mapping"] == "jw" or d.n_qubits in (14, 16)
        out.append(T.schedule_for(ctx, d, value_form=form) if known and d.n_qubits >= 10 else 0)
    return out


def prepare(case, seed):
    ctx = _use()
    kind, dtype = case["kind"], case["dtype"]
    systems = _systems(case, seed)
    sy = systems[0]
    if kind in ("compile", "pool"):
        return {"kind": kind, "ctx": ctx, "dtype": dtype,
                "packs": [sy.hamiltonian] if kind == "compile" else _scaled(sy.pool, seed)}
    if kind == "admit":
        pools = PB.PoolCache(ctx, matrix_free=True)
        probe = PB.device_system(ctx, sy, dtype, pools)
        return {"kind": kind, "ctx": ctx, "dtype": dtype, "system": sy, "pools": pools,
                "schedule": T.schedule_for(ctx, probe)}
    psis = _states(case, seed, systems)
    if kind in ("energy", "request"):
        H = B.csr_from_pack(ctx, sy.hamiltonian, dtype)
        psi = torch.from_numpy(psis[0]).to(ctx.torch_device)
        st = {"kind": kind, "ctx": ctx, "H": H, "psi": psi, "sigma": torch.empty_like(psi)}
        if kind == "request":
            st["pool"] = B.pool_from_packs(ctx, sy.pool, dtype)
            st["theta"] = float(_angles(case, seed)[0, 0])
        ctx.stream.synchronize()
        return st
    # plans: matrix-free pools, except that untuned full-precision plans use CSR pools
    pools = PB.PoolCache(ctx, matrix_free=case["tuned"] or dtype == "c64")
    ds = [PB.device_system(ctx, s, dtype, pools) for s in systems]
    flat = torch.from_numpy(np.concatenate(psis)).to(ctx.torch_device)
    at = 0
    for d in ds:                       # the states side by side in one buffer
        d.psi, at = flat[at:at + d.H.dim], at + d.H.dim
    plan = PB.make_batch(ctx, ds, schedules=_schedules(ctx, case, ds))
    st = {"kind": kind, "ctx": ctx, "plan": plan, "psi": flat, "steps": case["steps"],
          "tiled": case["start"] == "complex"}
    if kind == "batch":
        st["rows"] = torch.from_numpy(_angles(case, seed)).to(ctx.torch_device)
    elif kind == "linesearch":
        plan.set_line_search(THETA_MAX)
    else:
        st["refs"] = [d.psi.clone() for d in ds]
        st["ks"] = torch.from_numpy(_indices(case, seed)).to(ctx.torch_device)
        st["thetas"] = torch.from_numpy(_angles(case, seed).T.copy()).to(ctx.torch_device)
    ctx.stream.synchronize()
    return st


def _scaled(packs, seed):
    """A pool whose generators carry a seeded real scale each."""
    rng = np.random.default_rng([int(seed) & 0x7fffffff, 17])
    return [vs.PauliPack(p.n_qubits, p.xmask, p.zmask, p.coeff * s)
            for p, s in zip(packs, rng.uniform(0.5, 1.5, size=len(packs)))]


# ------------------------------------------------------------------ one pass
def _flat(ops):
    return [torch.cat([o.rowptr for o in ops]), torch.cat([o.col for o in ops]),
            torch.cat([o.val for o in ops])]


def run(st):
    ctx, kind = st["ctx"], st["kind"]
    if kind == "request":
        out = B.energy(ctx, st["H"], st["psi"], st["sigma"])
        g = B.pool_gradients(ctx, st["H"], st["pool"], st["psi"], st["sigma"])
        k, gmax = B.vqe_select(ctx, g)
        kk = int(k.cpu()[0])
        B.taylor5_apply(ctx, st["pool"].ops[kk], st["theta"], st["psi"], renormalize=True)
        return {"energy": out, "g": g, "gmax": gmax, "k": k, "psi": st["psi"], "sigma": st["sigma"]}
    if kind == "energy":
        out = B.energy(ctx, st["H"], st["psi"], st["sigma"])
        return {"energy": out, "sigma": st["sigma"]}
    if kind == "compile":
        H = B.csr_from_pack(ctx, st["packs"][0], st["dtype"])
        return {"rowptr": H.rowptr, "col": H.col, "val": H.val}
    if kind == "pool":
        pool = B.pool_from_packs(ctx, st["packs"], st["dtype"])
        rowptr, col, val = _flat(pool.ops)
        return {"rowptr": rowptr, "col": col, "val": val}
    if kind == "admit":
        ds = PB.device_system(ctx, st["system"], st["dtype"], st["pools"])
        layout = B.Layout(ctx, ds.H, st["schedule"])
        st["run"] = (ds, layout)       # the run stays resident; the previous one leaves
        return {"rowptr": ds.H.rowptr, "col": ds.H.col, "val": ds.H.val, "psi": ds.psi}
    plan = st["plan"]
    if kind == "batch":
        plan.run(st["rows"], tiled_screen=st["tiled"])
        return {"energy": plan.energies, "g": plan.g, "gmax": plan.gmax, "k": plan.k,
                "psi": st["psi"]}
    if kind == "linesearch":
        plan.run(None, line_search_steps=st["steps"])
        return {"k": plan.k, "psi": st["psi"]}
    plan.reoptimize(st["ks"], st["thetas"], st["steps"], st["refs"], 1, THETA_MAX)
    return {"psi": st["psi"]}


# ------------------------------------------------------------------ the same in 64 bits
def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _parity(v):
    for s in (16, 8, 4, 2, 1):
        v = v ^ (v >> s)
    return v & 1


def _groups(pack):
    """(flip mask, entries by row) of the Pauli sum, one flip mask after another."""
    dev = _dev()
    dim = 1 << pack.n_qubits
    x = np.asarray(pack.xmask, dtype=np.int64)
    z = torch.from_numpy(np.asarray(pack.zmask, dtype=np.int64).astype(np.int32)).to(dev)
    ph = np.array([1, 1j, -1, -1j])[[bin(int(a)).count("1") % 4 for a in
                                     (np.asarray(pack.xmask) & np.asarray(pack.zmask))]]
    c = np.asarray(pack.coeff) * ph
    c = torch.from_numpy(np.stack([c.real, c.imag])).to(dev)
    order = np.argsort(x, kind="stable")
    heads = np.flatnonzero(np.r_[True, np.diff(x[order]) != 0])
    rows = torch.arange(dim, device=dev, dtype=torch.int32)
    for a, b in zip(heads, np.r_[heads[1:], x.size]):
        t = torch.from_numpy(order[a:b].copy()).to(dev)
        col = rows ^ int(x[order[a]])
        v = torch.zeros(2, dim, dtype=torch.float64, device=dev)
        for i in range(0, t.numel(), 64):
            sub = t[i:i + 64]
            sign = 1.0 - 2.0 * _parity(z[sub][:, None] & col[None, :]).double()
            v += c[:, sub] @ sign
        yield int(x[order[a]]), torch.complex(v[0], v[1])


def _operator(pack):
    xs, vals = zip(*_groups(pack))
    vals = torch.stack([v.real for v in vals]) if all(float(v.imag.abs().max()) == 0 for v in vals) \
        else torch.stack(vals)
    return xs, vals


def _apply(op, psi):
    rows = torch.arange(psi.numel(), device=psi.device)
    out = torch.zeros_like(psi)
    for x, v in zip(*op):
        out += v * psi[rows ^ x]
    return out


def _generators(packs):
    """Every generator of a pool flips one mask: (masks, entries by generator and row)."""
    ops = [_operator(p) for p in packs]
    return torch.tensor([o[0][0] for o in ops], device=_dev()), torch.cat([o[1] for o in ops])


@lru_cache(maxsize=4)
def _pool(n, mapping):
    return _generators(vs.shared_pool(n, vs.ELECTRONS[n], mapping))


def _gradients(pool, psi, sigma):
    rows = torch.arange(psi.numel(), device=psi.device)
    return torch.stack([2.0 * torch.vdot(sigma, v * psi[rows ^ int(x)]).real
                        for x, v in zip(pool[0].tolist(), pool[1])])


def _generator_apply(pool, k, psi):
    rows = torch.arange(psi.numel(), device=psi.device)
    return pool[1][k] * psi[rows ^ int(pool[0][k])]


def _taylor(pool, k, theta, psi):
    acc, v, c = psi.clone(), psi, 1.0
    for n in range(1, 6):
        v, c = _generator_apply(pool, k, v), c * theta / n
        acc = acc + c * v
    return acc


def _select(g):
    gmax = float(g.abs().max())
    return int(torch.nonzero(g.abs() >= gmax * (1.0 - 1e-6))[0, 0]), gmax


def _minimum(K, G, t_alt):
    """The angle in [-THETA_MAX, THETA_MAX] of the lowest energy."""
    def parts(t):
        f = np.stack([np.ones_like(t), t - t ** 3 / 6 + t ** 5 / 120, t ** 2 / 2 - t ** 4 / 24])
        d = np.stack([np.zeros_like(t), 1 - t ** 2 / 2 + t ** 4 / 24, t - t ** 3 / 6])
        q = lambda a, M, b: np.einsum("it,ij,jt->t", a, M, b)  # noqa: E731
        num, den = q(f, K, f), q(f, G, f)
        return num / den, q(d, K, f) * den - num * q(d, G, f)

    grid = np.linspace(-THETA_MAX, THETA_MAX, 256)
    e, _ = parts(grid)
    i = int(np.argmin(e))
    lo, hi = grid[max(i - 1, 0)], grid[min(i + 1, 255)]
    best, eb = grid[i], e[i]
    slope = lambda t: parts(np.array([t]))[1][0]  # noqa: E731
    if slope(lo) < 0 < slope(hi):
        for _ in range(100):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if slope(mid) < 0 else (lo, mid)
        t = 0.5 * (lo + hi)
        if parts(np.array([t]))[0][0] < eb:
            best, eb = t, parts(np.array([t]))[0][0]
    return t_alt if parts(np.array([t_alt]))[0][0] < eb else best


def _forms(op, w):
    hw = [_apply(op, v) for v in w]
    K = np.array([[float(torch.vdot(a, b).real) for b in hw] for a in w])
    G = np.array([[float(torch.vdot(a, b).real) for b in w] for a in w])
    return 0.5 * (K + K.T), G


def _unit(v):
    return v / torch.linalg.vector_norm(v)


def _csr(pack, shift_row=None):
    """Row starts and values in row order, columns ascending, of the compiled sum."""
    xs, vals = _operator(pack)
    vals = vals.to(torch.complex128)
    dim = 1 << pack.n_qubits
    tol = DROP * float(np.abs(pack.coeff).max())
    keep = (vals.real.abs() > tol) | (vals.imag.abs() > tol)
    masks = torch.tensor(xs, device=vals.device)
    if shift_row is not None:          # every diagonal entry is stored, less the reference's
        at = int(torch.nonzero(masks == 0)[0, 0])
        keep[at] = True
        vals[at] = vals[at] - vals[at, shift_row].real
    key = []
    for g in range(masks.numel()):
        r = torch.nonzero(keep[g])[:, 0]
        key.append(torch.stack([r * dim + (r ^ masks[g]), g * dim + r]))
    key = torch.cat(key, dim=1)
    return vals.reshape(-1)[key[1][torch.argsort(key[0])]]


def exact(case, seed):
    kind = case["kind"]
    systems = _systems(case, seed)
    sy = systems[0]
    if kind == "compile":
        return {"rowptr": None, "col": None, "val": _csr(sy.hamiltonian)}
    if kind == "pool":
        return {"rowptr": None, "col": None,
                "val": torch.cat([_csr(p) for p in _scaled(sy.pool, seed)])}
    if kind == "admit":
        psi = torch.from_numpy(vs.reference_state(sy)).to(_dev())
        return {"rowptr": None, "col": None, "val": _csr(sy.hamiltonian, sy.reference_index),
                "psi": psi}
    thetas, outs = _angles(case, seed), []
    for i, (s, p) in enumerate(zip(systems, _states(case, seed, systems))):
        op = _operator(s.hamiltonian)
        psi = torch.from_numpy(p.astype(np.complex128)).to(_dev())
        outs.append(_exact_state(case, seed, i, s, op, psi, thetas[:, i if "states" in case else 0]))
    if "states" not in case:
        return outs[0]
    cat = lambda k: torch.cat([o[k] for o in outs])  # noqa: E731
    out = {"psi": cat("psi")}
    if kind != "reopt":
        out["k"] = None
    if kind == "batch":
        out.update(energy=cat("energy"), g=cat("g"), gmax=cat("gmax"))
    return out


def _exact_state(case, seed, i, s, op, psi, thetas):
    kind, dev = case["kind"], psi.device
    pool = None if kind == "energy" else _pool(s.spec.n_qubits, s.spec.mapping)
    if kind == "reopt":
        ks, ts, n = _indices(case, seed)[i].tolist(), thetas.tolist(), case["steps"]
        left = psi
        for m in range(n):
            v1 = _generator_apply(pool, ks[m], left)
            w = [left, v1, _generator_apply(pool, ks[m], v1)]
            for q in range(m + 1, n):
                w = [_taylor(pool, ks[q], ts[q], v) for v in w]
            ts[m] = _minimum(*_forms(op, w), ts[m])
            left = _taylor(pool, ks[m], ts[m], left)
        return {"psi": _unit(left)}
    for step in range(case.get("steps", 1)):
        sigma = _apply(op, psi)
        n2, e = float(torch.vdot(psi, psi).real), torch.vdot(psi, sigma)
        energy = torch.tensor([float(e.real) / n2, n2, 0.0], dtype=torch.float64, device=dev)
        if kind == "energy":
            return {"energy": energy, "sigma": sigma}
        g = _gradients(pool, psi, sigma)
        k, gmax = _select(g)
        if kind == "linesearch":
            v1 = _generator_apply(pool, k, psi)
            theta = _minimum(*_forms(op, [psi, v1, _generator_apply(pool, k, v1)]), 0.0)
        else:
            theta = float(thetas[step])
        psi = _unit(_taylor(pool, k, theta, psi))
    out = {"energy": energy, "g": g, "gmax": torch.tensor([gmax], dtype=torch.float64, device=dev),
           "k": None, "psi": psi}
    return dict(out, sigma=sigma) if kind == "request" else out
