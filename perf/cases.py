"""Performance cases: what a user of this package runs, over its real range.

A case is a dict of plain values.  ``prepare`` makes what a program holds
before the call (parameters drawn from the seed, a bound plan or the device
tables and a start state), ``run`` is one pass through the public entry
points and returns its outputs, ``work`` the bytes and operations the pass
cannot do without, and ``exact`` the same outputs in 64 bits from plain torch
(the true exp(-iHt), or its derivative), independent of the package.

The FP64 sums that a complex64 plan returns (occupations, gradients) carry
the precision of the complex64 state, so ``run`` hands them on as float32;
a complex128 plan's stay float64.
"""

import ctypes
import math

import numpy as np
import torch

from paper_1612_00746_amd import Plan, _lib, graph_evolve, graph_tables, lattice_edges, lattice_evolve, make_problem

_CHAIN = dict(kind="chain", m=2, stat="distinguishable", bc="open", inter="onsite", dtype="c64", n=64, n_max=0, R=8,
              dt=0.05, tol=1e-7, jn=0.1, ee=0.5, U=1.0, steps=10, every=0, pair=False, rho=False, fresh=False,
              cpl=1, persistent=0, graph=0, form=0)
_GRAD = dict(kind="gradient", m=2, stat="boson", bc="open", inter="onsite", dtype="c64", n=64, n_max=0, R=8, dt=0.05,
             tol=1e-7, jn=0.1, ee=0.5, U=1.0, steps=16, ckpt=8, loss="product")
_LATTICE = dict(kind="lattice", dtype="c64", lx=16, ly=16, px=False, py=False, R=8, dt=0.05, order=10, steps=4)
_GRAPH = dict(kind="graph", dtype="c128", lx=15, ly=15, per=False, m=2, stat="boson", R=8, dt=0.05, order=10, steps=4)


def _case(base, name=None, **kw):
    c = dict(base, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest walk (workload C1): two walkers on 16 nodes, 8 realisations, the whole run of 500
        # steps with the occupation every 10 -- a parameter study or a test, all launches and latency.
        _case(_CHAIN, "two_small_c128", dtype="c128", n=16, R=8, dt=0.01, tol=1e-14, jn=0.1, ee=0.0, U=0.0, steps=500,
              every=10, fresh=True),
        # The paper's ensemble size (workload C2): 1000 realisations of two bosons on 128 nodes in double
        # precision, occupation and pair correlation every 20 steps.
        _case(_CHAIN, "bosons_c128", stat="boson", dtype="c128", n=128, R=1000, tol=1e-14, jn=0.2, U=2.0, steps=40,
              every=20, pair=True),
        # The same ensemble in single precision with its full density matrix every 10 steps, the
        # post-processing the paper's Eq. 2 asks for.
        _case(_CHAIN, "bosons_density_c64", stat="boson", n=128, R=1000, jn=0.2, U=2.0, steps=10, rho=True),
        # The headline batch (workload C3): 4096 realisations on chains of 64 to 1024 nodes, the launch
        # shape the benchmark's tuner settles on, occupation at the end of a run of 8 steps.
        _case(_CHAIN, "uneven_c64", n=64, n_max=1024, R=4096, ee=0.0, U=4.0, steps=8, every=8, cpl=2, persistent=1,
              graph=1),
        # One realisation on a long chain, 100 steps: an interactive look at a single noisy walk.
        _case(_CHAIN, "single_c64", n=1024, R=1, U=2.0, steps=100, every=50, fresh=True, cpl=2, graph=1),
        # The gradient workload (C4): two bosons on 256 nodes, 512 realisations, the probability that both
        # are in the last quarter, single precision.
        _case(_GRAD, "gradient_c64", n=256, R=512, steps=48, ckpt=16),
        # A small gradient in double precision: distinguishable walkers on a ring of odd length, one-body loss.
        _case(_GRAD, "gradient_ring_c128", stat="distinguishable", bc="periodic", dtype="c128", n=129, R=24, tol=1e-14,
              steps=40, ckpt=8, loss="one_body"),
        # Three walkers at the stated size (workload C5), product form as the benchmark runs it.
        _case(_CHAIN, "three_c64", m=3, inter="nearest", n=256, R=64, dt=0.02, jn=0.0, ee=1.0, U=1.0, steps=4, every=4,
              form=1, graph=1),
        # Three walkers on a small ring of odd length in double precision, library defaults.
        _case(_CHAIN, "three_ring_c128", m=3, inter="nearest", bc="periodic", dtype="c128", n=61, R=8, dt=0.02, tol=1e-12,
              jn=0.1, ee=1.0, steps=20, every=10, pair=True),
        # One walker on the benchmark's 128 x 128 lattice, 4096 realisations, 10 terms.
        _case(_LATTICE, "lattice_c64", lx=128, ly=128, R=4096, steps=20),
        # Odd sides and a ring along x in double precision, a few realisations.
        _case(_LATTICE, "lattice_ring_c128", dtype="c128", lx=97, ly=65, px=True, R=64, order=9, steps=20),
        # Two bosons on the paper's 15 x 15 lattice as one walker on the pair graph (25425 states).
        _case(_GRAPH, "graph_pairs_c128", lx=15, ly=15, R=32, steps=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _amps(c):
    """Amplitudes of one realisation (mean over an uneven batch)."""
    if c["kind"] == "lattice":
        return c["lx"] * c["ly"]
    if c["kind"] == "graph":
        n = c["lx"] * c["ly"]
        return n if c["m"] == 1 else {"distinguishable": n * n, "boson": n * (n + 1) // 2,
                                      "fermion": n * (n - 1) // 2}[c["stat"]]
    n = c["n"]
    if c["n_max"]:
        return (c["n"] ** 2 + c["n"] * c["n_max"] + c["n_max"] ** 2) / 3.0
    if c["m"] == 2 and c["stat"] != "distinguishable":
        return n * (n + 1) // 2
    return n ** c["m"]


def _terms(c):
    """Taylor terms of a step, from the a-priori bound at typical noise."""
    if "order" in c:
        return c["order"]
    x = c["dt"] * (c["m"] * (2.0 + 4 * c["jn"] + c["ee"]) + c["U"] * c["m"] * (c["m"] - 1) / 2)
    t, n = x, 0
    while n < 40:
        n += 1
        t *= x / (n + 1)
        if x < n + 2 and t / (1 - x / (n + 2)) <= c["tol"]:
            break
    return n


def draw(rng):
    budget = math.exp(rng.uniform(math.log(2e7), math.log(1.5e10)))     # amplitude-terms of the pass
    dtype = rng.choice(["c64", "c128"])
    tol = 1e-7 if dtype == "c64" else 1e-14
    pick = rng.random()
    if pick < 0.5:      # two walkers (or one) on chains and rings
        m = 1 if rng.random() < 0.2 else 2
        stat = rng.choice(["distinguishable", "distinguishable", "boson", "fermion"]) if m == 2 else "distinguishable"
        bc = "periodic" if stat == "distinguishable" and rng.random() < 0.3 else "open"
        c = _case(_CHAIN, m=m, stat=stat, bc=bc, dtype=dtype, tol=tol, inter=rng.choice(["onsite", "nearest"]),
                  n=_log_int(rng, 16, 1024 if m == 2 else 4096), jn=round(rng.uniform(0.0, 0.2), 3),
                  ee=rng.choice([0.0, 0.5]), U=round(rng.uniform(0.0, 4.0), 2) if m == 2 else 0.0,
                  dt=rng.choice([0.01, 0.05]), pair=m == 2 and rng.random() < 0.3, fresh=rng.random() < 0.5,
                  cpl=rng.choice([1, 2]), persistent=rng.choice([0, 1]), graph=rng.choice([0, 1]))
        if rng.random() < 0.2 and not c["pair"]:
            c["n_max"] = min(1024, c["n"] * 4)
        c["steps"] = _log_int(rng, 5, 200)
        c["every"] = rng.choice([0, max(1, c["steps"] // 4), 10])
        cap = 1024 if c["n_max"] else 4096
    elif pick < 0.62:   # three walkers
        c = _case(_CHAIN, m=3, inter=rng.choice(["onsite", "nearest"]), bc=rng.choice(["open", "periodic"]), dtype=dtype,
                  tol=max(tol, 1e-12), n=_log_int(rng, 16, 160), dt=0.02, ee=1.0, steps=_log_int(rng, 4, 20),
                  form=rng.choice([0, 1]), graph=rng.choice([0, 1]), pair=rng.random() < 0.5)
        c["every"] = c["steps"]
        cap = 64
    elif pick < 0.75:   # gradients
        stat = rng.choice(["boson", "distinguishable"])
        bc = "periodic" if stat == "distinguishable" and rng.random() < 0.4 else "open"
        c = _case(_GRAD, stat=stat, bc=bc, dtype=dtype, tol=tol, n=_log_int(rng, 16, 256), steps=_log_int(rng, 8, 48),
                  ckpt=rng.choice([4, 8, 16]), loss=rng.choice(["product", "one_body"]))
        budget /= 6
        cap = 512
    elif pick < 0.9:    # one walker on a lattice
        c = _case(_LATTICE, dtype=dtype, lx=_log_int(rng, 9, 300), ly=_log_int(rng, 9, 300), px=rng.random() < 0.3,
                  py=rng.random() < 0.3, order=rng.randint(6, 10), steps=_log_int(rng, 4, 40))
        cap = 4096
    else:               # general graphs, one walker or pairs
        m = rng.choice([1, 2])
        c = _case(_GRAPH, dtype=dtype, m=m, lx=_log_int(rng, 4, 15 if m == 2 else 64),
                  ly=_log_int(rng, 4, 15 if m == 2 else 64), per=rng.random() < 0.3,
                  stat=rng.choice(["distinguishable", "boson", "fermion"]) if m == 2 else "distinguishable",
                  order=rng.randint(6, 12), steps=_log_int(rng, 2, 12))
        budget /= 8
        cap = 256
    c["R"] = max(1, min(cap, int(budget / (_amps(c) * _terms(c) * c["steps"]))))
    if c.get("n_max") and c["R"] < 4:
        c["n_max"] = 0
    return c


# ---------------------------------------------------------------- inputs
def _chain_inputs(c, seed):
    """Lattice sizes (the case's own) and the packed J, eps, U of every
    realisation (drawn from the seed)."""
    g = np.random.Generator(np.random.Philox(key=int(seed)))
    if c["n_max"]:
        fixed = np.random.Generator(np.random.Philox(key=c["R"]))
        sizes = fixed.integers(0, (c["n_max"] - c["n"]) // 32 + 1, size=c["R"]) * 32 + c["n"]
        sizes = np.minimum(sizes, c["n_max"])
    else:
        sizes = np.full(c["R"], c["n"])
    bonds = sizes if c["bc"] == "periodic" else sizes - 1
    J = 1.0 + c["jn"] * np.clip(g.standard_normal(int(bonds.sum())), -4, 4)
    eps = c["ee"] * g.uniform(-1.0, 1.0, int(sizes.sum()))
    # uneven batches draw U per realisation, as the headline batch does
    U = g.uniform(0.0, c["U"], c["R"]) if c["n_max"] else np.full(c["R"], c["U"])
    return sizes.astype(np.int32), bonds, J, eps, U


def _start(c):
    n = c["n"]
    if c.get("loss") == "product":      # at the edge of the block whose probability is the loss
        return [n - n // 4 - 1, n - n // 4]
    return [n // 2] if c["m"] == 1 else ([n // 2 - 1, n // 2] if c["m"] == 2 else [n // 2 - 1, n // 2, n // 2 + 1])


def _counts(c, sizes):
    s = sizes.astype(np.int64)
    if c["m"] == 2 and c["stat"] != "distinguishable":
        return s * (s + 1) // 2
    return s ** c["m"]


def _ctype(c):
    return torch.complex64 if c["dtype"] == "c64" else torch.complex128


def _random_state(c, sizes, seed):
    """A spread state, as after some evolution: every amplitude occupied,
    each realisation's norm close to 1 (fermions: the diagonal is 0)."""
    counts = _counts(c, sizes)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    psi = torch.randn(int(counts.sum()), dtype=_ctype(c), generator=gen, device="cuda")
    tri = c["m"] == 2 and c["stat"] != "distinguishable"
    w = 1.0 / np.sqrt(counts * (2.0 if tri else 1.0))
    if c["n_max"]:
        rt = torch.float32 if c["dtype"] == "c64" else torch.float64
        psi *= torch.repeat_interleave(torch.from_numpy(w).to("cuda", rt), torch.from_numpy(counts).to("cuda"))
    else:
        psi *= float(w[0])
    if c["stat"] == "fermion":
        o = 0
        for n in sizes:
            i = np.arange(int(n))
            psi[torch.from_numpy(o + i * int(n) - i * (i - 1) // 2).to("cuda")] = 0
            o += int(n) * (int(n) + 1) // 2
    return psi


def _site_weights(c):
    n = c["n"]
    if c["loss"] == "product":
        return (np.arange(n) >= n - max(1, n // 4)).astype(float)
    return np.arange(n) / float(n)


def _lattice_inputs(c, seed):
    real = torch.float32 if c["dtype"] == "c64" else torch.float64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    shape = (c["R"], c["ly"], c["lx"])
    Jx = 1.0 + 0.1 * torch.randn(shape, dtype=real, generator=gen, device="cuda")
    Jy = 1.0 + 0.1 * torch.randn(shape, dtype=real, generator=gen, device="cuda")
    eps = torch.rand(shape, dtype=real, generator=gen, device="cuda") - 0.5
    psi = torch.randn(shape, dtype=_ctype(c), generator=gen, device="cuda") / math.sqrt(c["lx"] * c["ly"])
    return Jx, Jy, eps, psi


def _graph_inputs(c, seed):
    g = np.random.Generator(np.random.Philox(key=int(seed)))
    n = c["lx"] * c["ly"]
    edges = lattice_edges((c["ly"], c["lx"]), c["per"])
    J = 1.0 + 0.1 * g.standard_normal((c["R"], len(edges)))
    eps = g.uniform(-0.5, 0.5, (c["R"], n))
    U = np.full(c["R"], 2.0)
    D = _amps(c)
    psi = (g.standard_normal((c["R"], D)) + 1j * g.standard_normal((c["R"], D))) / math.sqrt(2.0 * D)
    return n, edges, J, eps, U, psi


def prepare(case, seed):
    c = case
    s = {"case": c}
    if c["kind"] == "lattice":
        s["Jx"], s["Jy"], s["eps"], s["psi"] = _lattice_inputs(c, seed)
        need = ctypes.c_int64()
        code = _lib.C64 if c["dtype"] == "c64" else _lib.C128
        _lib.check(_lib.load().ctqw_lattice_workspace(c["lx"], c["ly"], c["R"], code, c["order"], int(c["px"]),
                                                      ctypes.byref(need)))
        s["ws"] = torch.empty(need.value, dtype=torch.uint8, device="cuda")
        s["norms"] = torch.zeros((c["steps"], c["R"]), dtype=torch.float64, device="cuda")
        return s
    if c["kind"] == "graph":
        real = torch.float32 if c["dtype"] == "c64" else torch.float64
        n, edges, J, eps, U, psi = _graph_inputs(c, seed)
        nbr, hop, on = graph_tables(n, edges, J, eps, U if c["m"] == 2 else None, m=c["m"], statistics=c["stat"])
        s["nbr"] = torch.from_numpy(nbr).to("cuda")
        s["hop"] = torch.from_numpy(hop).to("cuda", real)
        s["on"] = torch.from_numpy(on).to("cuda", real)
        s["psi"] = torch.from_numpy(psi).to("cuda", _ctype(c))
        s["ws"] = torch.empty(3 * s["psi"].numel() * s["psi"].element_size(), dtype=torch.uint8, device="cuda")
        s["norms"] = torch.zeros((c["steps"], c["R"]), dtype=torch.float64, device="cuda")
        return s
    sizes, _, J, eps, U = _chain_inputs(c, seed)
    obs = 3 if c.get("pair") else 1
    pr, keep = make_problem(c["m"], c["R"], [int(n) for n in sizes] if c["n_max"] else c["n"], c["dt"],
                            statistics=c["stat"], boundary=c["bc"], interaction=c["inter"], dtype=c["dtype"],
                            taylor_tol=c["tol"], observables=obs)
    plan = Plan(pr)
    if c["kind"] == "chain":
        plan.set_launch(cols_per_lane=c["cpl"], persistent=c["persistent"], use_graph=c["graph"], three_form=c["form"])
    plan.set_params(J, eps, U)
    plan.bind("cuda")
    s.update(plan=plan, keep=keep, obs=obs)
    if c["kind"] == "gradient":
        s["start"], s["w"] = _start(c), _site_weights(c)
        return s
    s["psi"] = torch.empty(int(_counts(c, sizes).sum()), dtype=_ctype(c), device="cuda")
    if c["fresh"]:
        s["start"] = np.array([_start(dict(c, n=int(n))) for n in sizes], dtype=np.int32)
    else:
        psi = _random_state(c, sizes, seed)
        torch.cuda.current_stream().synchronize()
        _lib.check(plan.lib.ctqw_set_state(plan.h, ctypes.c_void_p(psi.data_ptr()), 1), plan.h)
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "lattice":
        lattice_evolve(s["Jx"], s["Jy"], s["eps"], s["psi"], c["dt"], c["order"], c["steps"],
                       periodic=(c["px"], c["py"]), workspace=s["ws"], norms=s["norms"])
        return {"psi": s["psi"], "norms": _held(c, s["norms"])}
    if c["kind"] == "graph":
        graph_evolve(s["nbr"], s["hop"], s["on"], s["psi"], c["dt"], c["order"], c["steps"], workspace=s["ws"],
                     norms=s["norms"])
        return {"psi": s["psi"], "norms": _held(c, s["norms"])}
    plan = s["plan"]
    if c["kind"] == "gradient":
        plan.init_product_state(s["start"])
        loss, gJ, gE = plan.gradient(c["steps"], c["ckpt"], s["w"], c["loss"])
        return {"loss": _held(c, np.array([loss])), "gJ": _held(c, gJ), "gE": _held(c, gE)}
    if c["fresh"]:
        plan.init_product_state(s["start"])
    out = {"obs": _held(c, plan.propagate(c["steps"], c["every"], s["obs"] if c["every"] else 0))}
    if c["rho"]:
        out["rho"] = plan.density_matrix(0)
    _lib.check(plan.lib.ctqw_get_state(plan.h, ctypes.c_void_p(s["psi"].data_ptr()), 1), plan.h)
    out["psi"] = s["psi"]
    return out


def _held(c, x):
    """FP64 sums at the precision of the state they were formed from."""
    if x is None or c["dtype"] == "c128":
        return x
    return x.astype(np.float32) if isinstance(x, np.ndarray) else x.float()


def work(case):
    c = case
    amps, terms, e = _amps(c) * c["R"], _terms(c), 8 if c["dtype"] == "c64" else 16
    if c["kind"] == "lattice":
        return {"bytes": amps * (2 * e + 3 * e // 2), "flops": 24.0 * amps * terms * c["steps"]}
    if c["kind"] == "graph":
        w = 4 * c["m"]
        return {"bytes": amps * (2 * e + (w + 1) * e // 2) + 4 * w * _amps(c), "flops": (4.0 * w + 8) * amps * terms * c["steps"]}
    per_term = 8.0 * c["m"] + 8
    if c["kind"] == "gradient":
        # forward, the forward vectors and the adjoint recursion with its contractions
        return {"bytes": 2.0 * c["R"] * c["n"] * 8, "flops": amps * terms * c["steps"] * (3 * per_term + 16)}
    b, f = 2.0 * e * amps + 2.0 * c["R"] * c["n"] * 8, per_term * amps * terms * c["steps"]
    if c["rho"]:
        d = _amps(c)
        b, f = b + e * d * d, f + 4.0 * d * (d + 1) * c["R"]
    return {"bytes": b, "flops": f}


# ------------------------------------------------- the same in 64 bits
def _chain_ops(c, n, J, eps, U):
    """Functions of one equal-size batch: J [R, bonds], eps [R, n], U [R] as
    device FP64; apply(t) = H t on the full grid [R, n, .., n]."""
    m, R = c["m"], J.shape[0]
    if c["bc"] == "periodic":
        jr = J
    else:
        jr = torch.cat([J, J.new_zeros(R, 1)], 1)       # bond to the right of each node
    jl = torch.roll(jr, 1, 1)
    idx = torch.arange(n, device=J.device)
    diag = 0.0
    for a in range(m):
        diag = diag + eps.view([R] + [n if b == a else 1 for b in range(m)])
    for a in range(m):
        for b in range(a + 1, m):
            xa = idx.view([n if k == a else 1 for k in range(m)])
            xb = idx.view([n if k == b else 1 for k in range(m)])
            d = (xa - xb).abs()
            if c["inter"] == "nearest":
                hit = (d == 1) | (d == n - 1 if c["bc"] == "periodic" else torch.zeros_like(d, dtype=torch.bool))
            else:
                hit = d == 0
            diag = diag + U.view([R] + [1] * m) * hit.to(torch.float64)
    diag = diag.to(torch.complex128)

    def apply(t):
        h = diag * t
        for a in range(m):
            shape = [R] + [n if b == a else 1 for b in range(m)]
            h = torch.addcmul(h, jr.view(shape).to(torch.complex128), torch.roll(t, -1, a + 1))
            h = torch.addcmul(h, jl.view(shape).to(torch.complex128), torch.roll(t, 1, a + 1))
        return h
    return apply


def _series(apply, psi, dt, small):
    """exp(-i dt H) psi to `small`, relative."""
    out, t, size = psi, psi, None
    for k in range(1, 60):
        t = apply(t) * complex(0.0, -dt / k)
        out = out + t
        norm = float(torch.linalg.vector_norm(t.detach()))
        size = norm / dt if size is None else size
        if norm <= small * float(torch.linalg.vector_norm(psi.detach())):
            break
    return out


def _exact_chain(c, seed):
    sizes, bonds, J, eps, U = _chain_inputs(c, seed)
    counts = _counts(c, sizes)
    first = np.concatenate([[0], np.cumsum(counts)])
    jo = np.concatenate([[0], np.cumsum(bonds)])
    eo = np.concatenate([[0], np.cumsum(sizes)])
    tri = c["m"] == 2 and c["stat"] != "distinguishable"
    start = None if c["fresh"] else _random_state(c, sizes, seed)
    final = torch.empty(int(first[-1]), dtype=torch.complex128, device="cuda")
    small = 1e-12 if c["dtype"] == "c64" else 1e-17
    outs = [k for k in range(c["steps"] + 1) if c["every"] and k % c["every"] == 0]
    snaps = {k: [] for k in outs}
    rho = None
    for n in sorted(set(int(v) for v in sizes)):
        members = [r for r in range(c["R"]) if sizes[r] == n]
        occ = {k: torch.zeros(n, dtype=torch.float64, device="cuda") for k in outs}
        pair = {k: torch.zeros((n, n), dtype=torch.float64, device="cuda") for k in outs}
        step = max(1, int(6e7 // n ** c["m"]))
        if tri:
            upper = torch.triu_indices(n, n, device="cuda")
        for b in range(0, len(members), step):
            rs = members[b:b + step]
            dev = lambda rows: torch.from_numpy(np.stack(rows)).to("cuda")  # noqa: E731
            apply = _chain_ops(c, n, dev([J[jo[r]:jo[r + 1]] for r in rs]), dev([eps[eo[r]:eo[r + 1]] for r in rs]),
                               torch.from_numpy(U[rs]).to("cuda"))
            t = torch.zeros([len(rs)] + [n] * c["m"], dtype=torch.complex128, device="cuda")
            if c["fresh"]:
                at = _start(dict(c, n=n))
                if tri:
                    t[:, at[0], at[1]] = 0.5 ** 0.5
                    t[:, at[1], at[0]] = -0.5 ** 0.5 if c["stat"] == "fermion" else 0.5 ** 0.5
                else:
                    t[tuple([slice(None)] + at)] = 1.0
            else:
                for k, r in enumerate(rs):
                    v = start[first[r]:first[r + 1]].to(torch.complex128)
                    if tri:
                        t[k][upper[1], upper[0]] = -v if c["stat"] == "fermion" else v
                        t[k][upper[0], upper[1]] = v
                    else:
                        t[k] = v.view(t[k].shape)
            for k in range(c["steps"] + 1):
                if k in occ:
                    p = t.abs().square().sum(0)
                    for a in range(c["m"]):
                        occ[k] += p.sum([x for x in range(c["m"]) if x != a]) if c["m"] > 1 else p
                    if c["pair"]:
                        for a in range(c["m"]):
                            for d in range(a + 1, c["m"]):
                                q = p.sum([x for x in range(c["m"]) if x not in (a, d)]) if c["m"] > 2 else p
                                pair[k] += q + q.T
                if k < c["steps"]:
                    t = _series(apply, t, c["dt"], small)
            for k, r in enumerate(rs):
                final[first[r]:first[r + 1]] = t[k][upper[0], upper[1]] if tri else t[k].reshape(-1)
            if c["rho"]:
                v = torch.stack([final[first[r]:first[r + 1]] for r in rs])
                v = v * torch.where(upper[0] == upper[1], 1.0, 2.0 ** 0.5) if tri else v
                part = v.T.contiguous() @ v.conj().resolve_conj().contiguous()
                rho = part if rho is None else rho + part
        for k in outs:
            snaps[k].append((occ[k] / len(members)).cpu().numpy())
            if c["pair"]:
                snaps[k].append((pair[k] / len(members)).cpu().numpy().reshape(-1))
    out = {"obs": np.stack([np.concatenate(snaps[k]) for k in outs]) if outs else None}
    if c["rho"]:
        out["rho"] = rho / c["R"]
    out["psi"] = final
    return out


def _exact_gradient(c, seed):
    n, R = c["n"], c["R"]
    _, _, J, eps, U = _chain_inputs(c, seed)
    dev = lambda v: torch.from_numpy(v).to("cuda")  # noqa: E731
    J, eps, U = dev(J.reshape(R, -1)), dev(eps.reshape(R, n)), dev(U)
    w = dev(_site_weights(c))
    w = w.view(n, 1) * w.view(1, n) if c["loss"] == "product" else w.view(n, 1) + w.view(1, n)
    small = 1e-12 if c["dtype"] == "c64" else 1e-17
    gJ, gE, loss = torch.zeros_like(J[0]), torch.zeros_like(eps[0]), 0.0
    per = max(1, int(2.0e7 // (n * n)))
    for b in range(0, R, per):
        rs = slice(b, min(R, b + per))
        t = torch.zeros((J[rs].shape[0], n, n), dtype=torch.complex128, device="cuda")
        x, y = _start(c)
        if c["stat"] == "boson":
            t[:, x, y] = t[:, y, x] = 0.5 ** 0.5
        else:
            t[:, x, y] = 1.0
        apply = _chain_ops(c, n, J[rs], eps[rs], U[rs])
        states = [t]
        for _ in range(c["steps"]):
            states.append(_series(apply, states[-1], c["dt"], small))
        loss += float((w * states[-1].abs().square()).sum()) / R
        lam = 2.0 * w * states[-1] / R
        for k in range(c["steps"] - 1, -1, -1):
            psi = states[k].requires_grad_(True)
            dJ, dE = torch.zeros_like(gJ).requires_grad_(True), torch.zeros_like(gE).requires_grad_(True)
            stepped = _series(_chain_ops(c, n, J[rs] + dJ, eps[rs] + dE, U[rs]), psi, c["dt"], small)
            lam, a, e = torch.autograd.grad(stepped, (psi, dJ, dE), grad_outputs=lam)
            gJ, gE = gJ + a, gE + e
            states[k + 1] = None
    return {"loss": np.array([loss]), "gJ": gJ.cpu().numpy(), "gE": gE.cpu().numpy()}


def _exact_grid(c, apply, psi):
    norms = []
    flat = [1 + a for a in range(psi.dim() - 1)]
    for _ in range(c["steps"]):
        psi = _series(apply, psi, c["dt"], 1e-12 if c["dtype"] == "c64" else 1e-17)
        norms.append(psi.abs().square().sum(flat))
    return {"psi": psi, "norms": torch.stack(norms)}


def exact(case, seed):
    c = case
    if c["kind"] == "chain":
        return _exact_chain(c, seed)
    if c["kind"] == "gradient":
        if _amps(c) * c["R"] * c["steps"] * _terms(c) > 1e10:
            return None     # autograd in 64 bits would take minutes
        return _exact_gradient(c, seed)
    if c["kind"] == "lattice":
        Jx, Jy, eps, psi = (v.to(torch.complex128) for v in _lattice_inputs(c, seed))
        if not c["px"]:
            Jx[:, :, -1] = 0
        if not c["py"]:
            Jy[:, -1, :] = 0
        jl, ju = torch.roll(Jx, 1, 2), torch.roll(Jy, 1, 1)

        def apply(t):
            h = eps * t
            h = torch.addcmul(h, Jx, torch.roll(t, -1, 2))
            h = torch.addcmul(h, jl, torch.roll(t, 1, 2))
            h = torch.addcmul(h, Jy, torch.roll(t, -1, 1))
            return torch.addcmul(h, ju, torch.roll(t, 1, 1))
        return _exact_grid(c, apply, psi)
    n, edges, J, eps, U, psi = _graph_inputs(c, seed)
    e = torch.from_numpy(edges.astype(np.int64)).to("cuda")
    J, eps = torch.from_numpy(J).to("cuda"), torch.from_numpy(eps).to("cuda")
    if c["m"] == 1:
        grid = torch.from_numpy(psi).to("cuda")
    else:       # pairs on the full n x n grid, symmetric or antisymmetric
        v = torch.from_numpy(psi).to("cuda")
        if c["stat"] == "distinguishable":
            grid = v.view(c["R"], n, n)
        else:
            up = torch.triu_indices(n, n, 0 if c["stat"] == "boson" else 1, device="cuda")
            wt = torch.where(up[0] == up[1], 1.0, 0.5 ** 0.5).to(torch.complex128)
            grid = torch.zeros((c["R"], n, n), dtype=torch.complex128, device="cuda")
            grid[:, up[1], up[0]] = v * wt * (1.0 if c["stat"] == "boson" else -1.0)
            grid[:, up[0], up[1]] = v * wt
    if c["dtype"] == "c64":
        grid = grid.to(torch.complex64).to(torch.complex128)
    h1 = torch.zeros((c["R"], n, n), dtype=torch.complex128, device="cuda")
    h1[:, e[:, 0], e[:, 1]] = J.to(torch.complex128)
    h1[:, e[:, 1], e[:, 0]] = J.to(torch.complex128)
    h1[:, range(n), range(n)] = eps.to(torch.complex128)
    if c["m"] == 1:
        if n * n * c["R"] > 2e9:
            return None     # a dense H per realisation would not fit
        got = _exact_grid(c, lambda t: torch.bmm(h1, t.unsqueeze(2)).squeeze(2), grid)
        return got
    hit = torch.from_numpy(np.eye(n)).to("cuda", torch.complex128) * float(U[0])
    got = _exact_grid(c, lambda t: torch.bmm(h1, t) + torch.bmm(t, h1) + hit * t, grid)
    if c["stat"] != "distinguishable":
        got["psi"] = got["psi"][:, up[0], up[1]] / wt
    else:
        got["psi"] = got["psi"].reshape(c["R"], -1)
    return got
