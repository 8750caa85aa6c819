"""The workloads that a user of the particle library has it do, as measurable
cases: steps in every layout and integrator, fused steps, the transposes,
checkpointed advection with its adjoint, batches of uneven sets, removal and
fused array expressions, from calls on a thousand particles to 1e8.

Sizes, records and distributions are those of the benchmark and the tests:
positions U[0, 2 pi)^3, velocities and accelerations N(0, 1), field
amplitudes 0.5 to 1.5 and dt 1e-4 to 1e-2.  listed() names the standing
cases, draw() gives more of the same ranges, prepare() makes a case's inputs
on the GPU, run() is one call of a user's program, work() the bytes and
operations it cannot do without and exact() its results in plain float64.
"""
import ctypes
import math

import torch

import paper_1710_03462_amd as soax

BOX = 2.0 * math.pi

# Records of the workloads (name, type, components).
SCHEMAS = {
    "base": [("id", "i32", 1), ("pos", "f64", 3), ("vel", "f32", 3)],
    "f64": [("id", "i32", 1), ("pos", "f64", 3), ("vel", "f64", 3)],
    "wide": [("tag", "i64", 1), ("id", "i32", 1), ("pos", "f64", 3), ("vel", "f32", 3),
             ("acc", "f32", 3), ("mass", "f64", 1), ("flags", "u8", 1)],
    "particle0": [("pos", "f32", 3), ("vel", "f32", 3)],
    "particle8": [("pos", "f32", 3), ("vel", "f32", 3), ("temp0", "f32", 3), ("temp1", "f32", 3),
                  ("temp2", "f32", 2)],
}
TORCH = {"i8": torch.int8, "u8": torch.uint8, "i32": torch.int32, "i64": torch.int64,
         "f32": torch.float32, "f64": torch.float64}
SIZE = {"i8": 1, "u8": 1, "i32": 4, "i64": 8, "f32": 4, "f64": 8}
FIELD_INTEGRATORS = ("rk2_abc", "heun_abc", "rk4_abc")
# Field evaluations of one step (the stored velocity included), and the
# floating operations of one: six sines and cosines at about 20 operations and
# six multiplications and three additions, plus the stages' own updates.
EVALUATIONS = {"rk2_abc": 3, "heun_abc": 3, "rk4_abc": 5}
EVAL_FLOPS = 6 * 20 + 15


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # The headline of the benchmark: 1e8 particles, RK2 in the ABC field.
        {"name": "step_rk2_soa_1e8", "kind": "step", "schema": "base", "layout": "soa",
         "integrator": "rk2_abc", "n": 100_000_000, "nsteps": 20, "dt": 1e-3,
         "A": 1.0, "B": 1.0, "C": 1.0},
        # The same record kept as an array of structures, the Euler step.
        {"name": "step_euler_aos_1e8", "kind": "step", "schema": "base", "layout": "aos",
         "integrator": "euler", "n": 100_000_000, "nsteps": 10, "dt": 1e-3,
         "A": 0.0, "B": 0.0, "C": 0.0},
        # The benchmark's small workload: 1e5 particles, 100 Euler steps, in cache.
        {"name": "step_euler_soa_1e5", "kind": "step", "schema": "base", "layout": "soa",
         "integrator": "euler", "n": 100_000, "nsteps": 100, "dt": 1e-3,
         "A": 0.0, "B": 0.0, "C": 0.0},
        # The smallest call: one step of a thousand particles, as a program
        # makes it that does work of its own between steps.
        {"name": "step_rk2_soa_1e3", "kind": "step", "schema": "base", "layout": "soa",
         "integrator": "rk2_abc", "n": 1_000, "nsteps": 1, "dt": 1e-3,
         "A": 1.0, "B": 1.0, "C": 1.0},
        # A higher-order step of a ragged size with double velocities and a
        # larger time step.
        {"name": "step_rk4_soa_f64_ragged", "kind": "step", "schema": "f64", "layout": "soa",
         "integrator": "rk4_abc", "n": 6_000_017, "nsteps": 10, "dt": 1e-2,
         "A": 1.0, "B": 0.8, "C": 0.6},
        # Several steps with nothing between them, in one launch.
        {"name": "fused_rk2_1e7", "kind": "fused", "schema": "base", "integrator": "rk2_abc",
         "n": 10_000_000, "nsteps": 50, "dt": 1e-3, "A": 1.0, "B": 1.0, "C": 1.0},
        # The wide record brought from structures to arrays and back.
        {"name": "transpose_wide_3e7", "kind": "transpose", "schema": "wide", "n": 30_000_000},
        # The differentiable workload: 200 checkpointed steps, loss and adjoint.
        {"name": "adjoint_1e7_200", "kind": "adjoint", "route": "calls", "n": 10_000_000,
         "nsteps": 200, "k": 20, "dt": 5e-3, "A": 1.0, "B": 0.8, "C": 0.6},
        # A small fit through torch.autograd with a ragged size, a checkpoint
        # interval that does not divide the steps and a larger time step.
        {"name": "adjoint_autograd_ragged", "kind": "adjoint", "route": "autograd", "n": 60_001,
         "nsteps": 130, "k": 16, "dt": 1e-2, "A": 1.2, "B": 0.9, "C": 0.7},
        # 256 uneven sets stepped together, replayed from a graph.
        {"name": "batch_256_sets", "kind": "batch", "nsets": 256, "lo": 1_000, "hi": 1_000_000,
         "nsteps": 20},
        # One percent of the headline set leaves the domain.
        {"name": "remove_1e8", "kind": "remove", "schema": "base", "n": 100_000_000,
         "fraction": 0.01},
        # A fused expression over whole arrays of the headline set.
        {"name": "expr_speed_1e8", "kind": "expr", "expr": "speed", "n": 100_000_000},
    ]


def _log_int(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return v | 1 if rng.random() < 0.6 else v


def _field(rng):
    return {"dt": 10.0 ** rng.uniform(-4, -2), "A": rng.uniform(0.5, 1.5),
            "B": rng.uniform(0.5, 1.5), "C": rng.uniform(0.5, 1.5)}


def draw(rng):
    kind = rng.choice(["step", "step", "step", "fused", "transpose", "adjoint", "adjoint",
                       "batch", "remove", "expr"])
    if kind == "step":
        integrator = rng.choice(["rk2_abc", "rk2_abc", "heun_abc", "rk4_abc", "euler", "euler",
                                 "euler_acc", "symplectic_euler"])
        if integrator in FIELD_INTEGRATORS:
            schema = rng.choice(["base", "base", "f64"])
        elif integrator == "euler":
            schema = rng.choice(["base", "f64", "particle0", "particle8"])
        else:
            schema = "wide"
        n = _log_int(rng, 1_000, 50_000_000)
        return {"kind": kind, "schema": schema, "integrator": integrator, "n": n,
                "layout": rng.choice(["soa", "soa", "aos", "aosoa"]),
                "nsteps": max(1, min(rng.choice([1, 5, 20, 100]), 1_000_000_000 // n)),
                **_field(rng)}
    if kind == "fused":
        n = _log_int(rng, 1_000, 10_000_000)
        return {"kind": kind, "schema": rng.choice(["base", "f64"]),
                "integrator": rng.choice(["rk2_abc", "heun_abc", "rk4_abc", "euler"]), "n": n,
                "nsteps": max(1, min(rng.randint(10, 200), 500_000_000 // n)), **_field(rng)}
    if kind == "transpose":
        return {"kind": kind, "schema": rng.choice(["base", "wide", "f64", "particle8"]),
                "n": _log_int(rng, 1_000, 30_000_000)}
    if kind == "adjoint":
        n = _log_int(rng, 1_000, 10_000_000)
        nsteps = max(10, min(rng.choice([rng.randint(10, 200), 20 * rng.randint(1, 10)]),
                             2_000_000_000 // n))
        return {"kind": kind, "route": rng.choice(["calls", "autograd"]), "n": n, "nsteps": nsteps,
                "k": rng.choice([20, 20, 10, rng.randint(3, 40)]), **_field(rng)}
    if kind == "batch":
        hi = _log_int(rng, 3_000, 1_000_000)
        return {"kind": kind, "nsets": rng.randint(4, 256), "lo": 1_000, "hi": hi,
                "nsteps": rng.randint(5, 20)}
    if kind == "remove":
        return {"kind": kind, "schema": rng.choice(["base", "wide"]),
                "n": _log_int(rng, 1_000, 30_000_000), "fraction": 10.0 ** rng.uniform(-3, -0.5)}
    return {"kind": kind, "expr": rng.choice(["speed", "difference"]),
            "n": _log_int(rng, 1_000, 100_000_000)}


# ------------------------------------------------------------------ the inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _box(n, g):
    x = torch.rand(n, generator=g, dtype=torch.float64, device="cuda").mul_(BOX)
    return x.clamp_(max=math.nextafter(BOX, 0.0))


def _fields(fields, n, g):
    """One device tensor per (property, component), in schema order."""
    out = []
    for name, t, dim in fields:
        for _ in range(dim):
            if name == "id":
                a = torch.arange(n, dtype=TORCH[t], device="cuda")
            elif name == "pos":
                a = _box(n, g).to(TORCH[t])
                if t == "f32":
                    a.clamp_(max=6.2831850)
            elif name in ("vel", "acc"):
                a = torch.randn(n, generator=g, dtype=TORCH[t], device="cuda")
            elif name == "mass":
                a = torch.rand(n, generator=g, dtype=TORCH[t], device="cuda").mul_(1.5).add_(0.5)
            elif t in ("f32", "f64"):
                a = torch.rand(n, generator=g, dtype=TORCH[t], device="cuda")
            else:
                hi = 256 if t == "u8" else 2 ** 31 - 1
                a = torch.randint(0, hi, (n,), generator=g, dtype=TORCH[t], device="cuda")
            out.append(a)
    return out


def _set(fields, n, g, **options):
    ps = soax.ParticleSet(fields, n, **options)
    for dst, src in zip(ps.soa, _fields(fields, n, g)):
        dst.copy_(src)
    return ps


def _leaving(case):
    return max(1, int(case["n"] * case["fraction"]))


def _wrap_of(case):
    return SCHEMAS[case["schema"]][_index(case["schema"], "pos")][1] == "f64"


def _index(schema, name):
    return [f[0] for f in SCHEMAS[schema]].index(name)


def _abc(case):
    return [case["A"], case["B"], case["C"]]


def _batch_plan(case, seed):
    g = torch.Generator()
    g.manual_seed(int(seed))
    r = torch.rand(case["nsets"], 5, generator=g, dtype=torch.float64)
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    # the sizes are part of the case; dt and the amplitudes come from the seed
    s = torch.Generator()
    s.manual_seed(case["nsets"] * 1_000_003 + case["hi"])
    sizes = torch.exp(lo + (hi - lo) * torch.rand(case["nsets"], generator=s,
                                                  dtype=torch.float64)).to(torch.int64)
    return sizes.tolist(), 1e-4 + (1e-2 - 1e-4) * r[:, 0], 0.5 + r[:, 1:4]


class _Slice:
    """A set bound to its slice of arrays that many sets share."""

    def __init__(self, schema, n, arrays):
        self.schema = schema
        self.handle = ctypes.c_void_p()
        ptrs = (ctypes.c_void_p * len(arrays))(*[a.data_ptr() for a in arrays])
        soax.check(soax.lib().soax_bind(schema.ref, n, ptrs, None, ctypes.byref(self.handle)),
                   "soax_bind")

    def __del__(self):
        soax.lib().soax_destroy(self.handle)


def _batch_arrays(case, seed):
    """(offsets, total) of the sets' slices and their shared arrays."""
    sizes, dts, abc = _batch_plan(case, seed)
    offsets, total = [], 0
    for n in sizes:
        offsets.append(total)
        total += -(-n // 64) * 64
    return sizes, offsets, dts, abc, _fields(SCHEMAS["base"], total, _generator(seed))


def prepare(case, seed):
    kind, g = case["kind"], _generator(seed)
    if kind == "step":
        lay = case["layout"]
        ps = _set(SCHEMAS[case["schema"]], case["n"], g, aos=lay == "aos", aosoa=lay == "aosoa")
        if lay == "aos":
            ps.soa_to_aos()
        elif lay == "aosoa":
            ps.soa_to_aosoa()
        return {"case": case, "set": ps, "out": _step_outputs(case, ps)}
    if kind == "fused":
        ps = _set(SCHEMAS[case["schema"]], case["n"], g, aos=False)
        return {"case": case, "set": ps, "out": _soa_outputs(case, ps)}
    if kind == "transpose":
        ps = _set(SCHEMAS[case["schema"]], case["n"], g)
        ps.soa_to_aos()
        return {"case": case, "set": ps}
    if kind == "adjoint":
        n = case["n"]
        pos0 = torch.stack([_box(n, g) for _ in range(3)])
        target = torch.stack([_box(n, g) for _ in range(3)])
        state = {"case": case, "pos0": pos0, "target": target}
        if case["route"] == "autograd":
            pos0.requires_grad_(True)
            state["abc"] = torch.tensor(_abc(case), dtype=torch.float64, device="cuda",
                                        requires_grad=True)
        else:
            state["abc"] = (ctypes.c_double * 3)(*_abc(case))
        return state
    if kind == "batch":
        sizes, offsets, dts, abc, arrays = _batch_arrays(case, seed)
        schema = soax.Schema(SCHEMAS["base"])
        sets = [_Slice(schema, n, [a[o:o + n] for a in arrays]) for n, o in zip(sizes, offsets)]
        return {"case": case, "arrays": arrays, "batch": soax.Batch(sets),
                "dt": dts.numpy(), "abc": abc.numpy()}
    if kind == "remove":
        ps = _set(SCHEMAS[case["schema"]], case["n"], g)
        ps.soa_to_aos()
        flags = torch.zeros(case["n"], dtype=torch.uint8, device="cuda")
        flags[torch.randperm(case["n"], generator=g, device="cuda")[:_leaving(case)]] = 1
        return {"case": case, "set": ps, "flags": flags}
    ps = _set(SCHEMAS["base"], case["n"], g, aos=False)
    if case["expr"] == "difference":
        program = ps.arr("vel", 1) - ps.arr("vel", 2)
    else:
        v = [ps.arr("vel", d) for d in range(3)]
        program = ps.arr("pos", 0) + 1e-3 * soax.sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2])
    return {"case": case, "set": ps, "program": program}


# ------------------------------------------------------------------ one call

def _soa_outputs(case, ps):
    """The arrays a step changes."""
    return [ps.array(name, d) for name in ("pos", "vel") for d in range(3)]


def _step_outputs(case, ps):
    """Views of the positions and velocities in the layout that is stepped,
    [n, 3] for records and [tiles, 64] per component for tiles."""
    if case["layout"] == "soa":
        return _soa_outputs(case, ps)
    fields, n = SCHEMAS[case["schema"]], case["n"]
    out = []
    if case["layout"] == "aos":
        for name in ("pos", "vel"):
            i = _index(case["schema"], name)
            t = fields[i][1]
            es = SIZE[t]
            out.append(torch.as_strided(ps.aos.view(TORCH[t]), (n, 3), (ps.stride // es, 1),
                                        ps.offsets[i] // es))
        return out
    tiles = -(-n // 64)
    tile_bytes = ps.aosoa_tile_bytes
    off = 0
    for name, t, dim in fields:
        es = SIZE[t]
        for d in range(dim):
            if name in ("pos", "vel"):
                out.append(torch.as_strided(_typed(ps._aosoa_store, t), (tiles, 64),
                                            (tile_bytes // es, 1), off // es))
            off += 64 * es
    return out


def _typed(buf, t):
    es = SIZE[t]
    return buf[: buf.numel() // es * es].view(TORCH[t])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        abc = _abc(case) if case["integrator"] in FIELD_INTEGRATORS else None
        state["set"].step(case["layout"], case["integrator"], case["dt"], case["nsteps"], abc=abc,
                          wrap=_wrap_of(case))
        return state["out"]
    if kind == "fused":
        abc = _abc(case) if case["integrator"] in FIELD_INTEGRATORS else None
        state["set"].step_fused(case["integrator"], case["dt"], case["nsteps"], abc=abc, wrap=True)
        return state["out"]
    if kind == "transpose":
        ps = state["set"]
        ps.aos_to_soa()
        ps.soa_to_aos()
        return {"soa": list(ps.soa), "aos": ps.aos[: case["n"] * ps.stride]}
    if kind == "adjoint":
        if case["route"] == "autograd":
            xT = soax.rk2_advect(state["pos0"], state["abc"], case["dt"], case["nsteps"],
                                 case["k"])
            loss = ((xT - state["target"]) ** 2).sum()
            gx, gabc = torch.autograd.grad(loss, (state["pos0"], state["abc"]))
            return {"xT": xT, "loss": loss.reshape(1), "grad_x0": gx, "grad_abc": gabc}
        args = (state["abc"], case["dt"], case["nsteps"], case["k"])
        xT, tape = soax.forward_ckpt(state["pos0"], *args)
        loss, lam = soax.sqdist_loss(xT, state["target"])
        gx, gabc = soax.adjoint(tape, lam, *args)
        return {"xT": xT, "loss": loss, "grad_x0": gx, "grad_abc": gabc}
    if kind == "batch":
        state["batch"].step(state["dt"], state["abc"], case["nsteps"], mode=soax.GRAPH)
        return state["arrays"][1:]
    if kind == "remove":
        ps = state["set"]
        ps.resize(case["n"])  # the set is at its full size before particles leave
        n_new = ps.remove_flagged(state["flags"])
        return {"n": n_new, "soa": list(ps.soa), "aos": ps.aos[: n_new * ps.stride]}
    ps = state["set"]
    ps.assign(("pos", 0), state["program"])
    return ps.array("pos", 0)


# ------------------------------------------------------------------ the work

def _soa_bytes(fields):
    return sum(SIZE[t] * dim for _, t, dim in fields)


def _record_bytes(fields):
    """Size of one C record with natural alignment."""
    end, widest = 0, 1
    for _, t, dim in fields:
        es = SIZE[t]
        end = -(-end // es) * es + es * dim
        widest = max(widest, es)
    return -(-end // widest) * widest


def work(case):
    """Bytes and operations of one call.  A step is by definition one pass
    over the particles with the state written back, so a call of nsteps steps
    counts that many passes; fused steps count one."""
    kind = case["kind"]
    if kind in ("step", "fused"):
        types = {name: t for name, t, _ in SCHEMAS[case["schema"]]}
        p, v = 3 * SIZE[types["pos"]], 3 * SIZE[types["vel"]]
        integrator = case["integrator"]
        if integrator in FIELD_INTEGRATORS:
            nbytes, flops = 2 * p + v, EVALUATIONS[integrator] * EVAL_FLOPS
        elif integrator == "euler":
            nbytes, flops = 2 * p + v, 6
        else:
            nbytes, flops = 2 * p + 3 * v, 12
        passes = case["nsteps"] if kind == "step" else 1
        return {"bytes": case["n"] * passes * nbytes, "flops": case["n"] * case["nsteps"] * flops}
    if kind == "transpose":
        return {"bytes": 2 * case["n"] * (_soa_bytes(SCHEMAS[case["schema"]]) +
                                          _record_bytes(SCHEMAS[case["schema"]])), "flops": 0}
    if kind == "adjoint":
        # forward: x0 in, xT out; loss: target in; adjoint: gradient out; the
        # tape once out and once in.  Operations: two field evaluations a step
        # forward, the same again recomputed, and the transposed step.
        tape = -(-case["nsteps"] // case["k"]) * 72
        return {"bytes": case["n"] * (4 * 24 + 2 * tape),
                "flops": case["n"] * case["nsteps"] * (4 * EVAL_FLOPS + 80)}
    if kind == "batch":
        total = sum(_batch_plan(case, 0)[0])
        return {"bytes": 60 * total * case["nsteps"],
                "flops": total * case["nsteps"] * EVALUATIONS["rk2_abc"] * EVAL_FLOPS}
    if kind == "remove":
        fields = SCHEMAS[case["schema"]]
        moved = _leaving(case) * (1.0 - case["fraction"])
        return {"bytes": case["n"] + 2 * moved * (_soa_bytes(fields) + _record_bytes(fields)),
                "flops": 0}
    if case["expr"] == "difference":
        return {"bytes": 16 * case["n"], "flops": case["n"]}
    return {"bytes": 28 * case["n"], "flops": 8 * case["n"]}


# ------------------------------------------------------------------ exact results

def _wrap(x):
    lo = x + BOX
    lo = torch.where(lo >= BOX, torch.zeros_like(lo), lo)
    return torch.where(x >= BOX, x - BOX, torch.where(x < 0, lo, x))


def _u(x, A, B, C):
    return (A * torch.sin(x[2]) + C * torch.cos(x[1]), B * torch.sin(x[0]) + A * torch.cos(x[2]),
            C * torch.sin(x[1]) + B * torch.cos(x[0]))


def _moved(x, h, k):
    return [x[d] + h * k[d] for d in range(3)]


def _field_step(integrator, x, dt, A, B, C):
    k1 = _u(x, A, B, C)
    if integrator == "rk2_abc":
        return _moved(x, dt, _u(_moved(x, 0.5 * dt, k1), A, B, C))
    if integrator == "heun_abc":
        k2 = _u(_moved(x, dt, k1), A, B, C)
        return [x[d] + 0.5 * dt * (k1[d] + k2[d]) for d in range(3)]
    k2 = _u(_moved(x, 0.5 * dt, k1), A, B, C)
    k3 = _u(_moved(x, 0.5 * dt, k2), A, B, C)
    k4 = _u(_moved(x, dt, k3), A, B, C)
    return [x[d] + dt / 6.0 * (k1[d] + 2.0 * k2[d] + 2.0 * k3[d] + k4[d]) for d in range(3)]


def _exact_steps(case, seed):
    fields, n, dt = SCHEMAS[case["schema"]], case["n"], case["dt"]
    arrays = _fields(fields, n, _generator(seed))
    at = {}
    k = 0
    for name, _, dim in fields:
        at[name] = arrays[k:k + dim]
        k += dim
    pt, vt = at["pos"][0].dtype, at["vel"][0].dtype
    wrap = _wrap if _wrap_of(case) else (lambda y: y)
    x, v = at["pos"], at["vel"]
    if case["integrator"] in FIELD_INTEGRATORS:
        for _ in range(case["nsteps"]):
            x = [wrap(y) for y in _field_step(case["integrator"], x, dt, *_abc(case))]
        v = list(_u(x, *_abc(case)))
    else:
        # the state is kept in the record's types from step to step
        for _ in range(case["nsteps"]):
            if case["integrator"] == "symplectic_euler":
                v = [(v[d].double() + dt * at["acc"][d].double()).to(vt) for d in range(3)]
            x = [wrap(x[d].double() + dt * v[d].double()).to(pt) for d in range(3)]
            if case["integrator"] == "euler_acc":
                v = [(v[d].double() + dt * at["acc"][d].double()).to(vt) for d in range(3)]
        x, v = [y.double() for y in x], [y.double() for y in v]
    layout = case.get("layout", "soa")
    if layout == "soa":
        return x + v
    if layout == "aos":
        return [torch.stack(x, 1), torch.stack(v, 1)]
    tiles = -(-n // 64)
    return [torch.nn.functional.pad(y, (0, tiles * 64 - n)).reshape(tiles, 64) for y in x + v]


def _exact_adjoint(case, seed):
    n, nsteps, dt, (A, B, C) = case["n"], case["nsteps"], case["dt"], _abc(case)
    g = _generator(seed)
    pos0 = torch.stack([_box(n, g) for _ in range(3)])
    target = torch.stack([_box(n, g) for _ in range(3)])
    xT, gx = torch.empty_like(pos0), torch.empty_like(pos0)
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    gabc = torch.zeros(3, dtype=torch.float64, device="cuda")
    h = 0.5 * dt

    def back(s, c, l):
        """(J^T l, G^T l) of the field at a point with sines s and cosines c."""
        return ((B * (c[0] * l[1] - s[0] * l[2]), C * (c[1] * l[2] - s[1] * l[0]),
                 A * (c[2] * l[0] - s[2] * l[1])),
                (s[2] * l[0] + c[2] * l[1], s[0] * l[1] + c[0] * l[2], c[1] * l[0] + s[1] * l[2]))

    chunk = 2_500_000
    for i in range(0, n, chunk):
        x = [pos0[d, i:i + chunk] for d in range(3)]
        states = []
        for _ in range(nsteps):
            states.append(x)
            x = _field_step("rk2_abc", x, dt, A, B, C)
        lam = []
        for d in range(3):
            e = x[d] - target[d, i:i + chunk]
            loss += (e * e).sum()
            lam.append(2.0 * e)
            xT[d, i:i + chunk] = x[d]
        acc = [torch.zeros_like(lam[0]) for _ in range(3)]
        for x in reversed(states):
            s, c = [torch.sin(y) for y in x], [torch.cos(y) for y in x]
            xm = _moved(x, h, (A * s[2] + C * c[1], B * s[0] + A * c[2], C * s[1] + B * c[0]))
            jm, gm = back([torch.sin(y) for y in xm], [torch.cos(y) for y in xm], lam)
            mu = [dt * y for y in jm]
            jx, g0 = back(s, c, mu)
            for d in range(3):
                acc[d] += dt * gm[d] + h * g0[d]
                lam[d] = lam[d] + mu[d] + h * jx[d]
        for d in range(3):
            gx[d, i:i + chunk] = lam[d]
            gabc[d] += acc[d].sum()
        del states
    return {"xT": xT, "loss": loss, "grad_x0": gx, "grad_abc": gabc}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "fused"):
        return _exact_steps(case, seed)
    if kind == "adjoint":
        return _exact_adjoint(case, seed)
    if kind == "batch":
        sizes, offsets, dts, abc, arrays = _batch_arrays(case, seed)
        x, v = [a.clone() for a in arrays[1:4]], [a.double() for a in arrays[4:7]]
        for n, o, dt, (A, B, C) in zip(sizes, offsets, dts.tolist(), abc.tolist()):
            y = [a[o:o + n] for a in x]
            for _ in range(case["nsteps"]):
                y = [_wrap(p) for p in _field_step("rk2_abc", y, dt, A, B, C)]
            u = _u(y, A, B, C)
            for d in range(3):
                x[d][o:o + n] = y[d]
                v[d][o:o + n] = u[d]
        return x + v
    if kind == "expr":
        a = _fields(SCHEMAS["base"], case["n"], _generator(seed))
        vx, vy, vz = (y.double() for y in a[4:7])
        if case["expr"] == "difference":
            return vy - vz
        return a[1] + 1e-3 * torch.sqrt(vx * vx + vy * vy + vz * vz)
    return None  # moves of whole particles: every byte stays as it was
