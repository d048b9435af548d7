"""The work that users of libpwadv have it do, as cases to be timed: each is one
call (or one differentiated call) through the public Python entry points, on
inputs of a size and kind that real programs pass.

listed() gives the fixed cases, draw(rng) one more of the same ranges,
prepare(case, seed) what a program holds before the call, run(state) the call,
work(case) the bytes and operations it cannot do without, and
exact(case, seed) its outputs in 64 bits from plain torch.

Kinds of case:
  forward     su, sv, sw = advect(u, v, w): the source terms of one timestep
  fill        halo_fill of u, v, w (periodic x, y; free-slip lid), then advect
  step        one explicit time step with the boundary rules applied by
              addressing: advect_bc with an epilogue, x_next = x + dt * F(x),
              written into the interior of the next state's padded arrays
  accumulate  out = c + F on the x-fastest layout (advect_epilogue): other
              model components contribute to the same source terms
  zfast       the same on z-contiguous arrays (advect_zfast_epilogue), as a
              column-major host model stores them
  tangent     J d (advect_tangent): the inner product of 4D-Var minimisation
  grad        PWAdvect forward and backward: training through the operator
  coeffs      advect_adjoint_coeff_grad: gradients of the winds and of the
              vertical weights, the backward of a calibration run
  bc_grad     PWAdvectBC forward and backward: the same through the boundaries
  batch       many uneven subdomains replayed from a captured graph
"""
import math

import numpy as np
import torch

from paper_2301_13016_amd import binding as B

_TORCH = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16, "f16": torch.float16}
_SIZE = {"f32": 4, "f64": 8, "bf16": 2, "f16": 2}
_TCX = _TCY = float(np.float32(0.25 / 100.0))   # 0.25 / grid spacing (100 m)
_TZ = 0.25 / 50.0                                # per-level weights around 0.25 / 50 m
_DT = 0.5
_USEFUL = 63                                     # useful operations per point of the scheme

# Periodic in x and y; u and v zero-gradient at the surface and the lid, w zero there.
_LID = [("periodic", "periodic", "copy")] * 2 + [("periodic", "periodic", "zero")]


def listed():
    return [
        # the smallest subdomain of a decomposed model: latency and launches
        {"name": "forward_f32_32x32x64", "kind": "forward", "dtype": "f32", "nx": 32, "ny": 32, "nz": 64},
        # one rank's ragged subdomain on its own
        {"name": "forward_f32_201x143x117", "kind": "forward", "dtype": "f32", "nx": 201, "ny": 143, "nz": 117},
        # the benchmark's single-GPU timestep
        {"name": "forward_f32_512x512x64", "kind": "forward", "dtype": "f32", "nx": 512, "ny": 512, "nz": 64},
        # double precision on an ordinary grid that is no power of two
        {"name": "forward_f64_250x250x100", "kind": "forward", "dtype": "f64", "nx": 250, "ny": 250, "nz": 100},
        # the largest single grid, 16-bit storage
        {"name": "forward_bf16_1024x1024x256", "kind": "forward", "dtype": "bf16", "nx": 1024, "ny": 1024, "nz": 256},
        # a whole explicit step of a doubly periodic model under a lid
        {"name": "step_f32_512x512x64", "kind": "step", "dtype": "f32", "nx": 512, "ny": 512, "nz": 64},
        # accumulation in a column-major model with 75 levels
        {"name": "zfast_f32_300x300x75", "kind": "zfast", "dtype": "f32", "nx": 300, "ny": 300, "nz": 75},
        # differentiation: the benchmark's grid, then ragged ones
        {"name": "tangent_f32_256x256x128", "kind": "tangent", "dtype": "f32", "nx": 256, "ny": 256, "nz": 128},
        {"name": "grad_f32_256x256x128", "kind": "grad", "dtype": "f32", "nx": 256, "ny": 256, "nz": 128},
        {"name": "coeffs_f32_190x130x100", "kind": "coeffs", "dtype": "f32", "nx": 190, "ny": 130, "nz": 100},
        {"name": "bc_grad_f32_200x200x80", "kind": "bc_grad", "dtype": "f32", "nx": 200, "ny": 200, "nz": 80},
        # 64 uneven subdomains on one GPU, one graph launch per timestep
        {"name": "batch_f32_64_subdomains", "kind": "batch", "dtype": "f32", "n": 64, "shapes": 3},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward"] * 4 + ["step", "accumulate", "fill", "zfast", "tangent", "grad", "coeffs",
                                         "bc_grad", "batch"])
    if kind == "batch":
        return {"kind": kind, "dtype": "f32", "n": _log_int(rng, 4, 48), "shapes": rng.randrange(4, 1 << 20)}
    if kind == "forward":
        dtype = rng.choice(["f32", "f32", "f64", "bf16", "f16"])
    elif kind in ("tangent", "grad"):
        dtype = rng.choice(["f32", "f32", "f64"])
    else:
        dtype = "f32"
    # bytes of one pass at most about a quarter of the largest grid's
    most = (1 << 27) // _SIZE[dtype] if kind in ("forward", "step", "accumulate", "fill", "zfast") else 1 << 23
    while True:
        nx, ny, nz = _log_int(rng, 32, 1024), _log_int(rng, 32, 1024), _log_int(rng, 16, 256)
        if nx * ny * nz <= most:
            return {"kind": kind, "dtype": dtype, "nx": nx, "ny": ny, "nz": nz}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, shape, lo, hi, dtype):
    """Uniform values in [lo, hi), drawn in single precision (double for double
    storage) and rounded to the storage type."""
    draw_as = torch.float64 if dtype == torch.float64 else torch.float32
    x = torch.rand(shape, generator=g, device="cuda", dtype=draw_as)
    return x.mul_(hi - lo).add_(lo).to(dtype)


def _padded(c):
    return c["nz"] + 2, c["ny"] + 2, c["nx"] + 2


def _interior(c):
    return c["nz"], c["ny"], c["nx"]


def _winds(g, shape, dtype):
    """Winds in [-10, 10) m/s over the whole padded array."""
    return [_uniform(g, shape, -10.0, 10.0, dtype) for _ in range(3)]


def _vertical(g, nz, dtype):
    """tzc1, tzc2, tzd1, tzd2: density-like weights in [0.5, 1.5) times 0.25 / 50 m."""
    return [_uniform(g, (nz,), 0.5 * _TZ, 1.5 * _TZ, dtype) for _ in range(4)]


def _subdomain_shapes(c):
    """nx, ny in 32..256 and nz in 64..256, each subdomain from its own stream."""
    out = []
    for b in range(c["n"]):
        r = np.random.default_rng((c["shapes"], b))
        nx, ny = (int(x) for x in r.integers(32, 257, 2))
        out.append((nx, ny, int(r.integers(64, 257))))
    return out


def _offsets(shapes):
    """Where each subdomain's output starts in the pooled output arrays (256-byte
    pieces), and the pool's length."""
    at, out = 0, []
    for nx, ny, nz in shapes:
        out.append(at)
        at += -(-nx * ny * nz // 64) * 64
    return out, at


def _inputs(c, seed):
    """The arrays of a single-grid case, by name, from the seed."""
    g, dt = _gen(seed), _TORCH[c["dtype"]]
    odt = torch.float64 if dt == torch.float64 else torch.float32
    k = c["kind"]
    a = {}
    if k == "zfast":   # arrays indexed [i, j, k]
        pz, py, px = _padded(c)
        nz, ny, nx = _interior(c)
        a["x"] = _winds(g, (px, py, pz), dt)
        a["add"] = [_uniform(g, (nx, ny, nz), -1.0, 1.0, odt) for _ in range(3)]
    else:
        a["x"] = _winds(g, _padded(c), dt)
    a["tz"] = _vertical(g, c["nz"], odt)
    if k == "accumulate":
        a["add"] = [_uniform(g, _interior(c), -1.0, 1.0, odt) for _ in range(3)]
    if k in ("grad", "coeffs", "bc_grad"):
        a["r"] = [_uniform(g, _interior(c), -1.0, 1.0, odt) for _ in range(3)]
    if k == "tangent":
        a["d"] = [_uniform(g, _padded(c), -1.0, 1.0, dt) for _ in range(3)]
    return a


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "batch":
        shapes = _subdomain_shapes(c)
        at, total = _offsets(shapes)
        g = _gen(seed)
        pool = [torch.zeros(total, device="cuda") for _ in range(3)]
        subs = []
        for (nx, ny, nz), o in zip(shapes, at):
            x = _winds(g, (nz + 2, ny + 2, nx + 2), torch.float32)
            co = B.Coeffs(_TCX, _TCY, *_vertical(g, nz, torch.float32))
            outs = tuple(p[o:o + nx * ny * nz].view(nz, ny, nx) for p in pool)
            subs.append((*x, co, outs))
        batch = B.Batch(subs)
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        batch.capture(stream)
        return {"case": c, "batch": batch, "pool": pool}
    a = _inputs(c, seed)
    s = {"case": c, "x": a["x"], "coeffs": B.Coeffs(_TCX, _TCY, *a["tz"])}
    s.update({k: v for k, v in a.items() if k not in ("x", "tz")})
    if c["kind"] == "step":      # the next state, and the interiors of both
        s["next"] = [x.clone() for x in s["x"]]
        s["inner"] = [x[1:-1, 1:-1, 1:-1] for x in s["x"]]
        s["next_inner"] = tuple(x[1:-1, 1:-1, 1:-1] for x in s["next"])
    if c["kind"] in ("accumulate", "zfast"):
        s["out"] = tuple(torch.empty_like(x) for x in s["add"])
    if c["kind"] in ("grad", "bc_grad"):
        s["x"] = [x.requires_grad_(True) for x in s["x"]]
    return s


# -------------------------------------------------------------------- call

def run(s):
    k = s["case"]["kind"]
    if k == "batch":
        s["batch"].replay()
        return list(s["pool"])
    x, co = s["x"], s["coeffs"]
    if k == "forward":
        return B.advect(*x, co)
    if k == "fill":
        B.halo_fill(x, _LID)
        return list(x) + list(B.advect(*x, co))
    if k == "step":
        return B.advect_bc(*x, co, _LID, out=s["next_inner"], addends=s["inner"], alpha=_DT)
    if k == "accumulate":
        return B.advect_epilogue(*x, co, s["add"], out=s["out"])
    if k == "zfast":
        return B.advect_zfast_epilogue(*x, co, s["add"], out=s["out"])
    if k == "tangent":
        return B.advect_tangent(*x, co, *s["d"])
    if k == "coeffs":
        grads, g = B.advect_adjoint_coeff_grad(*x, co, *s["r"])
        return list(grads) + [g[n] for n in ("tzc1", "tzc2", "tzd1", "tzd2", "tcx", "tcy")]
    if k == "grad":
        y = B.PWAdvect().apply(*x, co)
    else:
        y = B.PWAdvectBC().apply(*x, co, _LID)
    g = torch.autograd.grad(y, x, grad_outputs=s["r"])
    return [t.detach() for t in y] + list(g)


# -------------------------------------------------------------------- work

def work(case):
    c = dict(case)
    if c["kind"] == "batch":
        b = f = 0
        for nx, ny, nz in _subdomain_shapes(c):
            p, n = (nx + 2) * (ny + 2) * (nz + 2), nx * ny * nz
            b += 3 * 4 * (p + n) + 4 * 4 * nz
            f += _USEFUL * n
        return {"bytes": b, "flops": f}
    es = _SIZE[c["dtype"]]
    os_ = 8 if c["dtype"] == "f64" else 4
    n = c["nx"] * c["ny"] * c["nz"]
    p = (c["nx"] + 2) * (c["ny"] + 2) * (c["nz"] + 2)
    fwd = 3 * p * es + 3 * n * os_
    tz = 4 * c["nz"] * os_
    k = c["kind"]
    if k == "forward":
        return {"bytes": fwd + tz, "flops": _USEFUL * n}
    if k == "fill":              # the halo is written once, then everything is read once
        return {"bytes": fwd + tz + 2 * 3 * (p - n) * es, "flops": _USEFUL * n}
    if k == "step":              # reads the interior only (the addends are the same values), writes the next one
        return {"bytes": 3 * n * es + 3 * n * os_ + tz, "flops": (_USEFUL + 6) * n}
    if k in ("accumulate", "zfast"):
        return {"bytes": fwd + 3 * n * os_ + tz, "flops": (_USEFUL + 3) * n}
    if k == "tangent":
        return {"bytes": fwd + 3 * p * es + tz, "flops": 2 * _USEFUL * n}
    back = 3 * p * es + 3 * n * es + 3 * p * es   # values and cotangents read, gradients written
    if k == "coeffs":
        return {"bytes": back + tz + 8 * (6 * c["nz"] + 2), "flops": 3 * _USEFUL * n}
    if k == "grad":
        return {"bytes": fwd + back + 2 * tz, "flops": 3 * _USEFUL * n}
    return {"bytes": 3 * n * es * 2 + 3 * n * os_ + 3 * n * es + 3 * p * es + 2 * tz, "flops": 3 * _USEFUL * n}


# ------------------------------------------------------------------- exact

def _fill64(x, rules):
    """x with its one-cell halo set by (x, y, z) rules, one axis after the other."""
    for dim, rule in zip((2, 1, 0), rules):
        n = x.shape[dim] - 2
        idx = torch.arange(n + 2, device=x.device)
        sign = torch.ones(n + 2, dtype=x.dtype, device=x.device)
        if rule == "periodic":
            idx[0], idx[-1] = n, 1
        else:
            idx[0], idx[-1] = 1, n
            sign[0] = sign[-1] = 0.0 if rule == "zero" else 1.0
        shape = [1, 1, 1]
        shape[dim] = n + 2
        x = x.index_select(dim, idx) * sign.view(shape)
    return x


def _forward64(u, v, w, tcx, tcy, tz):
    """The scheme's source terms on the interior of arrays indexed [k, j, i]."""
    def at(f, k, j, i):
        return f[1 + k:f.shape[0] - 1 + k, 1 + j:f.shape[1] - 1 + j, 1 + i:f.shape[2] - 1 + i]

    c1, c2, d1, d2 = (t.view(-1, 1, 1) for t in tz)
    u0, v0, w0 = at(u, 0, 0, 0), at(v, 0, 0, 0), at(w, 0, 0, 0)
    ul, ur, vs, vn = at(u, 0, 0, -1), at(u, 0, 0, 1), at(v, 0, -1, 0), at(v, 0, 1, 0)
    wb, wt = at(w, -1, 0, 0), at(w, 1, 0, 0)
    su = (tcx * (ul * (u0 + ul) - ur * (u0 + ur))
          + tcy * (at(u, 0, -1, 0) * (vs + at(v, 0, -1, 1)) - at(u, 0, 1, 0) * (v0 + at(v, 0, 0, 1)))
          + c1 * at(u, -1, 0, 0) * (wb + at(w, -1, 0, 1)) - c2 * at(u, 1, 0, 0) * (w0 + at(w, 0, 0, 1)))
    sv = (tcx * (at(v, 0, 0, -1) * (ul + at(u, 0, 1, -1)) - at(v, 0, 0, 1) * (u0 + at(u, 0, 1, 0)))
          + tcy * (vs * (v0 + vs) - vn * (v0 + vn))
          + c1 * at(v, -1, 0, 0) * (wb + at(w, -1, 1, 0)) - c2 * at(v, 1, 0, 0) * (w0 + at(w, 0, 1, 0)))
    sw = (tcx * (at(w, 0, 0, -1) * (ul + at(u, 1, 0, -1)) - at(w, 0, 0, 1) * (u0 + at(u, 1, 0, 0)))
          + tcy * (at(w, 0, -1, 0) * (vs + at(v, 1, -1, 0)) - at(w, 0, 1, 0) * (v0 + at(v, 1, 0, 0)))
          + d1 * wb * (w0 + wb) - d2 * wt * (w0 + wt))
    return su, sv, sw


def _forward64_slabs(x, tz, step=32):
    """_forward64 of storage-precision arrays, in slabs of levels."""
    nz = x[0].shape[0] - 2
    out = [torch.empty((nz, x[0].shape[1] - 2, x[0].shape[2] - 2), dtype=torch.float64, device=x[0].device)
           for _ in range(3)]
    for k in range(0, nz, step):
        e = min(nz, k + step)
        got = _forward64(*(f[k:e + 2].double() for f in x), _TCX, _TCY, [t[k:e].double() for t in tz])
        for o, s in zip(out, got):
            o[k:e] = s
    return out


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "batch":
        shapes = _subdomain_shapes(c)
        at, total = _offsets(shapes)
        g = _gen(seed)
        pool = [torch.zeros(total, dtype=torch.float64, device="cuda") for _ in range(3)]
        for (nx, ny, nz), o in zip(shapes, at):
            x = _winds(g, (nz + 2, ny + 2, nx + 2), torch.float32)
            tz = _vertical(g, nz, torch.float32)
            for p, s in zip(pool, _forward64_slabs(x, tz)):
                p[o:o + nx * ny * nz] = s.reshape(-1)
        return pool
    a = _inputs(c, seed)
    x, tz, k = a["x"], a["tz"], c["kind"]
    if k == "forward":
        return tuple(_forward64_slabs(x, tz))
    if k == "fill":
        f = [_fill64(t.double(), r) for t, r in zip(x, _LID)]
        return f + _forward64_slabs(f, tz)
    if k == "step":
        f = [_fill64(t.double(), r) for t, r in zip(x, _LID)]
        return tuple(t[1:-1, 1:-1, 1:-1] + _DT * s for t, s in zip(f, _forward64_slabs(f, tz)))
    if k == "accumulate":
        return tuple(d.double() + s for d, s in zip(a["add"], _forward64_slabs(x, tz)))
    if k == "zfast":
        t = [f.permute(2, 1, 0) for f in x]
        return tuple(d.double() + s.permute(2, 1, 0) for d, s in zip(a["add"], _forward64_slabs(t, tz)))
    x, tz = [t.double() for t in x], [t.double() for t in tz]
    if k == "tangent":           # the operator is quadratic: its central difference is its derivative
        d = [t.double() for t in a["d"]]
        hi = _forward64_slabs([p + q for p, q in zip(x, d)], tz)
        lo = _forward64_slabs([p - q for p, q in zip(x, d)], tz)
        return tuple((p - q) / 2 for p, q in zip(hi, lo))
    x = [t.requires_grad_(True) for t in x]
    r = [t.double() for t in a["r"]]
    if k == "coeffs":
        tz = [t.requires_grad_(True) for t in tz]
        tc = [torch.tensor(v, dtype=torch.float64, device="cuda", requires_grad=True) for v in (_TCX, _TCY)]
        return list(torch.autograd.grad(_forward64(*x, *tc, tz), x + tz + tc, grad_outputs=r))
    f = x if k == "grad" else [_fill64(t, rules) for t, rules in zip(x, _LID)]
    y = _forward64(*f, _TCX, _TCY, tz)
    g = torch.autograd.grad(y, x, grad_outputs=r)
    return [t.detach() for t in y] + list(g)
