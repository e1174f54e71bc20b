"""The work that users of this library have it do, as cases that can be timed and compared.

Every case is one call (or, for the gauge-field update, one short sequence of
calls) of the ctypes binding on device buffers that a program holds anyway:
packed links and fields, workspaces, network weights.  The sizes are those of
the repository's workloads, tests and benchmark legs or generic ones; links
and sources follow the distributions of hisq_inputs (Haar and smooth SU(3)
links, Gaussian sources) but are drawn on the GPU, since they are drawn often.

Operations:
  dslash        hisq_dslash, one parity, 1 to 16 right-hand sides, every format
  apply_m       hisq_apply_m, the normal operator
  cg            hisq_cg, FP64 and reliable-update, 1 to 16 right-hand sides
  multishift    hisq_multishift_cg, shifts log-spaced in [1e-5, 1]
  batch         hisq_cg_batch on lattices of several sizes
  ptc_forward   hisq_ptc_forward, one application of the preconditioner network
  ptc_train     hisq_ptc_train_step: forward, loss, backward, Adam
  gauge_update  hisq_smear_links and hisq_pack_links of the new links

Solves are asked to a relative residual of 1e-12 so that solutions, and not
only residuals, can be compared: at the 1e-10 of the headline the solution
itself is defined to about 1e-8 only.
"""
import math

import numpy as np
import torch

from paper_2306_01098_amd import hisq as h

DEV = "cuda"
AXIS = {0: 3, 1: 2, 2: 1, 3: 0}   # axis of (Nt, Nz, Ny, Nx) that direction mu moves along
FORMATS = ("fp64", "fp32", "fp16n", "fp64r12", "fp32r12", "fp64w14", "fp32w14")
REAL = {"fp64": 8, "fp32": 4, "fp16n": 2}
LEVEL1 = (1 / 8, 1 / 16, 1 / 64, 1 / 384, 0.0)      # 1-, 3-, 5-, 7-link, Lepage
LEVEL2 = (1.0, 1 / 16, 1 / 64, 1 / 384, -1 / 8)
C_NAIK = -1 / 24
CHANNELS = (1, 8, 8, 1)
# multiply-adds of 3x3 complex matrices per site in hisq_smear_links: 60 staple
# fields of four products in level 1, 72 in level 2, 8 in the Naik links; 3 more
# per link for the projection
SMEAR_PRODUCTS = 4 * 60 + 4 * 72 + 8 + 12


def _case(name, op, dims, **more):
    c = {"name": name, "op": op, "nx": dims[0], "ny": dims[1], "nz": dims[2], "nt": dims[3], "tbc": -1}
    c.update(more)
    return c


def listed():
    return [
        # the smallest ordinary lattice: one operator call of an interactive program or a test, all launch latency
        _case("dslash_fp64_8x8x8x8", "dslash", (8, 8, 8, 8), tbc=1, prec="fp64", nrhs=1, links="haar"),
        # the headline: the FP64 operator of a true residual at 32^3x8
        _case("dslash_fp64_32x32x32x8", "dslash", (32, 32, 32, 8), prec="fp64", nrhs=1, links="smooth"),
        # three colour sources of a point-source propagator on a lattice that no tile divides, compressed links
        _case("dslash_fp32r12_3rhs_20x12x14x10", "dslash", (20, 12, 14, 10), prec="fp32r12", nrhs=3, links="haar"),
        # the block of 16 sources that shares each link load, the largest operator call
        _case("dslash_fp32_16rhs_48x48x48x12", "dslash", (48, 48, 48, 12), prec="fp32", nrhs=16, links="smooth"),
        # the normal operator with binary16 links and vectors, the reduced-precision end of the formats
        _case("apply_m_fp16n_32x32x32x8", "apply_m", (32, 32, 32, 8), prec="fp16n", nrhs=1, mass=0.01, links="smooth"),
        # plain FP64 CG on a small lattice: some hundred dependent iterations of a few microseconds
        _case("cg_fp64_8x8x8x8", "cg", (8, 8, 8, 8), tbc=1, inner="fp64", nrhs=1, mass=0.1, links="haar", tol=1e-12),
        # the reliable-update solve of one block of 16 sources (a propagator, noise vectors of a condensate)
        _case("cg_fp32_16rhs_32x32x32x8", "cg", (32, 32, 32, 8), inner="fp32", nrhs=16, mass=0.01, links="smooth", tol=1e-12),
        # the rational function of a molecular-dynamics force: 14 shifts on one source
        _case("multishift_14_24x24x24x12", "multishift", (24, 24, 24, 12), inner="fp32", nshift=14, mass=0.005, links="smooth", tol=1e-12),
        # many small independent ensembles at once
        _case("batch_24_uneven", "batch", (24, 24, 24, 6), inner="fp32", mass=0.1,
              mix="8x8x8x8:8 12x12x12x4:8 16x16x16x8:4 24x24x24x6:4", links="haar", tol=1e-12),
        # one application of the learned preconditioner, as every iteration of flexible CG makes it
        _case("ptc_forward_32x32x32x32", "ptc_forward", (32, 32, 32, 32), links="smooth"),
        # one training step of the preconditioner on four (source, solution) pairs
        _case("ptc_train_4_16x16x16x16", "ptc_train", (16, 16, 16, 16), batch=4, mass=0.05, links="smooth"),
        # a new gauge field: fat and Naik links, packed for the operator
        _case("gauge_update_32x32x32x32", "gauge_update", (32, 32, 32, 32), prec="fp32w14", links="smooth"),
    ]


def _sizes(rng, lo, hi, longest, step=2):
    """Four even extents, their volume spread over its logarithm between lo and hi."""
    while True:
        want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        d = [step * max(4 // step, round(want ** 0.25 * math.exp(rng.uniform(-0.5, 0.5)) / step)) for _ in range(3)]
        d.append(2 * max(2, round(want / (d[0] * d[1] * d[2]) / 2)))
        if lo <= d[0] * d[1] * d[2] * d[3] <= hi and max(d) <= longest:
            return tuple(d)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _drawn(rng)
        if _cost(c) <= most:
            return c


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def _drawn(rng):
    op = rng.choice(("dslash", "dslash", "dslash", "apply_m", "cg", "cg", "multishift", "batch", "ptc_forward", "ptc_train", "gauge_update"))
    # production extents are multiples of 8 about half of the time
    step = rng.choice((2, 2, 4, 8))
    lo = 4096 if step == 8 else 256
    tbc = rng.choice((-1, -1, 1))
    links = rng.choice(("haar", "smooth"))
    if op in ("dslash", "apply_m"):
        prec, nrhs = rng.choice(FORMATS), rng.choice((1, 1, 1, 2, 3, 4, 5, 7, 8, 12, 16))
        dims = _sizes(rng, lo, min(1 << 20, 16 * 1327104 // nrhs), 64, step)
        c = _case("", op, dims, tbc=tbc, prec=prec, nrhs=nrhs, links=links)
        if op == "apply_m":
            c["mass"] = round(rng.uniform(0.005, 0.2), 4)
    elif op == "cg":
        inner, nrhs = rng.choice(FORMATS), rng.choice((1, 1, 2, 3, 8, 16))
        dims = _sizes(rng, lo, 262144 if nrhs <= 3 else 131072, 32, step)
        c = _case("", op, dims, tbc=tbc, inner=inner, nrhs=nrhs, mass=round(rng.uniform(0.1, 0.3), 4), links=links, tol=1e-12)
    elif op == "multishift":
        inner = rng.choice(("fp64", "fp32", "fp32r12"))
        c = _case("", op, _sizes(rng, lo, 165888, 32, step), tbc=tbc, inner=inner, nshift=rng.randint(1, 16), mass=round(rng.uniform(0.1, 0.3), 4),
                  links=links, tol=1e-12)
    elif op == "batch":
        kinds = [_sizes(rng, 256, 65536, 24, 2) for _ in range(rng.randint(1, 3))]
        mix = " ".join("%dx%dx%dx%d:%d" % (*d, rng.randint(1, 6)) for d in kinds)
        c = _case("", op, kinds[0], tbc=tbc, inner=rng.choice(("fp64", "fp32")), mass=round(rng.uniform(0.1, 0.2), 4), mix=mix, links=links, tol=1e-12)
    elif op == "ptc_forward":
        c = _case("", op, _sizes(rng, lo, 1 << 20, 48, step), tbc=tbc, links=links)
    elif op == "ptc_train":
        c = _case("", op, _sizes(rng, lo, 131072, 32, step), tbc=tbc, batch=rng.randint(1, 5), mass=round(rng.uniform(0.05, 0.3), 4), links=links)
    else:
        c = _case("", op, _sizes(rng, lo, 1 << 20, 48, step), prec=rng.choice(("fp64", "fp32", "fp16n", "fp64w14", "fp32w14")), links="smooth")
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _dims(c):
    return c["nx"], c["ny"], c["nz"], c["nt"]


def _vol(dims):
    return dims[0] * dims[1] * dims[2] * dims[3]


def _gen(seed, what):
    return torch.Generator(device=DEV).manual_seed(1000 * (seed % (1 << 40)) + what)


def _cnormal(g, *shape):
    return torch.view_as_complex(torch.randn(*shape, 2, dtype=torch.float64, device=DEV, generator=g) * math.sqrt(0.5))


def _mm(a, b):
    """Products of 3x3 matrices, written out."""
    r = a[..., :, 0, None] * b[..., None, 0, :]
    r += a[..., :, 1, None] * b[..., None, 1, :]
    r += a[..., :, 2, None] * b[..., None, 2, :]
    return r


def _dag(a):
    return a.conj().transpose(-1, -2)


def _haar(g, n):
    """Rows of a Ginibre matrix orthonormalised, the third from the other two: Haar in SU(3)."""
    z = _cnormal(g, n, 2, 3)
    a = z[:, 0] / torch.linalg.vector_norm(z[:, 0], dim=-1, keepdim=True)
    b = z[:, 1] - a * (a.conj() * z[:, 1]).sum(-1, keepdim=True)
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack((a, b, torch.linalg.cross(a, b, dim=-1).conj()), dim=-2)


def _smooth(g, n, eps=0.3):
    """exp(i eps H), H Gaussian in the traceless Hermitian matrices (h_a ~ N(0, 1) on lambda_a / 2)."""
    r = torch.randn(n, 8, dtype=torch.float64, device=DEV, generator=g) / 2
    m = torch.zeros(n, 3, 3, dtype=torch.complex128, device=DEV)
    d3, d8 = r[:, 6], r[:, 7] / math.sqrt(3.0)
    m[:, 0, 0], m[:, 1, 1], m[:, 2, 2] = (d8 + d3).to(m.dtype), (d8 - d3).to(m.dtype), (-2 * d8).to(m.dtype)
    for k, (i, j) in enumerate(((0, 1), (0, 2), (1, 2))):
        m[:, i, j] = torch.complex(r[:, 2 * k], -r[:, 2 * k + 1])
        m[:, j, i] = m[:, i, j].conj()
    m *= 1j * eps / 4                       # exp by its series on a quarter, squared twice
    e = torch.eye(3, dtype=m.dtype, device=DEV) + m / 14
    for k in range(13, 0, -1):
        e = torch.eye(3, dtype=m.dtype, device=DEV) + _mm(m, e) / k
    e = _mm(e, e)
    return _mm(e, e)


def _links(kind, dims, seed, what):
    nx, ny, nz, nt = dims
    one = _haar if kind == "haar" else _smooth
    return torch.stack([one(_gen(seed, what + mu), _vol(dims)).reshape(nt, nz, ny, nx, 3, 3) for mu in range(4)])


def _fat_naik(kind, dims, seed):
    fat, v = _links(kind, dims, seed, 10), _links(kind, dims, seed, 20)
    if kind == "smooth":                     # products of three links, as the Naik term is built
        v = torch.stack([_mm(_mm(v[mu], v[mu].roll(-1, AXIS[mu])), v[mu].roll(-2, AXIS[mu])) for mu in range(4)])
    return fat, v


def _source(dims, seed, what, nrhs):
    return _cnormal(_gen(seed, what), nrhs, _vol(dims) // 2, 3)


def _packed_links(lat, prec, fat, naik):
    packed = h.empty_links(lat, prec)
    h.hisq_pack_links(lat, prec, fat, naik, packed)
    return packed


def _packed_field(lat, prec, half):
    packed = torch.zeros(h.hisq_field_bytes(lat, prec, half.shape[0]), dtype=torch.uint8, device=DEV)
    h.hisq_pack_field(lat, prec, half.shape[0], half, packed)
    return packed


def _field_format(prec):
    return "fp16n" if prec == "fp16n" else prec[:4]


def _weights(seed):
    """Starting weights of the network: 1/sqrt(c_in c_out) on the identity path, Gaussian noise on all."""
    g, out = _gen(seed, 50), []
    for cin, cout in zip(CHANNELS[:-1], CHANNELS[1:]):
        w = _cnormal(g, cout, cin, 9) * (0.05 * math.sqrt(2.0) / math.sqrt(9 * cin))
        w[:, :, 0] += 1.0 / math.sqrt(cin * cout)
        out.append(w.reshape(-1))
    return torch.cat(out)


def _mix(c):
    got = []
    for word in c["mix"].split():
        d, n = word.split(":")
        got.append((tuple(int(v) for v in d.split("x")), int(n)))
    return got


def _problem(c, seed, k, dims):
    """Links, source and mass of problem k of a batch."""
    fat, naik = _fat_naik(c["links"], dims, seed * 300 + k)
    return fat, naik, _source(dims, seed * 300 + k, 30, 1), c["mass"] * (1.0 + 0.5 * ((k * 7) % 10) / 10)


def prepare(c, seed):
    op, dims = c["op"], _dims(c)
    lat = h.lattice(dims, c["tbc"])
    s = {"case": c, "lat": lat}
    if op == "batch":
        s["hold"], items = [], []
        for dims, count in _mix(c):
            lat = h.lattice(dims, c["tbc"])
            for _ in range(count):
                fat, naik, src, mass = _problem(c, seed, len(items), dims)
                it = {"lat": lat, "mass": mass, "tol": c["tol"], "links_f64": _packed_links(lat, "fp64", fat, naik),
                      "b": _packed_field(lat, "fp64", src), "x": h.empty_field(lat, "fp64")}
                if c["inner"] != "fp64":
                    it["links_inner"] = _packed_links(lat, c["inner"], fat, naik)
                items.append(it)
        s["items"], s["problems"] = items, h.make_problems(items)
        s["ws"] = h.empty_workspace(h.hisq_cg_batch_workspace_bytes(s["problems"], c["inner"]))
        return s
    if op == "gauge_update":
        s["thin"] = _links(c["links"], dims, seed, 10)
        s["fat"], s["naik"] = torch.empty_like(s["thin"]), torch.empty_like(s["thin"])
        s["packed"] = torch.zeros(h.hisq_links_bytes(lat, c["prec"]), dtype=torch.uint8, device=DEV)
        s["ws"] = h.empty_workspace(h.hisq_smear_workspace_bytes(lat))
        return s
    fat, naik = _fat_naik(c["links"], dims, seed)
    if op in ("dslash", "apply_m"):
        f = _field_format(c["prec"])
        s["links"] = _packed_links(lat, c["prec"], fat, naik)
        s["in"] = _packed_field(lat, f, _source(dims, seed, 30, c["nrhs"]))
        s["out"] = torch.zeros_like(s["in"])
        s["tmp"] = torch.zeros_like(s["in"]) if op == "apply_m" else None
        return s
    if op in ("cg", "multishift"):
        n = c.get("nrhs", 1)
        s["links"] = _packed_links(lat, "fp64", fat, naik)
        s["inner"] = None if c["inner"] == "fp64" else _packed_links(lat, c["inner"], fat, naik)
        s["b"] = _packed_field(lat, "fp64", _source(dims, seed, 30, n))
        if op == "cg":
            s["x"] = h.empty_field(lat, "fp64", n)
        else:
            s["shifts"] = [float(v) for v in _shifts(c)]
            s["x"] = [h.empty_field(lat, "fp64") for _ in s["shifts"]]
        s["ws"] = h.empty_workspace(h.hisq_cg_workspace_bytes(lat, c["inner"], n, c.get("nshift", 0)))
        return s
    s["links"] = _packed_links(lat, "fp32", fat, naik)
    s["ws"] = h.empty_workspace(h.hisq_ptc_workspace_bytes(lat))
    master = torch.view_as_real(_weights(seed)).reshape(-1).contiguous()
    s["w32"] = master.to(torch.float32)
    if op == "ptc_forward":
        s["in"] = _packed_field(lat, "fp32", _source(dims, seed, 30, 1))
        s["out"] = torch.zeros_like(s["in"])
        return s
    # training: fields of a converged solve are smooth; here the solution is drawn and its source follows from it
    x = _source(dims, seed, 30, c["batch"])
    s["master"], s["m"], s["v"], s["step"] = master, torch.zeros_like(master), torch.zeros_like(master), 0
    s["sol"] = _packed_field(lat, "fp64", x)
    l64, src, tmp = _packed_links(lat, "fp64", fat, naik), torch.zeros_like(s["sol"]), torch.zeros_like(s["sol"])
    h.hisq_apply_m(lat, "fp64", c["mass"], l64, s["sol"], src, tmp, c["batch"])
    b = torch.empty_like(x)
    h.hisq_unpack_field(lat, "fp64", c["batch"], src, b)
    s["src"] = _packed_field(lat, "fp32", b)
    return s


def _shifts(c):
    n = c["nshift"]
    return 10.0 ** (-5.0 + 5.0 * np.arange(n) / max(1, n - 1))


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def _values(packed, prec, nrhs):
    """The numbers of a packed field (layout: the head of include/hisq.h), without the unused column of an odd pair."""
    if prec == "fp64":
        return packed.view(torch.float64)
    if prec == "fp16n":
        return [packed.view(torch.float16).view(-1, 8)[:, :6], packed.view(torch.float32).view(-1, 4)[:, 3]]
    v = packed.view(torch.float32)
    if nrhs == 1 or nrhs % 2 == 0:
        return v
    pairs = v.view(nrhs // 2 + 1, -1, 2, 2)
    return [pairs[:-1], pairs[-1, :, 0]]


def run(s):
    c, lat = s["case"], s["lat"]
    op = c["op"]
    if op == "dslash":
        h.hisq_dslash(lat, c["prec"], 0, s["links"], s["in"], s["out"], c["nrhs"])
        return _values(s["out"], _field_format(c["prec"]), c["nrhs"])
    if op == "apply_m":
        h.hisq_apply_m(lat, c["prec"], c["mass"], s["links"], s["in"], s["out"], s["tmp"], c["nrhs"])
        return _values(s["out"], _field_format(c["prec"]), c["nrhs"])
    if op == "cg":
        s["x"].zero_()
        h.hisq_cg(lat, c["mass"], s["links"], s["inner"], c["inner"], c["nrhs"], s["b"], s["x"], c["tol"], 20000, s["ws"])
        return s["x"].view(torch.float64)
    if op == "multishift":
        h.hisq_multishift_cg(lat, c["mass"], s["links"], s["inner"], c["inner"], s["shifts"], s["b"], s["x"], c["tol"], 20000, s["ws"])
        return [x.view(torch.float64) for x in s["x"]]
    if op == "batch":
        for it in s["items"]:
            it["x"].zero_()
        h.hisq_cg_batch(s["problems"], c["inner"], 20000, s["ws"])
        return [it["x"].view(torch.float64) for it in s["items"]]
    if op == "ptc_forward":
        h.hisq_ptc_forward(lat, s["links"], s["w32"], s["in"], s["out"], s["ws"])
        return s["out"].view(torch.float32)
    if op == "ptc_train":
        s["step"] += 1
        loss = h.hisq_ptc_train_step(lat, c["mass"], s["links"], s["master"], s["w32"], s["m"], s["v"], s["step"], c["batch"],
                                     s["src"], s["sol"], s["ws"])
        # weights, moments (the first one is the gradient, scaled) and loss carry the accuracy of the FP32 network
        return {"w": s["w32"], "m": s["m"].to(torch.float32), "v": s["v"].to(torch.float32), "loss": np.float32(loss)}
    h.hisq_smear_links(lat, s["thin"], s["fat"], s["naik"], s["ws"])
    h.hisq_pack_links(lat, c["prec"], s["fat"], s["naik"], s["packed"])
    kind = torch.float64 if c["prec"].startswith("fp64") else torch.float16 if c["prec"] == "fp16n" else torch.float32
    return {"fat": s["fat"], "naik": s["naik"], "packed": s["packed"].view(kind)}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _link_reals(prec):
    return 8 * (12 if prec.endswith("r12") else 18) + 8 * (12 if prec.endswith("r12") else 14 if prec.endswith("w14") else 18)


def _real(prec):
    return REAL[_field_format(prec)]


def _dslash_work(vol, prec, nrhs):
    """One parity: both parities' links of its sites, the fields in and out once; 1146 operations a site and right-hand side."""
    vh, b = vol // 2, _real(prec)
    per_field = 16 if prec == "fp16n" else 6 * b
    return vh * (_link_reals(prec) * b + 2 * nrhs * per_field), 1146 * vh * nrhs


def _iterations(c, dims, mass):
    """About how many iterations plain CG takes for these links and this mass: half the root of the condition number a digit of ln(2/tol)."""
    gap = 1e-3 if c["links"] == "haar" or c["tbc"] > 0 else 0.41 * min(1.0, 8.0 / dims[3]) ** 4.8   # measured on the listed ones
    low = mass * mass + gap
    return math.ceil(0.5 * math.sqrt(60.0 / low) * math.log(2 / c["tol"]))


def _solve_work(c, dims, prec, nrhs, mass, nshift=0):
    """Iterations of two operator calls and six fields touched for each column (four more for every further shift)."""
    vol = _vol(dims)
    by, fl = _dslash_work(vol, prec, nrhs)
    vec = (vol // 2) * (6 * nrhs + 4 * max(0, nshift - 1)) * 6 * (8 if prec.startswith("fp64") else 4)
    its = _iterations(c, dims, mass)
    return its * (2 * by + vec), its * (2 * fl + vec)


def _ptc_flops(vol):
    """8->8 layer on all sites; of the first the hops on odd sites, of the last the even ones."""
    hop, mul = 66, 24                       # 3x3 matrix times vector; complex number times vector, added
    return vol * (8 * 8 * hop + 8 * 72 * mul) + vol // 2 * (8 * hop + 8 * 8 * mul + 8 * mul) + vol // 2 * (8 * 8 * hop + 72 * mul)


def work(c):
    op, dims = c["op"], _dims(c)
    vol = _vol(dims)
    if op == "dslash":
        b, f = _dslash_work(vol, c["prec"], c["nrhs"])
    elif op == "apply_m":
        b, f = _dslash_work(vol, c["prec"], c["nrhs"])
        b, f = 2 * b, 2 * f + vol // 2 * 24 * c["nrhs"]
    elif op in ("cg", "multishift"):
        b, f = _solve_work(c, dims, c["inner"], c.get("nrhs", 1), c["mass"], c.get("nshift", 0))
    elif op == "batch":
        b = f = 0
        for d, n in _mix(c):
            x, y = _solve_work(c, d, c["inner"], 1, 1.2 * c["mass"])
            b, f = b + n * x, f + n * y
    elif op == "ptc_forward":
        b, f = vol * 4 * 18 * 4 + vol * 24, _ptc_flops(vol)
    elif op == "ptc_train":
        # links once; the fields of each pair; forward, weight and input gradients (the first layer has no input gradient), M_e
        n = c["batch"]
        b = vol * 8 * 18 * 4 + n * (vol // 2) * (24 + 48)
        f = n * (3 * _ptc_flops(vol) + 2 * 1146 * (vol // 2))
    else:
        b = vol * 4 * 9 * 16 * 3 + vol * _link_reals(c["prec"]) // 2 * _real(c["prec"])
        f = vol * SMEAR_PRODUCTS * 198
    return {"bytes": float(b), "flops": float(f)}


# ---------------------------------------------------------------------------
# The same numbers in 64 bits, by plain torch
# ---------------------------------------------------------------------------

def _parity_masks(dims):
    nx, ny, nz, nt = dims
    a = [torch.arange(n, device=DEV) for n in (nt, nz, ny, nx)]
    p = (a[0][:, None, None, None] + a[1][None, :, None, None] + a[2][None, None, :, None] + a[3]) % 2
    return p == 0, p == 1


def _eta(dims):
    """Staggered phases 1, (-1)^x, (-1)^(x+y), (-1)^(x+y+z)."""
    nx, ny, nz, nt = dims
    x = torch.arange(nx, device=DEV)[None, None, None, :].expand(nt, nz, ny, nx)
    y = torch.arange(ny, device=DEV)[None, None, :, None].expand(nt, nz, ny, nx)
    z = torch.arange(nz, device=DEV)[None, :, None, None].expand(nt, nz, ny, nx)
    return [1.0 - 2.0 * (k % 2).to(torch.float64) for k in (0 * x, x, x + y, x + y + z)]


def _mv(u, v):
    return (u * v[..., None, :]).sum(-1)


def _hop(v, mu, n, tbc, off):
    """v(x + n mu) with the boundary sign in time; `off` leading axes before (Nt, Nz, Ny, Nx)."""
    r = v.roll(-n, AXIS[mu] + off)
    if mu == 3 and tbc < 0:
        wrapped = r.narrow(off, r.shape[off] - n if n > 0 else 0, abs(n))
        wrapped.neg_()
    return r


def _full_dslash(X, W, eta, tbc, v):
    """D v over the whole lattice, v: (columns, Nt, Nz, Ny, Nx, 3)."""
    out = torch.zeros_like(v)
    for k in range(v.shape[0]):
        for mu in range(4):
            a = _mv(X[mu], _hop(v[k], mu, 1, tbc, 0)) - _hop(_mv(_dag(X[mu]), v[k]), mu, -1, tbc, 0)
            a += _mv(W[mu], _hop(v[k], mu, 3, tbc, 0))
            a -= _hop(_mv(_dag(W[mu]), v[k]), mu, -3, tbc, 0)
            out[k] += eta[mu][..., None] * a
    return out


class _Operator:
    """D and M_e on half-lattice fields (columns, V/2, 3)."""

    def __init__(self, dims, tbc, X, W):
        self.dims, self.tbc, self.X, self.W = dims, tbc, X, W
        self.mask, self.eta = _parity_masks(dims), _eta(dims)

    def dslash(self, half, out_parity):
        nx, ny, nz, nt = self.dims
        out = torch.empty_like(half)
        for k in range(half.shape[0]):
            v = torch.zeros(1, nt, nz, ny, nx, 3, dtype=torch.complex128, device=DEV)
            v[0][self.mask[1 - out_parity]] = half[k]
            out[k] = _full_dslash(self.X, self.W, self.eta, self.tbc, v)[0][self.mask[out_parity]]
        return out

    def m(self, half, mass):
        return mass * mass * half - self.dslash(self.dslash(half, 1), 0)


class _Neighbours:
    """M_e by gathered neighbours, for solves: the links of each parity's sites in one table. Several lattices
    (dims, X, W, mass) stand one after another in it, each with its own Krylov scalars."""

    def __init__(self, tbc, lattices):
        self.U, self.at = [[], []], [[], []]
        seg, m2, done = [], [], 0
        for n, (dims, X, W, mass) in enumerate(lattices):
            self._add(dims, tbc, X, W, done)
            vh = _vol(dims) // 2
            done += vh
            seg.append(torch.full((vh,), n, device=DEV))
            m2.append(mass * mass)
        self.U, self.at = [torch.cat(u) for u in self.U], [torch.cat(a) for a in self.at]
        self.counts = [len(v) for v in seg]
        self.seg, self.m2 = torch.cat(seg), torch.tensor(m2, dtype=torch.float64, device=DEV)[:, None]

    def _add(self, dims, tbc, X, W, done):
        nx, ny, nz, nt = dims
        mask, vh, eta = _parity_masks(dims), _vol(dims) // 2, _eta(dims)
        place = torch.empty(nt, nz, ny, nx, dtype=torch.int64, device=DEV)
        for p in range(2):
            place[mask[p]] = torch.arange(done, done + vh, device=DEV)
        one = torch.ones(nt, nz, ny, nx, dtype=torch.float64, device=DEV)
        for p in range(2):
            us, ats = [], []
            for mu in range(4):
                for L, n in ((X, 1), (W, 3)):
                    f = eta[mu] * _hop(one, mu, n, tbc, 0)
                    us.append((L[mu] * f[..., None, None])[mask[p]])
                    ats.append(place.roll(-n, AXIS[mu])[mask[p]])
                    f = -eta[mu] * _hop(one, mu, -n, tbc, 0)
                    us.append((_dag(L[mu]).roll(n, AXIS[mu]) * f[..., None, None])[mask[p]])
                    ats.append(place.roll(n, AXIS[mu])[mask[p]])
            self.U[p].append(torch.stack(us, 1).permute(0, 2, 1, 3).reshape(vh, 3, 48))   # [site][row][hop, col]
            self.at[p].append(torch.stack(ats, 1).reshape(-1))

    def dslash(self, v, p):
        """v: (sites, 3, columns) on the other parity."""
        g = v[self.at[p]].reshape(v.shape[0], 48, v.shape[2])
        if v.shape[2] > 1:
            return torch.matmul(self.U[p], g)
        return (self.U[p] * g[:, None, :, 0]).sum(-1, keepdim=True)

    def a(self, v, add):
        return add[self.seg][:, None] * v - self.dslash(self.dslash(v, 1), 0)

    def dot(self, u, v):
        d = (u.real * v.real + u.imag * v.imag).sum(1)
        return torch.stack([part.sum(0) for part in d.split(self.counts)])

    def cg(self, b, add, tol):
        x, r, p = torch.zeros_like(b), b.clone(), b.clone()
        rr = self.dot(r, r)
        stop = rr * tol * tol
        for k in range(6000):
            q, go = self.a(p, add), rr > stop
            al = torch.where(go, rr / self.dot(p, q), torch.zeros_like(rr))[self.seg][:, None]
            x += al * p
            r -= al * q
            new = self.dot(r, r)
            p = r + torch.where(go, new / rr, torch.zeros_like(rr))[self.seg][:, None] * p
            rr = torch.where(go, new, rr)
            if k % 25 == 24 and bool((rr <= stop).all()):
                break
        return x

    def solve(self, b, shifts):
        """(m^2 + shift_k - D D) x_k = b_k for columns b (sites, 3, columns), corrected once from the residual formed anew."""
        add = self.m2 + torch.as_tensor(shifts, dtype=torch.float64, device=DEV)[None, :]
        x = self.cg(b, add, 1e-14)
        return x + self.cg(b - self.a(x, add), add, 1e-3)


def _rounded_links(prec, fat, naik):
    """The links that a format holds, in 64 bits."""
    real = torch.float16 if prec == "fp16n" else torch.float32 if prec.startswith("fp32") else torch.float64

    def cast(a):
        return torch.view_as_complex(torch.view_as_real(a).to(real).to(torch.float64).contiguous())

    def third(a, z=None):
        q = cast(a)
        c = torch.linalg.cross(q[..., 0, :], q[..., 1, :], dim=-1).conj()
        q[..., 2, :] = c if z is None else cast(z)[..., None] * c
        return q

    if prec.endswith("r12"):
        return third(fat), third(naik)
    if prec.endswith("w14"):
        c = torch.linalg.cross(naik[..., 0, :], naik[..., 1, :], dim=-1).conj()
        z = (c.conj() * naik[..., 2, :]).sum(-1) / (c.conj() * c).sum(-1)
        return cast(fat), third(naik, z)
    return cast(fat), cast(naik)


def _rounded_field(prec, half):
    v = torch.view_as_real(half)
    if prec == "fp64":
        return half
    if prec == "fp32":
        return torch.view_as_complex(v.to(torch.float32).to(torch.float64))
    n = v.abs().amax((-1, -2), keepdim=True).to(torch.float32).to(torch.float64)
    return torch.view_as_complex(((v / n).to(torch.float16).to(torch.float64) * n).contiguous())


def _like_packed(prec, half):
    """A half field (columns, V/2, 3) laid out as _values gives the packed one."""
    n = half.shape[0]
    v = torch.view_as_real(half).permute(0, 2, 1, 3)               # [column][colour][site][2]
    if prec == "fp64" or (prec == "fp32" and n == 1):
        return v.reshape(-1)
    if prec == "fp16n":
        w = torch.view_as_real(half).reshape(-1, 6)
        norm = w.abs().amax(1)
        return [w / norm[:, None], norm]
    even = v[:n // 2 * 2].reshape(n // 2, 2, -1, 2).transpose(1, 2)   # [pair][colour, site][2 columns][2]
    return even.reshape(-1) if n % 2 == 0 else [even, v[-1].reshape(-1, 2)]


def _half_to_columns(half):
    return half.permute(1, 2, 0).contiguous()


def _packed64(x):
    """(V/2, 3, columns) to the packed FP64 layout."""
    return torch.view_as_real(x.permute(2, 1, 0)).reshape(-1)


def _polar(v):
    """The unitary factor of v by Newton's iteration Y <- (Y + Y^-+) / 2."""
    for _ in range(40):
        a, b, c = v[..., 0, :], v[..., 1, :], v[..., 2, :]
        cof = torch.stack((torch.linalg.cross(b, c, dim=-1), torch.linalg.cross(c, a, dim=-1), torch.linalg.cross(a, b, dim=-1)), -2)
        det = (a * cof[..., 0, :]).sum(-1)
        new = 0.5 * (v + (cof / det[..., None, None]).conj())       # inverse transposed = cofactors / det
        far = float((new - v).abs().max())
        v = new
        if far < 1e-14:
            break
    return v


def _staple(L, A, mu, nu, s):
    if s > 0:
        return _mm(_mm(L[nu], A.roll(-1, AXIS[nu])), _dag(L[nu].roll(-1, AXIS[mu])))
    return _mm(_mm(_dag(L[nu]), A), L[nu].roll(-1, AXIS[mu])).roll(1, AXIS[nu])


def _smeared(L, k):
    c1, c3, c5, c7, cl = k
    out = []
    for mu in range(4):
        other = [d for d in range(4) if d != mu]
        one = {(nu, s): _staple(L, L[mu], mu, nu, s) for nu in other for s in (1, -1)}
        both = {nu: one[nu, 1] + one[nu, -1] for nu in other}

        def along(nu, a):
            return _staple(L, a, mu, nu, 1) + _staple(L, a, mu, nu, -1)
        acc = c1 * L[mu]
        for nu in other:
            r, q = [d for d in other if d != nu]
            # outermost staple along nu of: the two 3-link sums (5-link), and the staples of staples (7-link)
            inner = c5 * (both[r] + both[q]) + c7 * (along(r, both[q]) + along(q, both[r]))
            acc = acc + c3 * both[nu] + along(nu, inner)
            if cl:
                acc = acc + cl * (_staple(L, one[nu, 1], mu, nu, 1) + _staple(L, one[nu, -1], mu, nu, -1))
        out.append(acc)
    return torch.stack(out)


def _transport(X, tbc, v, path):
    """T_p v for a field (channels, Nt, Nz, Ny, Nx, 3)."""
    if path == 0:
        return v
    mu = (path - 1) // 2
    if path % 2:
        return _mv(X[mu], _hop(v, mu, 1, tbc, 1))
    return _hop(_mv(_dag(X[mu]), v), mu, -1, tbc, 1)


def _layer(X, tbc, w, v):
    out = 0
    for p in range(9):
        out = out + torch.tensordot(w[:, :, p], _transport(X, tbc, v, p), dims=1)
    return out


def _layer_back(X, tbc, w, v, g):
    """(input gradient, weight gradient) of a layer, each dL/dRe + i dL/dIm."""
    gw, gv = torch.empty_like(w), 0
    for p in range(9):
        t = _transport(X, tbc, v, p)
        gw[:, :, p] = torch.stack([(t.conj() * g[o][None]).reshape(t.shape[0], -1).sum(1) for o in range(w.shape[0])])
        back = 0 if p == 0 else p + 1 if p % 2 else p - 1
        gv = gv + _transport(X, tbc, torch.tensordot(w[:, :, p].conj().T.contiguous(), g, dims=1), back)
    return gv, gw


def _split_weights(flat):
    out, k = [], 0
    for cin, cout in zip(CHANNELS[:-1], CHANNELS[1:]):
        out.append(flat[k:k + cout * cin * 9].reshape(cout, cin, 9))
        k += cout * cin * 9
    return out


def exact(c, seed):
    op, dims, tbc = c["op"], _dims(c), c["tbc"]
    if op == "gauge_update":
        Y = _polar(_smeared(_links(c["links"], dims, seed, 10), LEVEL1))
        naik = torch.stack([C_NAIK * _mm(_mm(Y[mu], Y[mu].roll(-1, AXIS[mu])), Y[mu].roll(-2, AXIS[mu])) for mu in range(4)])
        return {"fat": _smeared(Y, LEVEL2), "naik": naik, "packed": None}
    if op == "batch":
        every = []
        for dims, count in _mix(c):
            for _ in range(count):
                fat, naik, src, mass = _problem(c, seed, len(every), dims)
                every.append(((dims, fat, naik, mass), _half_to_columns(src)))
        x = _Neighbours(tbc, [e[0] for e in every]).solve(torch.cat([e[1] for e in every]), [0.0])
        return [_packed64(v) for v in x.split([e[1].shape[0] for e in every])]
    fat, naik = _fat_naik(c["links"], dims, seed)
    if op in ("dslash", "apply_m"):
        f = _field_format(c["prec"])
        D = _Operator(dims, tbc, *_rounded_links(c["prec"], fat, naik))
        v = _rounded_field(f, _source(dims, seed, 30, c["nrhs"]))
        return _like_packed(f, D.dslash(v, 0) if op == "dslash" else D.m(v, c["mass"]))
    if op in ("cg", "multishift"):
        n = c.get("nrhs", 1)
        b = _half_to_columns(_source(dims, seed, 30, n))
        A = _Neighbours(tbc, [(dims, fat, naik, c["mass"])])
        if op == "cg":
            return _packed64(A.solve(b, [0.0] * n))
        sh = _shifts(c)
        x = A.solve(b.expand(-1, -1, len(sh)).contiguous(), sh)
        return [_packed64(x[:, :, k:k + 1]) for k in range(len(sh))]
    X = _rounded_links("fp32", fat, fat)[0]
    nx, ny, nz, nt = dims
    mask = _parity_masks(dims)[0]
    w64 = _weights(seed)
    w = _split_weights(torch.view_as_complex(torch.view_as_real(w64).to(torch.float32).to(torch.float64)))

    def whole(half):
        v = torch.zeros(1, nt, nz, ny, nx, 3, dtype=torch.complex128, device=DEV)
        v[0][mask] = half
        return v

    if op == "ptc_forward":
        v = whole(_rounded_field("fp32", _source(dims, seed, 30, 1))[0])
        for k in range(3):
            v = _layer(X, tbc, w[k], v)
        return _like_packed("fp32", v[0][mask][None])
    x = _source(dims, seed, 30, c["batch"])
    D64 = _Operator(dims, tbc, fat, naik)
    D32 = _Operator(dims, tbc, *_rounded_links("fp32", fat, naik))
    b = _rounded_field("fp32", D64.m(x, c["mass"]))
    loss, grad = 0.0, [torch.zeros_like(a) for a in w]
    for i in range(c["batch"]):
        acts = [whole(b[i])]
        for k in range(3):
            acts.append(_layer(X, tbc, w[k], acts[-1]))
        e = acts[3][0][mask][None] - x[i:i + 1]
        me = D32.m(e, c["mass"])
        scale = 1.0 / (c["batch"] * float((x[i].conj() * b[i]).real.sum()))
        loss += float((e.conj() * me).real.sum()) * scale
        g = whole((2 * scale * me)[0])
        for k in (2, 1, 0):
            g, gw = _layer_back(X, tbc, w[k], acts[k], g)
            grad[k] += gw
    g = torch.view_as_real(torch.cat([a.reshape(-1) for a in grad])).reshape(-1)
    m, v = 0.1 * g, 0.001 * g * g
    master = torch.view_as_real(w64).reshape(-1) - 1e-3 * g / (g.abs() + 1e-8)
    return {"w": master, "m": m, "v": v, "loss": np.float64(loss)}
