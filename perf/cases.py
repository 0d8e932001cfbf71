"""Performance cases of the solver: the calls that an all-mode-averaging
program makes, each through the package's public entry points.

A case is a dict of plain values.  "kind" names the path:

  dirac     one application of the Wilson-clover operator
  sap       one application of the Schwarz preconditioner
  lowmode   the low-mode part of a solution, Phi A^{-1} Phi^+ v (restriction,
            little solve, prolongation)
  gcr       one deflated exact solve to 1e-10
  ama       an all-mode-averaging set: truncated solves of every position and
            exact solves of the first
  contract  the measurement on one propagator: nucleon two-point function,
            sequential sources of both flavours, three-point function
  gauss     Gaussian smearing of vectors with APE-smeared links
  ape       APE smearing of a gauge field's spatial links

Inputs are synthetic: links U = exp(i 0.4 H) with H a Gaussian traceless
Hermitian matrix, Gaussian spinors, point sources, propagators that fall off
with the distance from their source.  `exact` evaluates the same maps in
complex128 with torch alone, from the definitions (sites in the order t, x,
y, z; Euclidean chiral basis).
"""

import math

import numpy as np
import torch

import paper_1605_00564_amd as dfl

STORAGE = {"f64": dfl.F64, "f32": dfl.F32, "f16": dfl.F16, "bf16": dfl.BF16}
EPS, KAPPA, CSW = 0.4, 0.124, 1.5
NCY, NMR = 5, 4


def listed():
    return [
        # the smallest call: the 4^4 test lattice, FP64, where launches count
        dict(name="dirac-4c4-f64-n1", kind="dirac", dims="4x4x4x4", block="2x2x2x2", storage="f64", n=1),
        # an ordinary lattice in 6^4 blocks (not a power of two), BF16 links, an odd count of right-hand sides
        dict(name="dirac-24c48-bf16-n7", kind="dirac", dims="48x24x24x24", block="6x6x6x6", storage="bf16", n=7),
        # the production batch: the operator of the sloppy solves on 24 right-hand sides at 32^3 x 64
        dict(name="dirac-32c64-f16-n24", kind="dirac", dims="64x32x32x32", block="4x4x4x4", storage="f16", n=24),
        # the preconditioner of one exact solve on a small lattice
        dict(name="sap-16c32-f32-n1", kind="sap", dims="32x16x16x16", block="4x4x4x4", storage="f32", vecs="f32", n=1),
        # BF16 links, 6^4 blocks: the preconditioner of the larger-block configuration
        dict(name="sap-24c48-bf16-n6", kind="sap", dims="48x24x24x24", block="6x6x6x6", storage="bf16", vecs="f16", n=6),
        # the preconditioner of the sloppy solves on the production batch
        dict(name="sap-32c64-f16-n24", kind="sap", dims="64x32x32x32", block="4x4x4x4", storage="f16", vecs="f16", n=24),
        # the deflated start of 12 spin-colour solves, in FP64 as the outer loop does it
        dict(name="lowmode-16c32-f64-n12", kind="lowmode", dims="32x16x16x16", block="4x4x4x4", ns=12, io="f64", n=12),
        # one exact bias-correction solve: many short launches
        dict(name="gcr-16c32-n1", kind="gcr", dims="32x16x16x16", block="4x4x4x4", ns=12, io="f64", n=1),
        # a whole set: 4 positions sloppily (48 right-hand sides in batches of 24), the first one exactly
        dict(name="ama-24c48-p4", kind="ama", dims="48x24x24x24", block="4x4x4x4", ns=12, positions=4, batch=24,
             fixed=0, vecs="f16"),
        # the measurement on one sloppy propagator (the many ones)
        dict(name="contract-24c48-f32", kind="contract", dims="48x24x24x24", block="4x4x4x4", io="f32"),
        # sources (or sinks) of one propagator smeared
        dict(name="gauss-24c48-f64-n12", kind="gauss", dims="48x24x24x24", block="4x4x4x4", io="f64", n=12, iters=10),
        # the smeared links of one gauge field at the production size
        dict(name="ape-32c64", kind="ape", dims="64x32x32x32", block="4x4x4x4", iters=4),
    ]


# ---------------------------------------------------------------------------
# drawn cases
# ---------------------------------------------------------------------------

BLOCKS = ("4x4x4x4", "4x4x4x4", "4x4x4x4", "6x6x6x6", "8x4x4x4", "2x2x2x2", "4x4x4x6")


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lattice(rng, vmin, vmax, blocks=BLOCKS):
    """A block shape and a lattice of an even number of blocks in every
    direction, of about vmin to vmax sites."""
    for _ in range(100):
        block = _ints(rng.choice(blocks))
        dims = [2 * b for b in block]
        target = _log(rng, vmin, vmax)
        if math.prod(dims) > vmax:
            continue
        while True:
            fit = [m for m in range(4) if math.prod(dims) // dims[m] * (dims[m] + 2 * block[m]) <= target
                   and dims[m] <= 3 * min(dims)]
            if not fit:
                break
            m = rng.choice(fit)
            dims[m] += 2 * block[m]
        return "x".join(map(str, dims)), "x".join(map(str, block))
    return "8x8x8x8", "4x4x4x4"


def draw(rng):
    kind = rng.choice(["dirac", "dirac", "sap", "sap", "lowmode", "gcr", "ama", "contract", "gauss", "ape"])
    if kind in ("dirac", "sap"):
        dims, block = _lattice(rng, 256 if kind == "dirac" else 4096, 1 << 20)
        n = _log(rng, 1, max(1, min(24, (24 << 20) // math.prod(_ints(dims)))))
        if kind == "dirac":
            return dict(kind=kind, dims=dims, block=block, storage=rng.choice(["f64", "f32", "f16", "bf16"]), n=n)
        storage = rng.choice(["f32", "f16", "bf16"])
        vecs = "f32" if storage == "f32" else rng.choice(["f32", "f16"])
        return dict(kind=kind, dims=dims, block=block, storage=storage, vecs=vecs, n=n)
    if kind in ("lowmode", "gcr", "ama"):
        blocks = ("4x4x4x4", "4x4x4x4", "8x4x4x4", "6x6x6x6")
        dims, block = _lattice(rng, 4096, 1 << 17 if kind == "gcr" else 1 << 18, blocks)
        ns = rng.randint(4, 20)
        if kind == "lowmode":
            return dict(kind=kind, dims=dims, block=block, ns=ns, io=rng.choice(["f64", "f32"]), n=_log(rng, 1, 24))
        if kind == "gcr":
            return dict(kind=kind, dims=dims, block=block, ns=ns, io=rng.choice(["f64", "f32"]), n=rng.randint(1, 3))
        return dict(kind=kind, dims=dims, block=block, ns=ns, positions=rng.randint(1, 3),
                    batch=rng.choice([6, 12, 13, 24]), fixed=rng.choice([0, 2]), vecs=rng.choice(["f32", "f16"]))
    dims, block = _lattice(rng, 4096, 1 << 19)
    if kind == "contract":
        return dict(kind=kind, dims=dims, block=block, io=rng.choice(["f64", "f32"]))
    if kind == "gauss":
        return dict(kind=kind, dims=dims, block=block, io=rng.choice(["f64", "f32"]), n=_log(rng, 1, 13),
                    iters=rng.randint(3, 10))
    return dict(kind=kind, dims=dims, block=block, iters=rng.randint(1, 6))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _ints(text):
    return tuple(int(v) for v in text.split("x"))


def _io(case):
    if case["kind"] == "dirac":
        return torch.complex128 if case["storage"] == "f64" else torch.complex64
    if case["kind"] in ("sap",):
        return torch.complex64
    return torch.complex128 if case["io"] == "f64" else torch.complex64


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + 17)


def _cnormal(shape, dtype, gen):
    real = torch.float64 if dtype == torch.complex128 else torch.float32
    return torch.view_as_complex(torch.randn((*shape, 2), dtype=real, device="cuda", generator=gen))


def _mul(a, b):
    """Products of 3 x 3 matrices, entry by entry."""
    return (a[..., :, 0:1] * b[..., 0:1, :]).add_(a[..., :, 1:2] * b[..., 1:2, :]).add_(a[..., :, 2:3] * b[..., 2:3, :])


def _links(dims, gen, eps=EPS):
    """[V, 4, 3, 3] links exp(i eps H), H = sum_a w_a lambda_a / 2, by the
    exponential's series (eps H is of order one)."""
    V = math.prod(dims)
    w = torch.randn((V, 4, 8), dtype=torch.float64, device="cuda", generator=gen) * (0.5 * eps)
    a = torch.zeros((V, 4, 3, 3), dtype=torch.complex128, device="cuda")   # i eps H
    d8 = w[..., 7] / math.sqrt(3.0)
    a[..., 0, 0].imag.copy_(w[..., 2] + d8)
    a[..., 1, 1].imag.copy_(d8 - w[..., 2])
    a[..., 2, 2].imag.copy_(-2 * d8)
    for (i, j), (p, q) in (((0, 1), (0, 1)), ((0, 2), (3, 4)), ((1, 2), (5, 6))):
        a[..., i, j] = torch.complex(w[..., q], w[..., p])
        a[..., j, i] = torch.complex(-w[..., q], w[..., p])
    eye = torch.eye(3, dtype=torch.complex128, device="cuda")
    u = eye + a / 20
    for k in range(19, 0, -1):
        u = _mul(a, u).div_(k).add_(eye)
    return u


def _site(dims, seed):
    """The source position, on even coordinates."""
    s = 2654435761 * (int(seed) + 1)
    out = []
    for extent in dims:
        s = (s * 6364136223846793005 + 1442695040888963407) % (1 << 64)
        out.append(2 * ((s >> 33) % (extent // 2)))
    return tuple(out)


def _propagator(dims, seed, dtype, gen):
    """[12, V, 4, 3] of the size of a propagator from the seed's site: near
    the unit matrix there, random with an exponential fall-off elsewhere."""
    src = _site(dims, seed)
    dist = 0.0
    for m, (extent, c) in enumerate(zip(dims, src)):
        x = torch.arange(extent, device="cuda", dtype=torch.float32)
        d = torch.minimum((x - c).abs(), extent - (x - c).abs())
        dist = dist + d.reshape([-1 if k == m else 1 for k in range(4)]) ** 2
    amp = torch.exp(-0.7 * dist.sqrt()).reshape(-1)
    p = _cnormal((12, math.prod(dims), 4, 3), dtype, gen)
    p *= (0.3 * amp)[None, :, None, None].to(p.real.dtype)
    return p


def _phi(case, links, gen):
    """Block-orthonormal fields [Nb, Ns, Vb, 4, 3]: Gaussian fields smoothed by
    a few relaxation steps of the operator, orthonormalised in each block."""
    dims, block, ns = _ints(case["dims"]), _ints(case["block"]), case["ns"]
    op = _Wilson(dims, links, torch.complex64)
    v = _cnormal((ns, *dims, 4, 3), torch.complex64, gen)
    for _ in range(6):
        v = v - 0.6 * op.m(v)
    p = _to_blocks(v, dims, block)
    nb, vb = p.shape[0], p.shape[2]
    p = p.reshape(nb, ns, vb * 12).to(torch.complex128)
    for _ in range(2):
        g = torch.bmm(p, p.conj().transpose(1, 2).resolve_conj().contiguous())
        p = torch.linalg.solve_triangular(torch.linalg.cholesky(g), p, upper=False)
    # the handle keeps the fields in FP32
    return p.to(torch.complex64).to(torch.complex128).reshape(nb, ns, vb, 4, 3).contiguous()


def _to_blocks(v, dims, block):
    """[n, T, X, Y, Z, 4, 3] -> [Nb, n, Vb, 4, 3], both in lexicographic order."""
    n = v.shape[0]
    shape = [n]
    for extent, b in zip(dims, block):
        shape += [extent // b, b]
    v = v.reshape(*shape, 4, 3).permute(1, 3, 5, 7, 0, 2, 4, 6, 8, 9, 10)
    return v.reshape(math.prod(dims) // math.prod(block), n, math.prod(block), 4, 3)


def _from_blocks(p, dims, block):
    n = p.shape[1]
    grid = [extent // b for extent, b in zip(dims, block)]
    return p.reshape(*grid, n, *block, 4, 3).permute(4, 0, 5, 1, 6, 2, 7, 3, 8, 9, 10).reshape(n, *dims, 4, 3)


def _sources(case, seed, gen):
    """gcr: the first spin-colour point sources; lowmode: Gaussian vectors."""
    dims = _ints(case["dims"])
    V, n = math.prod(dims), case["n"]
    if case["kind"] != "gcr":
        return _cnormal((n, V, 4, 3), _io(case), gen)
    b = torch.zeros((n, V, 12), dtype=_io(case), device="cuda")
    t, x, y, z = _site(dims, seed)
    lex = z + dims[3] * (y + dims[2] * (x + dims[1] * t))
    for r in range(n):
        b[r, lex, (5 * r + seed) % 12] = 1
    return b.reshape(n, V, 4, 3)


def _positions(case, seed):
    """Source positions related by an even number of block steps in time."""
    dims, block = _ints(case["dims"]), _ints(case["block"])
    t, x, y, z = _site(dims, seed)
    return [((t + 2 * block[0] * k) % dims[0], x, y, z) for k in range(case["positions"])]


P_PLUS = [[0.5 * ((i == j) - (abs(i - j) == 2)) for j in range(4)] for i in range(4)]   # (1 + gamma_0) / 2
GAMMA_OP = [[float((i == j) * (1 if i < 2 else -1)) for j in range(4)] for i in range(4)]  # gamma_5
GAUSS_KAPPA, APE_ALPHA = 3.0, 0.5


def prepare(case, seed):
    dims, block, kind = _ints(case["dims"]), _ints(case["block"]), case["kind"]
    V = math.prod(dims)
    gen = _gen(seed)
    links = _links(dims, gen)
    field = dfl.Field(dims, block, KAPPA, CSW, links)
    s = dict(case=dict(case), field=field)
    if kind == "dirac":
        s["x"] = _cnormal((case["n"], V, 4, 3), _io(case), gen)
        s["out"] = torch.empty_like(s["x"])
    elif kind == "sap":
        s["x"] = _cnormal((case["n"], V, 4, 3), _io(case), gen)
        s["out"] = torch.empty_like(s["x"])
        s["sap"] = dfl.SapParams(NCY, NMR, STORAGE[case["storage"]], STORAGE[case["vecs"]])
    elif kind == "lowmode":
        s["dfl"] = dfl.Deflation(field, case["ns"], ninv=0)
        s["dfl"].set_phi(_phi(case, links, gen))
        s["x"] = _sources(case, seed, gen)
    elif kind == "gcr":
        sap = dfl.SapParams(NCY, NMR, dfl.F32)
        s["dfl"] = dfl.Deflation(field, case["ns"], ninv=5, sap=sap)
        s["x"] = _sources(case, seed, gen)
        s["par"] = dfl.GcrParams(nkv=16, nmx=400, res=1e-10, sap=sap, dfl=s["dfl"], little_tol=1e-10, little_maxit=16)
    elif kind == "ama":
        sap_s = dfl.SapParams(NCY, NMR, dfl.F16, STORAGE[case["vecs"]])
        sap_e = dfl.SapParams(NCY, NMR, dfl.F32)
        s["dfl"] = dfl.Deflation(field, case["ns"], ninv=5, sap=sap_e)
        s["sloppy"] = dfl.GcrParams(nkv=8, nmx=24, fixed_iters=case["fixed"], res=3e-3, sap=sap_s, dfl=s["dfl"],
                                    little_tol=1e-6, little_maxit=4)
        s["exact"] = dfl.GcrParams(nkv=16, nmx=400, res=1e-10, sap=sap_e, dfl=s["dfl"], little_tol=1e-10,
                                   little_maxit=16)
        s["pos"] = _positions(case, seed)
        s["xs"] = [torch.empty((12, V, 4, 3), dtype=torch.complex64, device="cuda") for _ in s["pos"]]
        s["xe"] = [torch.empty((12, V, 4, 3), dtype=torch.complex128, device="cuda")]
    elif kind == "contract":
        s["prop"] = _propagator(dims, seed, _io(case), gen)
        s["seq"] = _propagator(dims, seed + 1, _io(case), gen)
        s["t0"] = _site(dims, seed)[0]
        s["proj"], s["op"] = np.array(P_PLUS, dtype=complex), np.array(GAMMA_OP, dtype=complex)
    elif kind == "gauss":
        field.ape_smear(APE_ALPHA, 2)
        s["x"] = _cnormal((case["n"], V, 4, 3), _io(case), gen)
        s["out"] = torch.empty_like(s["x"])
    return s


def run(s):
    case, field = s["case"], s["field"]
    kind = case["kind"]
    if kind == "dirac":
        return dfl.dirac_apply(field, s["x"], STORAGE[case["storage"]], out=s["out"])
    if kind == "sap":
        return dfl.sap_precond(field, s["x"], s["sap"], out=s["out"])
    if kind == "lowmode":
        c, _ = s["dfl"].little_solve(s["dfl"].restrict(s["x"]), tol=1e-10)
        return s["dfl"].prolong(c, dtype=s["x"].dtype)
    if kind == "gcr":
        return dfl.gcr_solve(field, s["x"], s["par"])[0]
    if kind == "ama":
        xs, xe, _, _ = dfl.ama_solve(field, s["pos"], [k == 0 for k in range(len(s["pos"]))], s["sloppy"], s["exact"],
                                     dtype=torch.complex128, sloppy_dtype=torch.complex64, batch=case["batch"],
                                     out_sloppy=s["xs"], out_exact=s["xe"])
        return {"sloppy": xs, "exact": xe}
    if kind == "contract":
        T = field.dims[0]
        sink = (s["t0"] + T // 4) % T
        return {"c2": dfl.nucleon_2pt(field, s["prop"], s["t0"]),
                "u": dfl.nucleon_seq_sources(field, s["prop"], sink, s["proj"], "u"),
                "d": dfl.nucleon_seq_sources(field, s["prop"], sink, s["proj"], "d"),
                "c3": dfl.nucleon_3pt(field, s["seq"], s["prop"], s["t0"], s["op"])}
    if kind == "gauss":
        return dfl.gauss_smear(field, s["x"], GAUSS_KAPPA, case["iters"], out=s["out"])
    field.ape_smear(APE_ALPHA, case["iters"])
    return field.ape_links()


# ---------------------------------------------------------------------------
# work: each input once, each output once, and the operations of the maps
# ---------------------------------------------------------------------------

def _hops(block):
    return sum(2.0 * (b - 1) / b for b in block)


def _sap_flops(block, V):
    """Five cycles of minimal-residual block solves (165 flop a hop, 504 a
    clover block pair) with the hops across the faces."""
    h, nf = 165.0 * _hops(block), sum(4.0 / b for b in block)
    pair = 504 + (h + 72) + NMR * (2 * h + 1392) + (h + 576) + 552 + nf * 192
    return NCY * pair * V / 2


def work(case):
    dims, block, kind = _ints(case["dims"]), _ints(case["block"]), case["kind"]
    V = math.prod(dims)
    link = {"f64": 4 * 144 + 576, "f32": 4 * 48 + 288, "f16": 4 * 24 + 144, "bf16": 4 * 24 + 144}
    if kind == "ape":
        return {"bytes": 2 * 432.0 * V, "flops": 3 * 6000.0 * V * case["iters"]}
    if kind == "contract":
        vec = (192 if case["io"] == "f64" else 96) * 12.0 * V
        return {"bytes": 4 * vec, "flops": 28800.0 * V + 12 * 500.0 * V}
    vec = 24 * (8 if _io_bytes(case) == 8 else 4) * V
    if kind == "ama":
        n, ne = 12 * case["positions"], 12
        it, ite = 2, 6
        phi = 8 * 12 * case["ns"] * V
        per = _sap_flops(block, V) + 2 * 1872.0 * V + 16.0 * 12 * case["ns"] * V
        flops = n * (it * per + 2 * 1872.0 * V) + ne * (ite * per + 2 * 1872.0 * V)
        return {"bytes": V * 1.5 * link["f16"] + V * link["f64"] + phi + n * 96.0 * V + ne * 192.0 * V, "flops": flops}
    n = case["n"]
    if kind == "dirac":
        return {"bytes": V * link[case["storage"]] + 2.0 * n * vec, "flops": 1872.0 * V * n}
    if kind == "sap":
        return {"bytes": V * 1.3 * link[case["storage"]] + 2.0 * n * vec, "flops": n * _sap_flops(block, V)}
    if kind == "lowmode":
        nlit = V // math.prod(block) * case["ns"]
        little = 10 * 8.0 * 10 * case["ns"] * nlit * n
        return {"bytes": 8.0 * 12 * case["ns"] * V + 9 * 16.0 * case["ns"] * nlit + 2.0 * n * vec,
                "flops": 2 * 8.0 * 12 * case["ns"] * V * n + little}
    if kind == "gcr":
        per = _sap_flops(block, V) + 2 * 1872.0 * V + 16.0 * 12 * case["ns"] * V
        return {"bytes": V * 1.3 * link["f32"] + V * link["f64"] + 8.0 * 12 * case["ns"] * V + 2.0 * n * vec,
                "flops": n * (6 * per + 2 * 1872.0 * V)}
    return {"bytes": 3 * 144.0 * V + 2.0 * n * vec, "flops": n * case["iters"] * V * (6 * 4 * 66.0 + 48)}


def _io_bytes(case):
    if case["kind"] == "ama":
        return 8
    return 8 if _io(case) == torch.complex128 else 4


# ---------------------------------------------------------------------------
# the same maps in 64 bits, from their definitions
# ---------------------------------------------------------------------------

def _gammas():
    i = 1j
    z, one = torch.zeros((2, 2), dtype=torch.complex128), torch.eye(2, dtype=torch.complex128)
    sig = [torch.tensor(m, dtype=torch.complex128) for m in ([[0, 1], [1, 0]], [[0, -i], [i, 0]], [[1, 0], [0, -1]])]
    g = [torch.cat([torch.cat([z, -one], 1), torch.cat([-one, z], 1)])]
    g += [torch.cat([torch.cat([z, -i * s], 1), torch.cat([i * s, z], 1)]) for s in sig]
    return g


def _spin(m, v):
    """A 4 x 4 spin matrix on [..., 4, 3], by its nonzero entries."""
    rows = []
    for a in range(4):
        acc = None
        for b in range(4):
            c = complex(m[a, b])
            if c != 0:
                t = v[..., b, :] if c == 1 else c * v[..., b, :]
                acc = t if acc is None else acc + t
        rows.append(torch.zeros_like(v[..., 0, :]) if acc is None else acc)
    return torch.stack(rows, -2)


class _Wilson:
    """M = A - kappa H on [n, T, X, Y, Z, 4, 3]; block: the hops that leave a
    block of that shape are left out (the Dirichlet block operator)."""

    def __init__(self, dims, links, dtype=torch.complex128, clover=True):
        self.dims, self.dtype = dims, dtype
        u = links.reshape(*dims, 4, 3, 3)
        self.g = _gammas()
        self.a = self._clover(u).to(dtype) if clover else None
        self.u = [u[..., mu, :, :].to(dtype) for mu in range(4)]
        edge = [torch.ones(e, device="cuda", dtype=torch.float64) for e in dims]
        edge[0][-1] = -1   # antiperiodic in time: the hop from the last to the first timeslice
        self.bc = edge[0].reshape(-1, 1, 1, 1, 1, 1).to(dtype)

    def _clover(self, u):
        """Two Hermitian 6 x 6 blocks per site, [..., 2, 6, 6]."""
        def sh(m, *steps):
            for mu, d in steps:
                m = torch.roll(m, -d, mu)
            return m
        dag = lambda m: m.conj().transpose(-1, -2)  # noqa: E731
        full = torch.zeros((*self.dims, 2, 6, 6), dtype=torch.complex128, device="cuda")
        full[..., range(6), range(6)] = 1
        for mu in range(4):
            for nu in range(mu + 1, 4):
                um, un = u[..., mu, :, :], u[..., nu, :, :]
                q = _mul(_mul(um, sh(un, (mu, 1))), _mul(dag(sh(um, (nu, 1))), dag(un)))
                q = q + _mul(_mul(un, dag(sh(um, (mu, -1), (nu, 1)))), _mul(dag(sh(un, (mu, -1))), sh(um, (mu, -1))))
                q = q + _mul(_mul(dag(sh(um, (mu, -1))), dag(sh(un, (mu, -1), (nu, -1)))),
                             _mul(sh(um, (mu, -1), (nu, -1)), sh(un, (nu, -1))))
                q = q + _mul(_mul(dag(sh(un, (nu, -1))), sh(um, (nu, -1))), _mul(sh(un, (mu, 1), (nu, -1)), dag(um)))
                f = (q - dag(q)) / 8
                s = 0.5j * (self.g[mu] @ self.g[nu] - self.g[nu] @ self.g[mu])
                for h in range(2):
                    for a in range(2):
                        for b in range(2):
                            c = complex(s[2 * h + a, 2 * h + b])
                            if c != 0:
                                full[..., h, 3 * a:3 * a + 3, 3 * b:3 * b + 3] += 1j * KAPPA * CSW * c * f
        return full

    def clover(self, v, a=None):
        a = self.a if a is None else a
        w = v.reshape(*v.shape[:-2], 2, 6)
        out = a[..., 0] * w[..., 0:1]
        for j in range(1, 6):
            out = out + a[..., j] * w[..., j:j + 1]
        return out.reshape(v.shape)

    def hop(self, v, block=None):
        out = torch.zeros_like(v)
        for mu in range(4):
            u = self.u[mu]
            if block is not None:
                x = torch.arange(self.dims[mu], device="cuda")
                inside = (x % block[mu] != block[mu] - 1).to(self.dtype)
                u = u * inside.reshape([-1 if k == mu else 1 for k in range(6)])
            one = torch.eye(4, dtype=torch.complex128)
            # forward: (1 - gamma) U(x) v(x + mu); backward: (1 + gamma) U(x - mu)^+ v(x - mu)
            w = torch.roll(v, -1, 1 + mu)
            if mu == 0:
                w = w * self.bc
            w = _spin(one - self.g[mu], w)
            out += sum(u[..., None, :, b] * w[..., b:b + 1] for b in range(3))
            w = _spin(one + self.g[mu], v)
            w = sum(u.conj()[..., None, b, :] * w[..., b:b + 1] for b in range(3))
            if mu == 0:
                w = w * self.bc
            out += torch.roll(w, 1, 1 + mu)
        return out

    def m(self, v):
        return self.clover(v) - KAPPA * self.hop(v)


def _parity(dims):
    x = [torch.arange(e, device="cuda").reshape([-1 if k == m else 1 for k in range(4)]) for m, e in enumerate(dims)]
    return ((x[0] + x[1] + x[2] + x[3]) % 2 == 0).reshape(1, *dims, 1, 1)


def _colour(dims, block):
    x = [(torch.arange(e, device="cuda") // b).reshape([-1 if k == m else 1 for k in range(4)])
         for m, (e, b) in enumerate(zip(dims, block))]
    return ((x[0] + x[1] + x[2] + x[3]) % 2).reshape(1, *dims, 1, 1)


def _block_dot(a, b, dims, block):
    """sum conj(a) b over each block, spread over the block's sites again."""
    p = (a.conj() * b).sum((-1, -2))
    shape = [p.shape[0]]
    for extent, k in zip(dims, block):
        shape += [extent // k, k]
    p = p.reshape(shape).sum((2, 4, 6, 8), keepdim=True).expand(shape)
    return p.reshape(-1, *dims, 1, 1)


def _sap(op, eta, block):
    even = _parity(op.dims)
    col = _colour(op.dims, block)
    ainv = torch.linalg.inv(op.a)
    psi = torch.zeros_like(eta)
    hop = lambda v: op.hop(v, block)  # noqa: E731
    for _ in range(NCY):
        for colour in range(2):
            rho = (eta - op.m(psi)) * (col == colour)
            rho_o = rho * ~even
            r = (rho + KAPPA * hop(op.clover(rho_o, ainv))) * even
            xe = torch.zeros_like(r)
            for _ in range(NMR):
                p = op.clover(r) - KAPPA ** 2 * hop(op.clover(hop(r) * ~even, ainv) * ~even) * even
                pr, pp = _block_dot(p, r, op.dims, block), _block_dot(p, p, op.dims, block)
                alpha = torch.where(pp.real > 0, pr / pp.real.clamp_min(1e-300), torch.zeros_like(pr))
                xe = xe + alpha * r
                r = r - alpha * p
            psi = psi + xe + op.clover((rho_o + KAPPA * hop(xe)) * ~even, ainv) * ~even
    return psi


def _solve(apply, b, tol=1e-13, most=400):
    """BiCGStab on every right-hand side at once."""
    dot = lambda p, q: (p.conj() * q).flatten(1).sum(1).reshape(-1, *[1] * (p.dim() - 1))  # noqa: E731
    bn = dot(b, b).real.sqrt().clamp_min(1e-300)
    x = torch.zeros_like(b)
    for _ in range(4):
        r = b - apply(x)
        if float((dot(r, r).real.sqrt() / bn).max()) <= tol:
            break
        r0, p = r.clone(), r.clone()
        rho = dot(r0, r)
        for _ in range(most):
            v = apply(p)
            alpha = rho / dot(r0, v)
            s = r - alpha * v
            t = apply(s)
            omega = dot(t, s) / dot(t, t)
            x = x + alpha * p + omega * s
            r = s - omega * t
            if float((dot(r, r).real.sqrt() / bn).max()) <= 0.3 * tol:
                break
            new = dot(r0, r)
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
    return x


def _eps():
    return [((a, b, c), (1.0 if (a, b, c) in ((0, 1, 2), (1, 2, 0), (2, 0, 1)) else -1.0))
            for a in range(3) for b in range(3) for c in range(3) if len({a, b, c}) == 3]


def _spin_mul(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _nucleon(u1, u2, d):
    """C(x) [S, 4, 4] of [S, 4, 3, 4, 3] lines (sink spin, sink colour, source
    spin, source colour); both u lines in both of their places."""
    g = _gammas()
    gam = (g[0] @ g[2] @ torch.diag(torch.tensor([1, 1, -1, -1], dtype=torch.complex128))).cuda()
    q = torch.einsum("ij,sjakb,kl->siabl", gam, d.contiguous(), gam)     # [S, i, b, b', l]
    out = 0
    for (a, b, c), e1 in _eps():
        for (ap, bp, cp), e2 in _eps():
            qb = q[:, :, b, bp, :]
            tr = (qb * u1[:, :, a, :, ap]).sum((1, 2))
            out = out + e1 * e2 * u2[:, :, c, :, cp] * tr[:, None, None]
            out = out - e1 * e2 * _spin_mul(_spin_mul(u1[:, :, c, :, ap], qb.transpose(1, 2)), u2[:, :, a, :, cp])
    return out


def _contract(case, seed, gen):
    dims = _ints(case["dims"])
    T, V = dims[0], math.prod(dims)
    L = V // T
    prop = _propagator(dims, seed, _io(case), gen)
    seq = _propagator(dims, seed + 1, _io(case), gen)
    t0 = _site(dims, seed)[0]
    # [12 = (source spin, colour), T, L, spin, colour] -> per timeslice [L, spin, colour, source spin, source colour]
    lines = lambda p, t: p.reshape(4, 3, T, L, 4, 3)[:, :, t].permute(2, 3, 4, 0, 1).to(torch.complex128)  # noqa: E731
    proj = torch.tensor(P_PLUS, dtype=torch.complex128, device="cuda")
    gop = torch.tensor(GAMMA_OP, dtype=torch.complex128, device="cuda")
    g5 = torch.tensor([1, 1, -1, -1], dtype=torch.float64, device="cuda")
    c2 = torch.zeros((T, 4, 4), dtype=torch.complex128, device="cuda")
    c3 = torch.zeros(T, dtype=torch.complex128, device="cuda")
    for t in range(T):
        s, q = lines(prop, t), lines(seq, t)
        c2[(t - t0) % T] = _nucleon(s, s, s).sum(0)
        w = torch.einsum("ab,sbcde->sacde", gop, s.contiguous())
        c3[(t - t0) % T] = ((q * g5[:, None, None, None]).conj() * w).sum()
    out = {"c2": c2, "c3": c3}
    sink = (t0 + T // 4) % T
    for flavour in ("u", "d"):
        # the derivative of Re tr(P C) by a line's entries is the conjugate of
        # that of tr(P C), as torch gives it
        s = lines(prop, sink).clone()
        u, d = s.clone().requires_grad_(flavour == "u"), s.clone().requires_grad_(flavour == "d")
        loss = (proj.t() * _nucleon(u, u, d).sum(0)).sum().real
        k, = torch.autograd.grad(loss, u if flavour == "u" else d)
        eta = torch.zeros((4, 3, T, L, 4, 3), dtype=torch.complex128, device="cuda")
        eta[:, :, sink] = (g5[:, None, None, None] * k).permute(3, 4, 0, 1, 2)
        out[flavour] = eta.reshape(12, V, 4, 3)
    return out


def _project(w):
    """Onto SU(3): the unitary polar factor over a cube root of its determinant."""
    def cof(m):
        rows = [torch.linalg.cross(m[..., (r + 1) % 3, :], m[..., (r + 2) % 3, :], dim=-1) for r in range(3)]
        return torch.stack(rows, -2)
    for _ in range(14):
        c = cof(w)
        det = (w[..., 0, :] * c[..., 0, :]).sum(-1)[..., None, None]
        w = 0.5 * (w + (c / det).conj())
    det = (w[..., 0, :] * cof(w)[..., 0, :]).sum(-1)[..., None, None]
    return w * torch.exp(-1j * torch.angle(det) / 3)


def _ape(u, iters):
    """u: three lists entry [T, X, Y, Z, 3, 3] of the spatial directions 1..3."""
    dag = lambda m: m.conj().transpose(-1, -2)  # noqa: E731
    for _ in range(iters):
        new = []
        for i in range(3):
            acc = (1 - APE_ALPHA) * u[i]
            for j in range(3):
                if j == i:
                    continue
                up = _mul(_mul(u[j], torch.roll(u[i], -1, j + 1)), dag(torch.roll(u[j], -1, i + 1)))
                dn = _mul(_mul(dag(u[j]), u[i]), torch.roll(u[j], -1, i + 1))
                acc = acc + 0.25 * APE_ALPHA * (up + torch.roll(dn, 1, j + 1))
            new.append(_project(acc))
        u = new
    return u


def exact(case, seed):
    dims, block, kind = _ints(case["dims"]), _ints(case["block"]), case["kind"]
    V = math.prod(dims)
    n = 12 * case["positions"] + 12 if kind == "ama" else case.get("n", 1)
    # what stays within some seconds and a few tens of GB
    if {"dirac": V * n > 6e7, "sap": V * n > 4e6, "gcr": V * n > 8e5, "ama": V * n > 1e6}.get(kind, False):
        return None
    gen = _gen(seed)
    links = _links(dims, gen)
    full = lambda v: v.reshape(-1, *dims, 4, 3).to(torch.complex128)  # noqa: E731
    if kind == "ape":
        u = _ape([links.reshape(*dims, 4, 3, 3)[..., i + 1, :, :] for i in range(3)], case["iters"])
        return torch.stack(u, -3).reshape(V, 3, 3, 3)
    if kind == "contract":
        return _contract(case, seed, gen)
    if kind == "gauss":
        u = _ape([links.reshape(*dims, 4, 3, 3)[..., i + 1, :, :] for i in range(3)], 2)
        v = full(_cnormal((n, V, 4, 3), _io(case), gen))
        for _ in range(case["iters"]):
            h = torch.zeros_like(v)
            for i in range(3):
                w = torch.roll(v, -1, i + 2)
                h += sum(u[i][..., None, :, b] * w[..., b:b + 1] for b in range(3))
                w = sum(u[i].conj()[..., None, b, :] * v[..., b:b + 1] for b in range(3))
                h += torch.roll(w, 1, i + 2)
            v = (v + GAUSS_KAPPA * h) / (1 + 6 * GAUSS_KAPPA)
        return v.reshape(n, V, 4, 3)
    op = _Wilson(dims, links)
    if kind in ("dirac", "sap"):
        v = _cnormal((n, V, 4, 3), _io(case), gen)
        if kind == "dirac":
            return torch.cat([op.m(full(v[r:r + 4])) for r in range(0, n, 4)]).reshape(n, V, 4, 3)
        return torch.cat([_sap(op, full(v[r:r + 4]), block) for r in range(0, n, 4)]).reshape(n, V, 4, 3)
    if kind == "lowmode":
        p = _phi(case, links, gen)
        v = full(_sources(case, seed, gen))
        nb, ns = p.shape[0], p.shape[1]
        pf = p.reshape(nb, ns, -1)
        down = lambda w: torch.bmm(pf.conj().resolve_conj(),  # noqa: E731
                                   _to_blocks(w, dims, block).reshape(nb, w.shape[0], -1).transpose(1, 2).contiguous())
        up = lambda c: _from_blocks(torch.bmm(c.transpose(1, 2).contiguous(), pf).reshape(nb, -1, pf.shape[2] // 12, 4, 3),  # noqa: E731,E501
                                    dims, block)
        little = lambda c: down(op.m(up(c.permute(1, 2, 0).contiguous()))).permute(2, 0, 1)  # noqa: E731
        c = _solve(little, down(v).permute(2, 0, 1).contiguous())
        return up(c.permute(1, 2, 0).contiguous()).reshape(n, V, 4, 3)
    if kind == "gcr":
        return _solve(op.m, full(_sources(case, seed, gen))).reshape(n, V, 4, 3)
    sols = []
    for t, x, y, z in _positions(case, seed):
        b = torch.zeros((12, V, 12), dtype=torch.complex128, device="cuda")
        b[range(12), z + dims[3] * (y + dims[2] * (x + dims[1] * t)), range(12)] = 1
        sols.append(_solve(op.m, full(b)).reshape(12, V, 4, 3))
    return {"sloppy": sols, "exact": [sols[0]]}
