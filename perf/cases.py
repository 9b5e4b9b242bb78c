"""The calls whose speed this library is judged by: what a lattice program has it do, through
the public entry points of paper_1210_7398_amd.sapq, from the smallest test lattice to the
32^3x64 one, in every storage precision and with every block solver.

A case is a dict: `kind` names the entry point, `L`, `block`, `sub` are extents as "x,y,z,t"
(sub "0,0,0,0" is the even-odd site order), `prec` the storage precision, `bct` the fermion
boundary sign in t.  Gauge fields are exp(i eps H) with Gaussian H (eps 0.25, plaquette about
0.85), clover fields and sources are made from them as the library's own workloads make theirs,
all on the GPU and from the seed alone.

Results that the library computes in its inner storage precision come back as complex128 (the
interchange layout); a program that keeps them keeps what they hold, so `run` hands them on in
that type (complex64, float16 or bfloat16 pairs: exact, every value is representable there).

`exact` computes the same results in 64 bits with torch alone: the operator, the SSOR and the
minimal-residual block solves, the SAP recurrence, the network and its gradients, and D^-1 b.
"""
import math

import torch

from paper_1210_7398_amd import sapq

KAPPA = {8: 0.120}  # hopping parameter on the smallest lattice; 0.125 elsewhere
EPS, CSW = 0.25, 1.0
N_SSOR, N_SAP = 4, 4  # the library's defaults
NN_SHAPES = [(1, 8), (8, 8), (8, 1)]  # (channels in, channels out) of the network's layers
BITS = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}


# ------------------------------------------------------------------ the cases
def listed():
    c = dict
    return [
        # the operator alone, FP64: residual checks and measurement code call it, on the smallest
        # lattice (latency) and on the lattice of the headline solve
        c(name="dslash_fp64_8^4", kind="dslash", L="8,8,8,8", block="4,4,4,4", sub="2,2,2,2", prec="fp64", bct=1),
        c(name="dslash_fp64_24^3x48", kind="dslash", L="24,24,24,48", block="6,6,6,12", sub="3,3,3,6", prec="fp64", bct=1),
        # the operator in a storage precision, on the largest lattice
        c(name="dslash_fp16_32^3x64", kind="dslash", L="32,32,32,64", block="4,4,4,4", sub="0,0,0,0", prec="fp16", bct=1),
        # the SAP preconditioner inside a program's own Krylov solver: the headline's blocks (split
        # over two workgroups), the batched workload's (4^4, even-odd order, FP16), and a ragged
        # lattice with odd sub-blocks and an antiperiodic boundary in BF16
        c(name="msap_fp32_24^3x48", kind="msap", L="24,24,24,48", block="6,6,6,12", sub="3,3,3,6", prec="fp32", bct=1),
        c(name="msap_fp16_32^3x64", kind="msap", L="32,32,32,64", block="4,4,4,4", sub="0,0,0,0", prec="fp16", bct=1),
        c(name="msap_bf16_ragged", kind="msap", L="12,8,20,36", block="6,4,10,6", sub="3,2,5,3", prec="bf16", bct=-1),
        # the same with the even-odd minimal-residual block solve
        c(name="msap_eomr_24^3x48", kind="eomr", L="24,24,24,48", block="6,6,6,6", sub="0,0,0,0", prec="fp32", bct=1),
        # whole solves to 1e-10: the smallest lattice, the headline
        c(name="solve_8^4", kind="solve", L="8,8,8,8", block="4,4,4,4", sub="2,2,2,2", prec="fp32", bct=1, tol=1e-10),
        c(name="solve_24^3x48", kind="solve", L="24,24,24,48", block="6,6,6,12", sub="3,3,3,6", prec="fp32", bct=1, tol=1e-10),
        # several sources of two fields of different size in one call, FP16 storage
        c(name="batch_16^3x32", kind="batch", L="16,16,16,32", L2="8,8,8,16", nrhs=6, block="4,4,4,4", sub="0,0,0,0",
          prec="fp16", bct=1, tol=1e-11),
        # the learned stage: the gradient a training loop takes (forward, weight and input
        # gradients) on the training lattice, and the preconditioner with the trained network
        c(name="nn_backward_16^3x32", kind="nn_grad", L="16,16,16,32", block="4,4,4,4", sub="0,0,0,0", prec="fp32", bct=1),
        c(name="nn_precond_24^3x48", kind="nn_precond", L="24,24,24,48", block="4,4,4,4", sub="0,0,0,0", prec="fp16", bct=1),
    ]


# block and sub-block shapes that programs use: the paper's and the workloads' own, the even-odd
# order, odd extents, unequal extents, and blocks too large for one workgroup's LDS
_SHAPES = [((4, 4, 4, 4), (2, 2, 2, 2)), ((4, 4, 4, 4), (0, 0, 0, 0)), ((6, 6, 6, 6), (3, 3, 3, 3)),
           ((6, 6, 6, 12), (3, 3, 3, 6)), ((6, 4, 10, 6), (3, 2, 5, 3)), ((5, 4, 3, 6), (0, 0, 0, 0)),
           ((4, 6, 8, 4), (2, 3, 4, 2)), ((8, 8, 8, 4), (4, 4, 4, 2)), ((4, 2, 2, 4), (2, 2, 2, 2))]
_EO_SHAPES = [((4, 4, 4, 4), (0, 0, 0, 0)), ((6, 6, 6, 6), (0, 0, 0, 0)), ((4, 6, 4, 8), (0, 0, 0, 0)),
              ((5, 4, 3, 6), (0, 0, 0, 0))]
_VMAX = {"dslash": 2 << 20, "msap": 900000, "eomr": 600000, "solve": 300000, "batch": 140000, "nn_grad": 140000,
         "nn_precond": 600000}


def _lattice(rng, block, target):
    """A lattice of an even number of blocks per direction with about `target` sites, at most that many
    (or two blocks per direction)."""
    nb = [2, 2, 2, 2]
    while True:
        m = rng.randrange(4)
        nb[m] += 2
        if math.prod(n * b for n, b in zip(nb, block)) > target:
            nb[m] -= 2
            return tuple(n * b for n, b in zip(nb, block))


def _txt(e):
    return ",".join(str(v) for v in e)


def draw(rng):
    kind = rng.choice(["dslash", "dslash", "msap", "msap", "msap", "eomr", "solve", "solve", "batch", "nn_grad", "nn_precond"])
    if kind in ("eomr", "batch"):
        block, sub = rng.choice(_EO_SHAPES)
    else:
        block, sub = rng.choice(_SHAPES)
    target = int(math.exp(rng.uniform(math.log(4096), math.log(_VMAX[kind]))))
    case = dict(kind=kind, L=_txt(_lattice(rng, block, target)), block=_txt(block), sub=_txt(sub),
                prec=rng.choice(["fp32", "fp16", "bf16"]), bct=rng.choice([1, -1]))
    if kind == "dslash" and rng.random() < 0.5:
        case["prec"] = "fp64"
    if kind == "nn_grad":
        case["prec"] = "fp32"
    if kind in ("solve", "batch"):
        case["prec"] = rng.choice(["fp32", "fp16"])
        case["tol"] = 1e-11
    if kind == "batch":
        case["nrhs"] = rng.randint(1, 6)
        case["L2"] = _txt(_lattice(rng, block, max(4096, target // 8)))
    return case


def _ext(t):
    return tuple(int(v) for v in t.split(","))


def _kappa(L):
    return KAPPA.get(max(L), 0.125)


# ------------------------------------------------------------------ inputs
def _mm(a, b):
    """Products of small matrices, by components (batched 3x3 library products are slow)."""
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _dag(a):
    return a.conj().transpose(-1, -2)


def _links(L, gen):
    """U = exp(i eps sum_a h_a lambda_a / 2), projected onto SU(3) to rounding; [V, 4, 3, 3]."""
    V = math.prod(L)
    h = torch.randn((V, 4, 8), generator=gen, device="cuda", dtype=torch.float64) * (0.5 * EPS)
    H = torch.zeros((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
    d8 = h[..., 7] / math.sqrt(3.0)
    H[..., 0, 0] = h[..., 2] + d8
    H[..., 1, 1] = -h[..., 2] + d8
    H[..., 2, 2] = -2 * d8
    for (a, b), k in (((0, 1), 0), ((0, 2), 3), ((1, 2), 5)):
        off = torch.complex(h[..., k], -h[..., k + 1])
        H[..., a, b] = off
        H[..., b, a] = off.conj()
    X = 1j * H / 16
    E = torch.eye(3, dtype=torch.complex128, device="cuda") + X
    term = X
    for k in range(2, 9):  # |X| < 0.1: the Taylor series to order 8, then 4 squarings
        term = _mm(term, X) / k
        E = E + term
    for _ in range(4):
        E = _mm(E, E)
    r0 = E[..., 0, :]
    r0 = r0 / torch.linalg.vector_norm(r0, dim=-1, keepdim=True)
    r1 = E[..., 1, :]
    r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    r2 = torch.linalg.cross(r0, r1).conj()
    return torch.stack([r0, r1, r2], dim=-2).contiguous()


def _gammas():
    s = torch.tensor([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=torch.complex128)
    g = torch.zeros((4, 4, 4), dtype=torch.complex128)
    for k in range(3):
        g[k, :2, 2:] = -1j * s[k]
        g[k, 2:, :2] = 1j * s[k]
    g[3, :2, 2:] = torch.eye(2)
    g[3, 2:, :2] = torch.eye(2)
    return g.cuda()


def _clover_inverse(L, U, kappa):
    """F = (1 - c_SW kappa sum_{mu<nu} sigma_mu_nu F_mu_nu)^-1 from the four-leaf clover, [V, 2, 6, 6]."""
    V, g = U.shape[0], _gammas()
    lat = tuple(reversed(L))
    A = torch.zeros((V, 2, 6, 12), dtype=torch.complex128, device="cuda")
    A[..., :6] = torch.eye(6, device="cuda")
    A[..., 6:] = torch.eye(6, device="cuda")

    def at(f, *steps):  # f(n + steps)
        f = f.reshape(lat + (3, 3))
        for m, k in steps:
            f = torch.roll(f, -k, dims=3 - m)
        return f.reshape(V, 3, 3)

    for mu in range(4):
        for nu in range(mu + 1, 4):
            a, b = U[:, mu], U[:, nu]
            am, bm = at(a, (mu, -1)), at(b, (mu, -1))
            an, bn = at(a, (nu, -1)), at(b, (nu, -1))
            Q = _mm(_mm(a, at(b, (mu, 1))), _mm(_dag(at(a, (nu, 1))), _dag(b)))
            Q += _mm(_mm(b, _dag(at(a, (mu, -1), (nu, 1)))), _mm(_dag(bm), am))
            Q += _mm(_mm(_dag(am), _dag(at(b, (mu, -1), (nu, -1)))), _mm(at(a, (mu, -1), (nu, -1)), bn))
            Q += _mm(_mm(_dag(bn), an), _mm(at(b, (mu, 1), (nu, -1)), _dag(a)))
            Fmn = (Q - _dag(Q)) / 8j
            Fmn = Fmn - (Fmn.diagonal(dim1=1, dim2=2).sum(-1) / 3.0)[:, None, None] * torch.eye(3, device="cuda")
            sig = 0.5j * (g[mu] @ g[nu] - g[nu] @ g[mu])
            for k in range(2):
                sk = sig[2 * k:2 * k + 2, 2 * k:2 * k + 2]
                A[:, k, :, :6] -= (CSW * kappa * sk[None, :, None, :, None] * Fmn[:, None, :, None, :]).reshape(V, 6, 6)
    for k in range(6):  # Gauss-Jordan; the pivots stay near 1
        A[..., k, :] = A[..., k, :] / A[..., k, k:k + 1]
        f = A[..., :, k:k + 1].clone()
        f[..., k, :] = 0
        A -= f * A[..., k:k + 1, :]
    return A[..., 6:].contiguous()


def _spinor(V, gen, n=None):
    shape = (V, 4, 3, 2) if n is None else (n, V, 4, 3, 2)
    return torch.view_as_complex(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64))


def _weights(gen):
    """Network weights, exactly representable in BF16 (the layers use them so rounded): small random
    numbers and a local term near the identity, as a training run starts from."""
    out = []
    for ci, co in NN_SHAPES:
        w = 0.02 * torch.randn((9, co, ci, 4, 4, 2), generator=gen, device="cuda", dtype=torch.float64)
        for c in range(min(ci, co)):
            w[0, c, c, :, :, 0] += torch.eye(4, device="cuda") * (1.0 / math.sqrt(8.0) if ci != co else 1.0)
        out.append(w.reshape(-1))
    return torch.cat(out).to(torch.bfloat16).to(torch.float32)


def _inputs(case, seed):
    """Everything the case is made of, from the seed alone: per lattice the links, the inverse
    clover field and the vectors; the network's weights."""
    gen = torch.Generator(device="cuda").manual_seed(1000003 * (seed + 1))
    kind, got = case["kind"], {"fields": []}
    for key in ("L", "L2") if kind == "batch" else ("L",):
        L = _ext(case[key])
        V, U = math.prod(L), _links(L, gen)
        F = _clover_inverse(L, U, _kappa(L))
        vec = _spinor(V, gen, case["nrhs"]) if kind == "batch" else _spinor(V, gen)
        got["fields"].append((L, U, F, vec))
    if kind in ("nn_grad", "nn_precond"):
        got["w"] = _weights(gen)
    if kind == "nn_grad":
        got["grad_out"] = _spinor(V, gen)
    return got


def prepare(case, seed):
    inp, kind = _inputs(case, seed), case["kind"]
    state = {"case": case, "solvers": [], "vecs": []}
    for L, U, F, vec in inp["fields"]:
        s = sapq.Solver(L, _ext(case["block"]), _ext(case["sub"]), _kappa(L), bc=(1, 1, 1, case["bct"]),
                        prec="fp32" if case["prec"] == "fp64" else case["prec"], nn=kind in ("nn_grad", "nn_precond"),
                        outer="defect" if kind == "batch" else "fbicgstab",
                        block_solver="eomr" if kind == "eomr" else "ssor")
        s.load_gauge(U)
        s.load_clover(F)
        state["solvers"].append(s)
        state["vecs"].append(vec)
    if "w" in inp:
        state["solvers"][0].nn_set_weights(inp["w"])
    if "grad_out" in inp:
        state["grad_out"] = inp["grad_out"]
    return state


def _kept(x, prec):
    """A result in the type of the values it holds."""
    if prec == "fp64":
        return x
    if prec == "fp32":
        return x.to(torch.complex64)
    return torch.view_as_real(x).to(torch.float16 if prec == "fp16" else torch.bfloat16)


def run(state):
    case, s, v = state["case"], state["solvers"][0], state["vecs"][0]
    kind, prec = case["kind"], case["prec"]
    if kind == "dslash":
        return _kept(s.dslash(v, prec), prec)
    if kind in ("msap", "eomr"):
        y, dy = s.sap_precondition(v)
        return _kept(y, prec), _kept(dy, prec)
    if kind == "solve":
        return s.solve(v, tol=case["tol"])[0]
    if kind == "batch":
        return sapq.solve_batch(state["solvers"], state["vecs"], tol=case["tol"])[0]
    if kind == "nn_grad":
        gw, gin = s.nn_backward(state["grad_out"], v)
        return gw, _kept(gin, "fp32")
    y, dy = s.precondition(v)
    return _kept(y, prec), _kept(dy, prec)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    L, kind, b = _ext(case["L"]), case["kind"], BITS[case["prec"]]
    V = math.prod(L)
    fields = V * b * (48 + 72)         # two rows of 4 links, the hermitian clover blocks
    vec = V * 24 * 8                   # a spinor field in the interchange layout
    kept = V * 24 * b                  # the same in the type of its values
    d_flops = V * 1944                 # one application of D
    msap = N_SAP * (2 * N_SSOR + 2) * d_flops
    nn_w = 2 * 4 * sum(9 * ci * co * 16 for ci, co in NN_SHAPES)
    nn_mm = 3 * 8 * 16 * 9 * sum(ci * co for ci, co in NN_SHAPES)  # per site: spin matrices on 3 colours
    nn_tr = 8 * 4 * 66 * sum(ci for ci, _ in NN_SHAPES)            # per site: link times colour vector
    if kind == "dslash":
        return {"bytes": vec + kept + fields, "flops": d_flops}
    if kind in ("msap", "eomr"):
        return {"bytes": vec + 2 * kept + fields, "flops": msap}
    if kind == "solve":  # about 12 applications of the preconditioner and 9 of the FP64 operator
        return {"bytes": 2 * vec + fields + V * 8 * 120, "flops": 12 * msap + 9 * d_flops}
    if kind == "batch":  # about 16 inner iterations' worth of preconditioner applications per source
        V2 = V + math.prod(_ext(case["L2"]))
        n = case["nrhs"]
        return {"bytes": V2 * (2 * n * 24 * 8 + 120 * (8 + b)), "flops": n * 16 * V2 * 1944 * N_SAP * (2 * N_SSOR + 2)}
    links = V * 4 * 48
    if kind == "nn_grad":  # forward, adjoint and weight gradient each contract and transport once
        return {"bytes": 2 * vec + kept + links + 2 * nn_w, "flops": 3 * V * (nn_mm + nn_tr)}
    return {"bytes": vec + 2 * kept + fields + nn_w, "flops": V * (nn_mm + nn_tr) + d_flops + msap}


# ------------------------------------------------------------------ the same in 64 bits, with torch alone
class _Lattice:
    """D, its parts inside the blocks, and the site orders, on complex128 fields [V, 4, 3]."""

    def __init__(self, L, U, F, kappa, block, sub, bct):
        self.V, self.U, self.F, self.kappa = math.prod(L), U, F, kappa
        n = torch.arange(self.V, device="cuda")
        c, stride, rest = [], [], n
        for m in range(4):
            c.append(rest % L[m])
            stride.append(math.prod(L[:m]))
            rest = rest // L[m]
        self.fwd = [n + torch.where(c[m] == L[m] - 1, -(L[m] - 1), 1) * stride[m] for m in range(4)]
        self.bwd = [n + torch.where(c[m] == 0, L[m] - 1, -1) * stride[m] for m in range(4)]
        one = torch.ones(self.V, dtype=torch.float64, device="cuda")
        self.pf = [torch.where(c[m] == L[m] - 1, float(bct), 1.0) if m == 3 else one for m in range(4)]
        self.pb = [torch.where(c[m] == 0, float(bct), 1.0) if m == 3 else one for m in range(4)]
        self.in_f = [c[m] % block[m] != block[m] - 1 for m in range(4)]
        self.in_b = [c[m] % block[m] != 0 for m in range(4)]
        self.colour = sum(c[m] // block[m] for m in range(4)) % 2
        nbk = [L[m] // block[m] for m in range(4)]
        self.blk = sum((c[m] // block[m]) * math.prod(nbk[:m]) for m in range(4))
        self.nblk = math.prod(nbk)
        if max(sub) == 0:
            self.plane = sum(c[m] % block[m] for m in range(4)) % 2
        else:
            self.plane = sum((c[m] % block[m]) % sub[m] for m in range(4))
        g = _gammas()
        eye = torch.eye(4, dtype=torch.complex128, device="cuda")
        self.Pf = [(eye - g[m])[None] for m in range(4)]
        self.Pb = [(eye + g[m])[None] for m in range(4)]

    def hop(self, x, sites=None, where="all"):
        """(H x) on `sites` (all): every hop, only those inside the block, or only those leaving it."""
        pick = (lambda t: t) if sites is None else (lambda t: t[sites])
        acc = 0
        for m in range(4):
            for nb, ph, ins, P, back in ((self.fwd[m], self.pf[m], self.in_f[m], self.Pf[m], False),
                                         (self.bwd[m], self.pb[m], self.in_b[m], self.Pb[m], True)):
                j, wt = pick(nb), pick(ph)
                if where == "in":
                    wt = wt * pick(ins)
                elif where == "out":
                    wt = wt * ~pick(ins)
                psi = x[j] * wt[:, None, None]
                u = _dag(self.U[j, m]) if back else pick(self.U[:, m])
                t = (u[:, None, :, :] * psi[:, :, None, :]).sum(-1)
                acc = acc + (P[:, :, :, None] * t[:, None, :, :]).sum(2)
        return acc

    def clover(self, h, sites=None):
        F = self.F if sites is None else self.F[sites]
        h = h.reshape(-1, 2, 6)
        return (F * h[:, :, None, :]).sum(-1).reshape(-1, 4, 3)

    def D(self, x):
        return x - self.kappa * self.clover(self.hop(x))

    def K(self, x, sites, where="in"):
        return self.kappa * self.clover(self.hop(x, sites, where), sites)

    def block_solve(self, v, colour, mr):
        x = torch.zeros_like(v)
        mine = self.colour == colour
        planes = [(mine & (self.plane == h)).nonzero()[:, 0] for h in range(int(self.plane.max()) + 1)]
        if not mr:
            for k in range(2 * N_SSOR):
                for s in planes if k % 2 == 0 else reversed(planes):
                    x[s] = v[s] + self.K(x, s)
            return x
        ev, od = planes
        t = torch.zeros_like(v)
        t[od] = v[od]
        r, xe = v[ev] + self.K(t, ev), torch.zeros_like(v[ev])
        blk = self.blk[ev]

        def total(f):  # per block
            f = f.sum((1, 2))
            z = torch.zeros(self.nblk, dtype=f.dtype, device="cuda").index_add_(0, blk, f)
            return z[blk][:, None, None]

        for _ in range(2 * N_SSOR):
            t = torch.zeros_like(v)
            t[ev] = r
            t[od] = self.K(t, od)
            p = r - self.K(t, ev)
            al = total(p.conj() * r) / total(p.abs().square())
            xe, r = xe + al * r, r - al * p
        x[ev] = xe
        x[od] = v[od] + self.K(x, od)
        return x

    def msap(self, v, mr=False):
        """(M v, D M v): N_SAP cycles of r <- r - D K r with K of Algorithm 1."""
        r, y = v, torch.zeros_like(v)
        for _ in range(N_SAP):
            x = self.block_solve(r, 0, mr)
            odd = (self.colour == 1).nonzero()[:, 0]
            w = r.clone()
            w[odd] = r[odd] + self.K(x, odd, "out")
            x = x + self.block_solve(w, 1, mr)
            y, r = y + x, r - self.D(x)
        return y, v - r

    def solve(self, b, tol=2e-13):
        """D^-1 b by BiCGStab."""
        dot = lambda p, q: (p.conj() * q).sum()  # noqa: E731
        x, r = torch.zeros_like(b), b.clone()
        r0, rho, p = r.clone(), dot(r, r), r.clone()
        goal = tol * b.norm()
        for _ in range(1000):
            v = self.D(p)
            al = rho / dot(r0, v)
            s = r - al * v
            t = self.D(s)
            om = dot(t, s) / dot(t, t)
            x = x + al * p + om * s
            r = s - om * t
            if r.norm() <= goal:
                return x
            new = dot(r0, r)
            p = r + (new / rho) * (al / om) * (p - om * v)
            rho = new
        raise RuntimeError("the reference solve did not converge")

    def network(self, w, x):
        """The three parallel-transport layers on x [V, 4, 3]; w: list of complex [9, co, ci, 4, 4]."""
        a = x[:, None]
        for W in w:
            out = 0
            for d in range(9):
                if d == 0:
                    t = a
                else:
                    m, back = (d - 1) // 2, (d - 1) % 2
                    j, ph = (self.bwd[m], self.pb[m]) if back else (self.fwd[m], self.pf[m])
                    u = _dag(self.U[j, m]) if back else self.U[:, m]
                    psi = a[j] * ph[:, None, None, None]
                    t = sum(u[:, None, None, :, k] * psi[:, :, :, k, None] for k in range(3))
                n, ci = t.shape[0], t.shape[1]
                M = W[d].permute(0, 2, 1, 3).reshape(W.shape[1] * 4, ci * 4)
                cols = t.permute(1, 2, 0, 3).reshape(ci * 4, n * 3)
                out = out + (M @ cols).reshape(W.shape[1], 4, n, 3).permute(2, 0, 1, 3)
            a = out
        return a[:, 0]


def _layers(w):
    out, at = [], 0
    for ci, co in NN_SHAPES:
        n = 9 * co * ci * 16 * 2
        out.append(torch.view_as_complex(w[at:at + n].double().reshape(9, co, ci, 4, 4, 2).contiguous()))
        at += n
    return out


def exact(case, seed):
    inp, kind, prec = _inputs(case, seed), case["kind"], case["prec"]
    lats = [_Lattice(L, U, F, _kappa(L), _ext(case["block"]), _ext(case["sub"]), case["bct"])
            for L, U, F, _ in inp["fields"]]
    lat, v = lats[0], inp["fields"][0][3]
    pairs = (lambda x: x) if prec in ("fp64", "fp32") else torch.view_as_real
    if kind == "dslash":
        return pairs(lat.D(v))
    if kind in ("msap", "eomr"):
        y, dy = lat.msap(v, kind == "eomr")
        return pairs(y), pairs(dy)
    if kind == "solve":
        return lat.solve(v)
    if kind == "batch":
        return [torch.stack([la.solve(b) for b in f[3]]) for la, f in zip(lats, inp["fields"])]
    if kind == "nn_grad":
        with torch.enable_grad():
            w, x = [W.requires_grad_() for W in _layers(inp["w"])], v.clone().requires_grad_()
            lat.network(w, x).backward(inp["grad_out"])
        return torch.cat([torch.view_as_real(W.grad).reshape(-1) for W in w]), x.grad
    z = lat.network(_layers(inp["w"]), v)
    y, dy = lat.msap(v - lat.D(z))
    return pairs(z + y), pairs(lat.D(z) + dy)
