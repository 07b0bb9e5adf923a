"""The workloads by which this framework's speed is judged: single calls of its public entry
points (``Process.sigma``, ``select``, ``sigma_channel``, ``sigma_alphas`` and ``sigma`` with
per-helicity output) on batches of phase-space points resident in device memory, as an event
generator or an integrator issues them.

A case names the process, the precision, the call and the number of events.  The points are
RAMBO points made here in torch from the seed alone; ``exact`` evaluates the same matrix elements
in 64 bits by colour-ordered off-shell recursion written in torch, or in closed form for
e+e- -> mu+mu-.
"""
import itertools
import math

import numpy as np
import torch

M_TOP, ALPHA_EM, ALPHA_S = 173.0, 1.0 / 132.507, 0.118

# process -> (final-state masses, sqrt(s) in GeV, gluons)
PROCESSES = {
    "ee_mumu": ((0.0, 0.0), 500.0, 0),
    "gg_tt": ((M_TOP, M_TOP), 1500.0, 2),
    "gg_ttg": ((M_TOP, M_TOP, 0.0), 1500.0, 3),
    "gg_ttgg": ((M_TOP, M_TOP, 0.0, 0.0), 1500.0, 4),
    "gg_ttggg": ((M_TOP, M_TOP, 0.0, 0.0, 0.0), 1500.0, 5),
}
N_DIAGRAMS = {"gg_tt": 3, "gg_ttg": 16, "gg_ttgg": 123}
# Floating-point operations that one event cannot do without, roughly: off-shell currents shared
# by the helicities that have them in common, one contraction per (helicity, colour flow), and the
# colour sum.
FLOPS_PER_EVENT = {"ee_mumu": 6e2, "gg_tt": 5e3, "gg_ttg": 6e4, "gg_ttgg": 5e5, "gg_ttggg": 4.5e6}


def case(name, process, events, precision="fp64", call="sigma"):
    return {"name": name, "process": process, "events": events, "precision": precision, "call": call}


def listed():
    return [
        # a driver that asks for a handful of points at a time: launches and host time
        case("gg_tt small call", "gg_tt", 256),
        # the e+e- configuration of the paper, 8192 events at 500 GeV
        case("ee_mumu configured batch", "ee_mumu", 8192),
        # the same process in a large integration batch
        case("ee_mumu large batch", "ee_mumu", 1 << 20),
        # gg -> t t~ at its configured batch, the largest single integrator call
        case("gg_tt configured batch", "gg_tt", 1 << 19),
        # one more gluon, configured batch
        case("gg_ttg configured batch", "gg_ttg", 1 << 20),
        # multichannel integration: |M|^2 times the channel weight, a ragged batch
        case("gg_ttg channel weights", "gg_ttg", 100003, call="channel"),
        # the headline configuration
        case("gg_ttgg configured batch", "gg_ttgg", 1 << 19),
        # event generation: |M|^2 with a helicity and a colour flow drawn for every event
        case("gg_ttgg event generation", "gg_ttgg", 9973, call="select"),
        # the headline configuration in the reduced-precision form
        case("gg_ttgg mixed fp16", "gg_ttgg", 1 << 18, precision="mixed_fp16"),
        # the largest process: half of its configured batch, and one serving request
        case("gg_ttggg large batch", "gg_ttggg", 1 << 17),
        case("gg_ttggg request", "gg_ttggg", 1531),
        # the largest process in the other reduced-precision form
        case("gg_ttggg mixed bf16", "gg_ttggg", 8192, precision="mixed_bf16"),
    ]


# the largest batch of a drawn case: plain calls, and calls with further outputs per event
LARGEST = {"ee_mumu": 1 << 20, "gg_tt": 1 << 19, "gg_ttg": 1 << 20, "gg_ttgg": 1 << 19, "gg_ttggg": 1 << 16}


def draw(rng):
    process = rng.choice(["ee_mumu", "gg_tt", "gg_ttg", "gg_ttgg", "gg_ttgg", "gg_ttggg"])
    precision = rng.choice(["fp64", "fp64", "fp64", "fp64", "mixed_fp16", "mixed_bf16"])
    calls = ["sigma", "sigma", "sigma"]
    if process != "ee_mumu":
        calls += ["alphas", "select"]
    if process in N_DIAGRAMS:
        calls.append("channel")
    if process in ("gg_ttg", "gg_ttgg"):
        calls.append("hel")
    call = rng.choice(calls)
    top = LARGEST[process] if call in ("sigma", "alphas") else LARGEST[process] // 8
    events = int(round(math.exp(rng.uniform(math.log(32), math.log(top)))))
    return {"process": process, "events": min(top, events), "precision": precision, "call": call}


# ---------------------------------------------------------------------------------------------
# inputs

def points(process, n, seed):
    """n RAMBO phase-space points [n][particle][4] on the GPU, beams along +-z"""
    masses, rs, _ = PROCESSES[process]
    nf = len(masses)
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + n)
    r = torch.rand((4, n, nf), generator=g, dtype=torch.float64, device="cuda").clamp_(1e-15, 1 - 1e-15)
    c = 2 * r[0] - 1
    s, phi = torch.sqrt(1 - c * c), 2 * math.pi * r[1]
    e = -torch.log(r[2] * r[3])
    q = torch.stack([e, e * s * torch.cos(phi), e * s * torch.sin(phi), e * c], dim=-1)
    tot = q.sum(dim=1)
    M = torch.sqrt(tot[:, 0] ** 2 - (tot[:, 1:] ** 2).sum(-1))
    b = -tot[:, 1:] / M[:, None]
    gam = tot[:, 0] / M
    a = 1 / (1 + gam)
    bq = (b[:, None, :] * q[:, :, 1:]).sum(-1)
    k = q[:, :, 1:] + b[:, None, :] * (q[:, :, 0] + a[:, None] * bq)[..., None]
    k = k * (rs / M)[:, None, None]
    m2 = torch.tensor([m * m for m in masses], dtype=torch.float64, device="cuda")
    k2 = (k * k).sum(-1)
    if any(masses):
        xi = torch.full((n,), math.sqrt(1 - (sum(masses) / rs) ** 2), dtype=torch.float64, device="cuda")
        for _ in range(30):
            E = torch.sqrt(m2 + xi[:, None] ** 2 * k2)
            xi = xi - (E.sum(1) - rs) / (xi[:, None] * k2 / E).sum(1)
        k = k * xi[:, None, None]
        k2 = k2 * xi[:, None] ** 2
    x = torch.zeros((n, nf + 2, 4), dtype=torch.float64, device="cuda")
    x[:, 0, 0] = x[:, 1, 0] = x[:, 0, 3] = rs / 2
    x[:, 1, 3] = -rs / 2
    x[:, 2:, 0] = torch.sqrt(m2 + k2)
    x[:, 2:, 1:] = k
    return x


def extras(case, seed):
    """the further inputs of the call: uniforms, channel ids or strong couplings per event"""
    n = case["events"]
    g = torch.Generator(device="cuda")
    g.manual_seed(7919 * int(seed) + 13)
    u = torch.rand((2, n), generator=g, dtype=torch.float64, device="cuda")
    if case["call"] == "select":
        return [u[0].contiguous(), u[1].contiguous()]
    if case["call"] == "channel":
        return [(u[0] * N_DIAGRAMS[case["process"]]).to(torch.int32)]
    if case["call"] == "alphas":
        return [(0.08 + 0.06 * u[0]).contiguous()]
    return []


def prepare(case, seed):
    from paper_2210_11122_amd import Process
    p = Process(case["process"], m_top=M_TOP, alpha_em=ALPHA_EM, alpha_s=ALPHA_S, precision=case["precision"])
    return {"call": case["call"], "process": p, "x": points(case["process"], case["events"], seed),
            "more": extras(case, seed)}


def run(state):
    p, x, more = state["process"], state["x"], state["more"]
    if state["call"] == "sigma":
        return p.sigma(x)
    if state["call"] == "alphas":
        return p.sigma_alphas(x, more[0])
    if state["call"] == "channel":
        return p.sigma_channel(x, more[0])
    if state["call"] == "select":
        return p.select(x, more[0], more[1])
    return p.sigma(x, per_helicity=True)


def work(case):
    npar = len(PROCESSES[case["process"]][0]) + 2
    extra = {"sigma": 0, "alphas": 8, "channel": 4, "select": 24, "hel": 8 * 2 ** npar}[case["call"]]
    return {"bytes": case["events"] * (32 * npar + 8 + extra), "flops": case["events"] * FLOPS_PER_EVENT[case["process"]]}


# ---------------------------------------------------------------------------------------------
# the same matrix elements in 64 bits.  A wavefunction is a list of four tensors of shape
# [helicity of gluon 1] ... [helicity of gluon n][quark spin][antiquark spin][event], with extent 1
# along the axes it does not depend on.

def mdot(a, b):
    return a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3]


def add(a, b):
    return [x + y for x, y in zip(a, b)]


def times(f, a):
    return [f * x for x in a]


def slash_row(u, G):
    """ubar gamma.G in the chiral representation (row spinor)"""
    a, b, c, d = G[0] + G[3], G[0] - G[3], G[1] + 1j * G[2], G[1] - 1j * G[2]
    return [u[2] * a + u[3] * c, u[2] * d + u[3] * b, u[0] * b - u[1] * c, u[1] * a - u[0] * d]


def rdot(u, s):
    return u[0] * s[0] + u[1] * s[1] + u[2] * s[2] + u[3] * s[3]


def spinors(p, antiquark):
    """row spinors ubar(p, -), ubar(p, +), or columns v(p, -), v(p, +), stacked over the spin"""
    E, x, y, z = p
    pp = torch.sqrt(x * x + y * y + z * z)
    nrm = 1 / torch.sqrt(2 * pp * (pp + z))
    chi = {1: [(pp + z) * nrm + 0j, (x + 1j * y) * nrm], -1: [(-x + 1j * y) * nrm, (pp + z) * nrm + 0j]}
    w = {1: torch.sqrt(E + pp), -1: M_TOP / torch.sqrt(E + pp)}
    out = []
    for lam in (-1, 1):
        if antiquark:
            cs = chi[-lam]
            out.append([-lam * w[lam] * cs[0], -lam * w[lam] * cs[1], lam * w[-lam] * cs[0], lam * w[-lam] * cs[1]])
        else:
            cs = [t.conj() for t in chi[lam]]
            out.append([w[lam] * cs[0], w[lam] * cs[1], w[-lam] * cs[0], w[-lam] * cs[1]])
    return [torch.stack([out[0][i], out[1][i]]) for i in range(4)]


def polarisations(k):
    """polarisation vectors of both helicities (-, +) of a gluon, stacked"""
    E, x, y, z = k
    kt = torch.sqrt(x * x + y * y)
    ok = kt > 0
    safe = torch.where(ok, kt, torch.ones_like(kt))
    cp, sp = torch.where(ok, x / safe, torch.ones_like(x)), torch.where(ok, y / safe, torch.zeros_like(y))
    ct, st = z / E, kt / E
    out = []
    for lam in (-1, 1):
        out.append([0 * E + 0j, (-lam * ct * cp + 1j * sp) / math.sqrt(2), (-lam * ct * sp - 1j * cp) / math.sqrt(2),
                    lam * st / math.sqrt(2) + 0j])
    return [torch.stack([out[0][i], out[1][i]]) for i in range(4)]


def colour_matrix(n):
    """Tr(t^{s1} ... t^{sn} t^{r_n} ... t^{r_1}) for all orderings s, r, from the Gell-Mann matrices"""
    t = np.zeros((8, 3, 3), complex)
    for k, (i, j) in enumerate([(0, 1), (0, 2), (1, 2)]):
        t[2 * k, i, j] = t[2 * k, j, i] = 0.5
        t[2 * k + 1, i, j], t[2 * k + 1, j, i] = -0.5j, 0.5j
    t[6] = np.diag([0.5, -0.5, 0])
    t[7] = np.diag([1, 1, -2]) / (2 * math.sqrt(3))
    prod = t
    for _ in range(n - 1):
        prod = np.einsum("...ij,ajk->...aik", prod, t)
    perms = list(itertools.permutations(range(n)))
    base = np.conj(prod).reshape(-1)
    # axis a of the product with ordering r carries gluon r[a]: bring gluon g to axis g
    c = {r: float(np.real(np.dot(base, np.transpose(prod, [r.index(g) for g in range(n)] + [n, n + 1]).reshape(-1))))
         for r in perms}
    C = np.empty((len(perms),) * 2)
    for i, s in enumerate(perms):
        inv = [s.index(g) for g in range(n)]
        for j, r in enumerate(perms):
            C[i, j] = c[tuple(inv[g] for g in r)]
    return C


def helicity_squares(process, x, C):
    """[2^npar or (gluon helicities, spins) flattened in particle order][event]: colour-summed |M_h|^2"""
    ng = PROCESSES[process][2]
    N = x.shape[0]
    p = x.permute(1, 2, 0).contiguous()
    gpar = [0, 1] + list(range(4, ng + 2))
    kin = [p[i] if i < 2 else -p[i] for i in gpar]          # incoming gluon momenta
    gs = math.sqrt(4 * math.pi * ALPHA_S)
    naxes = ng + 2

    def place(w, axis):
        shape = [1] * naxes + [N]
        shape[axis] = 2
        return [t.reshape(shape) for t in w]

    cur, mom = {}, {}
    for i in range(ng):
        w = polarisations(p[gpar[i]])
        cur[(i,)] = place(w if gpar[i] < 2 else [t.conj() for t in w], i)
        mom[1 << i] = kin[i]

    def K(s):
        m = sum(1 << i for i in s)
        if m not in mom:
            mom[m] = sum(kin[i] for i in s)
        return mom[m]

    def J(s):
        """colour-ordered gluon current of the ordering s"""
        if s in cur:
            return cur[s]
        P = K(s)
        v = None
        for c in range(1, len(s)):
            A, B, ka, kb = J(s[:c]), J(s[c:]), K(s[:c]), K(s[c:])
            ab, Ab, Ba = mdot(A, B), mdot(A, ka + 2 * kb), mdot(B, 2 * ka + kb)
            t = [ab * (ka[m] - kb[m]) + B[m] * Ab - A[m] * Ba for m in range(4)]
            v = t if v is None else add(v, t)
        for c in range(1, len(s) - 1):
            for d in range(c + 1, len(s)):
                A, B, D = J(s[:c]), J(s[c:d]), J(s[d:])
                ab, bd, ad = mdot(A, B), mdot(B, D), mdot(A, D)
                v = add(v, [gs * (A[m] * bd + D[m] * ab - 2 * B[m] * ad) for m in range(4)])
        cur[s] = times(-gs / mdot(P, P), v)
        return cur[s]

    ubar, vcol = place(spinors(p[2], False), ng), place(spinors(p[3], True), ng + 1)
    line = {(): ubar}

    def U(s):
        """quark string: ubar with the gluons s attached in order, propagated"""
        if s in line:
            return line[s]
        v = raw(s)
        q = p[2] - K(s)
        f = -gs / (mdot(q, q) - M_TOP ** 2)
        w = slash_row(v, q)
        line[s] = [f * (w[m] + M_TOP * v[m]) for m in range(4)]
        return line[s]

    def raw(s):
        v = None
        for c in range(len(s)):
            t = slash_row(U(s[:c]), J(s[c:]))
            v = t if v is None else add(v, t)
        return v

    amps = []
    for s in itertools.permutations(range(ng)):
        a = gs * rdot(raw(s), vcol)
        amps.append(a.expand([2] * naxes + [N]).reshape(-1))
        for key in [k for k in cur if len(k) == ng]:
            del cur[key]
    A = torch.stack(amps)
    C = torch.from_numpy(C).cuda()
    me = (A.real * (C @ A.real) + A.imag * (C @ A.imag)).sum(0)
    # axes: gluons 0, 1, 2 .., quark, antiquark -> particle order 0, 1, quark, antiquark, gluons
    me = me.reshape([2] * naxes + [N])
    order = [0, 1, ng, ng + 1] + list(range(2, ng))
    return me.permute(order + [naxes]).reshape(2 ** naxes, N)


def exact(case, seed):
    process, n = case["process"], case["events"]
    # single-diagram weights have no form independent of a diagram enumeration
    if case["call"] == "channel":
        return None
    x = points(process, n, seed)
    hel = None
    if process == "ee_mumu":
        # 2 e^4 (t^2 + u^2) / s^2, spin-averaged
        d = lambda i, j: x[:, i, 0] * x[:, j, 0] - (x[:, i, 1:] * x[:, j, 1:]).sum(-1)
        me = 2 * (4 * math.pi * ALPHA_EM) ** 2 * (d(0, 2) ** 2 + d(0, 3) ** 2) / d(0, 1) ** 2
    else:
        C = colour_matrix(PROCESSES[process][2])
        step = {"gg_tt": 1 << 16, "gg_ttg": 1 << 15, "gg_ttgg": 1 << 14, "gg_ttggg": 1 << 11}[process]
        parts, hels = [], []
        for i in range(0, n, step):
            h = helicity_squares(process, x[i:i + step], C)
            parts.append(h.sum(0) / 256)
            if case["call"] == "hel":
                hels.append(h.t().contiguous())
        me = torch.cat(parts)
        hel = torch.cat(hels) if hels else None
    if case["call"] == "alphas":
        me = me * (extras(case, seed)[0] / ALPHA_S) ** PROCESSES[process][2]
    if case["call"] == "select":
        return (me, None, None)
    if case["call"] == "hel":
        return (me, hel)
    return me
