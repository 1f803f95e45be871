"""Cases that stand for the work users of this package have it do, for timing and for comparing outputs.

A case is a plain dict; ``prepare`` makes the seeded inputs and handles a program would hold, ``run`` makes one pass
through the public entry points, ``work`` counts the bytes and operations the method cannot do without, and ``exact``
gives the same outputs in 64 bits from plain torch.

Ops:
  eval     RTT.evaluate: amplitudes, every single-flip ratio and local energies of all walkers (each measurement)
  sweep    RTT.sweep: one Metropolis sweep of all walkers (each sampling step; the larger half of a run)
  vmc      a sweep followed by local energies and their compensated sums (the step of a whole program)
  batch    Batch.step: many small uneven states stepped together in one captured graph
  learn    one learned multi-spin move of every walker and the gradient of its training step
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2604_22718_amd import lattice
from paper_2604_22718_amd import rtt as R
from paper_2604_22718_amd import workloads as wl

H_FIELD = 3.04


def _case(name, op, lx, ly, reps, chi, dtype, walkers, terms=1, path="site+perm", runs=1):
    c = dict(op=op, lx=lx, ly=ly, reps=reps, chi=chi, dtype=dtype, walkers=walkers, terms=terms, path=path, runs=runs)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the 4x4 exact-enumeration workload: a call whose cost is launches and latency
        _case("eval_4x4_chi8_f32_w64", "eval", 4, 4, 2, 8, "f32", 64),
        # a scan over fields and sizes: uneven small states stepped as one graph
        _case("batch_12_uneven_bf16", "batch", 8, 8, 2, 64, "bf16", 1000, runs=12),
        # the 8x8 workload, both core types it is benchmarked with: measurement and sampling
        _case("eval_8x8_chi64_f32_w4096", "eval", 8, 8, 2, 64, "f32", 4096),
        _case("sweep_8x8_chi64_f32_w4096", "sweep", 8, 8, 2, 64, "f32", 4096),
        _case("eval_8x8_chi64_bf16_w4096", "eval", 8, 8, 2, 64, "bf16", 4096),
        _case("sweep_8x8_chi64_bf16_w4096", "sweep", 8, 8, 2, 64, "bf16", 4096),
        # the 10x10 wide-bond workload
        _case("eval_10x10_chi128_bf16_w8192", "eval", 10, 10, 3, 128, "bf16", 8192),
        _case("sweep_10x10_chi128_bf16_w8192", "sweep", 10, 10, 3, 128, "bf16", 8192),
        # linear combinations of bond-256 FP8 states (the 16x16 workload's state at a size that is quick to make)
        _case("eval_9x9_chi256_fp8_t2_w8192", "eval", 9, 9, 2, 256, "fp8", 8192, terms=2),
        _case("sweep_9x9_chi256_fp8_t2_w8192", "sweep", 9, 9, 2, 256, "fp8", 8192, terms=2),
        # the bond-2 pipeline on the H+V+D+D' path: sample, measure, sum
        _case("vmc_10x10_hvdd_chi2_f32_w4096", "vmc", 10, 10, 4, 2, "f32", 4096, path="hvdd"),
        # online training of the learned proposal during burn-in, on the same kind of state
        _case("learn_10x10_hvdd_chi2_w4096", "learn", 10, 10, 4, 2, "f32", 4096, path="hvdd"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["eval", "eval", "sweep", "sweep", "vmc", "batch", "learn"])
    kind = rng.choice(["small", "medium", "wide", "huge", "narrow"])
    if op == "batch":
        return _case(None, op, 8, 8, 2, 64, "bf16", _log_int(rng, 200, 1000), runs=rng.randint(3, 12))
    if op in ("vmc", "learn") or kind == "narrow":
        lx, ly = rng.randint(3, 10), rng.randint(3, 10)
        return _case(None, op, lx, ly, 4, rng.choice([2, 2, 3, 4]), "f32", _log_int(rng, 50, 4096), path="hvdd")
    if kind == "small":
        lx, ly, chi = rng.randint(2, 5), rng.randint(2, 5), rng.randint(5, 32)
        dtype, terms, most = rng.choice(["f32", "bf16"]), rng.randint(1, 2), 4096
    elif kind == "medium":
        lx, ly, chi = rng.randint(4, 8), rng.randint(4, 8), rng.randint(33, 64)
        dtype, terms, most = rng.choice(["f32", "bf16", "fp8"]), rng.choice([1, 1, 2]), 4096
    elif kind == "wide":
        lx, ly, chi = rng.randint(5, 10), rng.randint(5, 10), rng.randint(65, 128)
        dtype, terms, most = rng.choice(["f32", "bf16", "bf16", "fp8"]), 1, 8192
        if dtype == "f32":
            lx, ly, most = min(lx, 7), min(ly, 7), 2048
    else:
        lx, ly, chi = rng.randint(5, 9), rng.randint(5, 9), rng.choice([200, 256])
        dtype, terms, most = rng.choice(["bf16", "fp8", "fp8"]), rng.randint(1, 2), 4096
    reps = 2 if kind == "huge" else rng.randint(2, 3)
    return _case(None, op, lx, ly, reps, chi, dtype, _log_int(rng, 30, most), terms)


# ---------------------------------------------------------------- inputs
def _path(case, seed):
    if case["path"] == "hvdd":
        return lattice.path(case["lx"], case["ly"])
    return wl.path_site_plus_perms(case["lx"] * case["ly"], case["reps"], seed)


def _cores(case, L, seed):
    """Cores of one term as float64 device tensors (2, a, b): Gaussian of variance 1 / bond for the wide states, a
    perturbed constant train for the narrow ones, already values of the core type (so that the library's own
    quantisation, which is exact on them, is no part of what is compared)."""
    chi, dtype = case["chi"], case["dtype"]
    gen = torch.Generator("cuda").manual_seed(int(seed))
    bond = wl.open_bonds(L, chi)
    out = []
    for k in range(L):
        x = torch.randn((2, int(bond[k]), int(bond[k + 1])), generator=gen, device="cuda")
        x = 1.0 + 0.4 * x if case["path"] == "hvdd" else x / math.sqrt(chi)
        if dtype == "bf16":
            x = x.bfloat16().float()
        elif dtype == "fp8":
            s = torch.exp2(torch.ceil(torch.log2(x.abs().max() / 448.0)))
            x = (x / s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).float() * s
        out.append(x.double())
    return out


def _coeffs(case):
    return [1.0, -0.6, 0.8, 0.3][: case["terms"]]


def _bits(case, seed):
    g = np.random.Generator(np.random.Philox(int(seed) + 17))
    return g.integers(0, 2, size=(case["walkers"], case["lx"] * case["ly"]), dtype=np.uint8)


def _terms(case, seed):
    L = case["lx"] * case["ly"] * case["reps"]
    return [_cores(case, L, seed + 7919 * t) for t in range(case["terms"])]


def _walkers(case, seed, terms):
    """Starting configurations.  Measurements are made on sampled walkers: each is one of eight random configurations,
    drawn in proportion to |psi|^2; the other ops start from random spins, as a chain does."""
    if case["op"] != "eval":
        return _bits(case, seed)
    W, N, pi = case["walkers"], case["lx"] * case["ly"], _path(case, seed)
    g = np.random.Generator(np.random.Philox(int(seed) + 41))
    cand = g.integers(0, 2, size=(W, 8, N), dtype=np.uint8)
    gumbel = g.gumbel(size=(W, 8))
    lab, _ = _amplitudes(terms, _coeffs(case), pi, torch.from_numpy(cand.reshape(W * 8, N)).cuda().bool())
    pick = np.argmax(2.0 * lab.reshape(W, 8).cpu().numpy() + gumbel, axis=1)
    return np.ascontiguousarray(cand[np.arange(W), pick])


def _state(case, seed, cores):
    """The RTT handle (a linear combination when the case has several terms)."""
    pi = _path(case, seed)
    N = case["lx"] * case["ly"]
    terms = []
    for dev in cores:
        flat = torch.cat([c.reshape(-1) for c in dev]).cpu().numpy()
        off, cores = 0, []
        for c in dev:
            cores.append(flat[off:off + c.numel()].reshape(c.shape))
            off += c.numel()
        terms.append(R.RTT.create(N, pi, cores, case["dtype"]))
    return terms[0] if len(terms) == 1 else R.RTT.lincomb(terms, _coeffs(case))


def _batch_members(case, seed):
    """Sizes of the states of a batch: sides 4-8, two or three orderings, bonds 16-64, uneven walker counts."""
    g = np.random.Generator(np.random.Philox(977 + case["runs"]))
    out = []
    for _ in range(case["runs"]):
        side = int(g.integers(4, 9))
        W = int(round(case["walkers"] * math.exp(g.uniform(math.log(0.2), 0.0))))
        out.append(_case(None, "vmc", side, side, int(g.integers(2, 4)), int([16, 32, 64][g.integers(0, 3)]), "bf16", W))
    return out


def _learn_inputs(case, seed):
    g = np.random.Generator(np.random.Philox(int(seed) + 29))
    N, W = case["lx"] * case["ly"], case["walkers"]
    moves = (g.integers(0, N, W) | (g.integers(1, 9, W) << 16)).astype(np.int32)
    return moves, g.uniform(0, 1, W).astype(np.float32)


def _params(seed):
    p = wl.net_init_params(int(seed) + 31)
    return torch.from_numpy(p).bfloat16().double().numpy()


def prepare(case, seed):
    seed = int(seed) % (1 << 30)
    if case["op"] == "batch":
        members = _batch_members(case, seed)
        psis = [_state(m, seed + 101 * i, _terms(m, seed + 101 * i)) for i, m in enumerate(members)]
        hams = [R.TFIM(m["lx"], m["ly"], 1.0, H_FIELD) for m in members]
        spins = [R.spins_to_device(wl.pack_spins(_bits(m, seed + 101 * i))) for i, m in enumerate(members)]
        return {"case": case, "batch": R.Batch(psis, hams, spins, seed)}
    terms = _terms(case, seed)
    s = {"case": case, "seed": seed, "psi": _state(case, seed, terms), "sweeps": 0,
         "ham": R.TFIM(case["lx"], case["ly"], 1.0, H_FIELD, periodic=case["path"] != "hvdd"),
         "spins": R.spins_to_device(wl.pack_spins(_walkers(case, seed, terms)))}
    W = case["walkers"]
    if case["op"] in ("sweep", "vmc"):
        s["logabs"] = torch.empty(W, dtype=torch.float64, device="cuda")
        s["sign"] = torch.empty(W, dtype=torch.int8, device="cuda")
        s["accepts"] = torch.zeros(W, dtype=torch.int32, device="cuda")
    if case["op"] == "learn":
        net = R.Net(case["lx"], case["ly"], _params(seed))
        s["chain"] = R.LearnedChain(s["psi"], net, s["spins"], seed)
        moves, ap = _learn_inputs(case, seed)
        s["states"] = R.spins_to_device(wl.pack_spins(_bits(case, seed + 1)))
        s["moves"], s["ap"] = torch.from_numpy(moves).cuda(), torch.from_numpy(ap).cuda()
        s["grad"] = torch.empty(R.N_NET_PARAMS, dtype=torch.float32, device="cuda")
    return s


def _sweep(s):
    s["psi"].sweep(s["spins"], s["seed"], sweep0=s["sweeps"], accepts=s["accepts"], logabs=s["logabs"], sign=s["sign"])
    s["sweeps"] += 1
    return {"spins": s["spins"], "logabs": s["logabs"], "sign": s["sign"], "accepts": s["accepts"]}


def run(s):
    op = s["case"]["op"]
    if op == "eval":
        return s["psi"].evaluate(s["spins"], s["ham"])
    if op == "sweep":
        return _sweep(s)
    if op == "vmc":
        out = _sweep(s)
        out["eloc"] = s["psi"].local_energy(s["spins"], s["ham"])
        out["esum"] = R.energy_reduce(out["eloc"])
        return out
    if op == "batch":
        b = s["batch"]
        b.step()
        return {"spins": b.spins, "eloc": b.eloc, "esum": b.esum}
    c = s["chain"]
    c.learned_step()
    R.rtt_net_grad(c.net.handle, s["states"], s["moves"], s["ap"], s["grad"])
    return {"spins": c.spins, "logabs": c.logabs, "sign": c.sign, "moves": c.moves, "accept_prob": c.aprob,
            "grad": s["grad"]}


# ---------------------------------------------------------------- counts
def _vector_flops(case, seed=0):
    """(amplitude, all flip ratios, sweep) flops per walker: row-vector times core products of 2 a b flops, a train's
    base row once and, for a flipped spin, the positions from its first to its last one."""
    pi = _path(case, seed)
    L, N = len(pi), case["lx"] * case["ly"]
    bond = wl.open_bonds(L, case["chi"]).astype(float)
    cost = np.concatenate([[0.0], np.cumsum(2.0 * bond[:-1] * bond[1:])])
    span = 0.0
    for j in range(N):
        at = np.flatnonzero(pi == j)
        span += cost[at[-1] + 1] - cost[at[0]]
    T = case["terms"]
    return T * cost[L], T * (cost[L] + span), T * (cost[L] + span)


def _core_bytes(case):
    L = case["lx"] * case["ly"] * case["reps"]
    b = wl.open_bonds(L, case["chi"]).astype(float)
    return float(np.sum(2 * b[:-1] * b[1:])) * {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]] * case["terms"]


def work(case):
    if case["op"] == "batch":
        parts = [work(m) for m in _batch_members(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    W, N = case["walkers"], case["lx"] * case["ly"]
    spins = 8 * W * ((N + 63) // 64)
    amp, flips, sweep = _vector_flops(case)
    ev = {"bytes": spins + W * (8 + 1 + 4 + 9 * N + 8), "flops": W * flips}
    sw = {"bytes": 2 * spins + W * (8 + 1 + 8), "flops": W * sweep}
    if case["op"] == "eval":
        return {"bytes": _core_bytes(case) + ev["bytes"], "flops": ev["flops"]}
    if case["op"] == "sweep":
        return {"bytes": _core_bytes(case) + sw["bytes"], "flops": sw["flops"]}
    if case["op"] == "vmc":
        return {"bytes": _core_bytes(case) + sw["bytes"] + spins + 16 * W, "flops": sw["flops"] + ev["flops"]}
    # learn: two forward passes (both directions of the move) and an amplitude per walker; forward, input gradients
    # and weight gradients per training sample
    layer = 2.0 * N * 9 * 32 * 32
    fwd = 2 * layer + 2.0 * N * 32 * (9 + 9)
    return {"bytes": _core_bytes(case) + 3 * spins + W * 40 + 8 * R.N_NET_PARAMS,
            "flops": W * (2 * fwd + amp + 3 * fwd)}


# ---------------------------------------------------------------- 64-bit values
def _step(x, slices, bits):
    """Rows x (n, a) times slice 0 or 1 of a core per row."""
    y0, y1 = x @ slices[0], x @ slices[1]
    return torch.where(bits[:, None], y1, y0)


def _renorm(x, e):
    m = x.abs().amax(dim=1)
    p = torch.where(m > 0, torch.floor(torch.log2(m)), torch.zeros_like(m))
    return x * torch.exp2(-p)[:, None], e + p


def _combine(vals, exps, coeffs):
    """log|sum| and sign of sum_t c_t v_t 2^e_t."""
    top = torch.stack(exps).amax(dim=0)
    s = sum(c * v * torch.exp2(e - top) for c, v, e in zip(coeffs, vals, exps))
    return torch.log(s.abs()) + top * math.log(2.0), torch.sign(s)


def _contract(cores, pi, bits, x, e, k0):
    """Rows x 2^e at bond k0 contracted to the end of the train."""
    for k in range(k0, len(pi)):
        x = _step(x, cores[k], bits[:, int(pi[k])])
        if k % 8 == 0:
            x, e = _renorm(x, e)
    x, e = _renorm(x, e)
    return x[:, 0], e


def _unit(n):
    return torch.ones((n, 1), dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")


def _amplitudes(terms, coeffs, pi, bits):
    got = [_contract(c, pi, bits, *_unit(len(bits)), 0) for c in terms]
    return _combine([g[0] for g in got], [g[1] for g in got], coeffs)


def _diagonal(case, bits):
    lx, ly, per = case["lx"], case["ly"], case["path"] != "hvdd"
    z = 1.0 - 2.0 * bits.double()
    out = torch.zeros(len(bits), dtype=torch.float64, device="cuda")
    for y in range(ly):
        for x in range(lx):
            i = y * lx + x
            if x + 1 < lx or (per and lx >= 3):
                out += z[:, i] * z[:, y * lx + (x + 1) % lx]
            if y + 1 < ly or (per and ly >= 3):
                out += z[:, i] * z[:, ((y + 1) % ly) * lx + x]
    return out


def _exact_eval(case, terms, coeffs, pi, bits):
    W, N = bits.shape
    chunk = max(1, min(W, int(2e8 / ((N + 1) * case["chi"]))))
    la, sg, lr, rs, el = [], [], [], [], []
    for w0 in range(0, W, chunk):
        b = bits[w0:w0 + chunk]
        n = len(b)
        rows = b[:, None, :].repeat(1, N + 1, 1)
        idx = torch.arange(N, device="cuda")
        rows[:, idx + 1, idx] ^= True
        lab, sgn = _amplitudes(terms, coeffs, pi, rows.reshape(n * (N + 1), N))
        lab, sgn = lab.reshape(n, N + 1), sgn.reshape(n, N + 1)
        la.append(lab[:, 0])
        lr.append(lab[:, 1:] - lab[:, :1])
        rs.append(sgn[:, 1:] * sgn[:, :1])
        el.append(_diagonal(case, b) - H_FIELD * (rs[-1] * torch.exp(lr[-1])).sum(dim=1))
    return {"logabs": torch.cat(la), "sign": None, "status": None, "logratio": torch.cat(lr), "rsign": None,
            "eloc": torch.cat(el)}


def _philox_uniforms(seed, walkers, sweep, spin):
    """Word 0 of Philox4x64-10 under key (seed, 0), counter (walker, sweep, spin, 0), as uniforms in [0, 1)."""
    m32 = np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)

    def mulhilo(a, b):
        a0, a1, b0, b1 = a & m32, a >> s32, b & m32, b >> s32
        p00, p01, p10, p11 = a0 * b0, a0 * b1, a1 * b0, a1 * b1
        mid = (p00 >> s32) + (p01 & m32) + (p10 & m32)
        return p11 + (p01 >> s32) + (p10 >> s32) + (mid >> s32), a * b

    c0 = np.arange(walkers, dtype=np.uint64)
    c1, c2 = np.full_like(c0, sweep), np.full_like(c0, spin)
    c3 = np.zeros_like(c0)
    k0, k1 = seed, 0
    for r in range(10):
        if r:
            k0 = (k0 + 0x9E3779B97F4A7C15) % (1 << 64)
            k1 = (k1 + 0xBB67AE8584CAA73B) % (1 << 64)
        hi0, lo0 = mulhilo(np.uint64(0xD2E7470EE14C6C93), c0)
        hi1, lo1 = mulhilo(np.uint64(0xCA5A826395121157), c2)
        c0, c1, c2, c3 = hi1 ^ c1 ^ np.uint64(k0), lo1, hi0 ^ c3 ^ np.uint64(k1), lo0
    return torch.from_numpy((c0 >> np.uint64(11)).astype(np.float64) * 2.0 ** -53).cuda()


def _exact_sweep(case, seed, terms, coeffs, pi, bits):
    """log|psi| after one sweep decided in 64 bits (walkers whose decisions differ at a near tie are further off)."""
    W, N = bits.shape
    bits = bits.clone()
    lab, _ = _amplitudes(terms, coeffs, pi, bits)
    prefix = [_unit(W) for _ in terms]
    pos, seen = 0, set()
    with np.errstate(over="ignore"):
        for k, j in enumerate(int(q) for q in pi):
            if j in seen:
                continue
            seen.add(j)
            while pos < k:
                prefix = [_renorm(_step(x, c[pos], bits[:, int(pi[pos])]), e) for (x, e), c in zip(prefix, terms)]
                pos += 1
            flipped = bits.clone()
            flipped[:, j] ^= True
            got = [_contract(c, pi, flipped, x, e, k) for (x, e), c in zip(prefix, terms)]
            lnew, _ = _combine([g[0] for g in got], [g[1] for g in got], coeffs)
            acc = _philox_uniforms(seed, W, 0, j) < torch.exp(2.0 * (lnew - lab))
            bits[:, j] ^= acc
            lab = torch.where(acc, lnew, lab)
    return bits, lab


def _exact_grad(case, seed):
    """Gradient of the training loss by autograd in 64 bits."""
    lx, ly, B = case["lx"], case["ly"], case["walkers"]
    N = lx * ly
    p = torch.from_numpy(_params(seed)).cuda().requires_grad_(True)
    off, blocks = 0, []
    for shp in wl.NET_BLOCKS:
        n = int(np.prod(shp))
        blocks.append(p[off:off + n].reshape(shp))
        off += n
    W1, b1, W2, b2, W3, b3, Wh, bh = blocks
    bits = torch.from_numpy(_bits(case, seed + 1)).cuda()
    moves, ap = _learn_inputs(case, seed)
    c = torch.from_numpy((moves & 0xFFFF).astype(np.int64)).cuda()
    k = torch.from_numpy((moves >> 16).astype(np.int64)).cuda()
    coef = -torch.from_numpy(ap.astype(np.float64)).cuda() * k / B

    def conv(x, W, b):
        out = b[None, :, None]
        x = x.reshape(B, -1, ly, lx)
        for t in range(9):
            sh = torch.roll(x, shifts=(1 - t // 3, 1 - t % 3), dims=(2, 3)).reshape(B, -1, N)
            out = out + torch.matmul(W[:, :, t // 3, t % 3], sh)
        return torch.nn.functional.silu(out)

    x = (1.0 - 2.0 * bits.double()).reshape(B, 1, N)
    h = conv(conv(conv(x, W1, b1), W2, b2), W3, b3)
    o = torch.matmul(Wh, h) + bh[None, :, None]
    r = torch.arange(B, device="cuda")
    lq = torch.log_softmax(o[:, 0], 1)[r, c] + torch.log_softmax(o[r, 1:9, c], 1)[r, k - 1]
    (coef * lq).sum().backward()
    return p.grad


def exact(case, seed):
    seed = int(seed) % (1 << 30)
    if case["op"] == "batch":
        return None  # its members are the single-state cases; they continue their chains from pass to pass
    if case["op"] == "learn":  # the move itself is a random draw from the network's probabilities
        return {"spins": None, "logabs": None, "sign": None, "moves": None, "accept_prob": None,
                "grad": _exact_grad(case, seed)}
    pi = _path(case, seed)
    terms = _terms(case, seed)
    bits = torch.from_numpy(_walkers(case, seed, terms)).cuda().bool()
    coeffs = _coeffs(case)
    if case["op"] == "eval":
        return _exact_eval(case, terms, coeffs, pi, bits)
    bits, lab = _exact_sweep(case, seed, terms, coeffs, pi, bits)
    out = {"spins": None, "logabs": lab, "sign": None, "accepts": None}
    if case["op"] == "vmc":
        el = _exact_eval(case, terms, coeffs, pi, bits)["eloc"]
        out["eloc"] = el
        out["esum"] = torch.stack([el.sum(), (el * el).sum(), torch.tensor(float(len(el)), dtype=torch.float64, device="cuda")])
    return out
