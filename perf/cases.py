"""The work that users of this framework have it do, as cases to time and to check.

A case names an entry point (``call``), the number of photons ``n``, the
precision of the amplitudes, the partonic kinematics (``mode`` 0: fixed
sqrt(shat), 1: uniform in [lo, hi], 2: pp with toy densities), the number of
points and the cuts.  Sizes and energies are those of this repository's
workloads (workloads.py, bench.py) and generic ones around them.

Calls:
  xsec         heget_xsec: generate, cut, evaluate, reduce; the record on the host
  xsec_device  heget_xsec_device: the same, the record left on the GPU
  hist         heget_xsec_hist: the cross section with a histogram of the leading pT
  batch        heget_xsec_batch: n = 2 .. n_max in one call, 2^(points_log2 - n) points each
  me2          heget_me2_device: |M|^2 of a program's own events
  frame        heget_me2_frame_device: the same for events in any frame

What a pass returns: FP64 results as they are; per-point |M|^2 of FP32
amplitudes in 32 bits, the precision they carry; and a cross section's record
without ``sum_w_comp``, the part of sum_w that the compensated sum carried
apart: it holds the rounding of the additions, not a result, and it is already
added into sum_w.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_0908_4403_amd as H

PAPER_CUTS = (20.0, 2.5, 0.4)
ALPHA, CHARGE = 1.0 / 137.0, 2.0 / 3.0
GEV2_FB = 0.3893793721e12


def _case(name, call, n, prec, points, mode=0, energy=1000.0, lo=0.0, dr_min=0.4, sampled=False, **more):
    return dict(name=name, call=call, n=n, prec=prec, points=points, mode=mode, energy=energy, lo=lo,
                dr_min=dr_min, sampled=sampled, **more)


def listed():
    return [
        # the smallest cross section: n = 2 against its closed form, where launches and latency count
        _case("xsec_2a_500GeV_16k", "xsec", 2, "fp32", 16384, energy=500.0, dr_min=0.0),
        # a handful of events evaluated between other work of a program: a single short launch
        _case("me2_3a_517_fp64", "me2", 3, "fp64", 517),
        # the headline: u ubar -> 4 photons at 1 TeV, 2^20 points, FP32 amplitudes
        _case("xsec_4a_1TeV_2p20", "xsec", 4, "fp32", 1 << 20),
        # the same process in FP64 with a ragged size, chained on the GPU with other work
        _case("xsec_4a_1TeV_1e6_fp64", "xsec_device", 4, "fp64", 1000003),
        # pp -> 5 photons at 14 TeV: convolution with parton densities, most points cut
        _case("xsec_5a_pp_14TeV_2p22", "xsec", 5, "fp32", 1 << 22, mode=2, energy=14000.0, lo=150.0),
        # several multiplicities in one call, uneven sizes (a scan over n)
        _case("batch_2to7_2p24", "batch", 7, "fp32", 0, mode=1, energy=2000.0, lo=200.0, points_log2=24),
        # u ubar -> 8 photons at 2 TeV: the most expensive amplitude, FP32
        _case("xsec_8a_2TeV_2p18", "xsec", 8, "fp32", 1 << 18, energy=2000.0),
        # reference-quality |M|^2 for an event sample of another generator
        _case("me2_6a_131101_fp64", "me2", 6, "fp64", 131101),
        # reweighting of a sample with fast amplitudes
        _case("me2_7a_65537_fp32", "me2", 7, "fp32", 65537, energy=2000.0),
        # reference values at the largest n: few points, long per point
        _case("me2_8a_2053_fp64", "me2", 8, "fp64", 2053, energy=2000.0),
        # distribution of the leading photon pT with the paper's per-event helicities
        _case("hist_5a_sampled_fp64", "hist", 5, "fp64", 300007, mode=1, energy=2000.0, lo=200.0,
              sampled=True, bins=50),
        # events in the lab frame (boosted and rotated), composed from the HELAS functions
        _case("frame_4a_20011_fp64", "frame", 4, "fp64", 20011),
    ]


# Points at most, per n, of drawn cross sections and of drawn events, so that
# none costs more than the largest listed case.
MOST_POINTS = {2: 1 << 22, 3: 1 << 22, 4: 1 << 21, 5: 1 << 21, 6: 1 << 19, 7: 1 << 17, 8: 1 << 15}
MOST_EVENTS = {2: 1 << 21, 3: 1 << 21, 4: 1 << 20, 5: 1 << 19, 6: 1 << 18, 7: 1 << 16, 8: 1 << 13}
MOST_FRAME = {2: 1 << 20, 3: 1 << 18, 4: 1 << 16, 5: 1 << 13}


def _spread(rng, lo, hi):
    """A size between lo and hi, spread over its logarithm; most are odd or ragged."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(["xsec", "xsec", "xsec", "xsec_device", "me2", "me2", "me2", "hist", "batch", "frame"])
    n = rng.randint(2, 8)
    prec = rng.choice(["fp32", "fp64"])
    energy = round(_spread(rng, 200 + 150 * n, 3000) * rng.uniform(0.95, 1.05), 1)
    if call == "batch":
        return dict(call=call, n=rng.randint(3, 7), prec="fp32", points=0, mode=1, energy=energy, lo=200.0,
                    dr_min=0.4, sampled=False, points_log2=rng.randint(14, 23))
    if call == "me2":
        return dict(call=call, n=n, prec=prec, points=_spread(rng, 200, MOST_EVENTS[n]), mode=0, energy=energy,
                    lo=0.0, dr_min=0.4, sampled=False)
    if call == "frame":
        n = 2 + n % 4
        return dict(call=call, n=n, prec=prec, points=_spread(rng, 200, MOST_FRAME[n]), mode=0, energy=energy,
                    lo=0.0, dr_min=0.4, sampled=False)
    mode = rng.choice([0, 0, 1, 2])
    lo = 0.0 if mode == 0 else 200.0
    if mode == 2:
        energy, lo = rng.choice([7000.0, 13000.0, 14000.0]), 150.0
    c = dict(call=call, n=n, prec="fp64" if call in ("xsec_device", "hist") else prec,
             points=_spread(rng, 2048, MOST_POINTS[n]), mode=mode, energy=energy, lo=lo,
             dr_min=rng.choice([0.0, 0.4, 0.4, 0.7]), sampled=rng.random() < 0.25)
    if c["prec"] == "fp64" and n >= 7:
        c["points"] = max(2048, c["points"] // 4)
    if call == "hist":
        c["bins"] = rng.choice([20, 50, 100, 333])
    return c


# ------------------------------------------------------------------ the passes

def _config(case, seed, n=None, points=None):
    mode = case["mode"]
    return H.Config(mode=mode, prec=H.FP32 if case["prec"] == "fp32" else H.FP64, seed=seed,
                    npoints=case["points"] if points is None else points,
                    sqrt_s=0.0 if mode == 1 else case["energy"], sqrt_shat_lo=case["lo"],
                    sqrt_shat_hi=case["energy"] if mode == 1 else 0.0, pt_min=PAPER_CUTS[0],
                    eta_max=PAPER_CUTS[1], dr_min=case["dr_min"], alpha=ALPHA, charge=CHARGE,
                    helicity_sampling=int(case["sampled"]))


def _batch_shape(case):
    return [(n, max(1, (1 << case["points_log2"]) >> n)) for n in range(2, case["n"] + 1)]


def prepare(case, seed):
    call, n = case["call"], case["n"]
    if call == "batch":
        shape = _batch_shape(case)
        return dict(call=call, ns=[m for m, _ in shape], cfgs=[_config(case, seed, m, p) for m, p in shape])
    if call in ("me2", "frame"):
        p = _events(case, seed, "cuda")[1 if call == "frame" else 0]
        soa = p.permute(1, 2, 0).reshape((n + 2) * 4, -1).contiguous()
        return dict(call=call, n=n, mom=soa, prec=H.FP32 if case["prec"] == "fp32" else H.FP64,
                    out=torch.empty(soa.shape[1], dtype=torch.float64, device="cuda"))
    s = dict(call=call, n=n, cfg=_config(case, seed))
    if call == "xsec_device":
        s["out"] = torch.zeros(7, dtype=torch.float64, device="cuda")
    if call == "hist":
        s["bins"], s["range"] = case["bins"], _hist_range(case)
    return s


def _record(r):
    return {k: r[k] for k in ("sigma_fb", "err_fb", "sum_w", "sum_w2", "n_gen", "n_acc")}


def run(state):
    call = state["call"]
    if call == "xsec":
        return _record(H.xsec(state["n"], state["cfg"]))
    if call == "xsec_device":
        out = state["out"]
        H.xsec_device(state["n"], state["cfg"], out)
        return dict(sigma_err_sum=out[:3], sum_w2=out[4:5], counts=out[5:].view(torch.int64))
    if call == "hist":
        h, r = H.xsec_hist(state["n"], state["cfg"], H.OBS_PT_MAX, state["bins"], *state["range"])
        return dict(hist=h, **_record(r))
    if call == "batch":
        return [_record(r) for r in H.xsec_batch(state["ns"], state["cfgs"])]
    evaluate = H.me2_device if call == "me2" else H.me2_frame_device
    evaluate(state["n"], state["mom"], state["out"], state["prec"])
    return state["out"] if state["prec"] == H.FP64 else state["out"].to(torch.float32)


# ------------------------------------------------------------------ its work

def _amplitude_flops(n, sampled):
    """Operations per point of the currents of every photon set from both ends,
    each value formed once for the helicities that it depends on, and of one
    contraction per set of K photons and helicity configuration."""
    K = (n + 1) // 2
    hel = (lambda m: 1) if sampled else (lambda m: 1 << m)

    def node(m):
        return 14.0 + (11.0 if m == 1 else 36.0 + 20.0 * (m - 1)) * hel(m)

    f = sum(math.comb(n, m) * node(m) for m in list(range(1, K + 1)) + list(range(1, n - K)))
    f += math.comb(n, K) * ((16.0 + 20.0 * (n - K - 1)) * hel(n - K) + 16.0 * hel(n))
    return f + 4.0 * n + 4.0 * hel(n)


def _one_work(case, n, points):
    # generation: per photon ten generator rounds, an azimuth, a logarithm, two
    # square roots, two maps and the cut variables; per pair one Delta R
    gen = points * (150.0 * n + 8.0 * n * (n - 1) / 2)
    few = dict(case, n=n, points=4096, seed=0)
    share = float(_sample(few, 0, torch.device("cpu"), 0, 4096)["ok"].double().mean())
    return gen + points * share * _amplitude_flops(n, case["sampled"])


def work(case):
    call, n, points = case["call"], case["n"], case["points"]
    if call == "batch":
        return dict(bytes=56 * (n - 1), flops=sum(_one_work(case, m, p) for m, p in _batch_shape(case)))
    if call in ("me2", "frame"):
        out = 8 if case["prec"] == "fp64" else 4
        return dict(bytes=points * (32 * (n + 2) + out), flops=points * _amplitude_flops(n, False))
    return dict(bytes=56 + 8 * (case["bins"] + 2 if call == "hist" else 0), flops=_one_work(case, n, points))


# ------------------------------------------------------------------ in 64 bits
# The same numbers from plain torch in FP64: Philox4x32-10, RAMBO, the cuts,
# the amplitudes from 2 x 2 matrices, the sums.

def _philox(point, block, stream, seed):
    """Four tensors of 32-bit words (in int64) for the points."""
    lo32 = 0xFFFFFFFF
    c = [point & lo32, point >> 32, torch.full_like(point, block), torch.full_like(point, stream)]
    k0, k1 = seed & lo32, (seed >> 32) & lo32
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57  # modulo 2^64
        c = [((b >> 32) & lo32) ^ c[1] ^ k0, b & lo32, ((a >> 32) & lo32) ^ c[3] ^ k1, a & lo32]
        k0, k1 = (k0 + 0x9E3779B9) & lo32, (k1 + 0xBB67AE85) & lo32
    return c


def _pair(point, block, stream, seed):
    w = _philox(point, block, stream, seed)
    return [((((w[i + 1] << 32) | w[i]) >> 11 & ((1 << 53) - 1)).double() + 0.5) * 2.0**-53 for i in (0, 2)]


def _conformal(k, e):
    """Boost k[points, n, 4] to its rest frame and scale its sum to e[points]."""
    Q = k.sum(1)
    M = torch.sqrt(Q[:, 0] ** 2 - (Q[:, 1:] ** 2).sum(1))
    b = -Q[:, 1:] / M[:, None]
    g = Q[:, 0] / M
    bq = (k[:, :, 1:] * b[:, None]).sum(2)
    r = torch.empty_like(k)
    r[:, :, 0] = g[:, None] * k[:, :, 0] + bq
    r[:, :, 1:] = k[:, :, 1:] + b[:, None] * (k[:, :, :1] + (bq / (1 + g)[:, None])[:, :, None])
    return r * (e / M)[:, None, None]


def _sample(case, seed, device, first, count):
    """Points first .. first + count - 1: events, weight without |M|^2, whether they pass."""
    n, mode = case["n"], case["mode"]
    point = torch.arange(first, first + count, dtype=torch.int64, device=device)
    e = torch.full((count,), case["energy"], dtype=torch.float64, device=device)
    y, f = torch.zeros_like(e), torch.ones_like(e)
    above = torch.ones(count, dtype=torch.bool, device=device)
    if mode == 1:
        e = case["lo"] + (case["energy"] - case["lo"]) * _pair(point, 1, 1, seed)[0]
    elif mode == 2:
        r = _pair(point, 0, 1, seed)
        xu, xub = r[0] ** 2, r[1] ** (1 / 0.7)
        e = torch.sqrt(xu * xub) * case["energy"]
        above = e >= case["lo"]
        e = torch.where(above, e, torch.full_like(e, case["lo"]))
        f = 2 * ((1 - xu) ** 3 / 0.5) * ((1 - xub) ** 6 / 0.7)
        y = 0.5 * torch.log(xu / xub)
    k = torch.empty(count, n, 4, dtype=torch.float64, device=device)
    for i in range(n):
        u = [(w.double() + 0.5) * 2.0**-32 for w in _philox(point, i, 0, seed)]
        c, phi, q = 2 * u[0] - 1, 2 * math.pi * u[1], -torch.log(u[2] * u[3])
        s = torch.sqrt(1 - c * c)
        k[:, i] = torch.stack([q, q * s * torch.cos(phi), q * s * torch.sin(phi), q * c], 1)
    for _ in range(2):
        k = _conformal(k, e)
        k[:, :, 0] = torch.sqrt((k[:, :, 1:] ** 2).sum(2))
    pt = torch.sqrt(k[:, :, 1] ** 2 + k[:, :, 2] ** 2)
    eta = torch.asinh(k[:, :, 3] / pt) + y[:, None]
    phi = torch.atan2(k[:, :, 2], k[:, :, 1])
    ok = above & (pt > PAPER_CUTS[0]).all(1) & (eta.abs() < PAPER_CUTS[1]).all(1)
    if case["dr_min"] > 0:
        for i in range(n):
            for j in range(i):
                d = (phi[:, i] - phi[:, j]).abs()
                d = torch.minimum(d, 2 * math.pi - d)
                ok &= (eta[:, i] - eta[:, j]) ** 2 + d**2 > case["dr_min"] ** 2
    volume = (2 * math.pi) ** (4 - 3 * n) * (math.pi / 2) ** (n - 1) / (math.factorial(n - 1) * math.factorial(n - 2))
    w = 0.5 * 0.25 * (3 / 9) / math.factorial(n) * volume * GEV2_FB * (e * e) ** (n - 3) * f
    half = torch.zeros(count, 2, 4, dtype=torch.float64, device=device)
    half[:, :, 0] = (e / 2)[:, None]
    half[:, 0, 3], half[:, 1, 3] = e / 2, -e / 2
    return dict(p=torch.cat([half, k], 1), w=w, ok=ok, point=point, pt_max=pt.max(1).values)


def _events(case, seed, device):
    """A program's own events: the first `points` ones that pass the cuts, in
    the partonic CM frame, and the same ones boosted and rotated."""
    want, got, first = case["points"], [], 0
    while want > 0:
        count = max(1024, min(1 << 20, 4 * want))
        s = _sample(case, seed, torch.device(device), first, count)
        got.append(s["p"][s["ok"]][:want])
        first, want = first + count, want - got[-1].shape[0]
    p = torch.cat(got)
    r = np.random.RandomState(seed % (1 << 31))
    turn, _ = np.linalg.qr(r.standard_normal((3, 3)))
    b = r.uniform(-0.4, 0.4, 3)
    g = 1 / math.sqrt(1 - float(b @ b))
    boost = np.eye(4)
    boost[0, 0], boost[0, 1:], boost[1:, 0] = g, g * b, g * b
    boost[1:, 1:] += (g - 1) / float(b @ b) * np.outer(b, b)
    if np.linalg.det(turn) < 0:
        turn[:, 0] *= -1
    full = np.eye(4)
    full[1:, 1:] = turn
    q = p @ torch.tensor((full @ boost).T.copy(), device=p.device)
    q[:, :, 0] = torch.sqrt((q[:, :, 1:] ** 2).sum(2))
    return p, q


def _sigma(v, sign):
    """v0 + sign sigma . v as 2 x 2 entries (a list of lists), v = (v0, v1, v2, v3)."""
    return [[v[0] + sign * v[3], sign * (v[1] - 1j * v[2])], [sign * (v[1] + 1j * v[2]), v[0] - sign * v[3]]]


def _me2_table(p):
    """|M|^2 of u(p1, helicity -) ubar(p2, +) -> photons at p[points, n + 2, 4]
    with unit charge, for every photon helicity configuration: [2^n, points],
    bit j of the first index set where photon j has helicity +1."""
    n, count = p.shape[1] - 2, p.shape[0]
    k = [p[:, j + 2] for j in range(n)]
    vert = []  # per photon [2 helicities][2][2]: (eps*) . sigmabar
    for v in k:
        pt = torch.sqrt(v[:, 1] ** 2 + v[:, 2] ** 2)
        cp, sp, ct, st = v[:, 1] / pt, v[:, 2] / pt, v[:, 3] / v[:, 0], pt / v[:, 0]
        theta = torch.stack([ct * cp, ct * sp, -st])
        azim = torch.stack([-sp, cp, torch.zeros_like(cp)])
        both = []
        for lam in (-1, 1):
            e = (-lam * theta + 1j * azim) / math.sqrt(2)
            m = _sigma([torch.zeros_like(e[0]), e[0], e[1], e[2]], 1)
            both.append(torch.stack([torch.stack(m[0]), torch.stack(m[1])]))
        vert.append(torch.stack(both))  # [2, 2, 2, points]
    row = torch.zeros(2, count, dtype=torch.complex128, device=p.device)
    row[0] = torch.sqrt(2 * p[:, 1, 0])  # the antiquark's spinor, momentum along -z
    level = {0: row}
    for size in range(1, n + 1):
        nxt = {}
        for mask in range(1 << n):
            if bin(mask).count("1") != size:
                continue
            have = [j for j in reversed(range(n)) if mask >> j & 1]  # axes: highest photon first
            total = None
            for at, j in enumerate(have):
                r = level[mask & ~(1 << j)].unsqueeze(at)           # [.., 1 at the photon, .., 2, points]
                v = vert[j].reshape([1] * at + [2] + [1] * (size - 1 - at) + [2, 2, count])
                t = (r.unsqueeze(-2) * v).sum(-3)                   # row times matrix
                total = t if total is None else total + t
            if size < n:
                q = sum(k[j] for j in have) - p[:, 1]
                q2 = q[:, 0] ** 2 - (q[:, 1:] ** 2).sum(1)
                m = _sigma([q[:, i].to(torch.complex128) / q2 for i in range(4)], -1)
                total = torch.stack([total[..., 0, :] * m[0][i] + total[..., 1, :] * m[1][i] for i in (0, 1)], -2)
            nxt[mask] = total
        level = nxt
    amp = level[(1 << n) - 1][..., 1, :] * torch.sqrt(2 * p[:, 0, 0])  # the quark's spinor, along +z
    return (amp.real**2 + amp.imag**2).reshape(1 << n, count)


def _coupling(n):
    return (4 * math.pi * ALPHA * CHARGE**2) ** n


def _exact_me2(p):
    """Summed over both quark pairs (each other's mirror image) and all photon helicities."""
    n, part = p.shape[1] - 2, max(64, 6_000_000 // 3 ** (p.shape[1] - 2))
    return torch.cat([2 * _coupling(n) * _me2_table(q).sum(0) for q in p.split(part)])


def _hist_range(case):
    return 20.0, 0.4 * (2000.0 if case["mode"] == 2 else case["energy"])


def _exact_xsec(case, seed, n, points, bins=None):
    case = dict(case, n=n)
    weights, largest, n_acc = [], [], 0
    part = 1 << 20
    for first in range(0, points, part):
        s = _sample(case, seed, torch.device("cuda"), first, min(part, points - first))
        ok = s["ok"]
        p, w = s["p"][ok], s["w"][ok]
        if case["sampled"]:
            drawn = _philox(s["point"][ok], 0, 2, seed)[0] & ((2 << n) - 1)
            lam = (drawn >> 1) ^ torch.where((drawn & 1) == 1, (1 << n) - 1, 0)
            few = max(64, 6_000_000 // 3**n)
            me2 = torch.cat([2 ** (n + 1) * _coupling(n) * _me2_table(q).gather(0, h[None])[0]
                             for q, h in zip(p.split(few), lam.split(few))]) if len(p) else w
        else:
            me2 = _exact_me2(p) if len(p) else w
        weights.append(w * me2)
        largest.append(s["pt_max"][ok])
        n_acc += int(ok.sum())
    w = torch.cat(weights)
    total, total2 = float(w.sum()), float((w * w).sum())
    sigma = total / points
    var = (total2 / points - sigma**2) / (points - 1) if points > 1 else 0.0
    r = dict(sigma_fb=sigma, err_fb=math.sqrt(max(var, 0.0)), sum_w=total, sum_w2=total2, n_gen=points, n_acc=n_acc)
    if bins is None:
        return r
    lo, hi = _hist_range(case)
    x = torch.cat(largest)
    at = torch.where(x < lo, 0, torch.where(x < hi, 1 + ((x - lo) * (bins / (hi - lo))).long().clamp(max=bins - 1), bins + 1))
    h = torch.zeros(bins + 2, dtype=torch.float64, device=w.device).index_add_(0, at, w) / points
    return dict(hist=h.cpu().numpy(), **r)


def exact(case, seed):
    call, n = case["call"], case["n"]
    if call in ("me2", "frame"):
        r = _exact_me2(_events(case, seed, "cuda")[0])
        return r if case["prec"] == "fp64" else r.to(torch.float32)
    if call == "batch":
        return [_exact_xsec(case, seed, m, p) for m, p in _batch_shape(case)]
    r = _exact_xsec(case, seed, n, case["points"], case.get("bins"))
    if call != "xsec_device":
        return r
    t = dict(dtype=torch.float64)
    return dict(sigma_err_sum=torch.tensor([r["sigma_fb"], r["err_fb"], r["sum_w"]], **t),
                sum_w2=torch.tensor([r["sum_w2"]], **t), counts=torch.tensor([r["n_gen"], r["n_acc"]]))
