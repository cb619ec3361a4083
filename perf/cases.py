"""Cases whose time is measured: the calls a search, a sensitivity campaign and
the learned proposer make, through the package's public entry points.

A case is a dict of plain values with a "kind":
  search    load a spectrogram per detector, set velocities (and antenna
            patterns), evaluate a cubic lattice, rank both statistics
  bank      evaluate a uniform random bank of explicit templates and rank it
  prep      strain -> normalised power
  batch     many uneven searches in one launch
  campaign  noise-only and injected realisations of a sensitivity campaign
  network   one training step of the ranking network
  propose   ingest a stack of realisations and propose templates on it
Inputs are drawn on the device from the seed: Exp(1) normalised power, U[0.5, 2]
noise-floor weights, detector velocities of a circular orbit plus rotation.
"""
import math

import numpy as np
import torch

from paper_2507_07816_amd import ltgw
from paper_2507_07816_amd.campaign import Campaign
from paper_2507_07816_amd.proposer import coarse_grid_for, init_params, nearest_coarse_groups

C_LIGHT = 299792458.0
RHO_TH = 1.6
K = 10  # candidates ranked per statistic
SKY0 = (1.0, 0.3)  # right ascension, declination of the first sky point
SITES = ((46.455, -119.408, 324.0), (30.563, -90.774, 252.3))  # latitude, longitude, arm azimuth


def listed():
    return [
        # the small search: 1024 segments of 4 s, 800 bins, 4800 templates; launches and host time count
        dict(name="search_small", kind="search", n_seg=1024, n_bins=800, k_lo=1600, t_sft=4.0, n_det=1, n_f0=400,
             f0_lo=400, n_tau=4, n_brake=3, n_sky=1, store="f32", weighted=False, antenna=False, tune=False),
        # a directed search over a day: 10800 segments of 8 s, 500-1500 Hz, 2.3 million templates
        dict(name="search_day", kind="search", n_seg=10800, n_bins=8000, k_lo=4000, t_sft=8.0, n_det=1, n_f0=8000,
             f0_lo=0, n_tau=32, n_brake=9, n_sky=1, store="f32", weighted=True, antenna=False, tune=True),
        # a sky patch with two detectors over six hours, BF16 power, sizes that fill no tile
        dict(name="search_patch_bf16", kind="search", n_seg=2699, n_bins=1601, k_lo=6003, t_sft=8.0, n_det=2,
             n_f0=1601, f0_lo=0, n_tau=4, n_brake=3, n_sky=17, store="bf16", weighted=False, antenna=False, tune=False),
        # antenna-pattern weights (moments summed with the statistic), FP8 power, half a day
        dict(name="search_antenna_fp8", kind="search", n_seg=5400, n_bins=4000, k_lo=4000, t_sft=8.0, n_det=1,
             n_f0=4000, f0_lo=0, n_tau=8, n_brake=5, n_sky=2, store="fp8", weighted=True, antenna=True, tune=False),
        # a random bank as the campaign uses it: one small realisation, 4800 templates
        dict(name="bank_small", kind="bank", n_seg=1024, n_bins=800, k_lo=1600, t_sft=4.0, n_tpl=4800, store="f32",
             weighted=True),
        # a random bank of a million templates over a day
        dict(name="bank_day", kind="bank", n_seg=10800, n_bins=8000, k_lo=4000, t_sft=8.0, n_tpl=1000000, store="f32",
             weighted=True),
        # an hour of strain at 2048 Hz, a band and a median window that fill no tile
        dict(name="prep_hour", kind="prep", n_seg=450, n_fft=16384, k_lo=803, n_bins=1205, window=51),
        # a day of strain at 4096 Hz -> the directed search's input
        dict(name="prep_day", kind="prep", n_seg=10800, n_fft=32768, k_lo=4000, n_bins=8000, window=101),
        # uneven searches of a follow-up in one launch: two detectors, sky patches
        dict(name="batch_uneven", kind="batch", n_searches=6, t_obs_max=43200.0, width_max=300.0, sky_max=64, store="f32"),
        # a campaign's stack: thresholds from noise, the templates near each injection
        dict(name="campaign_stack", kind="campaign", n_seg=1024, n_bins=800, k_lo=1600, t_sft=4.0, n_f0=400, n_tau=4,
             n_brake=3, R_noise=256, R_inj=256),
        # a training step of the ranking network
        dict(name="network_step", kind="network", B=256, c_in=8, c_out=24, L=200),
        # proposals for a stack of realisations, from the raw stack to the best templates
        dict(name="propose_stack", kind="propose", R=1024, n_seg=1024, n_bins=800, k_lo=1600, t_sft=4.0, n_f0=400,
             block=32, n_select=384, coarse_segments=8, store="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "bank", "prep", "batch", "campaign", "network", "propose"])
    if kind == "search":
        n_seg, n_bins = _log_int(rng, 200, 10800), _log_int(rng, 150, 8000)
        c = dict(kind=kind, n_seg=n_seg, n_bins=n_bins, k_lo=_log_int(rng, 1600, 12000), t_sft=rng.choice([4.0, 8.0]),
                 n_det=rng.choice([1, 1, 2]), n_f0=_log_int(rng, 90, n_bins), f0_lo=0, n_tau=_log_int(rng, 2, 32),
                 n_brake=_log_int(rng, 1, 9), n_sky=_log_int(rng, 1, 20), store=rng.choice(["f32", "f32", "bf16", "fp8"]),
                 weighted=rng.random() < 0.5, antenna=rng.random() < 0.25, tune=False)
        c["f0_lo"] = rng.randrange(0, n_bins - c["n_f0"] + 1)
        while c["n_sky"] > 1 and _evals(c) > 6e9:
            c["n_sky"] -= 1
        while c["n_tau"] > 1 and _evals(c) > 6e9:
            c["n_tau"] -= 1
        return c
    if kind == "bank":
        n_seg = _log_int(rng, 200, 10800)
        return dict(kind=kind, n_seg=n_seg, n_bins=_log_int(rng, 150, 8000), k_lo=_log_int(rng, 1600, 12000),
                    t_sft=rng.choice([4.0, 8.0]), n_tpl=_log_int(rng, 100, 1000000),
                    store=rng.choice(["f32", "bf16", "fp8"]), weighted=rng.random() < 0.5)
    if kind == "prep":
        n_fft, window = rng.choice([4096, 8192, 16384, 32768]), 2 * rng.randrange(12, 129) + 1
        n_bins = _log_int(rng, 100, n_fft // 2 - window)
        return dict(kind=kind, n_seg=_log_int(rng, 40, 10800), n_fft=n_fft,
                    k_lo=rng.randrange(window // 2, n_fft // 2 - n_bins - window // 2 + 1), n_bins=n_bins, window=window)
    if kind == "batch":
        return dict(kind=kind, n_searches=rng.randrange(2, 9), t_obs_max=rng.uniform(8000.0, 30000.0),
                    width_max=rng.uniform(110.0, 300.0), sky_max=_log_int(rng, 17, 64), store=rng.choice(["f32", "bf16"]))
    if kind == "campaign":
        return dict(kind=kind, n_seg=4 * _log_int(rng, 64, 256), n_bins=2 * _log_int(rng, 150, 400), k_lo=1600, t_sft=4.0,
                    n_f0=_log_int(rng, 100, 300), n_tau=4, n_brake=3, R_noise=_log_int(rng, 16, 256),
                    R_inj=_log_int(rng, 16, 256))
    if kind == "network":
        return dict(kind=kind, B=_log_int(rng, 16, 256), c_in=rng.choice([4, 8, 12]), c_out=24, L=_log_int(rng, 50, 200))
    return dict(kind=kind, R=_log_int(rng, 32, 1024), n_seg=8 * _log_int(rng, 32, 128), n_bins=800, k_lo=1600, t_sft=4.0,
                n_f0=2 * _log_int(rng, 50, 200), block=rng.choice([16, 32, 64]), n_select=_log_int(rng, 192, 400),
                coarse_segments=rng.choice([2, 4, 8]), store=rng.choice(["f32", "bf16"]))


# ---- inputs ----------------------------------------------------------------
def _exp_noise(shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) % (1 << 62))
    return torch.empty(shape, dtype=torch.float32, device="cuda").exponential_(1.0, generator=g)


def _times(n_seg, t_sft):
    return (np.arange(n_seg, dtype=np.float64) + 0.5) * t_sft


def _velocity(t, site):
    la, lo = math.radians(site[0]), math.radians(site[1])
    ob, phi, psi = math.radians(23.4393), 2 * np.pi * t / 3.156e7, 2 * np.pi * t / 86164.0 + lo
    orb = 29.8e3 * np.stack([-np.sin(phi), np.cos(phi) * math.cos(ob), np.cos(phi) * math.sin(ob)], axis=-1)
    rot = 465.0 * math.cos(la) * np.stack([-np.sin(psi), np.cos(psi), np.zeros_like(psi)], axis=-1)
    return np.ascontiguousarray(orb + rot)


def _arms(site):
    la, lo, az = (math.radians(x) for x in site)
    north = np.array([-math.sin(la) * math.cos(lo), -math.sin(la) * math.sin(lo), math.cos(la)])
    east = np.array([-math.sin(lo), math.cos(lo), 0.0])
    arms = [math.cos(a) * north + math.sin(a) * east for a in (az, az + math.pi / 2)]
    return np.ascontiguousarray([a / np.linalg.norm(a) for a in arms])


def _sky(n, r=None):
    """n unit vectors: the first at SKY0, the others within a few degrees of it."""
    out = []
    for i in range(n):
        ra, de = SKY0[0] + 0.01 * i, SKY0[1] + 0.05 * math.sin(2.4 * i)
        if r is not None:
            ra, de = ra + r.uniform(-1.0, 1.0), de + r.uniform(-0.5, 0.5)
        v = np.array([math.cos(de) * math.cos(ra), math.cos(de) * math.sin(ra), math.sin(de)])
        out.append(v / np.linalg.norm(v))
    return np.array(out)


def _geometry(c, seed, det=0):
    t = _times(c["n_seg"], c["t_sft"])
    r = np.random.Generator(np.random.PCG64([int(seed), 77, det]))
    w = r.uniform(0.5, 2.0, c["n_seg"]).astype(np.float32) if c.get("weighted") else None
    return dict(t=t, v=_velocity(t, SITES[det % 2]), w=w, k_lo=c["k_lo"], t_sft=c["t_sft"], n_bins=c["n_bins"])


def _grid(c, r):
    """The lattice: f0 at every bin from f0_lo, tau log-spaced, n linear; the
    seed moves the sky (a directed search's target)."""
    step = 1.0 / c["t_sft"]
    tau = np.geomspace(3500.0, 35000.0, c["n_tau"])
    brake = np.linspace(3.0, 7.0, c["n_brake"]) if c["n_brake"] > 1 else np.array([5.0])
    return dict(f0_min=(c["k_lo"] + c.get("f0_lo", 0)) * step, f0_step=step, n_f0=c["n_f0"], tau=tau, brake=brake,
                sky=_sky(c.get("n_sky", 1), r), t0=0.0)


def _bank(c, seed):
    r = np.random.Generator(np.random.PCG64([int(seed), 11]))
    n, k, T = c["n_tpl"], c["k_lo"], c["t_sft"]
    p = np.empty((n, 6))
    p[:, 0] = r.uniform(k / T, (k + c["n_bins"] - 1) / T, n)
    p[:, 1] = r.uniform(3500.0, 35000.0, n)
    p[:, 2] = r.uniform(3.0, 7.0, n)
    p[:, 3:] = _sky(1, r)[0]
    return p


def _batch_specs(c, seed):
    r = np.random.Generator(np.random.PCG64([int(seed), 5]))
    shape = np.random.Generator(np.random.PCG64([5, c["n_searches"]]))  # sizes are the case's, not the seed's
    out = []
    for _ in range(c["n_searches"]):
        n_seg = max(1, int(round(shape.uniform(7200.0, c["t_obs_max"]) / 8.0)))
        n_bins = int(round(shape.uniform(100.0, c["width_max"]) / 0.125))
        k_lo = int(shape.integers(4000, 24000 - n_bins))
        n_sky = int(round(math.exp(shape.uniform(math.log(16.0), math.log(c["sky_max"])))))
        grid = dict(f0_min=k_lo / 8.0, f0_step=0.125, n_f0=n_bins, tau=np.array([3500.0, 7000.0, 14000.0, 35000.0]),
                    brake=np.array([3.0, 5.0, 7.0]), sky=_sky(n_sky, r), t0=0.0)
        out.append(dict(n_seg=n_seg, n_bins=n_bins, k_lo=k_lo, t_sft=8.0, grid=grid))
    return out


def _load(ctx, slot, power, geo, store):
    ctx.load_spectrogram(slot, power, geo["k_lo"], geo["t_sft"], geo["t"], weights=geo["w"], rho_th=RHO_TH, store=store)
    ctx.set_velocity_table(slot, geo["v"])


def _propose_grids(c):
    step = 1.0 / c["t_sft"]
    tau, brake = np.array([3500.0, 7000.0, 14000.0, 35000.0]), np.array([3.0, 5.0, 7.0])
    fine = dict(f0_min=500.0, f0_step=step, n_f0=c["n_f0"], tau=tau, brake=brake, sky=_sky(1), t0=0.0)
    coarse = coarse_grid_for(fine, np.sqrt(tau[0::2] * tau[1::2]), np.array([4.0, 6.0]))
    return fine, coarse


def _network_params(c_in, c_out, seed, coarse_map=None):
    """He-uniform weights; with a coarse map, small ones around a network that
    passes each coarse power channel through to the fine groups it is nearest
    to (the ranking that training starts to learn)."""
    p = init_params(c_in, c_out, int(seed))
    if coarse_map is None:
        return p
    p *= 0.02
    at = [0, 32 * c_in * 5 + 32]
    at += [at[1] + 32 * 32 * 5 + 32, at[1] + 2 * (32 * 32 * 5 + 32)]
    W = [p[at[0]:at[0] + 32 * c_in * 5].reshape(32, c_in, 5), p[at[1]:at[1] + 5120].reshape(32, 32, 5),
         p[at[2]:at[2] + 5120].reshape(32, 32, 5), p[at[3]:at[3] + c_out * 32].reshape(c_out, 32)]
    for ch in range(c_in):
        for w in W[:3]:
            w[ch, ch, 2] += 1.0
    for o in range(c_out):
        W[3][o, coarse_map[o // 2][0]] += 1.0
    return p


def _injections(n, grid, amps, r):
    out = np.zeros((n, 4))
    out[:, 0] = r.uniform(grid["f0_min"], grid["f0_min"] + (grid["n_f0"] - 1) * grid["f0_step"], n)
    out[:, 1] = np.exp(r.uniform(math.log(3500.0), math.log(35000.0), n))
    out[:, 2] = r.uniform(3.0, 7.0, n)
    out[:, 3] = r.uniform(amps[0], amps[1], n)
    return out


def prepare(case, seed):
    c, kind = case, case["kind"]
    r = np.random.Generator(np.random.PCG64([int(seed), 1]))
    s = dict(case=c, kind=kind)
    if kind == "prep":
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed))
        s["strain"] = torch.randn(c["n_seg"] * c["n_fft"], generator=g, device="cuda", dtype=torch.float32)
        s["ctx"] = ltgw.Context(0)
        return s
    ctx = s["ctx"] = ltgw.Context(0)
    if kind == "search":
        s["grid"] = _grid(c, r)
        s["geo"] = [_geometry(c, seed, d) for d in range(c["n_det"])]
        s["power"] = [_exp_noise((c["n_seg"], c["n_bins"]), 1000 * int(seed) + d) for d in range(c["n_det"])]
        if c["antenna"]:
            s["arms"] = [_arms(SITES[d % 2]) for d in range(c["n_det"])]
            s["era"] = [2 * np.pi * g["t"] / 86164.0 for g in s["geo"]]
        if c["tune"]:
            for d in range(c["n_det"]):
                _load(ctx, d, s["power"][d], s["geo"][d], c["store"])
            ctx.autotune(**s["grid"])
    elif kind == "bank":
        s["geo"] = _geometry(c, seed)
        s["power"] = _exp_noise((c["n_seg"], c["n_bins"]), 1000 * int(seed))
        s["params"] = _bank(c, seed)
    elif kind == "batch":
        s["specs"] = []
        for i, b in enumerate(_batch_specs(c, seed)):
            for d in range(2):
                _load(ctx, 2 * i + d, _exp_noise((b["n_seg"], b["n_bins"]), 1000 * int(seed) + 2 * i + d),
                      _geometry(b, seed, d), c["store"])
            s["specs"].append(dict(b["grid"], dets=[2 * i, 2 * i + 1]))
    elif kind == "campaign":
        geo = _geometry(dict(c, weighted=True), seed)
        grid = dict(_grid(dict(c, n_sky=1), r), f0_min=500.0)
        s["camp"] = Campaign(ctx, dict(t_seg=geo["t"], v=geo["v"], weights=geo["w"], k_lo=c["k_lo"], t_sft=c["t_sft"],
                                       n_bins=c["n_bins"]), grid, seed=int(seed), stack_chunk=256)
        s["inj"] = _injections(c["R_inj"], grid, (0.5, 6.0), r)
    elif kind == "network":
        f = dict(dtype=torch.float32, device="cuda")
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed))
        B, ci, co, L = c["B"], c["c_in"], c["c_out"], c["L"]
        s["params"] = torch.from_numpy(_network_params(ci, co, seed)).cuda()
        n = s["params"].numel()
        # a state in mid-training: moments of past gradients
        s["m"] = 1e-3 * torch.randn(n, generator=g, **f)
        s["v"] = 1e-5 * (0.5 + torch.rand(n, generator=g, **f))
        s["x"] = torch.randn((B, ci, L), generator=g, **f)  # critical ratios: zero mean, unit variance
        t = torch.randint(0, co * L, (B,), generator=g, dtype=torch.int32, device="cuda")
        s["target"] = torch.where(torch.rand(B, generator=g, **f) < 0.9, t, torch.full_like(t, -1))
        s["n_valid"] = int((s["target"] >= 0).sum())
        s["act"], s["logits"] = torch.empty((3, B, 32, L), **f), torch.empty((B, co, L), **f)
        s["dlogits"], s["loss"] = torch.empty((B, co, L), **f), torch.empty(B, **f)
        s["work"] = torch.empty(ltgw.ltgw_cnn_work_floats(B, ci, co, L), **f)
        s["grads"] = torch.empty(n, **f)
    else:
        geo = _geometry(dict(c, weighted=False), seed)
        fine, coarse = _propose_grids(c)
        s["stack"] = _exp_noise((c["R"], c["n_seg"], c["n_bins"]), 1000 * int(seed))
        _load(ctx, 0, s["stack"][0], geo, "f32")
        ltgw.ltgw_inject_stack(ctx.h, 0, s["stack"], _injections(c["R"], fine, (0.3, 3.0), r), fine["sky"][0])
        s["fine"], s["coarse"] = (ltgw.make_grid(g["f0_min"], g["f0_step"], g["n_f0"], g["tau"], g["brake"], g["sky"])
                                  for g in (fine, coarse))
        s["params"] = torch.from_numpy(_network_params(8, 24, seed, nearest_coarse_groups(fine, coarse))).cuda()
    return s


# ---- one pass --------------------------------------------------------------
def _ranked(ctx, k=K):
    out = {}
    for stat in ("power", "count"):
        top = ctx.topk(stat, k)
        out[stat + "_index"] = np.array([q["index"] for q in top], np.int64)
        out[stat + "_psi"] = np.array([q["psi"] for q in top], np.float64)
    return out


def run(state):
    s, c, kind, ctx = state, state["case"], state["kind"], state["ctx"]
    if kind == "search":
        for d in range(c["n_det"]):
            _load(ctx, d, s["power"][d], s["geo"][d], c["store"])
            if c["antenna"]:
                ctx.set_antenna(d, s["arms"][d], s["era"][d])
        sums = ctx.eval_templates(**s["grid"])
        return dict(zip("scN", sums), **_ranked(ctx))
    if kind == "bank":
        _load(ctx, 0, s["power"], s["geo"], c["store"])
        sums = ctx.eval_list(s["params"])
        return dict(zip("scN", sums), **_ranked(ctx))
    if kind == "prep":
        return ctx.sft_normalise(s["strain"], c["n_fft"], c["k_lo"], c["n_bins"], c["window"])
    if kind == "batch":
        top_p, top_c, _ = ctx.eval_batch(s["specs"], k=K)
        out = {}
        for i, q in enumerate(s["specs"]):
            n = q["n_f0"] * len(q["tau"]) * len(q["brake"]) * len(q["sky"])
            out["r%d" % i] = dict(zip(("s", "c", "N", "psi_power", "psi_count"), ctx.batch_results(i, n)))
        out["power_index"] = np.array([[q["index"] for q in t] for t in top_p], np.int64)
        out["count_index"] = np.array([[q["index"] for q in t] for t in top_c], np.int64)
        return out
    if kind == "campaign":
        noise = s["camp"].noise_maxima(c["R_noise"])
        near = s["camp"].injected_maxima(s["inj"])
        return dict(noise_power=noise[0], noise_count=noise[1], near_power=near[0], near_count=near[1])
    if kind == "network":
        h = ctx.h
        ltgw.ltgw_cnn_forward(h, s["params"], s["x"], c["c_out"], s["act"], s["logits"])
        ltgw.ltgw_softmax_xent(h, s["logits"], s["target"], max(s["n_valid"], 1), s["loss"], s["dlogits"])
        ltgw.ltgw_cnn_backward(h, s["params"], s["x"], c["c_out"], s["act"], s["dlogits"], s["work"], s["grads"])
        ltgw.ltgw_adam_step(h, s["params"], s["grads"], s["m"], s["v"], 2e-4, 0.9, 0.999, 1e-8, 100)
        return {k: s[k] for k in ("logits", "loss", "grads", "params", "m", "v")}
    ltgw.ltgw_load_stack(ctx.h, 0, s["stack"], c["store"], coarse=c["coarse_segments"])
    out = ltgw.ltgw_propose(ctx.h, s["fine"][0], s["coarse"][0], s["params"], 8, 24, c["n_f0"] // 2, c["n_select"], 5.2,
                            4.7, c["R"], block=c["block"], return_blocks=True)
    return dict(zip(("best_index", "best_psi", "fallback", "blocks"), out))


# ---- what a pass cannot do without ------------------------------------------
def _groups(c):
    return c["n_tau"] * c["n_brake"] * c.get("n_sky", 1)


def _evals(c):
    return c["n_f0"] * _groups(c) * c["n_seg"] * c["n_det"]


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: per template
    and segment the product and shift that give the column, the weighted sum
    and the count (6); a random bank's own track factor (12 more); 2.5 N log2 N
    per real transform; a multiply-add per weight."""
    c, kind = case, case["kind"]
    if kind == "search":
        return dict(bytes=4.0 * c["n_seg"] * c["n_bins"] * c["n_det"] + 12.0 * c["n_f0"] * _groups(c), flops=6.0 * _evals(c))
    if kind == "bank":
        return dict(bytes=4.0 * c["n_seg"] * c["n_bins"] + 60.0 * c["n_tpl"], flops=18.0 * c["n_tpl"] * c["n_seg"])
    if kind == "prep":
        return dict(bytes=4.0 * c["n_seg"] * (c["n_fft"] + c["n_bins"]),
                    flops=2.5 * c["n_seg"] * c["n_fft"] * math.log2(c["n_fft"]))
    if kind == "batch":
        b = _batch_specs(c, 0)
        tpl = [q["n_bins"] * 12 * len(q["grid"]["sky"]) for q in b]
        return dict(bytes=sum(8.0 * q["n_seg"] * q["n_bins"] * (1 if c["store"] == "f32" else 0.5) + 28.0 * n
                              for q, n in zip(b, tpl)),
                    flops=sum(12.0 * n * q["n_seg"] for q, n in zip(b, tpl)))
    if kind == "campaign":
        px, n = c["n_seg"] * c["n_bins"], c["n_f0"] * _groups(c) * c["n_seg"]
        return dict(bytes=4.0 * px * (c["R_noise"] + c["R_inj"]),
                    flops=6.0 * n * c["R_noise"] + 6.0 * 45 * c["n_seg"] * c["R_inj"])
    if kind == "network":
        n = c["B"] * c["L"]
        macs = n * 32 * (5 * c["c_in"] + 2 * 160 + c["c_out"])
        return dict(bytes=4.0 * n * (c["c_in"] + 2 * 96 + 3 * c["c_out"]), flops=6.0 * macs - 2.0 * n * 160 * c["c_in"])
    n_cells = c["n_f0"] * 12
    e = c["R"] * c["n_seg"] * (min(c["n_select"], n_cells) + c["n_f0"] // 2 * 4 / c["coarse_segments"])
    return dict(bytes=4.0 * c["R"] * c["n_seg"] * c["n_bins"], flops=6.0 * e)


# ---- the same in 64 bits -----------------------------------------------------
def _antenna_response(arms, era, sky):
    """F+^2 + Fx^2 [n_sky][n_seg] from an explicit polarisation basis."""
    out = np.empty((len(sky), len(era)))
    for i, n in enumerate(sky):
        ra, de = math.atan2(n[1], n[0]), math.asin(max(-1.0, min(1.0, n[2])))
        ex = np.array([math.sin(ra), -math.cos(ra), 0.0])
        ey = np.array([-math.cos(ra) * math.sin(de), -math.sin(ra) * math.sin(de), math.cos(de)])
        co, si = np.cos(era), np.sin(era)
        rot = [np.stack([co * a[0] - si * a[1], si * a[0] + co * a[1], np.full_like(co, a[2])], axis=1) for a in arms]
        ax, ay, bx, by = rot[0] @ ex, rot[0] @ ey, rot[1] @ ex, rot[1] @ ey
        fp, fx = 0.5 * ((ax**2 - ay**2) - (bx**2 - by**2)), ax * ay - bx * by
        out[i] = fp**2 + fx**2
    return out


def _sums(dets, f0, tau, brake, sky, lattice):
    """s, W1, W2, c, N in 64 bits of templates over detectors [(power, geo,
    response or None)]: a lattice (f0 axis times groups (sky, n, tau)), or rows."""
    dev = dict(dtype=torch.float64, device="cuda")
    f0, tau, brake, sky = (torch.as_tensor(a, **dev) for a in (f0, tau, brake, sky))
    n_sky = sky.shape[0]
    shape = (n_sky * brake.numel() * tau.numel(), f0.numel()) if lattice else (f0.numel(),)
    s, w1, w2, cn, nn = (torch.zeros(shape, **dev) for _ in range(5))
    e = 1.0 / (1.0 - brake)
    for power, geo, resp in dets:
        t, v, T = (torch.as_tensor(a, **dev) for a in (geo["t"], geo["v"], geo["t_sft"]))
        w = torch.ones(len(geo["t"]), **dev) if geo["w"] is None else torch.as_tensor(geo["w"], **dev)
        resp = None if resp is None else torch.as_tensor(resp, **dev)
        nb = power.shape[1]
        for j in range(power.shape[0]):
            u = 1.0 + t[j] / tau
            D = 1.0 + ((v[j, 0] * sky[:, 0] + v[j, 1] * sky[:, 1]) + v[j, 2] * sky[:, 2]) / C_LIGHT
            if lattice:
                H = ((u[None, :] ** e[:, None]).reshape(1, -1) * D[:, None]).reshape(-1, 1) * T
                x = f0[None, :] * H
            else:
                x = f0 * ((u ** e) * D * T)
            b = torch.floor(x + 0.5).to(torch.int64) - geo["k_lo"]
            inb = ((b >= 0) & (b < nb)).to(torch.float64)
            p = power[j][b.clamp(0, nb - 1)].to(torch.float64) * inb
            wj = w[j] if resp is None else (w[j] * resp[:, j]).repeat_interleave(shape[0] // n_sky)[:, None]
            s += wj * p
            w1 += wj * inb
            w2 += wj * wj * inb
            cn += (p > RHO_TH).to(torch.float64)
            nn += inb
    return tuple(a.reshape(-1) for a in (s, w1, w2, cn, nn))


def _ratios(s, w1, w2, cn, nn):
    q = math.exp(-float(np.float32(RHO_TH)))
    return (s - w1) / torch.sqrt(w2), (cn - nn * q) / torch.sqrt(nn * q * (1 - q))


def _exact_ranked(sums, k=K):
    out = {}
    for stat, psi in zip(("power", "count"), _ratios(*sums)):
        psi = torch.where(torch.isnan(psi), torch.full_like(psi, -math.inf), psi)
        out[stat + "_index"] = None
        out[stat + "_psi"] = torch.topk(psi, min(k, int((psi > -math.inf).sum())))[0].cpu().numpy()
    return dict(out, s=sums[0], c=None, N=None)


def _exact_prep(c, strain):
    N, h = c["n_fft"], c["window"] // 2
    win = 0.5 - 0.5 * torch.cos(2 * math.pi * torch.arange(N, dtype=torch.float64, device="cuda") / N)
    out = torch.empty((c["n_seg"], c["n_bins"]), dtype=torch.float64, device="cuda")
    rows = max(1, (1 << 26) // (c["n_bins"] * c["window"]))
    for j in range(0, c["n_seg"], rows):
        x = strain[j * N:(j + rows) * N].reshape(-1, N).double() * win
        P = torch.fft.rfft(x).abs().square()[:, c["k_lo"] - h:c["k_lo"] + c["n_bins"] + h]
        med = P.unfold(1, c["window"], 1).sort(dim=2)[0][:, :, h]
        out[j:j + rows] = P[:, h:h + c["n_bins"]] * math.log(2.0) / med
    return out


def _exact_network(c, s):
    B, ci, co, L = c["B"], c["c_in"], c["c_out"], c["L"]
    p = s["params"].double().requires_grad_(True)
    at, W = 0, []
    for o, i, k in ((32, ci, 5), (32, 32, 5), (32, 32, 5), (co, 32, 1)):
        W.append((p[at:at + o * i * k].reshape(o, i * k), p[at + o * i * k:at + o * i * k + o], k))
        at += o * i * k + o
    x = s["x"].double()
    for n, (w, b, k) in enumerate(W):  # each convolution as one product over unfolded positions
        cols = torch.nn.functional.pad(x, (k // 2, k // 2)).unfold(2, k, 1).permute(0, 2, 1, 3).reshape(B * L, -1)
        x = (cols @ w.t() + b).reshape(B, L, -1).permute(0, 2, 1)
        x = torch.relu(x) if n < 3 else x
    logits, tg = x.reshape(B, -1), s["target"].long()
    loss = torch.where(tg >= 0, torch.logsumexp(logits, 1) - logits.gather(1, tg.clamp(min=0)[:, None])[:, 0],
                       torch.zeros(B, dtype=torch.float64, device="cuda"))
    (grad,) = torch.autograd.grad(loss.sum() / max(s["n_valid"], 1), p)
    m, v = 0.9 * s["m"].double() + 0.1 * grad, 0.999 * s["v"].double() + 0.001 * grad * grad
    step = (m / (1 - 0.9**100)) / (torch.sqrt(v / (1 - 0.999**100)) + 1e-8)
    return dict(logits=x.detach().contiguous(), loss=loss.detach(), grads=grad, params=p.detach() - 2e-4 * step, m=m, v=v)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "propose" or kind == "campaign":
        return None  # the outputs rest on choices of the network, and on the library's own noise
    if kind == "prep" and c["n_seg"] * c["n_bins"] * c["window"] > 4e9:
        return None
    s = prepare(dict(case, tune=False), seed)
    if kind == "search":
        g = s["grid"]
        resp = [_antenna_response(a, e, g["sky"]) for a, e in zip(s["arms"], s["era"])] if c["antenna"] else [None] * 2
        f0 = g["f0_min"] + np.arange(g["n_f0"]) * g["f0_step"]
        return _exact_ranked(_sums(list(zip(s["power"], s["geo"], resp)), f0, g["tau"], g["brake"], g["sky"], True))
    if kind == "bank":
        p = s["params"]
        return _exact_ranked(_sums([(s["power"], s["geo"], None)], p[:, 0], p[:, 1], p[:, 2], p[:1, 3:], False))
    if kind == "prep":
        return _exact_prep(c, s["strain"])
    if kind == "network":
        return _exact_network(c, s)
    out = dict(power_index=None, count_index=None)
    for i, b in enumerate(_batch_specs(c, seed)):
        g = b["grid"]
        dets = [(_exp_noise((b["n_seg"], b["n_bins"]), 1000 * int(seed) + 2 * i + d), _geometry(b, seed, d), None)
                for d in range(2)]
        f0 = g["f0_min"] + np.arange(g["n_f0"]) * g["f0_step"]
        sums = _sums(dets, f0, g["tau"], g["brake"], g["sky"], True)
        pp, pc = _ratios(*sums)
        out["r%d" % i] = dict(s=sums[0], c=None, N=None, psi_power=pp, psi_count=pc)
    return out
