"""In-band moments (N, W1, W2) of a lattice at the edges of their kernel: parts of
4096 f0 (uniform weights) or 1024 (weighted), a step of zero and one far below a bin
(where the in-band range is searched for, not computed), two detectors.  N is the
oracle's; both ratios, which carry W1 and W2, agree to the bars of the parity tests."""
import numpy as np
import pytest

import oracle
from gpu_util import psi_tolerance

pytestmark = pytest.mark.gpu

SKY = np.array([0.6, 0.0, 0.8])


@pytest.mark.parametrize("n_f0,step,weighted,dets", [
    (1, 0.25, False, 1),
    (1023, 0.25, True, 1),
    (1025, 0.25, True, 2),
    (4096, 0.0625, False, 2),
    (4097, 0.0625, False, 1),
    (2049, 0.03125, True, 2),
    (70, 0.0, True, 1),
    (300, 1e-13, False, 2),
])
def test_moments_at_part_edges(n_f0, step, weighted, dets):
    import torch
    from paper_2507_07816_amd import ltgw

    print(f"case: moments n_f0 {n_f0} step {step} weighted {weighted} dets {dets}", flush=True)
    ns, nb, k_lo, t_sft = 41, 230, 1880, 4.0
    r = np.random.default_rng(n_f0)
    ctx = ltgw.Context(0)
    od = []
    for d in range(dets):
        t = np.arange(ns) * 90.0 + 2.0 + d
        v = r.normal(size=(ns, 3))
        v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
        w = r.uniform(0.5, 2.0, ns).astype(np.float32) if weighted else None
        P = r.exponential(size=(ns, nb)).astype(np.float32)
        ctx.load_spectrogram(d, torch.from_numpy(P).cuda(), k_lo, t_sft, t, weights=w)
        ctx.set_velocity_table(d, v)
        od.append(oracle.Detector(P, t, v, k_lo, t_sft, weights=w))
    g = dict(f0_min=(k_lo + 20) / t_sft, f0_step=step, n_f0=n_f0, tau=[4000.0, 30000.0], brake=[3.0, 5.0], sky=[SKY],
             t0=0.0)
    s, c, N = ctx.eval_templates(**g, det_mask=(1 << dets) - 1)
    pp, pc = ctx.psi("power", n_f0 * 4).cpu().numpy(), ctx.psi("count", n_f0 * 4).cpu().numpy()
    got = N.cpu().numpy().reshape(-1)
    ctx.close()
    ref = oracle.evaluate(od if dets > 1 else od[0], oracle.Grid(*[g[k] for k in ("f0_min", "f0_step", "n_f0", "tau",
                                                                                "brake", "sky", "t0")]))
    assert np.array_equal(got, ref["N"].reshape(-1))
    po, co = oracle.psi_power(ref).reshape(-1), oracle.psi_count(ref).reshape(-1)
    ok = np.isfinite(po)
    assert np.array_equal(ok, np.isfinite(pp)) and np.array_equal(np.isfinite(co), np.isfinite(pc))
    assert np.all(np.abs(pp[ok] - po[ok]) <= psi_tolerance(ref).reshape(-1)[ok])
    okc = np.isfinite(co)
    assert np.all(np.abs(pc[okc] - co[okc]) <= 1e-12 * (1 + np.abs(co[okc])))


@pytest.mark.parametrize("n_f0,weighted,dets,ns,groups", [
    (1, False, 1, 41, 2048), (512, False, 2, 41, 2048), (513, False, 1, 300, 2048),  # parts of 512 f0
    (128, True, 1, 300, 2048), (129, True, 2, 41, 2048),                             # of 128 with weights
    (3, False, 1, 65, 4097), (2, True, 2, 41, 9000),        # a workgroup with one of its eight groups
    (4097, False, 1, 5, 2049), (1025, True, 1, 5, 2049),    # two parts, of 4096 and 1024
])
def test_moments_of_many_groups(n_f0, weighted, dets, ns, groups):
    """2048 groups, from which on a wavefront takes a group and a workgroup eight."""
    import torch
    from paper_2507_07816_amd import ltgw

    print(f"case: moments of {groups} groups, n_f0 {n_f0} weighted {weighted} dets {dets} segments {ns}", flush=True)
    nb, k_lo, t_sft = 60, 1880, 4.0
    r = np.random.default_rng(n_f0)
    ctx = ltgw.Context(0)
    od = []
    for d in range(dets):
        t = np.arange(ns) * (3600.0 / ns) + 2.0 + d
        v = r.normal(size=(ns, 3))
        v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
        w = r.uniform(0.5, 2.0, ns).astype(np.float32) if weighted else None
        P = r.exponential(size=(ns, nb)).astype(np.float32)
        ctx.load_spectrogram(d, torch.from_numpy(P).cuda(), k_lo, t_sft, t, weights=w)
        ctx.set_velocity_table(d, v)
        od.append(oracle.Detector(P, t, v, k_lo, t_sft, weights=w))
    g = dict(f0_min=(k_lo + 20) / t_sft, f0_step=20.0 / n_f0, n_f0=n_f0, tau=np.geomspace(2000.0, 60000.0, groups // 2 if groups % 2 == 0 else groups),
             brake=[3.0, 5.0] if groups % 2 == 0 else [4.0], sky=[SKY], t0=0.0)
    s, c, N = ctx.eval_templates(**g, det_mask=(1 << dets) - 1)
    pp = ctx.psi("power", n_f0 * groups).cpu().numpy()
    got, total = N.cpu().numpy().reshape(-1), ctx.diagnostics()["in_band"]
    ctx.close()
    ref = oracle.evaluate(od if dets > 1 else od[0], oracle.Grid(*[g[k] for k in ("f0_min", "f0_step", "n_f0", "tau",
                                                                                "brake", "sky", "t0")]))
    assert np.array_equal(got, ref["N"].reshape(-1)) and total == int(ref["N"].sum())
    po = oracle.psi_power(ref).reshape(-1)
    ok = np.isfinite(po)
    assert np.array_equal(ok, np.isfinite(pp))
    assert np.all(np.abs(pp[ok] - po[ok]) <= psi_tolerance(ref).reshape(-1)[ok])
