"""GPU tests of the learned proposer's path through the C-ABI.

- Exp(1) noise from the device's Philox4x32-10 equals the oracle's (the FP64
  logarithms may differ in their last bit: at most one FP32 ulp apart);
- injected stacks put amp * w at the oracle's track bins and nowhere else;
- fine and coarse critical ratios of a stack against the oracle per
  realisation; listed ratios bit-identical to the full ones, NaN for indices
  outside the grid;
- the network's forward and backward passes against the FP64 reference
  with the same BF16 operand rounding (and loosely against plain FP64);
  softmax cross-entropy, Adam and top-M selection against their definitions;
- propose: with every cell selected it finds the oracle's exhaustive best;
  with a partial selection it equals the composition of the public calls;
  the fallback rule and its exhaustive evaluation.
"""
import numpy as np
import pytest

import oracle
from oracle import cnn
from oracle import proposer as op
from gpu_util import psi_tolerance

pytestmark = pytest.mark.gpu

N_SEG, N_BINS, K_LO, T_SFT = 96, 192, 1880, 4.0
SKY = np.array([0.6, 0.0, 0.8])
FINE = dict(f0_min=478.0, f0_step=0.25, n_f0=48, tau=[4000.0, 15000.0], brake=[3.0, 5.0],
            sky=[SKY], t0=0.0)
COARSE = dict(f0_min=478.0, f0_step=0.5, n_f0=24, tau=[4000.0, 15000.0], brake=[3.0, 5.0],
              sky=[SKY], t0=0.0)


def _geometry(seed=0, weights=True):
    r = np.random.default_rng(seed)
    t = np.arange(N_SEG) * 40.0 + 2.0
    v = r.normal(size=(N_SEG, 3))
    v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
    w = r.uniform(0.5, 2.0, N_SEG).astype(np.float32) if weights else None
    return t, v, w


def _ctx(weights=True):
    import torch
    from paper_2507_07816_amd import ltgw

    ctx = ltgw.Context(0)
    t, v, w = _geometry(weights=weights)
    ctx.load_spectrogram(0, torch.zeros((N_SEG, N_BINS), dtype=torch.float32, device="cuda"), K_LO, T_SFT, t,
                         weights=w)
    ctx.set_velocity_table(0, v)
    return ctx, t, v, w


def _grid(d):
    from paper_2507_07816_amd import ltgw
    return ltgw.make_grid(d["f0_min"], d["f0_step"], d["n_f0"], d["tau"], d["brake"], d["sky"], d["t0"])


def _ogrid(d):
    return oracle.Grid(d["f0_min"], d["f0_step"], d["n_f0"], d["tau"], d["brake"], d["sky"], d["t0"])


def _stack(ctx, R, inj, seed=11):
    """Noise stack with injections inj[r] = (f0, tau, brake, amp) -> device tensor."""
    import torch
    from paper_2507_07816_amd import ltgw

    st = torch.empty((R, N_SEG, N_BINS), dtype=torch.float32, device="cuda")
    ltgw.ltgw_generate_noise(ctx.h, seed, 0, 0, st)
    ltgw.ltgw_inject_stack(ctx.h, 0, st, np.asarray(inj, np.float64), SKY, 0.0)
    return st


def _oracle_stack(R, inj, t, v, w, seed=11):
    out = []
    for r in range(R):
        P = oracle.exp_noise(seed, 0, r, N_SEG * N_BINS).reshape(N_SEG, N_BINS).copy()
        f0, tau, brake, amp = inj[r]
        if amp > 0:
            det = oracle.Detector(P, t, v, K_LO, T_SFT, weights=w)
            b = oracle.track_bins(det, f0, tau, brake, SKY, 0.0)
            ww = np.ones(N_SEG, np.float32) if w is None else w
            for j in range(N_SEG):
                if 0 <= b[j] < N_BINS:
                    P[j, b[j]] = np.float32(P[j, b[j]] + np.float32(np.float32(amp) * ww[j]))
        out.append(P)
    return out


# (f0, tau, n, amp): the first is a template of the fine grid and stays in
# band for about 60 of the 96 segments, the third is off the grid and leaves
# the band early; the second realisation is noise only
INJ = [(488.0, 15000.0, 5.0, 6.0), (0.0, 0.0, 0.0, 0.0), (486.25, 12000.0, 3.0, 2.0)]


def test_noise_matches_oracle():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    print("case: noise seed 987654321 stream 3 r0 5 R 3 n 10001", flush=True)
    out = torch.empty((3, 10001), dtype=torch.float32, device="cuda")
    ltgw.ltgw_generate_noise(ctx.h, 987654321, 3, 5, out)
    g = out.cpu().numpy()
    for i in range(3):
        ref = oracle.exp_noise(987654321, 3, 5 + i, 10001)
        diff = np.abs(g[i].view(np.int32).astype(np.int64) - ref.view(np.int32).astype(np.int64))
        assert diff.max() <= 1 and (diff > 0).sum() <= 2
    ctx.close()


@pytest.mark.parametrize("n,offset", [(1 << 20, 0), (1 << 18, 1), (4099, 2), (1, 0)])
def test_noise_layouts(n, offset):
    """Whole groups of four on and off a 16-byte boundary, and ragged rows; the bar is
    test_noise_matches_oracle's (the FP64 logarithms may round one value in 10^4
    differently), and nothing is written outside the rows."""
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    print(f"case: noise layout n {n} offset {offset}", flush=True)
    buf = torch.full((offset + 2 * n + 4,), -1.0, dtype=torch.float32, device="cuda")
    ltgw.ltgw_generate_noise(ctx.h, 24680, 1, 2, buf[offset:offset + 2 * n].view(2, n))
    g = buf.cpu().numpy()
    ctx.close()
    assert np.all(g[:offset] == -1.0) and np.all(g[offset + 2 * n:] == -1.0)
    for i in range(2):
        ref = oracle.exp_noise(24680, 1, 2 + i, n)
        diff = np.abs(g[offset + i * n:offset + (i + 1) * n].view(np.int32).astype(np.int64) -
                      ref.view(np.int32).astype(np.int64))
        assert diff.max() <= 1 and (diff > 0).sum() <= 1 + n // 10000


def test_inject_stack_matches_oracle_bins():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, t, v, w = _ctx()
    st = torch.zeros((3, N_SEG, N_BINS), dtype=torch.float32, device="cuda")
    ltgw.ltgw_inject_stack(ctx.h, 0, st, np.asarray(INJ, np.float64), SKY, 0.0)
    g = st.cpu().numpy()
    det = oracle.Detector(np.zeros((N_SEG, N_BINS), np.float32), t, v, K_LO, T_SFT, weights=w)
    for r, (f0, tau, brake, amp) in enumerate(INJ):
        ref = np.zeros((N_SEG, N_BINS), np.float32)
        if amp > 0:
            b = oracle.track_bins(det, f0, tau, brake, SKY, 0.0)
            for j in range(N_SEG):
                if 0 <= b[j] < N_BINS:
                    ref[j, b[j]] = np.float32(amp) * w[j]
        assert np.array_equal(g[r], ref), r
    ctx.close()


@pytest.mark.parametrize("weights,S", [(True, 2), (False, 2), (True, 4), (True, 8)])
def test_stack_psi_fine_and_coarse_vs_oracle(weights, S):
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, t, v, w = _ctx(weights)
    R = len(INJ)
    print(f"case: stack psi weights={weights} coarse segments {S}", flush=True)
    st = _stack(ctx, R, INJ)
    ref_stack = _oracle_stack(R, INJ, t, v, w)
    host = st.cpu().numpy()
    for r in range(R):   # the device stack is the oracle's up to the last bit of a logarithm
        d = np.abs(host[r].view(np.int32).astype(np.int64) - ref_stack[r].view(np.int32).astype(np.int64))
        assert d.max() <= 1
    ltgw.ltgw_load_stack(ctx.h, 0, st, "f32", coarse=S)
    fg, keep_f = _grid(FINE)
    cg, keep_c = _grid(COARSE)
    n_f, n_c = _ogrid(FINE).n_templates, _ogrid(COARSE).n_templates
    pf = torch.empty((R, n_f), dtype=torch.float64, device="cuda")
    pc = torch.empty((R, n_c), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi(ctx.h, fg, 0, pf)
    ltgw.ltgw_stack_psi(ctx.h, cg, 1, pc)
    x = torch.empty((R, 2 * 4, COARSE["n_f0"]), dtype=torch.float32, device="cuda")
    ltgw.ltgw_stack_features(ctx.h, cg, x, counts=True)
    x = x.cpu().numpy()
    pf, pc = pf.cpu().numpy(), pc.cpu().numpy()
    # the fine store written beside the coarse one is the fine store alone, bit
    # for bit, in every format (its ratios are identical)
    for store in ("bf16", "fp8", "f32"):
        a = torch.empty((R, n_f), dtype=torch.float64, device="cuda")
        b = torch.empty((R, n_f), dtype=torch.float64, device="cuda")
        ltgw.ltgw_load_stack(ctx.h, 0, st, store, coarse=0)
        ltgw.ltgw_stack_psi(ctx.h, fg, 0, a)
        ltgw.ltgw_load_stack(ctx.h, 0, st, store, coarse=S)
        ltgw.ltgw_stack_psi(ctx.h, fg, 0, b)
        assert np.array_equal(a.cpu().numpy().view(np.uint64), b.cpu().numpy().view(np.uint64)), store
    ltgw.ltgw_load_stack(ctx.h, 0, st, "f32", coarse=S)
    for r in range(R):
        det = oracle.Detector(ref_stack[r], t, v, K_LO, T_SFT, weights=w)
        ref = oracle.evaluate(det, _ogrid(FINE))
        psi = oracle.psi_power(ref)
        ok = np.isfinite(psi)
        assert np.array_equal(ok, np.isfinite(pf[r]))
        assert np.all(np.abs(pf[r][ok] - psi[ok]) <= psi_tolerance(ref)[ok])
        cref = op.coarse_psi(det, _ogrid(COARSE), ref_stack[r], S=S)
        okc = np.isfinite(cref)
        assert np.array_equal(okc, np.isfinite(pc[r]))
        assert np.allclose(pc[r][okc], cref[okc], rtol=0, atol=2e-5 * (1 + np.abs(cref[okc])))
        # the network's input: power ratios, then count ratios (integer counts:
        # the ratio is the oracle's up to its FP32 rounding)
        nref = op.coarse_psi_count(det, _ogrid(COARSE), ref_stack[r], nan_to_zero=True, S=S)
        xr = x[r].reshape(2, -1)
        assert np.array_equal(xr[0], np.where(np.isfinite(pc[r]), pc[r], 0.0).astype(np.float32))
        assert np.array_equal(xr[1], nref.astype(np.float32))
    # the injected realisation peaks near its injection (tau, n off the grid:
    # the best template trades a little f0 for them), far above the noise-only one
    f_idx = int(np.nanargmax(pf[0]))
    f0, tau, brake, _ = _ogrid(FINE).params(f_idx)
    assert abs(f0 - INJ[0][0]) <= 2.0 and np.nanmax(pf[0]) > 2 * np.nanmax(pf[1])
    ctx.close()


def test_stack_psi_list_is_bit_identical_and_nan_outside():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    R = len(INJ)
    st = _stack(ctx, R, INJ)
    for store in ("f32", "bf16", "fp8"):
        print(f"case: list psi store {store}", flush=True)
        ltgw.ltgw_load_stack(ctx.h, 0, st, store, coarse=False)
        fg, keep = _grid(FINE)
        n = _ogrid(FINE).n_templates
        full = torch.empty((R, n), dtype=torch.float64, device="cuda")
        ltgw.ltgw_stack_psi(ctx.h, fg, 0, full)
        rng = np.random.default_rng(4)
        idx = rng.integers(0, n, size=(R, 300)).astype(np.int32)
        idx[:, 7] = -1
        idx[:, 8] = n
        out = torch.empty((R, 300), dtype=torch.float64, device="cuda")
        ltgw.ltgw_stack_psi_list(ctx.h, fg, torch.from_numpy(idx).cuda(), out)
        f, o = full.cpu().numpy(), out.cpu().numpy()
        for r in range(R):
            good = (idx[r] >= 0) & (idx[r] < n)
            assert np.array_equal(o[r][good], f[r][idx[r][good]], equal_nan=True)
            assert np.all(np.isnan(o[r][~good]))
    with pytest.raises(ltgw.LtgwError):   # no coarse store loaded
        ltgw.ltgw_stack_psi(ctx.h, _grid(COARSE)[0], 1, torch.empty((R, 96), dtype=torch.float64, device="cuda"))
    ctx.close()


@pytest.mark.parametrize("ns,nb,store", [(94, 189, "bf16"), (94, 188, "bf16"), (96, 190, "fp8"), (94, 188, "f32")])
def test_stack_store_against_oracle_odd_shape(ns, nb, store):
    """Stacks of 94 or 96 segments x 188 to 190 bins (neither a multiple of
    16; odd bins take the one-row ingest, even ones the blocked ingest of 2 or
    4 rows per workgroup), a bright pixel in the last segment and bin, BF16,
    FP8 and FP32 stores: every template's ratio matches the oracle on the
    values the store holds, and the listed evaluation of every template
    equals the full one bit for bit."""
    import torch
    from paper_2507_07816_amd import ltgw

    print(f"case: stack store {store} {ns} x {nb}", flush=True)
    r = np.random.default_rng(31)
    t = np.arange(ns) * 40.0 + 2.0
    v = r.normal(size=(ns, 3))
    v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
    w = r.uniform(0.5, 2.0, ns).astype(np.float32)
    ctx = ltgw.Context(0)
    ctx.load_spectrogram(0, torch.zeros((ns, nb), dtype=torch.float32, device="cuda"), K_LO, T_SFT, t, weights=w)
    ctx.set_velocity_table(0, v)
    R = 3
    P = r.exponential(size=(R, ns, nb)).astype(np.float32)
    P[0, 10, 50] = 40.0
    P[2, ns - 1, nb - 1] = 30.0                      # the last segment's last bin
    ltgw.ltgw_load_stack(ctx.h, 0, torch.from_numpy(P).cuda(), store, coarse=False)
    fg, keep = _grid(FINE)
    g = _ogrid(FINE)
    n = g.n_templates
    full = torch.empty((R, n), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi(ctx.h, fg, 0, full)
    f = full.cpu().numpy()
    for q in range(R):
        vals, _ = oracle.dequantised(P[q], store)
        ref = oracle.evaluate(oracle.Detector(P[q], t, v, K_LO, T_SFT, weights=w, values=vals), g)
        psi = oracle.psi_power(ref)
        ok = np.isfinite(psi)
        assert ok.sum() > 50 and np.array_equal(ok, np.isfinite(f[q]))
        assert np.all(np.abs(f[q][ok] - psi[ok]) <= psi_tolerance(ref)[ok])
    idx = np.tile(np.arange(n, dtype=np.int32), (R, 1))
    out = torch.empty((R, n), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi_list(ctx.h, fg, torch.from_numpy(idx).cuda(), out)
    assert np.array_equal(out.cpu().numpy(), f, equal_nan=True)
    ctx.close()


@pytest.mark.parametrize("ns,nb,n_f0,R,store", [
    (1, 65, 1, 1, "f32"),
    (31, 190, 65, 3, "bf16"),
    (33, 189, 63, 2, "fp8"),
    (512, 190, 64, 5, "f32"),      # 16 chunks of segments
    (513, 64, 130, 3, "bf16"),     # and one segment more
    (1057, 131, 257, 9, "f32"),
    (37, 1022, 1000, 126, "f32"),  # two realisations per workgroup: the widest row it holds
    (66, 61, 1000, 211, "bf16"),   # an odd count of them
])
def test_stack_sums_over_segments_and_rows(ns, nb, n_f0, R, store):
    """Both ratios of every template, in full and as a list, at the edges of the
    chunks of segments, of the 64 f0 of a wavefront and of odd counts of realisations:
    the oracle's on the values the store holds (counts exact, so that ratio to 1e-12),
    and the list bit for bit what the whole grid gives."""
    import torch
    from paper_2507_07816_amd import ltgw

    print(f"case: stack sums {store} {R} x {ns} x {nb}, {n_f0} f0", flush=True)
    r = np.random.default_rng(ns)
    t = np.arange(ns) * (3840.0 / max(ns, 96)) + 2.0
    v = r.normal(size=(ns, 3))
    v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
    w = r.uniform(0.5, 2.0, ns).astype(np.float32)
    ctx = ltgw.Context(0)
    ctx.load_spectrogram(0, torch.zeros((ns, nb), dtype=torch.float32, device="cuda"), K_LO, T_SFT, t, weights=w)
    ctx.set_velocity_table(0, v)
    P = r.exponential(size=(R, ns, nb)).astype(np.float32)
    ltgw.ltgw_load_stack(ctx.h, 0, torch.from_numpy(P).cuda(), store, coarse=False)
    d = dict(f0_min=(K_LO - 2) / T_SFT, f0_step=0.25, n_f0=n_f0, tau=[4000.0, 15000.0, 60000.0], brake=[3.0, 5.0],
             sky=[SKY], t0=0.0)
    fg, keep = _grid(d)
    g = _ogrid(d)
    n = g.n_templates
    full = torch.empty((R, n), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi(ctx.h, fg, 0, full)
    f = full.cpu().numpy()
    idx = torch.from_numpy(np.tile(np.arange(n, dtype=np.int32), (R, 1))).cuda()
    lists = {}
    for stat in ("power", "count"):
        out = torch.empty((R, n), dtype=torch.float64, device="cuda")
        ltgw.ltgw_stack_psi_list(ctx.h, fg, idx, out, stat=stat)
        lists[stat] = out.cpu().numpy()
        bi = torch.empty(R, dtype=torch.int32, device="cuda")
        bp = torch.empty(R, dtype=torch.float64, device="cuda")
        ltgw.ltgw_stack_best(ctx.h, fg, bi, bp, stat=stat)
        best = np.where(np.isnan(lists[stat]), -np.inf, lists[stat])
        assert np.array_equal(bp.cpu().numpy(), best.max(axis=1))
        lists[stat + " best"] = bi.cpu().numpy(), bp.cpu().numpy()
    bi = torch.empty((2, R), dtype=torch.int32, device="cuda")
    bp = torch.empty((2, R), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_best_both(ctx.h, fg, bi[0], bp[0], bi[1], bp[1])
    for k, stat in enumerate(("power", "count")):
        assert np.array_equal(bi[k].cpu().numpy(), lists[stat + " best"][0])
        assert np.array_equal(bp[k].cpu().numpy(), lists[stat + " best"][1])
    assert np.array_equal(lists["power"], f, equal_nan=True)
    for q in range(R) if R < 16 else (0, R - 1):
        vals, _ = oracle.dequantised(P[q], store)
        ref = oracle.evaluate(oracle.Detector(P[q], t, v, K_LO, T_SFT, weights=w, values=vals), g)
        psi, pc = oracle.psi_power(ref), oracle.psi_count(ref)
        ok = np.isfinite(psi)
        assert ok.sum() >= min(n_f0 - 2, 1) and np.array_equal(ok, np.isfinite(f[q]))
        assert np.all(np.abs(f[q][ok] - psi[ok]) <= psi_tolerance(ref)[ok])
        okc = np.isfinite(pc)
        assert np.array_equal(okc, np.isfinite(lists["count"][q]))
        assert np.all(np.abs(lists["count"][q][okc] - pc[okc]) <= 1e-12 * (1 + np.abs(pc[okc])))
    ctx.close()


def _net(seed, c_in, c_out):
    p = cnn.init_params(c_in, c_out, seed).astype(np.float64)
    p += np.random.default_rng(seed + 1).normal(scale=0.05, size=p.size)
    return p.astype(np.float32)


def _rel(a, b):
    return np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30)


def test_cnn_forward_backward_vs_oracle():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    B, c_in, c_out, L = 3, 4, 6, 37
    print(f"case: cnn B={B} c_in={c_in} c_out={c_out} L={L}", flush=True)
    assert ltgw.ltgw_cnn_param_count(c_in, c_out) == cnn.n_params(c_in, c_out)
    params = _net(5, c_in, c_out)
    rng = np.random.default_rng(8)
    x = rng.normal(size=(B, c_in, L)).astype(np.float32)
    dz = rng.normal(scale=0.1, size=(B, c_out, L)).astype(np.float32)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    pd, xd, dzd = T(params), T(x), T(dz)
    act = torch.empty((3, B, 32, L), dtype=torch.float32, device="cuda")
    logits = torch.empty((B, c_out, L), dtype=torch.float32, device="cuda")
    ltgw.ltgw_cnn_forward(ctx.h, pd, xd, c_out, act, logits)
    work = torch.empty(ltgw.ltgw_cnn_work_floats(B, c_in, c_out, L), dtype=torch.float32, device="cuda")
    grads = torch.empty(params.size, dtype=torch.float32, device="cuda")
    ltgw.ltgw_cnn_backward(ctx.h, pd, xd, c_out, act, dzd, work, grads)
    z = logits.cpu().numpy().astype(np.float64)
    g = grads.cpu().numpy().astype(np.float64)
    zr, cache = cnn.forward(params, x, c_in, c_out, rnd=cnn.bf16_operands)
    gr = cnn.backward(params, cache, dz.astype(np.float64), c_in, c_out, rnd=cnn.bf16_operands)
    assert _rel(z, zr) < 2e-3
    z64, c64 = cnn.forward(params, x, c_in, c_out)
    assert _rel(z, z64) < 5e-2
    off = 0
    for shp in cnn.layer_shapes(c_in, c_out):
        n = int(np.prod(shp))
        assert _rel(g[off:off + n], gr[off:off + n]) < 5e-3, shp
        off += n
    g64 = cnn.backward(params, c64, dz.astype(np.float64), c_in, c_out)
    assert _rel(g, g64) < 0.15          # BF16 operands against exact FP64: a sanity bound
    # deterministic
    grads2 = torch.empty_like(grads)
    ltgw.ltgw_cnn_backward(ctx.h, pd, xd, c_out, act, dzd, work, grads2)
    assert torch.equal(grads, grads2)
    # inference without activations (one fused pass): the same logits bit for bit,
    # up to the largest supported shape; beyond it the call is refused
    for (Bi, ci, co, Li) in ((B, c_in, c_out, L), (5, 4, 24, 200), (2, 32, 32, 256), (3, 7, 9, 1)):
        print(f"case: fused inference B={Bi} c_in={ci} c_out={co} L={Li}", flush=True)
        pi = T(_net(9, ci, co))
        xi = T(rng.normal(size=(Bi, ci, Li)).astype(np.float32))
        ai = torch.empty((3, Bi, 32, Li), dtype=torch.float32, device="cuda")
        z1 = torch.empty((Bi, co, Li), dtype=torch.float32, device="cuda")
        z2 = torch.full((Bi, co, Li), float("nan"), dtype=torch.float32, device="cuda")
        ltgw.ltgw_cnn_forward(ctx.h, pi, xi, co, ai, z1)
        ltgw.ltgw_cnn_forward(ctx.h, pi, xi, co, None, z2)
        assert torch.equal(z1, z2)
    with pytest.raises(ltgw.LtgwError):
        ltgw.ltgw_cnn_forward(ctx.h, T(_net(9, 4, 6)), T(np.zeros((1, 4, 257), np.float32)), 6, None,
                              torch.empty((1, 6, 257), dtype=torch.float32, device="cuda"))
    ctx.close()


@pytest.mark.parametrize("B,c_in,c_out,L", [
    (1, 1, 1, 1),        # the work area holds no partial vector: the layer-by-layer kernels
    (1, 1, 1, 255),      # one channel each, one position short of the on-chip limit
    (2, 32, 32, 256),    # every limit of the on-chip pass
    (2, 8, 24, 257),     # past it: the layer-by-layer kernels
    (7, 3, 5, 16),       # one tile of positions
    (5, 12, 24, 17),     # a remainder of one position
    (40, 8, 24, 50),     # several samples per workgroup
])
def test_cnn_gradients_at_shape_limits(B, c_in, c_out, L):
    """The bound is that of the product's BF16 operands (2^-8 of a term, of
    random sign): 5e-3 of the layer's largest gradient, as above."""
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    print(f"case: cnn gradients B={B} c_in={c_in} c_out={c_out} L={L}", flush=True)
    params = _net(15, c_in, c_out)
    rng = np.random.default_rng(B * 1000 + L)
    x = rng.normal(size=(B, c_in, L)).astype(np.float32)
    dz = rng.normal(scale=0.1, size=(B, c_out, L)).astype(np.float32)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    act = torch.empty((3, B, 32, L), dtype=torch.float32, device="cuda")
    logits = torch.empty((B, c_out, L), dtype=torch.float32, device="cuda")
    ltgw.ltgw_cnn_forward(ctx.h, T(params), T(x), c_out, act, logits)
    work = torch.full((ltgw.ltgw_cnn_work_floats(B, c_in, c_out, L),), float("nan"), dtype=torch.float32, device="cuda")
    grads = torch.full((params.size,), float("nan"), dtype=torch.float32, device="cuda")
    ltgw.ltgw_cnn_backward(ctx.h, T(params), T(x), c_out, act, T(dz), work, grads)
    zr, cache = cnn.forward(params, x, c_in, c_out, rnd=cnn.bf16_operands)
    gr = cnn.backward(params, cache, dz.astype(np.float64), c_in, c_out, rnd=cnn.bf16_operands)
    assert _rel(logits.cpu().numpy().astype(np.float64), zr) < 2e-3
    g, off = grads.cpu().numpy().astype(np.float64), 0
    for shp in cnn.layer_shapes(c_in, c_out):
        n = int(np.prod(shp))
        assert _rel(g[off:off + n], gr[off:off + n]) < 5e-3, shp
        off += n
    ctx.close()


def test_softmax_xent_adam_and_select_top():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    rng = np.random.default_rng(21)
    B, n = 5, 300
    z = rng.normal(scale=3.0, size=(B, n)).astype(np.float32)
    tg = np.array([4, -1, 299, 0, 150], np.int32)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    loss = torch.empty(B, dtype=torch.float32, device="cuda")
    dz = torch.empty((B, n), dtype=torch.float32, device="cuda")
    ltgw.ltgw_softmax_xent(ctx.h, T(z), T(tg), 4, loss, dz)
    l_g, d_g = loss.cpu().numpy(), dz.cpu().numpy()
    for b in range(B):
        lr_, dr = cnn.softmax_xent(z[b:b + 1].astype(np.float64), tg[b:b + 1])
        assert abs(l_g[b] - lr_) <= 1e-5 * max(1.0, abs(lr_))
        assert np.allclose(d_g[b] * 4, dr[0], atol=1e-6)    # the device divides by n_valid = 4
    # Adam against its FP64 definition
    p = rng.normal(size=1000).astype(np.float32)
    g = rng.normal(size=1000).astype(np.float32)
    pd, gd = T(p), T(g)
    md, vd = torch.zeros_like(pd), torch.zeros_like(pd)
    pr, mr, vr = p.astype(np.float64), np.zeros(1000), np.zeros(1000)
    for step in (1, 2, 3):
        ltgw.ltgw_adam_step(ctx.h, pd, gd, md, vd, 1e-3, 0.9, 0.999, 1e-8, step)
        pr, mr, vr = cnn.adam(pr, g.astype(np.float64), mr, vr, 1e-3, 0.9, 0.999, 1e-8, step)
    assert np.allclose(pd.cpu().numpy(), pr, rtol=0, atol=1e-6)
    # top-M with ties and NaN: one wavefront per row up to 1024 scores (slots of
    # 1 .. 16 per lane; 5 rows, so the last workgroup is partly empty), one
    # workgroup per row above; a row mostly NaN takes NaN entries, lowest first
    for n_sc, M in ((1000, 50), (8192, 200), (7, 7), (300, 15), (130, 3), (100, 1), (64, 64), (2000, 40),
                    (600, 400)):
        s = rng.integers(0, 40, size=(5, n_sc)).astype(np.float32)
        s[0, 3] = np.nan
        s[1, : (n_sc * 3) // 4] = np.nan
        out = torch.empty((5, M), dtype=torch.int32, device="cuda")
        ltgw.ltgw_select_top(ctx.h, T(s), M, out)
        o = out.cpu().numpy()
        for r in range(5):
            # the M best (score desc, ties to the lower index, NaN last), in index order
            key = np.where(np.isnan(s[r]), -np.inf, s[r])
            ref = np.sort(np.lexsort((np.arange(n_sc), np.isnan(s[r]), -key))[:M])
            assert np.array_equal(o[r], ref)
    ctx.close()


def _propose_setup(weights=True):
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, t, v, w = _ctx(weights)
    R = len(INJ)
    st = _stack(ctx, R, INJ)
    ltgw.ltgw_load_stack(ctx.h, 0, st, "f32", coarse=True)
    L = COARSE["n_f0"]
    c_in = 4
    c_out = 2 * 4
    params = torch.from_numpy(_net(9, c_in, c_out)).cuda()
    return ctx, st, t, v, w, R, L, c_in, c_out, params


def test_propose_all_cells_finds_the_exhaustive_best():
    from paper_2507_07816_amd import ltgw

    ctx, st, t, v, w, R, L, c_in, c_out, params = _propose_setup()
    ref_stack = _oracle_stack(R, INJ, t, v, w)
    fg, kf = _grid(FINE)
    cg, kc = _grid(COARSE)
    n_cells = c_out * L
    bi, bp, fb = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, n_cells, 1e9, 1e9, R)
    assert np.all(fb == 0)
    g = _ogrid(FINE)
    for r in range(R):
        det = oracle.Detector(ref_stack[r], t, v, K_LO, T_SFT, weights=w)
        ref = oracle.evaluate(det, g)
        psi = oracle.psi_power(ref)
        i, p = op.best_template(psi, np.arange(g.n_templates))
        tol = psi_tolerance(ref)
        assert abs(bp[r] - p) <= tol[i]
        # equal best, or a near-tie within the FP32 accumulation tolerance
        assert bi[r] == i or abs(psi[bi[r]] - p) <= 2 * tol[i]
    # every realisation falls back: the exhaustive fine grid decides
    bi2, bp2, fb2 = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, 4, 1e9, -1e9, R)
    assert np.all(fb2 == 1)
    assert np.array_equal(bi2, bi) and np.array_equal(bp2, bp)
    # blocks of 16 f0 (the last of each group ragged: 48 = 3 x 16 is not, so use 20):
    # all blocks at once, or half of them and the other half as the second tier
    # (no cell passes the threshold, so every realisation takes it), cover the grid
    for W in (16, 20):
        nb = 4 * ((2 * L + W - 1) // W)
        print(f"case: propose blocks of {W}", flush=True)
        bi3, bp3, fb3 = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, nb * W, 1e9, 1e9, R, block=W)
        assert np.all(fb3 == 0) and np.array_equal(bi3, bi) and np.array_equal(bp3, bp)
        h = nb // 2
        bi4, bp4, fb4, bl4 = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, h * W, 1e9, 1e9, R,
                                               block=W, n_select2=(nb - h) * W, return_blocks=True)
        assert np.all(fb4 == 0) and np.array_equal(bi4, bi) and np.array_equal(bp4, bp)
        # the reported blocks: each tier ascending, together every block once
        assert bl4.shape == (R, nb)
        for r in range(R):
            assert np.all(np.diff(bl4[r, :h]) > 0) and np.all(np.diff(bl4[r, h:]) > 0)
            assert sorted(bl4[r].tolist()) == list(range(nb))
    # a BF16 store: blocks of 16 evaluated in place, the exhaustive fallback
    # and the exhaustive best find the same template and ratio
    print("case: propose on a BF16 store", flush=True)
    import torch
    ltgw.ltgw_load_stack(ctx.h, 0, st, "bf16", coarse=True)
    bb = torch.empty(R, dtype=torch.int32, device="cuda")
    bpp = torch.empty(R, dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_best(ctx.h, fg, bb, bpp)
    nb16 = 4 * ((2 * L + 15) // 16)
    bi5, bp5, fb5 = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, nb16 * 16, 1e9, 1e9, R, block=16)
    bi6, bp6, fb6 = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, 16, 1e9, -1e9, R, block=16)
    assert np.all(fb5 == 0) and np.all(fb6 == 1)
    assert np.array_equal(bi5, bb.cpu().numpy()) and np.array_equal(bp5, bpp.cpu().numpy())
    assert np.array_equal(bi6, bi5) and np.array_equal(bp6, bp5)
    ctx.close()


def test_propose_partial_selection_equals_composed_calls():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, st, t, v, w, R, L, c_in, c_out, params = _propose_setup()
    fg, kf = _grid(FINE)
    cg, kc = _grid(COARSE)
    M = 12
    bi, bp, fb, bl = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, M, 1e9, 1e9, R, return_blocks=True)
    # the same steps through the public calls
    pc = torch.empty((R, c_in * L), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi(ctx.h, cg, 1, pc, nan_to_zero=True)
    x = pc.float().reshape(R, c_in, L).contiguous()
    act = torch.empty((3, R, 32, L), dtype=torch.float32, device="cuda")
    logits = torch.empty((R, c_out, L), dtype=torch.float32, device="cuda")
    ltgw.ltgw_cnn_forward(ctx.h, params, x, c_out, act, logits)
    cells = torch.empty((R, M), dtype=torch.int32, device="cuda")
    ltgw.ltgw_select_top(ctx.h, logits.reshape(R, -1).contiguous(), M, cells)
    tpl = op.cell_to_template(cells.cpu().numpy(), L).astype(np.int32)
    out = torch.empty((R, M), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi_list(ctx.h, fg, torch.from_numpy(tpl).cuda(), out)
    o = out.cpu().numpy()
    for r in range(R):
        i, p = op.best_template(o[r], tpl[r])
        assert bi[r] == i and bp[r] == p
        # blocks of one cell are fine templates (group * 2 L + f0 index)
        assert bl[r].tolist() == sorted(tpl[r].tolist())
    # the fallback rule: coarse maximum above the threshold, best below the detection threshold
    cmax = np.nanmax(pc.cpu().numpy(), axis=1)
    thr = float(np.max(bp)) + 1.0
    bi3, bp3, fb3 = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, M, thr, float(np.median(cmax)), R)
    assert np.array_equal(fb3, (cmax > np.median(cmax)).astype(np.int32))
    ctx.close()


def test_propose_block_selection_equals_composed_scores():
    """Blocks of 16, 32 and 64 f0 take the fused network + block-score pass;
    the reported first-tier blocks must be the best blocks by the largest
    logit of their cells (ties to the lower block), from the layer-by-layer
    network, and the first tier's best its exact ratios' best."""
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, st, t, v, w, R, L, c_in, c_out, params = _propose_setup()
    fg, kf = _grid(FINE)
    cg, kc = _grid(COARSE)
    pc = torch.empty((R, c_in * L), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi(ctx.h, cg, 1, pc, nan_to_zero=True)
    x = pc.float().reshape(R, c_in, L).contiguous()
    act = torch.empty((3, R, 32, L), dtype=torch.float32, device="cuda")
    logits = torch.empty((R, c_out, L), dtype=torch.float32, device="cuda")
    ltgw.ltgw_cnn_forward(ctx.h, params, x, c_out, act, logits)
    z = logits.cpu().numpy()
    G = c_out // 2
    for W in (16, 32, 64):
        print(f"case: fused block scores W={W}", flush=True)
        nbg = -(-2 * L // W)
        score = np.full((R, G * nbg), -np.inf)
        for g in range(G):
            for k in range(nbg):
                for i in range(k * W, min(k * W + W, 2 * L)):
                    score[:, g * nbg + k] = np.maximum(score[:, g * nbg + k], z[:, 2 * g + i % 2, i // 2])
        K1 = 2
        bi, bp, fb, bl = ltgw.ltgw_propose(ctx.h, fg, cg, params, c_in, c_out, L, K1 * W, 1e9, 1e9, R, block=W,
                                           return_blocks=True)
        for r in range(R):
            order = np.lexsort((np.arange(G * nbg), -score[r]))
            assert bl[r].tolist() == sorted(order[:K1].tolist())
            tpl = [g * 2 * L + i for b in bl[r] for g in [b // nbg] for i in range((b % nbg) * W,
                                                                                   min((b % nbg) * W + W, 2 * L))]
            one = torch.empty((R, len(tpl)), dtype=torch.int32, device="cuda")
            one[:] = torch.tensor(tpl, dtype=torch.int32)
            allp = torch.empty((R, len(tpl)), dtype=torch.float64, device="cuda")
            ltgw.ltgw_stack_psi_list(ctx.h, fg, one, allp)
            i, p = op.best_template(allp.cpu().numpy()[r], np.array(tpl))
            assert bi[r] == i and bp[r] == p
    ctx.close()


def test_propose_coarse_only_equals_composed_scores():
    """Without a network the blocks are ranked by the coarse power ratios of
    the nearest coarse groups (the method alone): the reported blocks are the
    best by that score (ties to the lower block), the best template is their
    exact ratios' best, and the count channels of the input do not change it."""
    import torch
    from paper_2507_07816_amd import ltgw
    from paper_2507_07816_amd.proposer import nearest_coarse_groups

    ctx, st, t, v, w, R, L, c_in, c_out, params = _propose_setup()
    fg, kf = _grid(FINE)
    cg, kc = _grid(COARSE)
    cmap = nearest_coarse_groups(FINE, COARSE)
    assert cmap.shape == (4, 2) and np.array_equal(cmap[:, 0], np.arange(4)) and np.all(cmap[:, 1] == -1)
    # a second map: every fine group scored by two coarse groups
    cmap2 = np.array([[0, 1], [1, 2], [2, 3], [3, 0]], np.int32)
    x = torch.empty((R, c_in, L), dtype=torch.float32, device="cuda")
    ltgw.ltgw_stack_features(ctx.h, cg, x)
    z = x.cpu().numpy()
    G = c_out // 2
    for m, W, counts in ((cmap, 16, False), (cmap2, 16, True), (cmap2, 64, False)):
        print(f"case: coarse-only blocks W={W} counts={counts}", flush=True)
        nbg = -(-2 * L // W)
        score = np.full((R, G * nbg), -np.inf, np.float32)
        for g in range(G):
            for k in range(nbg):
                for i in range(k * W, min(k * W + W, 2 * L)):
                    for ch in m[g]:
                        if ch >= 0:
                            score[:, g * nbg + k] = np.maximum(score[:, g * nbg + k], z[:, ch, i // 2])
        K1 = 2
        bi, bp, fb, bl = ltgw.ltgw_propose(ctx.h, fg, cg, None, 2 * c_in if counts else c_in, c_out, L, K1 * W,
                                           1e9, 1e9, R, block=W, return_blocks=True, coarse_map=m)
        assert np.all(fb == 0)
        for r in range(R):
            order = np.lexsort((np.arange(G * nbg), -score[r]))
            assert bl[r].tolist() == sorted(order[:K1].tolist())
            tpl = [g * 2 * L + i for b in bl[r] for g in [b // nbg] for i in range((b % nbg) * W,
                                                                                   min((b % nbg) * W + W, 2 * L))]
            one = torch.empty((R, len(tpl)), dtype=torch.int32, device="cuda")
            one[:] = torch.tensor(tpl, dtype=torch.int32)
            allp = torch.empty((R, len(tpl)), dtype=torch.float64, device="cuda")
            ltgw.ltgw_stack_psi_list(ctx.h, fg, one, allp)
            i, p = op.best_template(allp.cpu().numpy()[r], np.array(tpl))
            assert bi[r] == i and bp[r] == p
    E = ltgw.LtgwError
    with pytest.raises(E):   # a map is needed without a network
        ltgw.ltgw_propose(ctx.h, fg, cg, None, c_in, c_out, L, 16, 1e9, 1e9, R, block=16)
    with pytest.raises(E):   # coarse group out of range
        ltgw.ltgw_propose(ctx.h, fg, cg, None, c_in, c_out, L, 16, 1e9, 1e9, R, block=16,
                          coarse_map=np.array([[0, -1], [1, -1], [2, -1], [4, -1]], np.int32))
    ctx.close()


def test_proposer_errors():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    E = ltgw.LtgwError
    fg, kf = _grid(FINE)
    cg, kc = _grid(COARSE)
    params = torch.zeros(cnn.n_params(4, 8), dtype=torch.float32, device="cuda")
    with pytest.raises(E) as ei:   # no stack yet
        ltgw.ltgw_propose(ctx.h, fg, cg, params, 4, 8, 24, 8, 1.0, 1.0, 1)
    assert ei.value.code == ltgw.LTGW_E_STATE
    st = torch.ones((2, N_SEG, N_BINS), dtype=torch.float32, device="cuda")
    st[1, 3, 4] = float("nan")
    with pytest.raises(E):
        ltgw.ltgw_load_stack(ctx.h, 0, st, "f32", coarse=True)
    with pytest.raises((E, TypeError)):
        ltgw.ltgw_load_stack(ctx.h, 0, st.cpu(), "f32", coarse=True)   # host pointer
    st[1, 3, 4] = 1.0
    ltgw.ltgw_load_stack(ctx.h, 0, st, "f32", coarse=True)
    with pytest.raises(E):       # channel mismatch
        ltgw.ltgw_propose(ctx.h, fg, cg, params, 3, 8, 24, 8, 1.0, 1.0, 2)
    with pytest.raises(E):       # fine grid not twice the coarse positions
        ltgw.ltgw_propose(ctx.h, cg, cg, params, 4, 8, 24, 8, 1.0, 1.0, 2)
    with pytest.raises(E):
        ltgw.ltgw_inject_stack(ctx.h, 0, st, np.array([[480.0, 5000.0, 0.5, 1.0]] * 2), SKY, 0.0)
    ctx.close()


def test_stack_best_features_and_cells():
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, t, v, w = _ctx()
    R = len(INJ)
    st = _stack(ctx, R, INJ)
    ref_stack = _oracle_stack(R, INJ, t, v, w)
    ltgw.ltgw_load_stack(ctx.h, 0, st, "f32", coarse=True)
    fg, kf = _grid(FINE)
    cg, kc = _grid(COARSE)
    bi = torch.empty(R, dtype=torch.int32, device="cuda")
    bp = torch.empty(R, dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_best(ctx.h, fg, bi, bp)
    bi_h, bp_h = bi.cpu().numpy(), bp.cpu().numpy()
    g = _ogrid(FINE)
    for r in range(R):
        ref = oracle.evaluate(oracle.Detector(ref_stack[r], t, v, K_LO, T_SFT, weights=w), g)
        psi = oracle.psi_power(ref)
        i, p = op.best_template(psi, np.arange(g.n_templates))
        tol = psi_tolerance(ref)
        assert abs(bp_h[r] - p) <= tol[i]
        assert bi_h[r] == i or abs(psi[bi_h[r]] - p) <= 2 * tol[i]
    # the number count: best template and ratio identical to the oracle's
    # (integer counts; the ratio's arithmetic is the oracle's, ties to the lower index)
    ltgw.ltgw_stack_best(ctx.h, fg, bi, bp, stat="count")
    bi_h, bp_h = bi.cpu().numpy(), bp.cpu().numpy()
    for r in range(R):
        ref = oracle.evaluate(oracle.Detector(ref_stack[r], t, v, K_LO, T_SFT, weights=w), g)
        i, p = op.best_template(oracle.psi_count(ref), np.arange(g.n_templates))
        assert bi_h[r] == i and bp_h[r] == pytest.approx(p, rel=1e-13, abs=1e-13)
    # listed count ratios equal the single search's ratios bit for bit
    # (realisation 0 loaded as an ordinary spectrogram)
    ctx2 = ltgw.Context(0)
    ctx2.load_spectrogram(0, st[0].contiguous(), K_LO, T_SFT, t, weights=w)
    ctx2.set_velocity_table(0, v)
    ctx2.eval_templates(FINE["f0_min"], FINE["f0_step"], FINE["n_f0"], FINE["tau"], FINE["brake"], FINE["sky"],
                        0.0, outputs=False)
    single = ctx2.psi("count", g.n_templates).cpu().numpy()
    ctx2.close()
    idx = np.tile(np.arange(g.n_templates, dtype=np.int32), (R, 1))
    cl = torch.empty(idx.shape, dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi_list(ctx.h, fg, torch.from_numpy(idx).cuda(), cl, stat="count")
    assert np.array_equal(cl.cpu().numpy()[0], single, equal_nan=True)
    with pytest.raises(ltgw.LtgwError):
        ltgw.ltgw_stack_best(ctx.h, fg, bi, bp, stat=3)
    # features: the coarse ratios with NaN -> 0, in FP32
    L = COARSE["n_f0"]
    x = torch.empty((R, 4, L), dtype=torch.float32, device="cuda")
    ltgw.ltgw_stack_features(ctx.h, cg, x)
    pc = torch.empty((R, 4 * L), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi(ctx.h, cg, 1, pc, nan_to_zero=True)
    assert np.array_equal(x.cpu().numpy().reshape(R, -1), pc.cpu().numpy().astype(np.float32))
    # cells of templates, masked
    tpl = np.array([0, 1, 2 * L - 1, 2 * L, 4 * 2 * L - 1, -1, 37], np.int32)
    mask = np.array([1, 1, 1, 1, 1, 1, 0], np.int32)
    cells = torch.empty(tpl.size, dtype=torch.int32, device="cuda")
    ltgw.ltgw_cells_from_templates(ctx.h, torch.from_numpy(tpl).cuda(), L, cells,
                                   mask=torch.from_numpy(mask).cuda())
    want = np.where((tpl >= 0) & (mask == 1), op.template_to_cell(np.maximum(tpl, 0), L), -1)
    assert np.array_equal(cells.cpu().numpy(), want)
    ctx.close()


def test_training_learns_and_proposer_recalls(tmp_path):
    """A short training run on device-generated data lowers the loss well below
    the uniform-guess value log(n_cells); the trained proposer recalls the
    injections the exhaustive search detects (fallback included).  Saved to a
    file and loaded into another proposer in a fresh context, the network
    gives the same proposals bit for bit."""
    from paper_2507_07816_amd import ltgw
    from paper_2507_07816_amd.proposer import Proposer, coarse_grid_for

    ctx, t, v, w = _ctx()
    fine = dict(FINE, tau=np.array(FINE["tau"]), brake=np.array(FINE["brake"]), sky=np.array([SKY]))
    coarse = coarse_grid_for(fine, [6000.0], [4.0])
    pr = Proposer(ctx, 0, (N_SEG, N_BINS), fine, coarse, seed=3, select_frac=0.1)
    assert pr.c_in == 2 and pr.c_out == 8 and pr.L == 24
    losses = [pr.train_step(64, amp_range=(3.0, 6.0), lr=3e-3) for _ in range(200)]
    print(f"case: training loss {np.mean(losses[:10]):.3f} -> {np.mean(losses[-10:]):.3f}", flush=True)
    assert np.mean(losses[:5]) > 0.8 * np.log(pr.n_cells)
    assert np.mean(losses[-10:]) < 0.85 * np.mean(losses[:10])
    ev = pr.evaluate(R_noise=128, R_signal=256, amp_range=(3.0, 6.0), reps=1)
    print("case: evaluation", ev, flush=True)
    assert ev["detectable"] > 64
    assert ev["recall"] >= 0.75
    # the same budget ranked by the coarse power ratios alone (one coarse group
    # here: it cannot tell the fine groups apart) recalls no more
    assert ev["recall_no_fallback"] >= ev["coarse_only"]["recall_no_fallback"]
    # file round trip: train -> save -> load in a fresh context -> same proposals
    import torch

    path = str(tmp_path / "ranker.ltgwcnn")
    pr.save(path)
    assert ltgw.ltgw_proposer_load(ctx.h, path) == (pr.c_in, pr.c_out)
    R = 64
    inj, _ = pr.draw_injections(R, 1.0, (3.0, 6.0), rng=np.random.Generator(np.random.PCG64(99)))
    pr.make_batch(R, 5, 0, inj, with_labels=False)
    want = pr.propose(5.0, 6.0, R)
    ctx2, _, _, _ = _ctx()
    # the same seed draws the same noise; its network is the untrained one
    other = Proposer(ctx2, 0, (N_SEG, N_BINS), fine, coarse, seed=3, select_frac=0.1)
    assert not torch.equal(other.params, pr.params)
    other.load(path)
    assert torch.equal(other.params.view(torch.int32), pr.params.view(torch.int32))
    other.make_batch(R, 5, 0, inj, with_labels=False)
    got = other.propose(5.0, 6.0, R)
    for a, b in zip(got, want):
        assert np.array_equal(np.asarray(a), np.asarray(b))
    bad = Proposer(ctx2, 0, (N_SEG, N_BINS), fine, coarse_grid_for(fine, [5000.0, 9000.0], [4.0]), seed=6)
    with pytest.raises(ValueError):
        bad.load(path)
    ctx2.close()
    ctx.close()


@pytest.mark.slow
def test_trained_network_beats_coarse_ranking_at_equal_budget():
    """What the trained network gains over the method without it, on the
    small workload's shape (1024 segments x 800 bins, 4800 templates): the
    same budget (5% of the cells in blocks of 32 f0, no second tier, no
    fallback) ranked by the network after a short training recalls more of
    the injections the exhaustive search detects than ranked by the coarse
    power ratios of the nearest coarse groups."""
    import torch
    import synth
    from paper_2507_07816_amd import ltgw
    from paper_2507_07816_amd.proposer import Proposer, coarse_grid_for

    wl = synth.tiny(with_noise=False)
    d, g = wl.dets[0], wl.grid
    ctx = ltgw.Context(0)
    ctx.load_spectrogram(0, torch.zeros(d["rho"].shape, dtype=torch.float32, device="cuda"), d["k_lo"], d["t_sft"],
                         d["t_seg"], weights=d["weights"])
    ctx.set_velocity_table(0, d["v"])
    tau, brake = np.asarray(g["tau"]), np.asarray(g["brake"])
    coarse = coarse_grid_for(dict(g), np.sqrt(tau[0::2] * tau[1::2]),
                             np.array([(brake[0] + brake[1]) / 2, (brake[-2] + brake[-1]) / 2]))
    pr = Proposer(ctx, 0, d["rho"].shape, dict(g), coarse, seed=5, select_frac=0.05, store="f32", block=32,
                  coarse_segments=8)
    assert pr.c_in == 8
    print("case: training 12800 realisations x 4 epochs", flush=True)
    pr.train(12800, batch=256, epochs=4, p_signal=0.9, amp_range=(0.3, 3.0), lr=2e-3, label_psi=4.5, label="near")
    ev = pr.evaluate(R_noise=512, R_signal=1024, amp_range=(0.3, 3.0), fine_store="bf16", reps=1,
                     coarse_quantiles=(None,))
    print(f"case: trained {ev['recall_no_fallback']:.4f} coarse only {ev['coarse_only']['recall_no_fallback']:.4f} "
          f"over {ev['detectable']} detectable", flush=True)
    ctx.close()
    assert ev["detectable"] > 200
    assert ev["fallback_frac"] == 0.0 and ev["coarse_only"]["fallback_frac"] == 0.0
    assert ev["recall_no_fallback"] >= ev["coarse_only"]["recall_no_fallback"] + 0.1


@pytest.mark.parametrize("ns,nb,n_f0,R,store,t_sft", [
    (133, 1022, 1000, 256, "f32", 4.0),   # the widest row; a last batch of one segment
    (99, 61, 1000, 255, "bf16", 4.0),     # of three, and an odd count of realisations
    (41, 2046, 1000, 255, "bf16", 8.0),   # the widest row, f0 in steps of two bins
    (38, 1021, 1000, 255, "f32", 8.0),
])
def test_stack_sums_two_realisations_at_a_time(ns, nb, n_f0, R, store, t_sft, monkeypatch):
    """The same at sizes that the kernel for two realisations takes."""
    monkeypatch.setitem(globals(), "T_SFT", t_sft)
    test_stack_sums_over_segments_and_rows(ns, nb, n_f0, R, store)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 511, 512, 513, 2049, 3072, 3073, 8192, 8193, 20000])
def test_softmax_xent_row_lengths(n):
    """Rows at and around the lengths that a wavefront, four of them and sixteen take and
    hold in registers, some logits masked to -inf; the bars of the test above (an FP32
    sum of n terms in a tree and 20 in line)."""
    import torch
    from paper_2507_07816_amd import ltgw

    ctx, *_ = _ctx()
    print(f"case: softmax of {n}", flush=True)
    rng = np.random.default_rng(n)
    B = 7
    z = rng.normal(scale=3.0, size=(B, n)).astype(np.float32)
    z[1, : n // 2] = -np.inf
    tg = np.array([0, n - 1, n // 2, -1, n - 1, n // 3, 0], np.int32)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    loss = torch.empty(B, dtype=torch.float32, device="cuda")
    dz = torch.full((B, n), float("nan"), dtype=torch.float32, device="cuda")
    ltgw.ltgw_softmax_xent(ctx.h, T(z), T(tg), 6, loss, dz)
    l_g, d_g = loss.cpu().numpy(), dz.cpu().numpy()
    ctx.close()
    for b in range(B):
        lr_, dr = cnn.softmax_xent(z[b:b + 1].astype(np.float64), tg[b:b + 1])
        assert abs(l_g[b] - lr_) <= 1e-5 * max(1.0, abs(lr_))
        assert np.allclose(d_g[b] * 6, dr[0], atol=1e-6)


@pytest.mark.parametrize("ns,R,m,store", [
    (33, 70, 65, "f32"),       # a wavefront per 64 templates, the rows dealt to XCDs, the last deal not full
    (96, 63, 64, "bf16"),      # not dealt
    (97, 64, 63, "fp8"),       # four share them, with a last chunk of one segment
    (300, 70, 700, "f32"),     # 770 workgroups: four
    (300, 64, 768, "bf16"),    # 768: sixteen
    (225, 1, 1, "f32"),        # sixteen with eight chunks
])
def test_stack_list_shapes(ns, R, m, store):
    """Listed templates, some outside the grid, at the edges of how many wavefronts share
    them and of how rows go to workgroups: the whole grid's ratios bit for bit."""
    import torch
    from paper_2507_07816_amd import ltgw

    print(f"case: stack list {store} {R} x {ns}, {m} templates", flush=True)
    nb, n_f0 = 70, 90
    r = np.random.default_rng(ns + m)
    t = np.arange(ns) * (3840.0 / ns) + 2.0
    v = r.normal(size=(ns, 3))
    v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
    ctx = ltgw.Context(0)
    ctx.load_spectrogram(0, torch.zeros((ns, nb), dtype=torch.float32, device="cuda"), K_LO, T_SFT, t,
                         weights=r.uniform(0.5, 2.0, ns).astype(np.float32))
    ctx.set_velocity_table(0, v)
    P = torch.from_numpy(r.exponential(size=(R, ns, nb)).astype(np.float32)).cuda()
    ltgw.ltgw_load_stack(ctx.h, 0, P, store, coarse=False)
    fg, keep = _grid(dict(f0_min=(K_LO - 2) / T_SFT, f0_step=0.25, n_f0=n_f0, tau=[4000.0, 15000.0, 60000.0],
                          brake=[3.0, 5.0], sky=[SKY], t0=0.0))
    n = n_f0 * 6
    full = torch.empty((R, n), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi(ctx.h, fg, 0, full)
    idx = r.integers(-1, n + 1, (R, m)).astype(np.int32)
    out = torch.empty((R, m), dtype=torch.float64, device="cuda")
    ltgw.ltgw_stack_psi_list(ctx.h, fg, torch.from_numpy(idx).cuda(), out)
    f, o = full.cpu().numpy(), out.cpu().numpy()
    ctx.close()
    inside = (idx >= 0) & (idx < n)
    want = np.where(inside, np.take_along_axis(f, np.clip(idx, 0, n - 1), axis=1), np.nan)
    assert np.array_equal(o, want, equal_nan=True) and (m == 1 or np.isfinite(o).any())


@pytest.mark.parametrize("B,c_in,c_out,L", [
    (4, 8, 24, 50), (8, 8, 24, 50),       # by layers, and two workgroups of four samples
    (40, 8, 24, 16), (128, 8, 24, 16),    # by layers, and ten of thirteen
    (1000, 1, 2, 7),                      # 43 of 24
])
def test_cnn_gradients_of_short_samples(B, c_in, c_out, L):
    """Samples so short that the work area holds few partial parameter vectors."""
    test_cnn_gradients_at_shape_limits(B, c_in, c_out, L)
