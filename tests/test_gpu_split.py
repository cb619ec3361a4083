"""The statistic with a workgroup's wavefronts sharing the segments: bit for bit what the
forced tile shapes give, at the edges of its chunks (32 segments), of the 64 f0 of a
workgroup, and for each number of wavefronts (16, 8, 4 by the size of the lattice), with
and without antenna weights (moments in the loop), for one and two detectors."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SKY = np.array([0.6, 0.0, 0.8])


@pytest.mark.parametrize("ns,n_f0,n_tau,dets,store,antenna", [
    (1, 1, 1, 1, "f32", False),
    (31, 65, 2, 2, "bf16", False),
    (33, 64, 2, 1, "fp8", True),
    (513, 130, 3, 1, "f32", False),      # 16 wavefronts and one segment more than their chunks
    (1100, 63, 2, 2, "f32", True),
    (300, 180, 200, 1, "bf16", False),   # 600 workgroups: 8 wavefronts
    (70, 180, 300, 1, "fp8", True),
    (90, 130, 700, 2, "f32", False),     # 2100: 4 wavefronts
    (90, 130, 700, 1, "bf16", True),
])
def test_split_equals_tile_shapes(ns, n_f0, n_tau, dets, store, antenna):
    import torch
    from paper_2507_07816_amd import ltgw

    print(f"case: split {store} {dets} x {ns}, {n_f0} f0 x {n_tau}, antenna {antenna}", flush=True)
    nb, k_lo, t_sft = 150, 1880, 4.0
    r = np.random.default_rng(ns + n_f0)
    ctx = ltgw.Context(0)
    for d in range(dets):
        t = np.arange(ns) * (3600.0 / max(ns, 60)) + 2.0 + d
        v = r.normal(size=(ns, 3))
        v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
        ctx.load_spectrogram(d, torch.from_numpy(r.exponential(size=(ns, nb)).astype(np.float32)).cuda(), k_lo, t_sft, t,
                             weights=r.uniform(0.5, 2.0, ns).astype(np.float32), store=store)
        ctx.set_velocity_table(d, v)
        if antenna:
            a = np.array([[0.36, 0.48, 0.8], [-0.8, 0.6, 0.0]])
            ctx.set_antenna(d, a, np.linspace(0.1, 2.0, ns))
    g = dict(f0_min=(k_lo - 3) / t_sft, f0_step=0.25, n_f0=n_f0, tau=np.geomspace(3000.0, 60000.0, n_tau), brake=[5.0],
             sky=[SKY], t0=0.0, det_mask=(1 << dets) - 1)
    n = n_f0 * n_tau
    out = []
    for shape in (-1, 0, 3):
        ctx.set_tile_shape(shape)
        out.append([x.cpu().numpy() for x in ctx.eval_templates(**g)] +
                   [ctx.psi(s, n).cpu().numpy() for s in ("power", "count")] + [ctx.diagnostics()["in_band"]])
    ctx.close()
    assert out[0][5] > 0 or n == 1  # the single template starts below the band
    for o in out[1:]:
        for x, y in zip(out[0], o):
            assert np.array_equal(x, y, equal_nan=True)


def test_untuned_large_lattice_in_slabs():
    """2000 f0 x 160 tau over 4100 segments, where an untuned lattice is walked in slabs
    (four and a remainder): bit for bit the one-pass shape, which a forced 1 is."""
    import torch
    from paper_2507_07816_amd import ltgw

    print("case: untuned 2000 x 160 over 4100 segments", flush=True)
    ns, nb, k_lo, t_sft = 4100, 2100, 4000, 8.0
    r = np.random.default_rng(9)
    t = np.arange(ns) * 8.0 + 4.0
    v = r.normal(size=(ns, 3))
    v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
    ctx = ltgw.Context(0)
    ctx.load_spectrogram(0, torch.from_numpy(r.exponential(size=(ns, nb)).astype(np.float32)).cuda(), k_lo, t_sft, t)
    ctx.set_velocity_table(0, v)
    g = dict(f0_min=k_lo / t_sft, f0_step=1.0 / t_sft, n_f0=2000, tau=np.geomspace(20000.0, 90000.0, 160), brake=[5.0],
             sky=[SKY], t0=0.0)
    out = []
    for shape in (-1, 1):
        ctx.set_tile_shape(shape)
        out.append([x.cpu().numpy() for x in ctx.eval_templates(**g)])
        d = ctx.diagnostics()
        assert (d["tile_shape"], d["eval_launches"]) == ((9, 5) if shape < 0 else (1, 1))
    ctx.close()
    for x, y in zip(*out):
        assert np.array_equal(x, y)


def _lattice(ns, nb, k_lo, t_sft, n_f0, n_tau, store="f32"):
    import torch
    from paper_2507_07816_amd import ltgw

    r = np.random.default_rng(ns + n_f0)
    v = r.normal(size=(ns, 3))
    v = v / np.linalg.norm(v, axis=1, keepdims=True) * 3.0e4
    ctx = ltgw.Context(0)
    ctx.load_spectrogram(0, torch.from_numpy(r.exponential(size=(ns, nb)).astype(np.float32)).cuda(), k_lo, t_sft,
                         np.arange(ns) * 40.0 + 2.0, store=store)
    ctx.set_velocity_table(0, v)
    return ctx, dict(f0_min=(k_lo - 3) / t_sft, f0_step=1.0 / t_sft, n_f0=n_f0, tau=np.geomspace(3000.0, 60000.0, n_tau),
                     brake=[5.0], sky=[SKY], t0=0.0)


@pytest.mark.parametrize("ns,n_f0,n_tau,waves", [
    (65, 1, 1, 16), (64, 1, 1, 0),              # three chunks of segments, and two
    (70, 64, 512, 16), (70, 64, 513, 8),        # two workgroups a CU of 256
    (70, 64, 1280, 8), (70, 64, 1281, 4),       # five
    (70, 2500, 100, 4), (70, 2500, 101, 0),     # 40 MB of the lattice's columns
])
def test_which_kernel_an_untuned_lattice_runs(ns, n_f0, n_tau, waves):
    import torch

    print(f"case: untuned {n_f0} f0 x {n_tau} tau, {ns} segments", flush=True)
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 CUs")
    ctx, g = _lattice(ns, 150, 1880, 4.0, n_f0, n_tau)
    ctx.eval_templates(**g)
    assert ctx.shared_wavefronts() == waves and ctx.diagnostics()["tile_shape"] == 1
    ctx.set_tile_shape(2)  # a shape asked for is the one that runs
    ctx.eval_templates(**g)
    assert ctx.shared_wavefronts() == 0 and ctx.diagnostics()["tile_shape"] == 2
    ctx.close()


@pytest.mark.parametrize("store,nb,shape", [("f32", 2000, 9), ("f32", 1999, 1), ("bf16", 2100, 1), ("fp8", 2100, 1)])
def test_slabs_are_for_rows_the_caches_do_not_hold(store, nb, shape):
    import torch

    n_tau = {"f32": 160, "bf16": 330, "fp8": 650}[store]  # 40 MB of columns and more
    print(f"case: {nb} {store} columns of 4100 segments, 2000 x {n_tau} templates", flush=True)
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 CUs")
    ctx, g = _lattice(4100, nb, 8000, 8.0, 2000, n_tau, store)
    ctx.eval_templates(**g)
    d = ctx.diagnostics()
    assert (d["tile_shape"], d["eval_launches"], ctx.shared_wavefronts()) == (shape, 5 if shape == 9 else 1, 0)
    ctx.close()


def test_a_tuned_shape_runs(tmp_path):
    """A tuned lattice runs what the tuning found faster: its shape where the file says so
    (one that knows the shapes alone, or 0 for the shared segments), those where it says 1,
    and what ltgw_autotune measured after it."""
    import json

    from paper_2507_07816_amd import ltgw

    print("case: tuned lattice", flush=True)
    ctx, g = _lattice(1024, 300, 1880, 4.0, 130, 3)
    ref = [x.cpu().numpy() for x in ctx.eval_templates(**g)]
    assert ctx.shared_wavefronts() == 16
    best = ctx.autotune(**g)
    path = tmp_path / "tune.json"
    ctx.tune_save(str(path))
    saved = json.loads(path.read_text())["ltgw_tune"]
    (key,) = [k for k in saved if k.startswith("eval/")]
    shared = "shared/" + key[5:]
    assert saved[key] == best and saved[shared] in (0, 1)
    # a lane walking 1024 segments alone against 16 wavefronts sharing them: a factor of five
    assert saved[shared] == 1
    for entries, want in (({key: 3}, (3, 0)), ({key: 2, shared: 0}, (2, 0)), ({key: 0, shared: 1}, (0, 16)),
                          ({key: 3}, (3, 0)), (saved, (best, 16))):
        path.write_text(json.dumps({"ltgw_tune": entries}))
        ctx.tune_load(str(path))
        out = [x.cpu().numpy() for x in ctx.eval_templates(**g)]
        assert (ctx.diagnostics()["tile_shape"], ctx.shared_wavefronts()) == want
        for x, y in zip(out, ref):
            assert np.array_equal(x, y)
    ctx.close()
