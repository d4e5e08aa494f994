"""GPU parity: libseedinf through its C ABI against the CPU oracle on the same
seeded inputs (see tests/parity.py for the rule).  fp32 mode: 1e-4; bf16
mode: 2e-2."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_1910_06591_amd import seedinf, workloads as wl
from tests.parity import check_against_oracle, random_arch, supported_random_arch, to_device
from tests.test_layerwise_plans import ROUTES

pytestmark = pytest.mark.gpu
TOL = {"fp32": 1e-4, "bf16": 2e-2}
CORE_KEYS = ("prev_action", "prev_reward", "h_in", "c_in", "uniforms")


def run_case(orc, cfg, B, precision, max_batch=None, weights=None, seed_shift=0, intermediates=True):
    import torch
    weights = wl.make_weights(cfg, bf16_representable=(precision == "bf16")) if weights is None else weights
    batch = wl.make_batch(cfg, B, seed_shift=seed_shift)
    print(f"case {cfg['label']} B={B} {precision}", flush=True)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=max_batch or B, precision=precision), weights)
    out = net.step(**to_device(batch))
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    ref = orc.forward(oracle.make_arch(cfg), weights, batch["obs"], want_intermediates=intermediates,
                      **{k: batch[k] for k in CORE_KEYS})
    tol = TOL[precision]
    if intermediates:
        for which, key in ((0, "torso_feat"), (1, "fc_act")):
            g = net.read_intermediate(which, B).cpu().numpy().astype(np.float64)
            o = ref[key].astype(np.float64)
            sc = np.maximum(1.0, np.abs(o).max(axis=1))
            err = np.abs(g - o).max(axis=1) / sc
            assert err.max() <= tol, f"{key}: worst row err {err.max():.3e}"
    rep = check_against_oracle(got, ref, tol, batch["uniforms"])
    print("   ", rep, flush=True)
    net.close()
    return got, ref, rep


def test_c1_fp32_full(orc):
    cfg = wl.CONFIGS["C1"]
    run_case(orc, cfg, cfg["batch"], "fp32")


@pytest.mark.parametrize("name,B", [("C2", 5), ("C3", 3), ("C4", 2)])
def test_fp32_mode_every_family(orc, name, B):
    """Every network family in fp32 mode at a small ragged batch: tight
    tolerance, so an indexing slip anywhere cannot hide behind bf16 rounding."""
    run_case(orc, wl.CONFIGS[name], B, "fp32")


def test_fp32_odd_shapes(orc):
    """Shapes that are not multiples of any tile: odd image, odd channels,
    odd pooled sizes (pool padding before = 1), A not a power of two."""
    cfg = dict(label="odd resnet", obs_h=13, obs_w=19, obs_c=5, torso=1, sections=[6, 10], fc_units=37,
               lstm_units=21, num_actions=7, head=0, head_hidden=0, select=1, precision="fp32", obs_kind="uniform",
               index=11)
    run_case(orc, cfg, 3, "fp32")
    cfg2 = dict(label="odd stack", obs_h=23, obs_w=17, obs_c=3, torso=0, convs=[(7, 5, 2), (9, 3, 1)], fc_units=50,
                lstm_units=0, num_actions=33, head=1, head_hidden=29, select=0, precision="fp32", obs_kind="uniform",
                index=12)
    run_case(orc, cfg2, 2, "fp32")


@pytest.mark.parametrize("case", ["stack_mult4", "stack_k5", "resnet_mult4", "stack_generic_lanes"])
def test_fp32_convolution_kernels(orc, case):
    """Both fp32 convolution kernels against the oracle: the one with four output channels per lane and the taps
    over the block's wavefronts (channel counts in multiples of four; tap counts 9, 16 and 25, which do and do not
    divide by eight; SAME padding and the residual add in the ResNet), and the generic one with the taps over
    adjacent lanes (other channel counts)."""
    base = dict(fc_units=24, lstm_units=0, num_actions=5, head=0, head_hidden=0, select=1, precision="fp32",
                obs_kind="uniform")
    cfgs = {
        "stack_mult4": dict(base, label="fp32 stack x4", obs_h=29, obs_w=31, obs_c=4, torso=0, convs=[(8, 4, 2), (12, 3, 1)], index=71),
        "stack_k5": dict(base, label="fp32 stack k5", obs_h=21, obs_w=23, obs_c=8, torso=0,
                                                 convs=[(4, 5, 2), (20, 3, 2)], index=72),
        "resnet_mult4": dict(base, label="fp32 resnet x4", obs_h=21, obs_w=27, obs_c=4, torso=1, sections=[8, 12], index=73),
        "stack_generic_lanes": dict(base, label="fp32 stack generic", obs_h=20, obs_w=17, obs_c=3, torso=0,
                                    convs=[(6, 4, 2), (7, 3, 1)], index=74),
    }
    run_case(orc, cfgs[case], 5, "fp32")


def test_fp32_b1_and_max_batch_larger_than_b(orc):
    cfg = wl.CONFIGS["C1"]
    run_case(orc, cfg, 1, "fp32", max_batch=16)


def test_repeatable_and_row_independent(orc):
    """Same inputs twice give bit-identical outputs (no atomics anywhere), and
    a row's result does not depend on its neighbours."""
    import torch
    cfg = wl.CONFIGS["C1"]
    w = wl.make_weights(cfg)
    batch = wl.make_batch(cfg, 8)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=8), w)
    dev = to_device(batch)
    o1 = {k: v.clone() for k, v in net.step(**dev).items()}
    o2 = net.step(**dev)
    torch.cuda.synchronize()
    for k in o1:
        assert torch.equal(o1[k], o2[k]), k
    sub = {k: (None if v is None else v[3:4].contiguous()) for k, v in dev.items()}
    o3 = net.step(**sub)
    torch.cuda.synchronize()
    for k in o1:
        assert torch.equal(o1[k][3:4], o3[k]), k
    net.close()


def test_error_paths_on_device(orc):
    import torch
    cfg = wl.CONFIGS["C3"]
    w = wl.make_weights(cfg, bf16_representable=False)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=4, precision="fp32"), w)
    batch = to_device(wl.make_batch(cfg, 4))
    A, Hn = cfg["num_actions"], cfg["lstm_units"]
    act = torch.full((4,), -7, dtype=torch.int32, device="cuda")
    logits = torch.full((4, A), 123.0, device="cuda")
    value = torch.zeros(4, device="cuda")
    ho, co = torch.zeros(4, Hn, device="cuda"), torch.zeros(4, Hn, device="cuda")
    p = lambda t: C.c_void_p(t.data_ptr())
    args = [p(batch["obs"]), p(batch["prev_action"]), p(batch["prev_reward"]), p(batch["h_in"]), p(batch["c_in"]),
            p(batch["uniforms"]), p(act), p(logits), p(value), p(ho), p(co), None]
    st, msg = net.step_raw(5, *args)
    assert st == 3 and "max_batch" in msg
    st, _ = net.step_raw(-1, *args)
    assert st == 1
    bad = list(args); bad[9] = p(batch["h_in"])          # h_out aliases h_in
    st, _ = net.step_raw(4, *bad)
    assert st == 4
    bad = list(args); bad[0] = C.c_void_p(batch["obs"].data_ptr() + 4)   # obs not 16-byte aligned
    assert net.step_raw(3, *bad)[0] == 1
    bad = list(args); bad[0] = None                      # obs missing
    assert net.step_raw(4, *bad)[0] == 1
    bad = list(args); bad[5] = None                      # uniforms missing for Gumbel selection
    assert net.step_raw(4, *bad)[0] == 1
    bad = list(args); bad[3] = None                      # recurrent arch without h_in
    assert net.step_raw(4, *bad)[0] == 1
    torch.cuda.synchronize()
    # no output was written by any failed call
    assert (act == -7).all() and (logits == 123.0).all()
    assert net.step_raw(0, *args)[0] == 0                # B = 0 is a no-op
    torch.cuda.synchronize()
    assert (act == -7).all()
    assert net.step_raw(4, *args)[0] == 0
    torch.cuda.synchronize()
    assert (act >= 0).all()
    # out-of-range previous action behaves as an all-zero one-hot (oracle does the same)
    b2 = wl.make_batch(cfg, 4)
    b2["prev_action"][:] = [-1, A, 3, 10**6]
    out = net.step(**to_device(b2))
    torch.cuda.synchronize()
    ref = orc.forward(oracle.make_arch(cfg), w, b2["obs"], **{k: b2[k] for k in CORE_KEYS})
    check_against_oracle({k: v.cpu().numpy() for k, v in out.items()}, ref, 1e-4, b2["uniforms"])
    net.close()


# ------------------------------------------------------------------ bf16 mode

@pytest.mark.parametrize("name,B", [("C2", 7), ("C3", 5), ("C4", 3)])
def test_bf16_small_ragged(orc, name, B):
    """bf16 matrix-core path, small ragged batches (fewer rows than one MFMA
    row tile; several images per persistent workgroup are covered below)."""
    run_case(orc, wl.CONFIGS[name], B, "bf16")


def _rows(batch, idx):
    return {k: (None if v is None else v[idx]) for k, v in batch.items()}


def run_full(orc, cfg, B, sample=None):
    """GPU on the full batch (the launch configuration bench.py times); oracle on all rows, or on a seeded
    sample of rows when B is large (rows are independent, so a row's oracle value does not depend on B)."""
    import torch
    weights = wl.make_weights(cfg)
    batch = wl.make_batch(cfg, B)
    print(f"full-size {cfg['label']} B={B} sample={sample}", flush=True)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=B), weights)
    out = net.step(**to_device(batch))
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    idx = np.arange(B) if sample is None else np.sort(np.random.default_rng(B).choice(B, sample, replace=False))
    if sample is not None:
        idx = np.unique(np.concatenate([idx, [0, B - 1]]))          # always the first and the last row
    sub = _rows(batch, idx)
    ref = orc.forward(oracle.make_arch(cfg), weights, sub["obs"], **{k: sub[k] for k in CORE_KEYS})
    rep = check_against_oracle({k: v[idx] for k, v in got.items()}, ref, TOL[cfg["precision"]], sub["uniforms"])
    print("   ", rep, flush=True)
    # properties that hold at any size: every action in range, probabilities normalised, finite state
    A = cfg["num_actions"]
    assert ((got["action"] >= 0) & (got["action"] < A)).all()
    assert np.abs(got["probs"].sum(1) - 1).max() < 1e-5
    for k in ("logits", "value", "h", "c"):
        if k in got:
            assert np.isfinite(got[k]).all(), k
    net.close()
    return rep


def test_full_size_c2(orc):
    run_full(orc, wl.CONFIGS["C2"], 256)


def test_full_size_c3(orc):
    run_full(orc, wl.CONFIGS["C3"], 1024)


def test_full_size_c4(orc):
    run_full(orc, wl.CONFIGS["C4"], 2048)


@pytest.mark.parametrize("B,sample", [(64, None), (256, None), (4096, 256), (8192, 256), (4099, 96)])
def test_full_size_c5_sweep(orc, B, sample):
    """The batch sweep of the headline workload; 4099 = a ragged last 64-row tile of the linear layer's
    wide-batch launch shape (three rows in its last block)."""
    run_full(orc, wl.CONFIGS["C5"], B, sample)


@pytest.mark.parametrize("label,base,over,B,sample", [
    ("R2D2 net at batch 4096", "C2", {}, 4096, 96),
    ("R2D2 net at ragged batch 2050", "C2", {}, 2050, 64),
    ("Football torso + LSTM-128 at batch 2100", "C4", dict(lstm_units=128), 2100, 64),
    ("DMLab net, 96 linear units, batch 2048", "C3", dict(fc_units=96), 2048, 48),
    ("R2D2 net at batch 1600", "C2", {}, 1600, 48),
    ("Football net at batch 1537", "C4", {}, 1537, 48),
    ("DMLab net at batch 1536", "C3", {}, 1536, 48),
])
def test_large_batch_dense_layers(orc, label, base, over, B, sample):
    """From 1536 rows on the linear layer, the recurrent core and the dueling hidden layers run LDS-staged GEMM
    kernels; these cases cover the tilings the C5 sweep does not reach (512 linear units, 128 x 256 tiles for
    the 512-unit core, hidden layers fed by fp32 rows only, a ragged last tile, a 128-unit core) and a linear
    width whose odd chunk count keeps the direct kernels."""
    cfg = dict(wl.CONFIGS[base], label=label, index=41, **over)
    run_full(orc, cfg, B, sample)


@pytest.mark.parametrize("B", [1, 257, 300, 512, 513, 770])
def test_bf16_persistent_grid_edges(orc, B):
    """B = 1; one more image than there are compute units (one workgroup takes two, as a group); a ragged count;
    exactly two images per workgroup; a workgroup with a group and then a single image; groups and singles mixed
    in the second round."""
    run_full(orc, wl.CONFIGS["C3"], B, sample=None if B == 1 else 64)


@pytest.mark.parametrize("name,B", [("C3", 300), ("C3", 4096), ("C2", 256), ("C2", 4096), ("C4", 2048)])
def test_bf16_repeatable(orc, name, B):
    """Bit-identical outputs on the same inputs, at batches on both sides of every kernel choice (no atomics and
    every cross-wavefront sum is taken in a fixed order), and a row's result does not depend on the batch it
    travels in when that leaves the kernel choice alone (its own row alone vs its place in a batch of 16)."""
    import torch
    cfg = wl.CONFIGS[name]
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=B), wl.make_weights(cfg))
    dev = to_device(wl.make_batch(cfg, B))
    o1 = {k: v.clone() for k, v in net.step(**dev).items()}
    o2 = {k: v.clone() for k, v in net.step(**dev).items()}
    torch.cuda.synchronize()
    for k in o1:
        assert torch.equal(o1[k], o2[k]), k
    if B <= 300:
        first16 = {k: (None if v is None else v[:16].contiguous()) for k, v in dev.items()}
        row5 = {k: (None if v is None else v[5:6].contiguous()) for k, v in dev.items()}
        a = {k: v.clone() for k, v in net.step(**first16).items()}
        b = net.step(**row5)
        torch.cuda.synchronize()
        for k in a:
            assert torch.equal(a[k][5:6], b[k]), k
    net.close()


def test_bf16_head_and_core_variants(orc):
    """Combinations the five configurations do not cover: conv stack without a core and with policy heads,
    ResNet with dueling heads and greedy selection, Football torso with an LSTM core."""
    a = dict(wl.CONFIGS["C2"], label="R2D2 torso, no core, policy heads", lstm_units=0, head=0, head_hidden=0,
             select=1, index=21)
    run_case(orc, a, 9, "bf16")
    b = dict(wl.CONFIGS["C3"], label="DMLab torso, dueling greedy", head=1, head_hidden=64, select=0, index=22)
    run_case(orc, b, 6, "bf16")
    c = dict(wl.CONFIGS["C4"], label="Football torso + LSTM-128", lstm_units=128, index=23)
    run_case(orc, c, 4, "bf16")


@pytest.mark.parametrize("label,over,B", [
    ("DMLab torso, filters x2", dict(sections=[32, 64, 64]), 5),
    ("DMLab torso, filters x4", dict(sections=[64, 128, 128]), 3),
    ("Football torso, medium map 120x90", dict(obs_h=90, obs_w=120), 4),
    ("Football torso, large map 144x108", dict(obs_h=108, obs_w=144), 2),
    ("odd frame 50x70x3, two sections, 48 channels", dict(obs_h=50, obs_w=70, sections=[16, 48]), 7),
    ("4-plane minimap 72x96x4", dict(obs_c=4, sections=[16, 32, 32, 32]), 6),
    ("odd frame 46x62x3, 32 then 96 channels", dict(obs_h=46, obs_w=62, sections=[32, 96]), 5),
    # the per-section kernels (first layer + pool, conv0 + pool, residual blocks) on maps that leave ragged tiles and odd
    # pooled sizes; with so few rows on tiles or, for small maps and at 128 channels, on strips
    ("odd frame 45x61x3, sections 64/128/128", dict(obs_h=45, obs_w=61, sections=[64, 128, 128]), 3),
    ("odd frame 37x53x1, sections 16/16/32/64", dict(obs_h=37, obs_w=53, obs_c=1, sections=[16, 16, 32, 64]), 4),
    ("frame 67x41x8, sections 32/32/64/64", dict(obs_h=67, obs_w=41, obs_c=8, sections=[32, 32, 64, 64]), 3),
    ("frame 33x99x2, sections 16/32", dict(obs_h=33, obs_w=99, obs_c=2, sections=[16, 32]), 5),
    ("16-plane map 59x83, sections 64/64", dict(obs_h=59, obs_w=83, obs_c=16, sections=[64, 64]), 3),
])
def test_bf16_model_size_variants_run_layer_by_layer(orc, label, over, B):
    """Model-size variants (Section 4.1: wider filters; Section 4.2: larger minimaps) have no fused kernel and
    take the layer-by-layer bf16 path; same tolerance as the fused torso."""
    base = wl.CONFIGS["C4"] if "Football" in label or "minimap" in label else wl.CONFIGS["C3"]
    cfg = dict(base, label=label, index=31, **over)
    got, ref, rep = run_case(orc, cfg, B, "bf16")
    assert rep["max_rel_err"] <= 2e-2


@pytest.mark.parametrize("B", [37, 300, 1100, 2100])
def test_bf16_odd_widths_through_the_dense_layer_tilings(orc, B):
    """Widths that are not whole tile groups (48 linear units = 3 feature tiles, 48 LSTM units = 3 gate groups,
    7 actions) at batches on both sides of the small-batch tilings' limits; a one-layer conv stack (layer by
    layer)."""
    cfg = dict(label="odd widths", obs_h=23, obs_w=24, obs_c=8, torso=0, convs=[(16, 4, 2)], fc_units=48,
               lstm_units=48, num_actions=7, head=0, head_hidden=0, select=1, precision="bf16", obs_kind="uniform",
               index=43)
    run_case(orc, cfg, B, "bf16")


@pytest.mark.parametrize("B", [3, 256, 700])
def test_bf16_atari_agent_without_frame_stacking(orc, B):
    """The recurrent Atari agent on single 84x84 frames (Section 4.3: the run without frame stacking): the fused
    conv stack's one-channel first layer, at a ragged small batch, one image per compute unit and several."""
    cfg = dict(wl.CONFIGS["C2"], label="Atari agent, no frame stacking", obs_c=1, index=42)
    run_case(orc, cfg, B, "bf16")


def test_bf16_unsupported_arch_is_reported():
    cfg = dict(wl.CONFIGS["C3"], sections=[16, 32, 40])
    with pytest.raises(seedinf.SeedError) as e:
        seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=2, precision="bf16"), wl.make_weights(cfg))
    assert e.value.status == 2 and "fp32" in e.value.message


@pytest.mark.parametrize("seed", range(24))
def test_fp32_random_architectures(orc, seed):
    """Seeded random architectures in fp32 mode (the reference mode covers every valid shape): both torso kinds,
    with and without core, both heads, both selections, at a ragged batch."""
    cfg = random_arch(seed, "fp32")
    st, msg = seedinf.validate(seedinf.make_arch(cfg, max_batch=5))
    assert st == 0, (cfg, msg)
    run_case(orc, cfg, 5, "fp32")


@pytest.mark.parametrize("seed", range(24))
def test_bf16_random_architectures(orc, seed):
    """Seeded random architectures within the widths the bf16 kernels cover (layer-by-layer torsos, direct dense
    kernels, every head / core / selection combination), at batches on both sides of the small-batch tilings' limits."""
    cfg = supported_random_arch(seed, "bf16")
    st, msg = seedinf.validate(seedinf.make_arch(cfg, max_batch=21, precision="bf16"))
    assert st == 0, (cfg, msg)
    run_case(orc, cfg, (21, 1, 16, 17, 100, 257, 600, 1030)[seed % 8], "bf16")


@pytest.mark.parametrize("fc_units,B", [(160, 21), (352, 40), (160, 300)])
def test_bf16_direct_dense_kernels_with_chunk_counts_of_every_residue(orc, fc_units, B):
    """The direct dense kernels walk K in stages of two 32-value chunks, three stages in flight: K segments of
    5, 11, 21 ... chunks (one more than two whole stages left at the end) through both the whole-K and the
    K-split kernels.  Linear layer K = 6 * 7 * 16 = 672 = 21 chunks; LSTM feature segment fc_units / 32 = 5 or 11."""
    cfg = dict(label=f"chunk residues fc{fc_units}", obs_h=23, obs_w=26, obs_c=5, torso=1, sections=[48, 16],
               fc_units=fc_units, lstm_units=32, num_actions=8, head=1, head_hidden=16, select=0, precision="bf16",
               obs_kind="uniform", index=71)
    run_case(orc, cfg, B, "bf16")


@pytest.mark.parametrize("seed", range(16))
def test_bf16_random_dense_widths_at_large_batch(orc, seed):
    """Seeded random widths of the linear layer, the core and the heads behind a small conv layer, at batches
    from 1536 rows (LDS-staged dense kernels where their shape rules allow, direct kernels elsewhere), with
    ragged last tiles; oracle on a sample of rows."""
    for attempt in range(50):           # redraw (seeded) until the widths are ones the kernels cover
        rng = np.random.default_rng(500 + seed + 1000 * attempt)
        B = int(rng.choice([1536, 1700, 2048, 2049, 2200, 3000, 4100]))
        head = int(rng.integers(0, 2))
        cfg = dict(label=f"random dense widths {seed}", obs_h=int(rng.choice([10, 11, 14, 15, 18])), obs_w=int(rng.choice([16, 24])),
                   obs_c=8, torso=0, convs=[(int(rng.choice([16, 32, 48])), 4, 2)], fc_units=16 * int(rng.integers(1, 25)),
                   lstm_units=0 if rng.integers(0, 4) == 0 else 16 * int(rng.integers(1, 20)),
                   num_actions=int(rng.integers(2, 33)), head=head, head_hidden=16 * int(rng.integers(1, 20)) if head else 0,
                   select=int(rng.integers(0, 2)), precision="bf16", obs_kind="uniform", index=80 + seed)
        st, msg = seedinf.validate(seedinf.make_arch(cfg, max_batch=B, precision="bf16"))
        if st == 0:
            break
    assert st == 0, (cfg, msg)
    run_full(orc, cfg, B, sample=48)


@pytest.mark.parametrize("name,B", [("C4", 257), ("C4", 600), ("C2", 257), ("C2", 515), ("C2", 1100)])
def test_bf16_persistent_grid_edges_of_the_other_fused_torsos(orc, name, B):
    """The Football torso and the fused conv stack with one more image than compute units, a ragged count and
    several images per workgroup (the conv stack double-buffers its frames across images)."""
    run_full(orc, wl.CONFIGS[name], B, sample=48)


@pytest.mark.parametrize("seed", range(16))
def test_bf16_random_layerwise_resnets(orc, seed):
    """Layer-by-layer ResNets with random odd image sizes and random channel counts in multiples of 16 and of 32
    (the LDS-tiled 3x3 kernel takes layers whose input channels are a multiple of 32, the gather kernel the rest),
    uint8 inputs of 1 .. 16 planes."""
    rng = np.random.default_rng(900 + seed)
    mult = 32 if seed % 2 == 0 else 16
    cfg = dict(label=f"random layer-by-layer resnet {seed}", obs_h=int(rng.integers(17, 64)), obs_w=int(rng.integers(17, 64)),
               obs_c=int(rng.choice([1, 3, 4, 8, 16])), torso=1,
               sections=[mult * int(rng.integers(1, 4)) for _ in range(int(rng.integers(1, 4)))],
               fc_units=64, lstm_units=32, num_actions=9, head=0, head_hidden=0, select=1, precision="bf16",
               obs_kind="uniform", index=90 + seed)
    st, msg = seedinf.validate(seedinf.make_arch(cfg, max_batch=8, precision="bf16"))
    assert st == 0, (cfg, msg)
    run_case(orc, cfg, int(rng.integers(1, 8)), "bf16")


@pytest.mark.parametrize("seed", range(32))
def test_bf16_random_conv_stacks_and_wide_action_sets(orc, seed):
    """Layer-by-layer bf16 conv stacks over the (channels, kernel) pairs their implicit-GEMM kernel covers
    (k * Cin and stride * Cin multiples of 8, k * k * Cin of 32), up to three layers; heads with up to 64
    actions (every lane-group width of the heads kernels), inputs of the widths both heads kernels take."""
    menu = {2: [4], 4: [4, 8], 8: [2, 4, 6], 16: [2, 4], 32: [1, 2, 3, 4], 48: [2, 4]}
    for attempt in range(50):           # redraw (seeded) until the stack is one the kernels cover, e.g. a flattened output of whole chunks
        rng = np.random.default_rng(700 + seed + 1000 * attempt)
        c = int(rng.choice([2, 4, 8]))
        h, w = int(rng.integers(20, 48)), 8 * int(rng.integers(3, 7))
        cfg = dict(label=f"random conv stack {seed}", obs_h=h, obs_w=w, obs_c=c, torso=0, precision="bf16", obs_kind="uniform",
                   index=110 + seed, num_actions=int(rng.choice([2, 3, 5, 9, 17, 31, 33, 50, 64])), select=int(rng.integers(0, 2)),
                   head=int(rng.integers(0, 2)), fc_units=16 * int(rng.choice([2, 4, 8, 16, 5])),
                   lstm_units=int(rng.choice([0, 32, 64, 128, 256, 48])))
        cfg["head_hidden"] = int(rng.choice([32, 64, 128, 512, 80])) if cfg["head"] == 1 else 0
        convs = []
        for _ in range(int(rng.integers(1, 4))):
            k = int(rng.choice(menu[c]))
            s = int(rng.choice([t for t in range(1, min(k, 4) + 1) if (t * c) % 8 == 0]))   # pixel step of 8 elements
            if (h - k) // s + 1 < 2 or (w - k) // s + 1 < 2:
                break
            ch = int(rng.choice([16, 32, 48]))
            convs.append((ch, k, s))
            h, w, c = (h - k) // s + 1, (w - k) // s + 1, ch
        if not convs:
            continue
        cfg["convs"] = convs
        st, msg = seedinf.validate(seedinf.make_arch(cfg, max_batch=64, precision="bf16"))
        if st == 0:
            break
    assert st == 0, (cfg, msg)
    run_case(orc, cfg, int(rng.choice([3, 16, 40, 64])), "bf16")


def test_two_instances_on_two_streams_do_not_interfere():
    """Two networks alive at once, stepped alternately on two streams: each gives bit for bit what it gives alone
    (the library keeps no state outside its handles)."""
    import torch
    res = {}
    for name, B in (("C3", 300), ("C2", 130)):
        cfg = wl.CONFIGS[name]
        net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=B), wl.make_weights(cfg))
        dev = to_device(wl.make_batch(cfg, B))
        res[name] = ({k: v.clone() for k, v in net.step(**dev).items()}, dev, cfg, B)
        torch.cuda.synchronize()
        net.close()
    nets = {n: seedinf.SeedInfer(seedinf.make_arch(c, max_batch=B), wl.make_weights(c)) for n, (_, _, c, B) in res.items()}
    streams = {n: torch.cuda.Stream() for n in res}
    outs = {}
    for rep in range(3):
        for n in res:
            with torch.cuda.stream(streams[n]):
                outs[n] = nets[n].step(**res[n][1])
    torch.cuda.synchronize()
    for n in res:
        for k, v in res[n][0].items():
            assert torch.equal(v, outs[n][k]), (n, k)
        nets[n].close()


def test_create_destroy_returns_device_memory():
    """Handles free what they allocate: device memory in use is back where it was after 25 create / step /
    destroy rounds of the headline network at batch 1024 (each holds > 100 MB of buffers and weights)."""
    import torch
    cfg = wl.CONFIGS["C3"]
    w = wl.make_weights(cfg)
    dev = to_device(wl.make_batch(cfg, 64))
    def round_():
        net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=1024), w)
        net.step(**dev)
        torch.cuda.synchronize()
        net.close()
    round_()
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    for _ in range(25):
        round_()
    torch.cuda.synchronize()
    free1, _ = torch.cuda.mem_get_info()
    assert free0 - free1 < 32 * 1024 * 1024, (free0, free1)


@pytest.mark.parametrize("precision", ["fp32", "fp32_channels_x4", "bf16"])
def test_largest_batch_the_interface_allows(orc, precision):
    """B = max_batch = 2^20 rows, the limit of the interface, on small networks: 8.6e9 activation values per
    layer in fp32 mode (more than 2^32 elements: the elementwise kernels' capped grids) and an 11 GB feature
    matrix in bf16 mode (element and byte offsets beyond 2^32); oracle on a sample of rows that includes the last one."""
    B = 1 << 20
    if precision == "fp32":
        cfg = dict(label="largest batch, fp32", obs_h=18, obs_w=18, obs_c=1, torso=0, convs=[(32, 3, 1)], fc_units=16,
                   lstm_units=8, num_actions=4, head=0, head_hidden=0, select=1, precision="fp32", obs_kind="uniform",
                   index=120)
    elif precision == "fp32_channels_x4":
        # the convolution kernel with four output channels per lane walks the images beyond the grid's 65535 rows
        cfg = dict(label="largest batch, fp32, channels x4", obs_h=10, obs_w=10, obs_c=4, torso=0, convs=[(8, 3, 1)], fc_units=16,
                   lstm_units=0, num_actions=4, head=0, head_hidden=0, select=1, precision="fp32", obs_kind="uniform",
                   index=122)
    else:
        cfg = dict(label="largest batch, bf16", obs_h=12, obs_w=16, obs_c=8, torso=0, convs=[(32, 2, 1)], fc_units=32,
                   lstm_units=16, num_actions=5, head=1, head_hidden=16, select=0, precision="bf16", obs_kind="uniform",
                   index=121)
    run_full(orc, cfg, B, sample=64)


@pytest.mark.parametrize("label,over", [
    # 34 x 22 frames: maps of 17 x 11 and 9 x 6, whole images, stacked where a round does not hold the batch; every width
    ("16/32/64", dict(obs_h=34, obs_w=22, sections=[16, 32, 64])),
    ("32/64/128", dict(obs_h=34, obs_w=22, sections=[32, 64, 128])),
    ("64/128/128", dict(obs_h=33, obs_w=21, sections=[64, 128, 128])),
])
def test_bf16_strip_kernels_stack_small_images(orc, label, over):
    """A batch large enough to stack images (a ragged last stack included) gives the same bits as the same rows in
    a batch too small for it, and those match the oracle."""
    cfg = dict(wl.CONFIGS["C3"], label=f"stacked strips {label}", index=120, **over)
    B, few = 1029 + 512, 5
    weights, batch = wl.make_weights(cfg), wl.make_batch(cfg, B)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=B), weights)
    net.step(**to_device(batch))
    big = net.read_intermediate(0, B).cpu().numpy()
    rows = [0, 1, 2, B - 2, B - 1]
    part = {k: None if v is None else np.ascontiguousarray(v[rows]) for k, v in batch.items()}
    net.step(**to_device(part))
    small = net.read_intermediate(0, few).cpu().numpy()
    net.close()
    np.testing.assert_array_equal(big[rows], small)
    run_case(orc, cfg, few, "bf16")


@pytest.mark.parametrize("label,over", [
    ("16/32/64", dict(obs_h=34, obs_w=22, sections=[16, 32, 64])),
    ("64/128/128", dict(obs_h=21, obs_w=33, sections=[64, 128, 128])),
])
def test_bf16_stacks_of_four_images(orc, label, over):
    """The largest stacks (one round of 256 workgroups, where four images fit): all four places of a stack and a ragged
    last one of three images."""
    cfg = dict(wl.CONFIGS["C3"], label=f"stacks of four {label}", index=125, **over)
    B, rows = 4 * 256 - 1, [0, 1, 2, 3, 1020, 1021, 1022]
    weights, batch = wl.make_weights(cfg), wl.make_batch(cfg, B)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=B), weights)
    net.step(**to_device(batch))
    big = net.read_intermediate(0, B).cpu().numpy()
    net.step(**to_device({k: None if v is None else np.ascontiguousarray(v[rows]) for k, v in batch.items()}))
    small = net.read_intermediate(0, len(rows)).cpu().numpy()
    net.close()
    np.testing.assert_array_equal(big[rows], small)
    run_case(orc, cfg, len(rows), "bf16")


@pytest.mark.parametrize("label,over,B", [
    # strips of one section that end in a shorter one, two strips (one halo side each) and many; rows of one pixel column
    ("64 channels, 58 x 50 maps", dict(obs_h=116, obs_w=100, obs_c=3, sections=[64]), 2),
    ("128 channels, 31 x 30 maps", dict(obs_h=124, obs_w=119, obs_c=1, sections=[64, 128]), 2),
    ("128 channels, too wide for a strip", dict(obs_h=18, obs_w=520, obs_c=1, sections=[64, 128, 128]), 2),
    ("16 channels, 70 x 61 maps", dict(obs_h=139, obs_w=121, obs_c=4, sections=[16, 16]), 2),
    ("one column", dict(obs_h=40, obs_w=2, obs_c=4, sections=[32, 64]), 3),
])
def test_bf16_strip_kernels_at_the_edges_of_their_plans(orc, label, over, B):
    cfg = dict(wl.CONFIGS["C3"], label=f"strips: {label}", index=121, fc_units=32, **over)
    run_case(orc, cfg, B, "bf16")


@pytest.mark.parametrize("label,over", [
    ("16/16/32", dict(obs_h=8, obs_w=2060, sections=[16, 16, 32])),
    ("32/32/64/64", dict(obs_h=6, obs_w=2060, sections=[32, 32, 64, 64])),
    ("64/64/128/128", dict(obs_h=9, obs_w=1030, sections=[64, 64, 128, 128])),
])
def test_bf16_maps_wider_than_any_strip(orc, label, over):
    """Frames whose maps fit no strip (more than 510 / 254 / 126 / 62 columns at 16 / 32 / 64 / 128 channels): the tile
    kernels' first layer, conv0 + pooling and blocks at every channel pair they are built for, whatever the batch."""
    cfg = dict(wl.CONFIGS["C3"], label=f"wide maps {label}", index=126, obs_c=3, fc_units=32, **over)
    run_case(orc, cfg, 2, "bf16")


@pytest.mark.parametrize("frame,sections,routes", ROUTES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_bf16_strips_and_tiles_give_the_same_bits(orc, frame, sections, routes):
    """Which kernels a section runs on depends on the batch: rows of a large batch equal the same rows in a small one, and
    the oracle."""
    h, w, c = frame
    cfg = dict(wl.CONFIGS["C3"], label=f"{h}x{w}x{c}, sections {sections}", index=124, obs_h=h, obs_w=w, obs_c=c,
               sections=list(sections), fc_units=16)
    B, few = max(b for b in routes if b <= 300), min(routes)
    weights, batch = wl.make_weights(cfg), wl.make_batch(cfg, B)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=B), weights)
    net.step(**to_device(batch))
    big = net.read_intermediate(0, B).cpu().numpy()
    for row in (0, B // 2, B - 1):
        part = {k: None if v is None else np.ascontiguousarray(v[[row] * few]) for k, v in batch.items()}
        net.step(**to_device(part))
        np.testing.assert_array_equal(net.read_intermediate(0, few).cpu().numpy(), big[[row] * few])
    net.close()
    run_case(orc, cfg, 2, "bf16")


def test_bf16_one_row_frames_wider_than_a_strip(orc):
    """Frames of one row: the residual stream between a section's blocks is larger than the conv0 map it lies over, so
    the last rows of a large batch would meet the first rows' outputs if anything live lay behind it.  Every row sampled
    equals the same row in a batch of its own, and the oracle."""
    cfg = dict(wl.CONFIGS["C3"], label="one row of 1199 pixels", index=123, obs_h=1, obs_w=1199, sections=[16, 16], fc_units=32)
    B, rows = 2048, [0, 1, 2, 3, 2044, 2045, 2046, 2047]
    weights, batch = wl.make_weights(cfg), wl.make_batch(cfg, B)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=B), weights)
    net.step(**to_device(batch))
    big = net.read_intermediate(0, B).cpu().numpy()
    net.step(**to_device({k: None if v is None else np.ascontiguousarray(v[rows]) for k, v in batch.items()}))
    small = net.read_intermediate(0, len(rows)).cpu().numpy()
    net.close()
    np.testing.assert_array_equal(big[rows], small)
    run_case(orc, cfg, len(rows), "bf16")
