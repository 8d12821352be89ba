"""The 256-column many-row GEMM through the C ABI: every tile height and both
pipeline depths, at shapes that leave a ragged last row tile (R not a multiple
of any of them), more and fewer column tiles than one band, K of 4 to 7 k-blocks
(every way the four-stage pipeline ends) and of 16, and each epilogue (QKV with and without RoPE and bias, K|V of the DiT
features with invalid rows, GeGLU with and without a second term, GELU, plain
stores, residual adds, K slices).  The bars are those of the other parity tests:
the operands are rounded to bf16 once per stage whatever the kernel."""
import os

import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_helpers import compare, cross_case, run_gpu, small_cfg, tolerance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILES = ["2x4", "3x4", "4x4", "4x2", "7x2", "8x2", "9x2"]


@pytest.fixture
def tile(request):
    os.environ["PHYAI_WIDE_TILE"] = request.param
    yield request.param
    del os.environ["PHYAI_WIDE_TILE"]


@pytest.mark.parametrize("tile", TILES, indirect=True)
@pytest.mark.parametrize("variant,kw", [
    ("pi0", dict(batch=7, n_q_heads=2, d_mlp=1024)),
    ("pi0", dict(batch=7, n_q_heads=2, d_mlp=1024, weight_dtype="fp8")),
    ("pi05", dict(batch=7, n_q_heads=3, n_kv_heads=1, head_dim=256)),
    ("dit", dict(batch=5, d_feat=256, prefix_cap=90, prefix_min=31, prefix_max=90, horizon=60, n_q_heads=4,
                 n_kv_heads=4)),
])
def test_wide_gemm_expert(tile, variant, kw):
    import paper_2608_03682_amd as px
    cfg = small_cfg(variant, **kw)
    print(f"[case] wide tile {tile} {variant} {kw}", flush=True)
    case = wl.make_case(cfg, seed=11)
    ex = px.Expert(cfg, case.weights)
    gpu = run_gpu(ex, case)
    ex.close()
    ref = oracle.denoise(cfg, case.weights, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)
    compare(f"wide tile {tile} {variant} {kw}", gpu, ref, cfg)


@pytest.mark.parametrize("tile", TILES, indirect=True)
@pytest.mark.parametrize("wdt", ["bf16", "fp8"])
def test_wide_gemm_keys_of_several_cross_blocks(tile, wdt):
    """As test_dit_keys_of_several_cross_blocks, 450 feature rows; rows a request
    does not have leave zero keys whatever they hold."""
    import paper_2608_03682_amd as px
    cfg = small_cfg("dit", n_layers=4, weight_dtype=wdt, batch=5, prefix_cap=90, prefix_min=31, prefix_max=90)
    print(f"[case] wide tile {tile} dit, two cross blocks {wdt}", flush=True)
    case = cross_case(cfg, 17)
    ex = px.Expert(cfg, case.weights)
    gpu = run_gpu(ex, case)
    assert case.prefix_len.min() < cfg.prefix_cap
    case.prefix = wl.make_prefix(cfg, case.prefix_len, 17, pad_value=float("nan"))
    assert np.array_equal(run_gpu(ex, case), gpu)
    ex.close()
    ref = oracle.denoise(cfg, case.weights, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)
    compare(f"wide tile {tile} dit, two cross blocks {wdt}", gpu, ref, cfg)


@pytest.mark.parametrize("tile", TILES[:3], indirect=True)
@pytest.mark.parametrize("variant,wdt", [("pi0", "bf16"), ("pi0", "fp8"), ("pi05", "bf16")])
@pytest.mark.parametrize("kb", [5, 6, 7])
def test_wide_gemm_pipeline_tails(tile, variant, wdt, kb):
    """The four-stage pipeline ends with 3, 4, 5 or 6 k-blocks left: 5, 6 and 7
    k-blocks in the output projection (heads of 64; pi0) and in the down
    projection (with a second operand term in pi0.5)."""
    import paper_2608_03682_amd as px
    kw = dict(n_q_heads=kb) if variant == "pi0" else {}
    cfg = small_cfg(variant, batch=7, d_mlp=64 * kb, weight_dtype=wdt, **kw)
    print(f"[case] wide tile {tile} {variant} {wdt} {kb} k-blocks", flush=True)
    case = wl.make_case(cfg, seed=19)
    ex = px.Expert(cfg, case.weights)
    gpu = run_gpu(ex, case)
    ex.close()
    ref = oracle.denoise(cfg, case.weights, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)
    compare(f"wide tile {tile} {variant} {wdt} {kb} k-blocks", gpu, ref, cfg)


@pytest.mark.parametrize("tile", TILES, indirect=True)
@pytest.mark.parametrize("wdt", ["bf16", "fp8"])
def test_wide_gemm_vision(tile, wdt):
    import paper_2608_03682_amd as px
    cfg = wl.ExpertConfig(
        name="wide_vit", cfg_id=71, variant="vision", n_layers=2, d_model=512, n_q_heads=8, n_kv_heads=8, head_dim=64,
        d_mlp=1024, horizon=0, action_dim=0, n_steps=0, prefix_cap=0, prefix_min=0, prefix_max=0, batch=3,
        state_token=False, rope=False, weight_dtype=wdt, kv_dtype="bf16", time_dim=0, n_images=2, n_patches=71,
        patch_dim=1024, d_out=768)
    print(f"[case] wide tile {tile} vision {wdt}", flush=True)
    case = wl.make_vision_case(cfg, seed=12)
    for k, t in case.weights.items():             # biases that decide the result (see test_gpu_vision.py)
        if k.endswith((".bq", ".bv")):
            rng = np.random.default_rng(len(k))
            t.data[:] = wl.bf16_bits_from_f32(rng.standard_normal(t.data.shape).astype(np.float32))
    m = px.VisionTower(cfg, case.weights)
    out = m.encode(torch.from_numpy(case.patches).cuda())
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    m.close()
    ref = oracle.encode_images(cfg, case.weights, case.patches)
    rms = float(np.sqrt(np.mean(ref ** 2)))
    # six deviations of L + 2 roundings to bf16 in quadrature, as for the tower at large
    bar = 6 * 2.0 ** -8 * np.sqrt(cfg.n_layers + 2) * max(1.0, rms)
    err = float(np.abs(got - ref).max())
    print(f"[parity] wide tile {tile} vision {wdt}: max_abs={err:.3e} bar={bar:.1e}", flush=True)
    assert np.isfinite(got).all() and err <= bar


@pytest.mark.parametrize("variant", ["pi0", "pi05", "dit"])
def test_schedule_tables_of_many_steps(variant):
    """From 256 Euler steps on the timestep tables come from the many-row GEMMs
    too.  300 steps, of which the last ten take all but 1e-3 of the way, and
    timestep weights of 0.6: in the oracle, actions without them are off by ten
    bars and more."""
    import paper_2608_03682_amd as px
    cfg = small_cfg(variant, n_layers=1, n_steps=300, horizon=5, batch=1)
    print(f"[case] 300 steps {variant}", flush=True)
    name = "time_w1" if variant == "pi0" else "cond_w1"
    w = 0.02 * np.random.default_rng(20).standard_normal(wl.weight_specs(cfg)[name])
    w[-cfg.time_dim:] *= 30
    case = wl.make_case(cfg, seed=20, weights=wl.make_weights(cfg, 20, overrides={name: w}))
    case.timesteps = np.concatenate([np.linspace(1, 0.999, 290, endpoint=False),
                                     np.linspace(0.999, 0, 11)]).astype(np.float32)
    ex = px.Expert(cfg, case.weights)
    gpu = run_gpu(ex, case)
    ex.close()

    def run(weights):
        return oracle.denoise(cfg, weights, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)

    ref = run(case.weights)
    compare(f"300 steps {variant}", gpu, ref, cfg)
    w[-cfg.time_dim:] = 0
    off = np.abs(run(wl.make_weights(cfg, 20, overrides={name: w})) - ref).max()
    assert off > 10 * tolerance(cfg) * max(1.0, float(np.sqrt(np.mean(ref ** 2))))
