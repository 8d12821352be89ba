"""The kernels at both ends of a denoising call: the prefix relayout (every
remainder of a key range mod the 16-byte run, key ranges left behind by an
earlier call) and the readout fused with the next step's embedding at four rows
per block (a partial last block, with and without pending slices, and the
residual stream it leaves).  Bars as in the other parity tests."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_helpers import compare, run_gpu, small_cfg, to_device, tolerance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kw", [
    dict(horizon=49, batch=21),                                    # 1029 rows: one row in the last block
    dict(horizon=50, batch=21, weight_dtype="f32", kv_dtype="f32"),
    dict(horizon=41, batch=26, d_model=1024, action_dim=7),        # 1066 rows of width 1024: two
    dict(horizon=41, batch=26, d_model=1024, weight_dtype="fp8"),
])
@pytest.mark.parametrize("variant", ["pi0", "pi05"])
def test_readout_four_rows(variant, kw):
    import paper_2608_03682_amd as px
    kw = dict(kw)
    if kw.get("weight_dtype") in ("f32", "fp8") and variant == "pi05":
        kw.update(weight_dtype="bf16", kv_dtype="bf16", d_mlp=2048)    # K slices of the down projection
    cfg = small_cfg(variant, n_layers=1, **kw)
    print(f"[case] readout of four rows {variant} {kw}", flush=True)
    case = wl.make_case(cfg, seed=5)
    ex = px.Expert(cfg, case.weights)
    gpu = run_gpu(ex, case)
    ex.close()
    ref = oracle.denoise(cfg, case.weights, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)
    compare(f"readout of four rows {variant} {kw}", gpu, ref, cfg)


@pytest.mark.parametrize("kw", [dict(batch=65), dict(batch=65, d_model=1024, action_dim=14)])
def test_readout_four_rows_dit(kw):
    """The same with the DiT's LayerNorm, position rows and state token (1,040
    rows), under weights that let the position rows decide: in the oracle,
    dropping them moves the actions past the bar."""
    import paper_2608_03682_amd as px
    cfg = small_cfg("dit", n_layers=1, **kw)
    print(f"[case] readout of four rows dit {kw}", flush=True)
    pos = np.random.default_rng(21).standard_normal((cfg.horizon, cfg.d_model))
    case = wl.make_case(cfg, seed=21, weights=wl.make_weights(cfg, 21, overrides={"pos_emb": pos}))
    ex = px.Expert(cfg, case.weights)
    gpu = run_gpu(ex, case)
    ex.close()

    def run(w):
        return oracle.denoise(cfg, w, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)

    ref = run(case.weights)
    compare(f"readout of four rows dit {kw}", gpu, ref, cfg)
    flat = wl.make_weights(cfg, 21, overrides={"pos_emb": 0 * pos})
    assert np.abs(run(flat) - ref).max() > 2 * tolerance(cfg) * max(1.0, float(np.sqrt(np.mean(ref ** 2))))


@pytest.mark.parametrize("variant,kw", [
    ("pi0", dict(batch=21)), ("pi05", dict(batch=21)), ("pi0", dict(batch=21, d_model=1024, n_steps=1)),
])
def test_hidden_rows_after_four_row_readout(variant, kw):
    """phyai_debug_hidden's action rows hold the last block's down projection
    also where that is split over K and the readout adds its slices four rows
    at a time (1,050 rows, the last block half empty): against the same requests
    at batch 3, whose rows other kernels finish.  Without it they are off by the
    block's MLP output, 0.1 and more; the two batches' bf16 roundings of one
    block's operands differ by up to 2e-3."""
    import paper_2608_03682_amd as px
    cfg = small_cfg(variant, n_layers=1, d_mlp=2048, **{"n_steps": 2, **kw})
    print(f"[case] hidden rows {variant} {kw}", flush=True)
    case = wl.make_case(cfg, seed=9)
    prefix, noise, state = to_device(case)
    ex = px.Expert(cfg, case.weights)

    def hidden(n):
        pick = slice(cfg.batch - n, cfg.batch)
        ex.denoise(prefix[:, :, pick].contiguous(), case.prefix_len[pick], noise[pick].contiguous(), case.timesteps,
                   None if state is None else state[pick].contiguous())
        h = ex.debug_hidden(n).cpu().numpy().astype(np.float64).reshape(n, cfg.tokens, cfg.d_model)
        return h[-3:, cfg.tokens - cfg.horizon:]

    compare(f"hidden rows {variant} {kw}", hidden(cfg.batch), hidden(3), cfg)
    ex.close()


@pytest.mark.parametrize("kw", [
    dict(head_dim=64), dict(head_dim=256, n_q_heads=2), dict(head_dim=64, weight_dtype="f32", kv_dtype="f32"),
])
def test_relayout_leaves_no_stale_key(kw):
    """An earlier call fills every key range with NaN; the next one's ranges end
    at each remainder of a run, and their masked keys have to be zeros again."""
    import paper_2608_03682_amd as px
    cfg = small_cfg("pi0", batch=9, prefix_cap=130, prefix_min=40, prefix_max=130, n_steps=2, **kw)
    print(f"[case] relayout {kw}", flush=True)
    case = wl.make_case(cfg, seed=8)
    case.prefix_len[:] = 64 + 13 - cfg.horizon - 1 + np.arange(9)      # key ranges end at 77 .. 85
    case.prefix_len[8] = 77                                            # ... and at 128, a whole tile
    prefix, noise, state = to_device(case)
    ex = px.Expert(cfg, case.weights)
    nan = torch.full_like(prefix, float("nan")) if prefix.is_floating_point() else torch.full_like(prefix, 0x7fc0)
    ex.denoise(nan, np.full(9, 130, np.int32), noise, case.timesteps, state)
    gpu = run_gpu(ex, case, dev=(prefix, noise, state))
    ex.close()
    ref = oracle.denoise(cfg, case.weights, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)
    compare(f"relayout {kw}", gpu, ref, cfg)
