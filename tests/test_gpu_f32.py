"""The fp32 path's attention and GEMMs at the edges of their launch rules:
one and several key chunks (512 keys each), a last chunk that is no multiple of
four keys, no prefix at all (the state token then sees one key), every
head_dim, and enough rows for both GEMM block heights.  Bar: the fp32 path's
own (1e-4), three decades above fp32 accumulation over these sums."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_helpers import compare, run_gpu, small_cfg, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kw", [
    dict(head_dim=64, prefix_cap=1100, prefix_min=455, prefix_max=1100),
    dict(head_dim=128, n_q_heads=2, prefix_cap=520, prefix_min=461, prefix_max=463),
    dict(head_dim=256, n_q_heads=2, prefix_cap=600, prefix_min=500, prefix_max=600, batch=2),
    dict(head_dim=64, prefix_cap=8, prefix_min=0, prefix_max=0, horizon=5, batch=1),
    dict(head_dim=64, batch=1, horizon=2, state_token=False),
    dict(head_dim=64, batch=9, d_mlp=1024),
    dict(head_dim=64, prefix_cap=12, prefix_min=0, prefix_max=12, horizon=19),        # 32 keys: D threads a block
    dict(head_dim=128, n_q_heads=2, prefix_cap=12, prefix_min=3, prefix_max=12, horizon=19),
    dict(head_dim=64, prefix_cap=13, prefix_min=13, prefix_max=13, horizon=19),       # 33: 256
])
def test_fp32_path(kw):
    import paper_2608_03682_amd as px
    cfg = small_cfg("pi0", weight_dtype="f32", kv_dtype="f32", **kw)
    print(f"[case] fp32 {kw}", flush=True)
    case = wl.make_case(cfg, seed=13)
    ex = px.Expert(cfg, case.weights)
    gpu = run_gpu(ex, case)
    ex.close()
    ref = oracle.denoise(cfg, case.weights, case.prefix, case.prefix_len, case.noise, case.timesteps, case.state)
    compare(f"fp32 {kw}", gpu, ref, cfg)


@pytest.mark.parametrize("lo,hi", [(0.0, 1.0), (1.0, 4.0), (-0.5, 0.0), (-4.0, -0.5)])
def test_fp32_gelu_is_as_accurate_as_its_tanh_form(lo, hi):
    """A DiT block on a zero residual stream whose MLP-in is its bias z, MLP-out
    the identity and gate 1 leaves gelu(z) itself in every row: its error against
    64 bits is no larger than that of z/2 (1 + tanh u) in 32-bit steps with a
    correctly rounded tanh, in the rms over 1,024 values (known to 2 %) and, within
    a tenth, at the worst of them."""
    import paper_2608_03682_amd as px
    cfg = small_cfg("dit", weight_dtype="f32", kv_dtype="f32", n_layers=1, n_steps=1, batch=1, d_model=1024,
                    d_mlp=1024, horizon=2, n_q_heads=8, n_kv_heads=8)
    print(f"[case] fp32 gelu {lo} .. {hi}", flush=True)
    d, p = cfg.d_model, "layers.0."
    z = np.random.default_rng(16).uniform(lo, hi, d).astype(np.float32)
    zero = {k: np.zeros(s) for k, s in wl.weight_specs(cfg).items()
            if k in ("in_w", "in_b", "state_w", "state_b", "pos_emb") or k in (p + "wo", p + "ada_w", p + "mlp_w1",
                                                                               p + "mlp_b2")}
    gates = np.zeros((1, 6 * d))
    gates[0, 5 * d:] = 1.0                        # shift, scale and gate of the two halves: the MLP's gate
    case = wl.make_case(cfg, seed=16, weights=wl.make_weights(cfg, 16, overrides={
        **zero, p + "ada_b": gates, p + "mlp_b1": z, p + "mlp_w2": np.eye(d)}))
    ex = px.Expert(cfg, case.weights)
    h = _hidden(ex, to_device(case), case, 1)
    ex.close()
    assert (h == h[0]).all()
    t = z.astype(np.float64)
    u = np.sqrt(2 / np.pi) * (t + 0.044715 * t ** 3)
    ref = t / (1 + np.exp(-2 * u))
    f = np.float32
    u32 = f(0.7978845608028654) * (z + f(0.044715) * z * z * z)
    tanh_form = f(0.5) * z * (f(1) + np.tanh(u32.astype(np.float64)).astype(f))
    rel = [np.abs(y.astype(np.float64) - ref) / np.abs(ref) for y in (h[0], tanh_form)]
    rms, worst = [np.sqrt((e ** 2).mean()) for e in rel], [e.max() for e in rel]
    print(f"[parity] fp32 gelu {lo} .. {hi}: rms {rms[0]:.2e} (tanh form {rms[1]:.2e}), worst {worst[0]:.2e} "
          f"({worst[1]:.2e})", flush=True)
    assert rms[0] <= rms[1] and worst[0] <= 1.1 * worst[1]


def _hidden(ex, dev, case, batch):
    prefix, noise, state = dev
    ex.denoise(prefix, case.prefix_len, noise, case.timesteps, state)
    return ex.debug_hidden(batch).cpu().numpy()


@pytest.mark.parametrize("plen", [70, 600])
def test_fp32_state_token_never_reads_masked_keys(plen):
    """The state token sees the prefix and itself, so its row of the residual
    stream stays bit for bit the same when the other suffix tokens (and with
    them their keys and values) are infinite or NaN."""
    import paper_2608_03682_amd as px
    cfg = small_cfg("pi0", weight_dtype="f32", kv_dtype="f32", n_layers=1, n_steps=1, batch=1, prefix_cap=600)
    print(f"[case] fp32 masked keys, prefix {plen}", flush=True)
    case = wl.make_case(cfg, seed=14)
    case.prefix_len[:] = plen
    prefix, noise, state = to_device(case)
    ex = px.Expert(cfg, case.weights)
    ref = _hidden(ex, (prefix, noise, state), case, 1)[0]
    assert np.isfinite(ref).all()
    for bad in (float("inf"), float("nan")):
        noise[0, 3] = bad
        np.testing.assert_array_equal(_hidden(ex, (prefix, noise, state), case, 1)[0], ref)
    ex.close()


@pytest.mark.parametrize("first,last", [(0, 1), (0, 512), (512, 600)])
def test_fp32_nan_keys_are_not_skipped(first, last):
    """NaN among the keys spoils every softmax that covers them, wherever they
    lie among the chunks of 512 and also where a chunk holds nothing else: each
    such query's attention is replaced by zeros, as with one NaN key at 40."""
    import paper_2608_03682_amd as px
    cfg = small_cfg("pi0", weight_dtype="f32", kv_dtype="f32", n_layers=1, n_steps=1, batch=1, prefix_cap=600)
    print(f"[case] fp32 NaN keys {first}..{last}", flush=True)
    case = wl.make_case(cfg, seed=15)
    case.prefix_len[:] = 600
    prefix, noise, state = to_device(case)
    ex = px.Expert(cfg, case.weights)
    one, many = prefix.clone(), prefix.clone()
    one[:, 0, :, 40] = float("nan")
    many[:, 0, :, first:last] = float("nan")
    ref = _hidden(ex, (one, noise, state), case, 1)
    assert np.isfinite(ref).all()
    np.testing.assert_array_equal(_hidden(ex, (many, noise, state), case, 1), ref)
    ex.close()
