"""End-to-end parity of vla_prefix_kv_build + vla_denoise against the fp64
oracle on the seeded workloads, plus the closed-form special cases run on the
GPU (zero / constant velocity field), determinism, graph-vs-stream identity
and batch independence.

Tolerances on the final action chunk: max|d| <= 1e-4 for the fp32 workload,
<= 2e-2 for the bf16 and W2A8 workloads, always against the plain fp64
oracle.  The 24-layer W2A8 workload is compared element-wise with a small
static residual gate that makes the random-weight stack contractive (at its
own gates a single flipped int8 code anywhere moves the chunk by more than
the tolerance, so two correct evaluations cannot agree there); at its own
gates it is checked against the oracle's rounding-noise envelope.
"""
import os

import numpy as np
import pytest

import workloads as wl
from oracle import vla_oracle as O

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2, "ternary": 2e-2}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def _pipe(cfg, W, inp, loop_mode=1):
    from vla_testlib import Pipeline
    return Pipeline(cfg, W, inp, loop_mode)


def _oracle(cfg, W, inp, tau, mean=None, std=None):
    cache = O.prefix_kv_build(cfg, W, inp["prefix"])
    return cache, O.denoise(cfg, W, cache, inp["noise"], inp["state"], tau, mean, std)


def _check_cache(pipe, cache_ref, cfg):
    got = pipe.cache_array()
    tol = 1e-5 if cfg.wtype == "f32" else 1e-2 * max(1.0, np.abs(cache_ref).max())
    if cfg.wtype == "ternary":
        tol = 3e-2 * np.abs(cache_ref).max()
    err = np.abs(got - cache_ref).max()
    assert err <= tol, f"cache max err {err} > {tol}"


@pytest.mark.parametrize("name", ["tiny_f32", "smolvla_bf16", "pi0_bf16", "gr00t_alt_bf16", "evo1_cross_bf16"])
def test_end_to_end(torch, name):
    from vla_testlib import workload
    cfg, W, inp = workload(name, 1)
    tau = wl.uniform_schedule(cfg.n_steps)
    mean = np.linspace(-0.5, 0.5, cfg.d_action).astype(np.float32)
    std = np.linspace(0.5, 2.0, cfg.d_action).astype(np.float32)
    cache_ref, ref = _oracle(cfg, W, inp, tau, mean, std)
    pipe = _pipe(cfg, W, inp)
    try:
        pipe.build_cache()
        from vla_testlib import to_device
        out = pipe.denoise(tau, to_device(mean), to_device(std))
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        _check_cache(pipe, cache_ref, cfg)
        err = np.abs(got - ref).max()
        print(f"{name}: max|d| = {err:.3e} (tol {TOL[cfg.wtype]})")
        assert np.all(np.isfinite(got))
        assert err <= TOL[cfg.wtype], f"{name}: max|d| {err}"
    finally:
        pipe.close()


@pytest.mark.parametrize("name", ["tiny_f32", "smolvla_bf16", "pi0_bf16"])
def test_end_to_end_causal_variant(torch, name):
    """The causal action-token variant (VLA_OPT_CAUSAL_SELF) end to end against
    the oracle with the same mask, under the default loop driver (for pi0 the
    persistent kernel); the mask changes the chunk."""
    from vla_testlib import workload
    cfg0, W, inp = workload(name, 1)
    cfg = cfg0.with_(n_steps=3, causal_self=True)
    tau = wl.uniform_schedule(cfg.n_steps)
    _, ref = _oracle(cfg, W, inp, tau)
    _, ref0 = _oracle(cfg.with_(causal_self=False), W, inp, tau)
    pipe = _pipe(cfg, W, inp, loop_mode=2)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
        err = np.abs(got - ref).max()
        print(f"{name} causal: max|d| = {err:.3e} (tol {TOL[cfg.wtype]}), mask effect {np.abs(ref - ref0).max():.3e}")
        assert np.all(np.isfinite(got))
        assert err <= TOL[cfg.wtype], f"{name}: max|d| {err}"
        # the mask was applied: the chunk is much closer to the masked oracle than
        # the unmasked oracle is
        assert err < 0.5 * np.abs(ref - ref0).max()
    finally:
        pipe.close()


@pytest.mark.parametrize("name,extra", [
    ("tiny_f32", {}), ("smolvla_bf16", {}), ("pi0_bf16", {}),
    ("tiny_f32", dict(causal_self=True, rope_base=10000.0)),
    ("smolvla_bf16", dict(causal_self=True)),
])
def test_end_to_end_state_token_variant(torch, name, extra):
    """The prepended state-token variant (VLA_OPT_STATE_TOKEN) end to end
    against the oracle: n + 1 token rows per request, the state row feeding
    attention only, actions_out in the [B, n, d_action] layout; also combined
    with the causal mask and RoPE, where the state row is token 0."""
    from vla_testlib import workload
    cfg0, W, inp = workload(name, 1)
    cfg = cfg0.with_(n_steps=3, state_token=True, **extra)
    tau = wl.uniform_schedule(cfg.n_steps)
    _, ref = _oracle(cfg, W, inp, tau)
    _, ref0 = _oracle(cfg.with_(state_token=False), W, inp, tau)
    pipe = _pipe(cfg, W, inp, loop_mode=2)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
        err = np.abs(got - ref).max()
        print(f"{name} {extra} state token: max|d| = {err:.3e} (tol {TOL[cfg.wtype]}), "
              f"variant effect {np.abs(ref - ref0).max():.3e}")
        assert got.shape == ref.shape == ref0.shape
        assert np.all(np.isfinite(got))
        assert err <= TOL[cfg.wtype], f"{name}: max|d| {err}"
        assert err < 0.5 * np.abs(ref - ref0).max()   # the state token was used
    finally:
        pipe.close()


@pytest.mark.parametrize("name,batch", [("tiny_f32", 3), ("smolvla_bf16", 2)])
def test_state_token_batched_requests(torch, name, batch):
    """State token with several requests: request b's token rows sit at
    b (n + 1) .. b (n + 1) + n on the device and its actions at b n .. b n + n - 1
    in actions_out. Stream and graph drivers, a non-uniform schedule."""
    cfg = wl.CONFIGS[name].with_(state_token=True, batch=batch)
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, batch)
    tau = np.array([1.0, 0.7, 0.35, 0.0], np.float32)
    _, ref = _oracle(cfg, W, inp, tau)
    for mode in (0, 1):
        pipe = _pipe(cfg, W, inp, loop_mode=mode)
        try:
            pipe.build_cache()
            got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
            err = np.abs(got - ref).max()
            print(f"{name} B={batch} mode {mode} state token: max|d| = {err:.3e}")
            assert got.shape == ref.shape
            assert err <= TOL[cfg.wtype], f"{name} mode {mode}: max|d| {err}"
        finally:
            pipe.close()


@pytest.mark.parametrize("name", ["tiny_f32", "smolvla_bf16", "pi0_bf16"])
def test_end_to_end_rope_variant(torch, name):
    """The rotary position embedding variant (VLA_OPT_ROPE_BASE) end to end
    against the oracle with the same rotation: the cached prefix keys of joint
    layers (rotated to positions 0 .. P-1) and the chunk, under the default
    loop driver (the graph driver runs it)."""
    from vla_testlib import workload
    cfg0, W, inp = workload(name, 1)
    cfg = cfg0.with_(n_steps=3, rope_base=10000.0)
    tau = wl.uniform_schedule(cfg.n_steps)
    cache_ref, ref = _oracle(cfg, W, inp, tau)
    _, ref0 = _oracle(cfg.with_(rope_base=0.0), W, inp, tau)
    pipe = _pipe(cfg, W, inp, loop_mode=2)
    try:
        pipe.build_cache()
        _check_cache(pipe, cache_ref, cfg)
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
        err = np.abs(got - ref).max()
        print(f"{name} rope: max|d| = {err:.3e} (tol {TOL[cfg.wtype]}), rotation effect {np.abs(ref - ref0).max():.3e}")
        assert np.all(np.isfinite(got))
        assert err <= TOL[cfg.wtype], f"{name}: max|d| {err}"
        assert err < 0.5 * np.abs(ref - ref0).max()   # the rotation was applied
    finally:
        pipe.close()


def test_tiny_nonuniform_schedule_and_batch(torch):
    """fp32 workload, B = 3, a non-uniform schedule, stream and graph drivers."""
    cfg = wl.TINY_F32
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 3)
    tau = np.array([1.0, 0.8, 0.45, 0.3, 0.05, 0.0], np.float32)
    _, ref = _oracle(cfg, W, inp, tau)
    for mode in (0, 1):
        pipe = _pipe(cfg, W, inp, loop_mode=mode)
        try:
            pipe.build_cache()
            got = pipe.denoise(tau).cpu().numpy()
            assert np.abs(got - ref).max() <= 1e-4
        finally:
            pipe.close()


def test_zero_and_constant_velocity_on_gpu(torch):
    """W_out = 0: b_out = 0 returns the noise bit-exactly; b_out = c gives the
    Euler endpoint noise + (tau_T - tau_0) c."""
    cfg = wl.SMOLVLA_BF16.with_(n_layers=2)
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 2)
    W["W_out"] = np.zeros_like(W["W_out"])
    W["b_out"] = np.zeros_like(W["b_out"])
    tau = wl.uniform_schedule(cfg.n_steps)
    pipe = _pipe(cfg, W, inp)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy()
        assert np.array_equal(got, inp["noise"])
    finally:
        pipe.close()
    c = np.linspace(-1, 1, cfg.d_action).astype(np.float32)
    W["b_out"] = c
    pipe = _pipe(cfg, W, inp)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy()
        expect = inp["noise"] + (float(tau[-1]) - float(tau[0])) * c
        np.testing.assert_allclose(got, expect, atol=2e-6)
    finally:
        pipe.close()


def test_determinism_and_graph_equals_stream(torch):
    from vla_testlib import workload
    cfg, W, inp = workload("smolvla_bf16", 1)
    tau = wl.uniform_schedule(cfg.n_steps)
    outs = []
    for mode in (1, 0):
        pipe = _pipe(cfg, W, inp, loop_mode=mode)
        try:
            pipe.build_cache()
            a = pipe.denoise(tau).clone()
            pipe.build_cache()       # rebuilt cache: same bits
            b = pipe.denoise(tau).clone()
            assert torch.equal(a, b)
            outs.append(a)
        finally:
            pipe.close()
    assert torch.equal(outs[0], outs[1])


def test_stress_batch_independence_and_parity(torch):
    """pi0-shaped stress workload (P = 2048, n = 100, 2 solver steps): in a
    B = 4 call, requests 0 and 3 each match their own oracle chunk at the bf16
    bar, and agree with separate B = 1 calls to the same bar (not bitwise:
    the K-split of a GEMM depends on its row count, so fp32 summation order
    differs with the batch)."""
    from vla_testlib import Pipeline
    cfg = wl.STRESS_PI0.with_(n_steps=2)
    W = wl.make_weights(cfg)
    inp4 = wl.make_batch(cfg, 4)
    tau = wl.uniform_schedule(cfg.n_steps)
    p4 = Pipeline(cfg, W, inp4)
    try:
        p4.build_cache()
        out4 = p4.denoise(tau).cpu().numpy()
    finally:
        p4.close()
    for r in (0, 3):
        one = {k: v[r:r + 1] for k, v in inp4.items()}
        p1 = Pipeline(cfg, W, one)
        try:
            p1.build_cache()
            out1 = p1.denoise(tau).cpu().numpy()
        finally:
            p1.close()
        _, ref = _oracle(cfg, W, one, tau)
        e4 = np.abs(out4[r] - ref[0]).max()
        e1 = np.abs(out1[0] - ref[0]).max()
        dev = np.abs(out1[0] - out4[r]).max()
        print(f"stress request {r}: B=4 vs oracle {e4:.3e}, B=1 vs oracle {e1:.3e}, B=4 vs B=1 {dev:.3e}")
        assert e4 <= 2e-2 and e1 <= 2e-2 and dev <= 2e-2


def test_stress_batch16_full_size_matches_single_requests(torch):
    """The batch-16 stress workload at its full size and launch configuration
    (P = 2048, n = 100, T = 20, the library's default driver: tiled GEMMs and
    tiled attention): sampled requests match the same requests run alone at
    B = 1 (untiled attention, other GEMM tiles) to the bf16 bar.  The oracle
    is too slow at this size; the B = 1 path is itself oracle-checked above."""
    from vla_testlib import Pipeline
    cfg = wl.STRESS_PI0
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 16)
    tau = wl.uniform_schedule(cfg.n_steps)
    p16 = Pipeline(cfg, W, inp, loop_mode=2)
    try:
        p16.build_cache()
        out16 = p16.denoise(tau).cpu().numpy()
    finally:
        p16.close()
    assert np.isfinite(out16).all()
    for r in (0, 7, 15):
        one = {k: v[r:r + 1] for k, v in inp.items()}
        p1 = Pipeline(cfg, W, one, loop_mode=2)
        try:
            p1.build_cache()
            out1 = p1.denoise(tau).cpu().numpy()
        finally:
            p1.close()
        dev = np.abs(out1[0] - out16[r]).max()
        scale = np.abs(out1[0]).max()
        print(f"stress B=16 request {r}: max |B=16 - B=1| {dev:.3e} (max |a| {scale:.2f})")
        assert dev <= 2e-2


def test_cache_reuse_equals_rebuild_per_call(torch):
    """The cached K/V serve every solver step: a T-step call equals the same
    call after rebuilding the cache (bitwise)."""
    cfg = wl.PI0_BF16.with_(n_layers=3, n_steps=4)
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 1)
    tau = wl.uniform_schedule(cfg.n_steps)
    pipe = _pipe(cfg, W, inp)
    try:
        pipe.build_cache()
        a = pipe.denoise(tau).clone()
        b = pipe.denoise(tau).clone()
        pipe.build_cache()
        c = pipe.denoise(tau).clone()
        assert torch.equal(a, b) and torch.equal(a, c)
        _, ref = _oracle(cfg, W, inp, tau)
        assert np.abs(a.cpu().numpy() - ref).max() <= 2e-2
    finally:
        pipe.close()


def _ternary_run(torch, cfg, W, inp):
    """GPU chunk (prefix K/V build + one regression pass) and the plain fp64
    oracle's chunk on the same inputs."""
    from vla_testlib import Pipeline
    tau = wl.uniform_schedule(1)
    pipe = Pipeline(cfg, W, inp)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
        cache_ref = O.prefix_kv_build(cfg, W, inp["prefix"])
        _check_cache(pipe, cache_ref, cfg)
    finally:
        pipe.close()
    ref = O.denoise(cfg, W, cache_ref, inp["noise"], inp["state"], tau)
    return got, ref


def _set_gates(cfg, W, alphas):
    """Static modulation table with residual gate alphas[j] in sublayer j of
    every layer (gamma, beta unchanged)."""
    d = cfg.d_model
    W = dict(W)
    for l in range(cfg.n_layers):
        m = W[f"L{l}.mod"].copy()
        for j, a in enumerate(alphas):
            m[(3 * j + 2) * d:(3 * j + 3) * d] = a
        W[f"L{l}.mod"] = m
    return W


@pytest.mark.parametrize("branch,alpha", [("attention", 0.25), ("mlp", 0.5)])
def test_ternary_single_branch(torch, branch, alpha):
    """Full W2A8 widths (d = 2560, F = 6912, 20 x 128 heads, 5 K/V heads,
    P = 512), one layer, one residual branch gated on and the other off,
    against the plain fp64 oracle at 2e-2: every ternary projection, quantiser
    and epilogue of the branch runs.  The attention branch's gate is 0.25: the
    kernel stores Q, K, V and the cache in bf16, which moves some int8 codes of
    the O-projection input by one (a CPU study of the oracle with those values
    rounded to bf16 puts that at 1.3e-2 for a gate of 0.5, half that at 0.25);
    the MLP branch's quantiser inputs are fp32 on both sides."""
    cfg = wl.TERNARY_W2A8.with_(n_layers=1)
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 1)
    gates = (alpha, 0.0) if branch == "attention" else (0.0, alpha)
    got, ref = _ternary_run(torch, cfg, _set_gates(cfg, W, gates), inp)
    ref0 = O.denoise(cfg, _set_gates(cfg, W, (0.0, 0.0)), O.prefix_kv_build(cfg, W, inp["prefix"]),
                     inp["noise"], inp["state"], wl.uniform_schedule(1))
    err = np.abs(got - ref).max()
    eff = np.abs(ref - ref0).max()
    print(f"ternary {branch} branch (alpha {alpha}): max|d| = {err:.3e}, branch effect {eff:.3f}")
    assert np.all(np.isfinite(got)) and err <= 2e-2
    assert eff > 0.25


def test_ternary_full_depth_contractive(torch):
    """All 24 W2A8 layers, every ternary GEMM active, against the plain fp64
    oracle element-wise at 2e-2.  The gate is a static 0.02 on every sublayer
    and the learned position table is N(0, 2^2), so the residual stream is
    dominated by its input and the stack is contractive: on this random-weight
    stack at gate 0.05 or more a single flipped int8 code anywhere moves the
    chunk by 3e-2 to 0.2 (CPU study of the oracle against itself with 1e-7
    quantiser-input jitter), so two correct evaluations cannot agree at 2e-2.
    The layers still move the chunk by far more than the tolerance (checked
    against the same expert with every gate at 0)."""
    cfg = wl.TERNARY_W2A8
    W = wl.make_weights(cfg)
    W["E_pos"] = wl.random_matrix(W["E_pos"].shape, 4242, 2.0, bf16=True)
    inp = wl.make_batch(cfg, 1)
    Wc = _set_gates(cfg, W, (0.02, 0.02))
    got, ref = _ternary_run(torch, cfg, Wc, inp)
    ref0 = O.denoise(cfg, _set_gates(cfg, W, (0.0, 0.0)), O.prefix_kv_build(cfg, W, inp["prefix"]),
                     inp["noise"], inp["state"], wl.uniform_schedule(1))
    err = np.abs(got - ref).max()
    eff = np.abs(ref - ref0).max()
    print(f"ternary 24 layers, gate 0.02: max|d| = {err:.3e}, mean {np.abs(got - ref).mean():.2e}, "
          f"layers' effect {eff:.3f}")
    assert np.all(np.isfinite(got)) and err <= 2e-2
    assert eff > 0.1


def test_ternary_full_depth_envelope(torch):
    """Supplement to the element-wise test above: the 24-layer W2A8 workload at
    its own gates (alpha = 1), where two correct evaluations differ by the
    stack's quantisation noise.  The GPU chunk lies within a few times the
    oracle's own noise envelope (tests/golden/ternary_envelope.txt: the plain
    oracle against itself with 1e-5 quantiser-input jitter) around the oracle
    chunk."""
    from vla_testlib import workload
    cfg, W, inp = workload("ternary_w2a8", 1)
    env_max, env_mean, ref_rms = np.loadtxt(os.path.join(os.path.dirname(__file__), "golden",
                                                         "ternary_envelope.txt"))
    got, ref = _ternary_run(torch, cfg, W, inp)
    d = np.abs(got - ref)
    print(f"ternary 24 layers: max|d| = {d.max():.3e} (envelope {env_max:.3e}), "
          f"mean|d| = {d.mean():.3e} (envelope {env_mean:.3e}), rms ref {ref_rms:.3f}")
    assert np.all(np.isfinite(got))
    assert abs(np.sqrt(np.mean(ref ** 2)) - ref_rms) < 1e-6 * max(1.0, ref_rms) + 1e-9
    assert d.mean() <= 2 * env_mean and d.max() <= 3 * env_max


@pytest.mark.timeout(900)
def test_stress_t20_single_request_vs_oracle(torch):
    """The stress workload at its real solver-step count: one request (P =
    2048, n = 100, T = 20) under the library's default driver against the fp64
    oracle at the bf16 bar."""
    from vla_testlib import Pipeline
    cfg = wl.STRESS_PI0
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 1)
    tau = wl.uniform_schedule(cfg.n_steps)
    pipe = Pipeline(cfg, W, inp, loop_mode=2)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
    finally:
        pipe.close()
    print("stress T=20: GPU done, oracle (about a minute) ...", flush=True)
    _, ref = _oracle(cfg, W, inp, tau)
    err = np.abs(got - ref).max()
    print(f"stress T=20 single request: max|d| = {err:.3e} (max |a| {np.abs(ref).max():.2f})")
    assert np.all(np.isfinite(got)) and err <= 2e-2


@pytest.mark.timeout(600)
def test_stress_batch16_sampled_requests_vs_oracle(torch):
    """Batch 16 of the stress workload (P = 2048, n = 100; the tiled GEMMs and
    tiled attention run at this size) at T = 2: requests 0, 9 and 15 of the
    B = 16 call against their own oracle chunks at the bf16 bar."""
    from vla_testlib import Pipeline
    cfg = wl.STRESS_PI0.with_(n_steps=2)
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 16)
    tau = wl.uniform_schedule(cfg.n_steps)
    pipe = Pipeline(cfg, W, inp, loop_mode=2)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
    finally:
        pipe.close()
    for r in (0, 9, 15):
        one = {k: v[r:r + 1] for k, v in inp.items()}
        _, ref = _oracle(cfg, W, one, tau)
        err = np.abs(got[r] - ref[0]).max()
        print(f"stress B=16 request {r} (T=2): max|d| vs oracle = {err:.3e}", flush=True)
        assert np.all(np.isfinite(got[r])) and err <= 2e-2


# Degenerate and limit shapes: one action token and one prefix row (every
# attention has a single query or a single prefix key, every row tile is
# ragged), action and state width 1, one or two solver steps; and the
# persistent kernel's largest chunk (64 action tokens) over a 1000-row prefix
# (18 key splits).  Loop mode 2 runs the persistent kernel where the model
# fits it and the graph driver otherwise.
_PI0_SMALL = wl.PI0_BF16.with_(n_layers=2, d_model=512, head_dim=64, d_ff=2048, d_prefix=512)
EDGE = {
    "f32_single": wl.TINY_F32.with_(name="edge_f32", n_action=1, prefix_len=1, d_action=1, d_state=1,
                                    n_steps=1, seed_base=9100),
    "alt_single": wl.SMOLVLA_BF16.with_(name="edge_alt", n_layers=2, n_action=1, prefix_len=1, d_action=1,
                                        d_state=1, n_steps=2, seed_base=9200),
    "joint_single": _PI0_SMALL.with_(name="edge_joint", n_action=1, prefix_len=1, d_action=1, d_state=1,
                                     n_steps=2, seed_base=9300),
    "joint_max_chunk": _PI0_SMALL.with_(name="edge_joint_max", n_action=64, prefix_len=1000, n_steps=2,
                                        seed_base=9400),
}


@pytest.mark.parametrize("loop_mode", [1, 2])
@pytest.mark.parametrize("name", sorted(EDGE))
def test_degenerate_and_limit_shapes(torch, name, loop_mode):
    cfg = EDGE[name]
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, 1)
    tau = wl.uniform_schedule(cfg.n_steps)
    cache_ref, ref = _oracle(cfg, W, inp, tau)
    pipe = _pipe(cfg, W, inp, loop_mode)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
        _check_cache(pipe, cache_ref, cfg)
    finally:
        pipe.close()
    err = np.abs(got - ref).max()
    print(f"{name} (loop mode {loop_mode}): max|d| = {err:.3e} (tol {TOL[cfg.wtype]})")
    assert np.all(np.isfinite(got))
    assert err <= TOL[cfg.wtype]


# Above 128 token rows (where the tiled GEMM kernel takes over): widths that are padded to whole 64-value slices
# (720, 712 and 1360), gate/up projections that stay on the skinny kernel (150 rows) and ones that do not (408), the
# state token's extra row of every request, and fp32 (136 rows).
ROWS = {
    "smolvla_3": (wl.SMOLVLA_BF16.with_(name="rows_3", n_layers=2, prefix_len=65, n_steps=2, seed_base=9500), 3),
    "smolvla_8_variants": (wl.SMOLVLA_BF16.with_(name="rows_8", n_layers=2, prefix_len=33, n_steps=2, causal_self=True,
                                                 state_token=True, seed_base=9510), 8),
    "ragged_widths_4": (wl.SMOLVLA_BF16.with_(name="rows_4", n_layers=2, d_model=712, d_ff=1360, mlp="gelu",
                                              prefix_len=40, n_steps=2, seed_base=9520), 4),
    "f32_17": (wl.TINY_F32.with_(name="rows_17", n_steps=2, seed_base=9530), 17),
}


@pytest.mark.parametrize("name", sorted(ROWS))
def test_many_token_rows(torch, name):
    cfg, batch = ROWS[name]
    W = wl.make_weights(cfg)
    inp = wl.make_batch(cfg, batch)
    tau = wl.uniform_schedule(cfg.n_steps)
    cache_ref, ref = _oracle(cfg, W, inp, tau)
    pipe = _pipe(cfg, W, inp)
    try:
        pipe.build_cache()
        got = pipe.denoise(tau).cpu().numpy().astype(np.float64)
        _check_cache(pipe, cache_ref, cfg)
    finally:
        pipe.close()
    err = np.abs(got - ref).max()
    print(f"{name}: max|d| = {err:.3e} (tol {TOL[cfg.wtype]})")
    assert np.all(np.isfinite(got))
    assert err <= TOL[cfg.wtype]
