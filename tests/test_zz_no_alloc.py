"""The allocation-free denoise entry point against the ordinary one.

reflex_denoise_chunk_static keeps the chunk's transient buffers in the
library's static device array and enqueues its launches without a graph; it
runs the same kernels in the same order as reflex_denoise_chunk, so the two
must agree bit for bit, and both must match the float64 oracle within the
bf16 tolerance (relative-L2 1e-2, max-abs 5e-2) or the fp32 one (max-abs
1e-4).  Two calls in a row on different contexts, the second with a smaller
input (fewer envs, fewer dynamic tokens), check that what the first call left
in the shared array does not leak into the second.
"""
import ctypes

import numpy as np
import pytest
import torch

from oracle import reflex_oracle as O
from paper_2607_14695_amd import reflex as R
from paper_2607_14695_amd import workloads as WL
from tests import plan_model as P

pytestmark = pytest.mark.gpu

BASE = WL.CONFIGS["tiny_fp32"].replace(
    name="noalloc", static_len=40, frame_tokens=24, window_frames=3, n_q_heads=3, head_dim=128, width=128,
    mlp_dim=192, cond_hidden=64, state_dim=8, action_dim=5, frame_dim=72, n_layers=2, num_steps=3)


def _static_call(eng, state, noise):
    """reflex_denoise_chunk_static through the C ABI, output into a fresh tensor."""
    s = torch.from_numpy(np.ascontiguousarray(state, dtype=np.float32)).to(eng.device)
    n = torch.from_numpy(np.ascontiguousarray(noise, dtype=np.float32)).to(eng.device)
    out = torch.full_like(n, float("nan"))
    eng.stream.wait_stream(torch.cuda.current_stream(eng.device))
    st = eng.lib.reflex_denoise_chunk_static(eng.ctx, s.data_ptr(), n.data_ptr(), eng.cfg.num_steps, None,
                                             out.data_ptr())
    assert st == R.REFLEX_OK, R.strerror(st)
    eng.stream.synchronize()
    return out.cpu().numpy()


def _check_oracle(cfg, got, ref):
    if cfg.bf16:
        rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
        mx = float(np.max(np.abs(got - ref)))
        assert rel <= 1e-2 and mx <= 5e-2, (rel, mx)
    else:
        assert float(np.max(np.abs(got - ref))) <= 1e-4


def _run(cfg, ticks):
    print(f"no-alloc: {cfg.name} batch {cfg.batch} T {cfg.dyn_tokens} dtype {cfg.dtype}", flush=True)
    w = WL.make_weights(cfg)
    sk, sv = WL.make_static_kv(cfg)
    frames = {t: WL.make_frame(cfg, t) for t in range(ticks)}
    eng = R.ReflexEngine(cfg, w, sk, sv)
    for t in range(ticks):
        eng.write_frame(frames[t])
    state, noise = WL.make_state(cfg, ticks - 1), WL.make_noise(cfg, ticks - 1)
    ref_gpu = eng.denoise(state, noise).cpu().numpy()
    eng.synchronize()
    got = _static_call(eng, state, noise)
    assert np.array_equal(got, ref_gpu), float(np.max(np.abs(got - ref_gpu)))
    ref = O.denoise_chunk(cfg, w, sk, sv, frames, ticks, state, noise, cfg.taus())
    _check_oracle(cfg, got, ref)
    # the ordinary entry point still works after the static one on this context
    again = eng.denoise(state, noise).cpu().numpy()
    eng.synchronize()
    assert np.array_equal(again, ref_gpu)
    eng.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_static_entry_equals_graph_entry_two_calls(dtype):
    # first call: three envs and 21 dynamic tokens; second: one env and 6
    # dynamic tokens (both pad the dynamic values to 64 columns, so columns
    # 6..20 hold the first call's values unless the call clears them)
    big = BASE.replace(name=f"noalloc_big_{dtype}", dtype=dtype, batch=3, action_horizon=20)
    small = BASE.replace(name=f"noalloc_small_{dtype}", dtype=dtype, batch=1, action_horizon=5)
    _run(big, 5)
    _run(small, 2)


def test_static_entry_with_plain_split_counts():
    """A chunk that fits the static array only with the plain split counts (4 key splits instead of 10 for the team
    kernel, 66.5 of 67.1 MB): accepted, equal to the graph entry, both against the oracle."""
    cfg = BASE.replace(name="noalloc_plain_splits", dtype="bf16", batch=14, width=3328, mlp_dim=128, n_q_heads=1,
                       head_dim=128, action_horizon=121, static_len=32, frame_tokens=112, window_frames=4, frame_dim=0,
                       n_layers=1, num_steps=2, mod_mode="scale_only")
    ap = P.attention_plan(cfg)
    assert P.plans(cfg)[3] and ap.kernel == 4 and ap.splits > ap.few_splits > 1
    _run(cfg, 5)


def test_static_entry_rejects_oversized_chunks():
    # 32 envs at the pi0 widths need more transient memory than the array holds
    cfg = WL.CONFIGS["pi0_chunk_bf16"].replace(name="noalloc_oversized", batch=32, n_layers=1)
    w = WL.make_weights(cfg)
    sk, sv = WL.make_static_kv(cfg)
    eng = R.ReflexEngine(cfg, w, sk, sv)
    eng.write_frame(WL.make_frame(cfg, 0))
    state, noise = WL.make_state(cfg, 0), WL.make_noise(cfg, 0)
    s = torch.from_numpy(state).cuda()
    n = torch.from_numpy(noise).cuda()
    out = torch.empty_like(n)
    st = eng.lib.reflex_denoise_chunk_static(eng.ctx, s.data_ptr(), n.data_ptr(), cfg.num_steps, None,
                                             out.data_ptr())
    assert st == R.REFLEX_ESCRATCH, st
    assert "static device array" in R.strerror(st)
    eng.close()
