"""GPU parity of the projections at the row counts, K ranges and widths where the weight-streaming and the
tiled GEMMs change form (bf16), the whole chunk against the float64 oracle."""
import numpy as np
import pytest

from oracle import reflex_oracle as O
from paper_2607_14695_amd import reflex as R
from paper_2607_14695_amd import workloads as WL

pytestmark = pytest.mark.gpu

BF16_REL, BF16_ABS = 1e-2, 5e-2  # the bar of the other bf16 parity tests

# ungated branches (scale-only): every projection enters the residual stream in full
BASE = WL.CONFIGS["tiny_fp32"].replace(
    name="rows", dtype="bf16", n_layers=2, cond_hidden=64, state_dim=8, action_dim=5, num_steps=2, static_len=16,
    frame_tokens=24, window_frames=2, frame_dim=0, mod_mode="scale_only", batch=1)


def _check(cfg):
    w = WL.make_weights(cfg)
    for name in ("w_o", "w_down", "w_aout"):
        w[name] *= np.float32(4)  # exact in bf16; the actions depend on every projection
    sk, sv = WL.make_static_kv(cfg)
    frames = {t: WL.make_frame(cfg, t) for t in range(2)}
    eng = R.ReflexEngine(cfg, w, sk, sv)
    for t in range(2):
        eng.write_frame(frames[t])
    state, noise = WL.make_state(cfg, 1), WL.make_noise(cfg, 1)
    envs = sorted({0, cfg.batch - 1})
    ref = O.denoise_chunk(cfg, w, sk, sv, frames, 2, state, noise, cfg.taus(), envs=envs)
    for mode in ("reflex", "unfused"):
        got = eng.denoise(state, noise, mode=mode).cpu().numpy()
        rel = float(np.linalg.norm(got[envs] - ref) / np.linalg.norm(ref))
        mx = float(np.max(np.abs(got[envs] - ref)))
        print(f"{cfg.batch * cfg.dyn_tokens} rows, width {cfg.width}, mlp {cfg.mlp_dim}, {mode}: rel-L2 {rel:.2e} "
              f"max-abs {mx:.2e}", flush=True)
        assert np.isfinite(got).all() and rel <= BF16_REL and mx <= BF16_ABS, (mode, rel, mx)
    eng.close()


@pytest.mark.parametrize("rows", [16, 17, 32, 33, 64, 65, 96, 97, 128])
def test_streamed_rows(rows):
    """Row counts around the workgroups' 32, 64, 96 and 128 rows; K ranges of 192 and 320 (one and a half and
    two and a half stages of 128), split unevenly over the workgroups; 64- and 128-wide heads."""
    _check(BASE.replace(action_horizon=rows - 1, width=192, mlp_dim=320, n_q_heads=3, head_dim=64))
    _check(BASE.replace(action_horizon=rows - 1, width=320, mlp_dim=1728, n_q_heads=5, head_dim=128))


@pytest.mark.parametrize("batch,tokens", [(2, 65), (3, 64), (2, 100), (2, 128), (3, 86)])
def test_streamed_row_chunks(batch, tokens):
    """130, 192, 200 and 256 rows as several row ranges per strip (258 rows: tiles), K ranges on either side
    of the longest one that is streamed; rows of several envs in one range."""
    _check(BASE.replace(batch=batch, action_horizon=tokens - 1, width=320, mlp_dim=640, n_q_heads=3, head_dim=128))
    _check(BASE.replace(batch=batch, action_horizon=tokens - 1, width=128, mlp_dim=4160, n_q_heads=2, head_dim=64))


@pytest.mark.parametrize("changes", [
    # 300 rows, 64-row tiles: 5, 6 and 27 stages of 64, a last row tile of 44 rows, 320 columns
    dict(batch=5, action_horizon=59, width=320, mlp_dim=1728, n_q_heads=3, head_dim=128, frame_dim=320),
    # 2,100 rows, 128-row tiles for the gate|up projection: 15 stages; 64-row ones for the others
    dict(batch=25, action_horizon=83, width=960, mlp_dim=896, n_q_heads=2, head_dim=128, n_layers=1, num_steps=1),
])
def test_odd_stage_counts(changes):
    """More than 256 rows with K ranges of no power-of-two stage count: every epilogue of the two-group tiles
    (fp32, RoPE, gated GELU, and the frame K/V projection of 320 rows with 5 stages)."""
    _check(BASE.replace(frame_tokens=64, **changes))
