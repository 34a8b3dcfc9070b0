"""GPU parity of the projections at the row counts, K ranges and widths where the weight-streaming and the
tiled GEMMs change form (bf16), the whole chunk against the float64 oracle."""
import numpy as np
import pytest

from oracle import reflex_oracle as O
from paper_2607_14695_amd import reflex as R
from paper_2607_14695_amd import workloads as WL
from tests import plan_model as P

pytestmark = pytest.mark.gpu

BF16_REL, BF16_ABS = 1e-2, 5e-2  # the bar of the other bf16 parity tests

# ungated branches (scale-only): every projection enters the residual stream in full
BASE = WL.CONFIGS["tiny_fp32"].replace(
    name="rows", dtype="bf16", n_layers=2, cond_hidden=64, state_dim=8, action_dim=5, num_steps=2, static_len=16,
    frame_tokens=24, window_frames=2, frame_dim=0, mod_mode="scale_only", batch=1)


def _check(cfg, head=4, branch=4, mod=1):
    w = WL.make_weights(cfg)
    for name, scale in (("w_o", branch), ("w_down", branch), ("w_aout", head), ("w_mod2", mod)):
        w[name] *= np.float32(scale)  # exact in bf16; the actions depend on every projection
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
    # 2,100 rows: 15 stages, 128-row tiles for gate|up (17 x 14), output and down (17 x 8) projections; QKV
    # (4 x 33) on 64-row ones
    dict(batch=25, action_horizon=83, width=960, mlp_dim=896, n_q_heads=2, head_dim=128, n_layers=1, num_steps=1),
])
def test_odd_stage_counts(changes):
    """More than 256 rows with K ranges of no power-of-two stage count, on the two-group tiles: the fp32, RoPE and
    gated-GELU epilogues, and the frame K/V projection of 320 rows with 5 stages."""
    _check(BASE.replace(frame_tokens=64, **changes))


def test_two_group_tiles_split_k():
    """300 rows on the two-group tiles with two K splits of 9 stages (down projection of 1,152 columns)."""
    cfg = BASE.replace(batch=5, action_horizon=59, width=320, mlp_dim=1152, n_q_heads=3, head_dim=128)
    assert P.pick_splits(cfg, cfg.width, cfg.mlp_dim) == 2
    _check(cfg)


@pytest.mark.parametrize("mod_mode", ["scale_only", "full"])
@pytest.mark.parametrize("n_layers", [1, 3, 10])
def test_two_group_tiles_conditioning(n_layers, mod_mode):
    """288 conditioning rows (nine steps of 32 envs): the first MLP has 6 stages of K, the second 5 and one slice
    per site (3, 7 and 21 of them).  Modulations on 64-row tiles with 3 sites (120 tiles), on 128-row ones with 7
    (168), on the two-stage kernel with 21; the first MLP on 64-row tiles up to 7 sites, on 128-row ones with 21
    (53 x 5 64-row tiles)."""
    _check(BASE.replace(batch=32, num_steps=9, n_layers=n_layers, width=320, state_dim=64, cond_hidden=320,
                        mlp_dim=64, n_q_heads=1, head_dim=64, action_horizon=3, static_len=0, frame_tokens=16,
                        mod_mode=mod_mode), branch=4 if n_layers < 10 else 1, mod=4)


@pytest.mark.parametrize("changes", [
    dict(batch=6, action_horizon=49, width=320, n_q_heads=3, frame_tokens=104, frame_dim=96),   # 300 and 624 rows
    dict(batch=2, action_horizon=127, width=192, n_q_heads=5, frame_tokens=136, frame_dim=160),  # 256 and 272
    dict(batch=13, action_horizon=100, width=576, n_q_heads=2, frame_tokens=24, frame_dim=320),  # 1,313 and 312
])
def test_streamed_64_wide_heads(changes):
    """64-wide heads: QKV and the frame K/V projection are streamed at every row count, in row ranges of 128."""
    _check(BASE.replace(mlp_dim=320, head_dim=64, **changes))


@pytest.mark.parametrize("rows", [17, 32, 33, 64])
def test_streamed_strips_beyond_one_wave(rows):
    """More streaming workgroups than CUs (small rings, two workgroups per CU): gate|up of 4,160 columns (260
    strips), the output and down projections as 40 strips by seven K ranges of 448 and 608 (3.5 and 4.75
    stages, more than the ring's), and QKV with 64 heads of 128 (264 strips).  The action head is scaled by 2 at 1,280
    columns: a velocity is about scale * 0.02 * sqrt(width), 1.4 here as in the cases of 320, and the absolute
    bar is meant for actions of order one (with 4, actions of 5.6 differed by 5.6e-2 at rel-L2 5.8e-3)."""
    _check(BASE.replace(action_horizon=rows - 1, width=1280, mlp_dim=4160, n_q_heads=12, head_dim=256, n_layers=1),
           head=2)
    _check(BASE.replace(action_horizon=rows - 1, width=704, mlp_dim=128, n_q_heads=64, head_dim=128, n_layers=1))


@pytest.mark.parametrize("batch,tokens", [(1, 24), (1, 40), (2, 32)])
def test_streamed_frame_projection_beyond_one_wave(batch, tokens):
    """The K/V projection of 17 layers of 256-wide heads as 272 strips over 24, 40 and 64 frame rows: the cache
    rows against the oracle's (results rounded to bf16, 2^-9 each; sums in fp32)."""
    cfg = BASE.replace(batch=batch, n_layers=17, width=64, mlp_dim=64, n_q_heads=1, head_dim=256, frame_tokens=tokens,
                       frame_dim=736)
    w = WL.make_weights(cfg)
    frame = WL.make_frame(cfg, 0)
    eng = R.ReflexEngine(cfg, w, *WL.make_static_kv(cfg))
    eng.write_frame(frame)
    K, Vt = [x.float().cpu().numpy() for x in eng.cache_views()]
    rows = slice(cfg.static_len, cfg.static_len + tokens)
    for env in range(batch):
        for l in range(cfg.n_layers):
            kf, vf = O.frame_kv(cfg, w, frame[env], 0, l)
            for got, ref in ((K[env, l, rows], kf[:, 0]), (Vt[env, l, :, rows], vf[:, 0].T)):
                assert np.linalg.norm(got - ref) <= 4e-3 * np.linalg.norm(ref), (env, l)
    eng.close()


@pytest.mark.parametrize("rows", [17, 33, 64])
@pytest.mark.parametrize("offset", [1, 2, 4])
def test_operands_at_any_address(rows, offset):
    """Weights and frames that start 2, 4 and 8 bytes past a 16-byte boundary (views into a larger buffer): the
    copies into LDS do not take them, the fragment loads do.  Equal to the oracle as aligned ones are."""
    import torch

    cfg = BASE.replace(action_horizon=rows - 1, width=192, mlp_dim=320, n_q_heads=3, head_dim=64, frame_dim=96)

    def shifted(a):
        flat = torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16).cuda().flatten()
        buf = torch.empty(flat.numel() + 16, dtype=torch.bfloat16, device="cuda")
        view = buf[offset:offset + flat.numel()].view(a.shape)
        view.copy_(flat.view(a.shape))
        assert view.data_ptr() % 16 == 2 * offset and view.is_contiguous()
        return view

    w = WL.make_weights(cfg)
    for name in ("w_o", "w_down", "w_aout"):
        w[name] *= np.float32(4)
    sk, sv = WL.make_static_kv(cfg)
    frames = {t: WL.make_frame(cfg, t) for t in range(2)}
    eng = R.ReflexEngine(cfg, {n: shifted(a) for n, a in w.items()}, sk, sv)
    for n, a in eng.w.items():
        assert a.data_ptr() % 16 == 2 * offset, n  # the engine takes them as they are
    for t in range(2):
        eng.write_frame(shifted(frames[t]))
    state, noise = WL.make_state(cfg, 1), WL.make_noise(cfg, 1)
    got = eng.denoise(state, noise).cpu().numpy()
    ref = O.denoise_chunk(cfg, w, sk, sv, frames, 2, state, noise, cfg.taus())
    rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    mx = float(np.max(np.abs(got - ref)))
    print(f"{rows} rows, operands {2 * offset} bytes off: rel-L2 {rel:.2e} max-abs {mx:.2e}", flush=True)
    assert np.isfinite(got).all() and rel <= BF16_REL and mx <= BF16_ABS, (rel, mx)
    eng.close()
