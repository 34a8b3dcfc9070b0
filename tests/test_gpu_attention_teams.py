"""GPU parity of the attention launches with wave teams and up to 64 key splits (a few envs, more keys than
one tile per workgroup) and of the split merge that follows them: against the float64 oracle, and against the
16-row kernel, which is held to the oracle by other tests."""
import numpy as np
import pytest

from oracle import reflex_oracle as O
from paper_2607_14695_amd import reflex as R
from paper_2607_14695_amd import workloads as WL

pytestmark = pytest.mark.gpu

# bf16 operands (2^-9 each), fp32 accumulation: the bar of the other bf16 parity tests.  The two kernels
# read the same bf16 q, K and V and round the probabilities and the split partials, 2^-9 each: the same bar.
BF16_REL, BF16_ABS = 1e-2, 5e-2

# ungated branches (scale-only), so that the attention enters the residual stream in full
BASE = WL.CONFIGS["tiny_fp32"].replace(
    name="teams", dtype="bf16", n_layers=2, width=128, mlp_dim=192, cond_hidden=64, state_dim=8, action_dim=5,
    num_steps=2, frame_dim=0, mod_mode="scale_only")

# name -> (changes, scale of the q projection, ticks at which the chunk is compared)
CASES = {
    # one workgroup per env (3 row blocks of 32: teams of 2 and 1), one tile per split, partial cached tile;
    # from an empty ring (every split but one or two without keys) over a partial one to a wrapped one
    "one_tile": (dict(batch=4, n_q_heads=4, head_dim=128, action_horizon=20, static_len=40, frame_tokens=152,
                      window_frames=9), 1, (0, 1, 4, 10)),
    # several tiles per split, uneven rows (13 blocks over 4 workgroups)
    "many_tiles": (dict(batch=3, n_q_heads=8, head_dim=256, action_horizon=50, static_len=0, frame_tokens=496,
                        window_frames=8), 1, (3, 9)),
    # two dynamic tiles (T = 101), a spare slot the tiles straddle
    "two_dynamic_tiles_hole": (dict(batch=5, n_q_heads=1, head_dim=256, action_horizon=100, static_len=24,
                                    frame_tokens=344, window_frames=10, spare_slot=1), 1, (0, 11, 15)),
    # one row block: the second team has no rows
    "one_block": (dict(batch=9, n_q_heads=1, head_dim=128, action_horizon=31, static_len=8, frame_tokens=1000,
                       window_frames=3), 1, (4,)),
    # scores of 11 nats rms: the running maxima move in most tiles.  q and K are rounded to 2^-9 of such
    # scores, which alone moves the probabilities by several percent: compared with the 16-row kernel only,
    # and over one layer and one step, since the next layer's scores would turn the two kernels' 2^-8
    # difference into 11 * 2^-8 of the probabilities (over two layers and two steps 1.4e-2 was seen)
    "rescale": (dict(n_layers=1, num_steps=1, batch=3, n_q_heads=8, head_dim=256, action_horizon=50, static_len=0, frame_tokens=496,
                     window_frames=8), 64, (3, 9)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_team_attention(case):
    changes, q_scale, checks = CASES[case]
    cfg = BASE.replace(**changes)
    rows = cfg.dyn_tokens * cfg.n_q_heads
    base = cfg.batch * -(-rows // 128)
    tiles = -(-cfg.cache_rows // 64) + 1
    assert base < 16 and cfg.batch * -(-rows // 32) * tiles > 256, "not a launch with teams"
    w = WL.make_weights(cfg)
    w["w_qkv"][:, :cfg.n_q_heads * cfg.head_dim] *= np.float32(q_scale)
    w["w_o"] *= np.float32(8)  # the actions move by their own norm without the attention
    w["w_aout"] *= np.float32(8)
    sk, sv = WL.make_static_kv(cfg)
    frames = {}
    engines = [R.ReflexEngine(cfg.replace(attn_kernel=k), w, sk, sv) for k in ("auto", "rows16")]
    envs = [0, cfg.batch - 1]
    for t in range(max(checks) + 1):
        if t in checks:
            state, noise = WL.make_state(cfg, t), WL.make_noise(cfg, t)
            got, rows16 = [e.denoise(state, noise).cpu().numpy() for e in engines]
            refs = [("rows16", got, rows16)]
            if q_scale == 1:
                ref = O.denoise_chunk(cfg, w, sk, sv, frames, t, state, noise, cfg.taus(), envs=envs)
                refs.append(("oracle", got[envs], ref))
            for name, a, b in refs:
                rel = float(np.linalg.norm(a - b) / np.linalg.norm(b))
                mx = float(np.max(np.abs(a - b)))
                print(f"{case} after {t} frames: rel-L2 to {name} {rel:.2e} max-abs {mx:.2e}", flush=True)
                assert np.isfinite(a).all() and rel <= BF16_REL and mx <= BF16_ABS, (t, name, rel, mx)
        frames[t] = WL.make_frame(cfg, t)
        for e in engines:
            e.write_frame(frames[t])
    for e in engines:
        e.close()


# name -> (changes, key splits)
MERGES = {
    # 64-wide heads, wide merge: wave pairs with 11 splits of one tile; 16-row waves with 10 splits
    "wide_64_pairs": (dict(batch=1, n_q_heads=3, head_dim=64, action_horizon=37, static_len=32, frame_tokens=200,
                           window_frames=3), 11),
    "wide_64_rows16": (dict(batch=25, n_q_heads=5, head_dim=64, action_horizon=24, static_len=0, frame_tokens=520,
                            window_frames=2), 10),
    # 256-wide heads, nine and ten splits in at least 256 16-byte blocks, and eleven (wide)
    "full_256_9": (dict(batch=28, n_q_heads=4, head_dim=256, action_horizon=31, static_len=0, frame_tokens=264,
                        window_frames=3), 9),
    "full_256_10": (dict(batch=25, n_q_heads=3, head_dim=256, action_horizon=27, static_len=0, frame_tokens=648,
                         window_frames=1), 10),
    "wide_256_11": (dict(batch=23, n_q_heads=4, head_dim=256, action_horizon=31, static_len=0, frame_tokens=328,
                         window_frames=2), 11),
}


@pytest.mark.parametrize("case", sorted(MERGES))
def test_merge_forms(case):
    """Split merges of nine and more splits on either side of the rule that picks their form, from a partly filled
    ring (splits without keys) and from a full one, against the oracle."""
    changes, splits = MERGES[case]
    cfg = BASE.replace(**changes)
    rows = cfg.dyn_tokens * cfg.n_q_heads
    tiles = -(-cfg.cache_rows // 64) + 1
    base = cfg.batch * -(-rows // 128)
    groups = cfg.batch * -(-rows // 32) if 256 // base >= tiles else base
    assert min(256 // groups, tiles, 16) == splits, "not a launch of that many splits"
    w = WL.make_weights(cfg)
    for name in ("w_o", "w_aout"):
        w[name] *= np.float32(8)
    sk, sv = WL.make_static_kv(cfg)
    frames = {}
    eng = R.ReflexEngine(cfg, w, sk, sv)
    envs = sorted({0, cfg.batch // 2, cfg.batch - 1})
    for t in range(cfg.window_frames):
        frames[t] = WL.make_frame(cfg, t)
        eng.write_frame(frames[t])
        if t not in (0, cfg.window_frames - 1):
            continue
        state, noise = WL.make_state(cfg, t), WL.make_noise(cfg, t)
        got = eng.denoise(state, noise).cpu().numpy()
        ref = O.denoise_chunk(cfg, w, sk, sv, frames, t + 1, state, noise, cfg.taus(), envs=envs)
        rel = float(np.linalg.norm(got[envs] - ref) / np.linalg.norm(ref))
        mx = float(np.max(np.abs(got[envs] - ref)))
        print(f"{case} after {t + 1} frames: rel-L2 {rel:.2e} max-abs {mx:.2e}", flush=True)
        assert np.isfinite(got).all() and rel <= BF16_REL and mx <= BF16_ABS, (t, rel, mx)
    eng.close()
