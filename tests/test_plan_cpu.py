"""The planner's split counts and buffer sizes over random configurations, on the host: the workspace is exactly
what the written-out layout gives, and the allocation-free entry point accepts every chunk that it accepts with the
plain split counts (at most 16 key splits, K splits of the tiles)."""
import random

import pytest

from paper_2607_14695_amd import reflex as R
from paper_2607_14695_amd import workloads as WL
from tests import plan_model as P


def draw(rng):
    bf16 = rng.random() < 0.8
    return WL.CONFIGS["tiny_fp32"].replace(
        name="plan", dtype="bf16" if bf16 else "f32", n_layers=rng.choice([1, 2, 3, 6, 18]), width=64 * rng.randint(1, 64),
        mlp_dim=64 * rng.choice([1, 3, 8, 16, 27, 64, 96, 128, 200]), n_q_heads=rng.randint(1, 16),
        head_dim=rng.choice([64, 128, 256] if bf16 else [64, 128]), state_dim=8 * rng.randint(1, 8),
        action_dim=rng.randint(1, 64), action_horizon=rng.randint(1, 127), cond_hidden=64 * rng.randint(1, 16),
        static_len=8 * rng.randint(0, 64), frame_tokens=8 * rng.randint(1, 128), window_frames=rng.randint(1, 50),
        frame_dim=0, batch=rng.choice([1, 1, 1, 2, 3, 4, 5, 8, 12, 15, 16, 32]), num_steps=rng.randint(1, 12),
        spare_slot=rng.randint(0, 1), attn_kernel=rng.choice(["auto"] * 6 + ["rows16", "pair", "rows16p"]))


def test_layout_and_accepted_calls():
    rng = random.Random(4)
    seen = {"fits": 0, "too_large": 0, "fallback": 0, "team_fallback": 0, "more": 0}
    for _ in range(30000):
        cfg = draw(rng)
        ws, static, plain, fallback = P.plans(cfg)
        assert R.query_sizes(cfg)[1] == ws, cfg
        # accepted exactly when the plain counts are
        assert (static <= P.SCRATCH) == (plain <= P.SCRATCH), cfg
        seen["fits" if plain <= P.SCRATCH else "too_large"] += 1
        seen["more"] += static > plain
        seen["fallback"] += fallback
        seen["team_fallback"] += fallback and P.attention_plan(cfg).kernel == 4
    print(seen)
    assert min(seen.values()) >= 5, seen


@pytest.mark.parametrize("heads,tokens", [(2, 126), (8, 101), (4, 65), (8, 51)])
def test_one_split_per_tile_counts_every_dynamic_tile(heads, tokens):
    """Where the chip has room for one key tile per split, no split of the team kernel takes two: 64 and more
    dynamic tokens are two tiles."""
    teams = 0
    for batch in range(1, 16):
        for keys in range(64, 4096, 200):
            cfg = WL.CONFIGS["tiny_fp32"].replace(name="tiles", dtype="bf16", batch=batch, head_dim=256, n_q_heads=heads,
                                                  action_horizon=tokens - 1, static_len=0, frame_tokens=keys,
                                                  window_frames=1)
            ap = P.attention_plan(cfg)
            if ap.kernel != 4:
                continue
            teams += 1
            tiles = P.ceil(keys, 64) + P.ceil(tokens, 64)
            room = min(256 // (batch * P.ceil(tokens * heads, 128)), 64)
            assert P.ceil(tiles, ap.splits) == P.ceil(tiles, min(room, tiles)), (batch, keys, ap.splits)
    assert teams >= 20


@pytest.mark.parametrize("batch,tokens,heads,head_dim,keys,kernel,splits", [
    (11, 15, 8, 128, 432, 2, 5),   # two tiles per split in five splits: wave pairs
    (5, 36, 7, 128, 696, 2, 6),
    (2, 87, 9, 128, 296, 2, 5),
    (11, 15, 8, 128, 960, 4, 16),  # more than two tiles per split: teams
    (1, 55, 10, 128, 928, 4, 16),  # nine and more splits as pairs
    (11, 15, 8, 256, 432, 4, 8),   # wider heads
    (1, 51, 8, 256, 816, 2, 14),   # one tile per pair
    (4, 51, 8, 256, 1584, 3, 16),  # 16 workgroups of 128 rows
])
def test_attention_kernel_of_a_few_envs(batch, tokens, heads, head_dim, keys, kernel, splits):
    cfg = WL.CONFIGS["tiny_fp32"].replace(name="few", dtype="bf16", batch=batch, head_dim=head_dim, n_q_heads=heads,
                                          action_horizon=tokens - 1, static_len=0, frame_tokens=keys, window_frames=1)
    ap = P.attention_plan(cfg)
    assert (ap.kernel, ap.splits) == (kernel, splits)
