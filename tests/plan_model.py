"""The chunk planner's buffer sizes, written out a second time: split counts of the plain rules (up to 16 key
splits, K splits of the tiles), the workspace layout, and the library's own split counts.  Host arithmetic only."""
import ctypes

from paper_2607_14695_amd import reflex as R

SCRATCH = 64 << 20  # the static device array of the allocation-free entry point


class AttnPlan(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_int), ("splits", ctypes.c_int), ("few_splits", ctypes.c_int)]


def ceil(a, b):
    return -(-a // b)


def elem(cfg):
    return 2 if cfg.bf16 else 4


def slots_rows(cfg):
    return cfg.static_len + (cfg.window_frames + cfg.spare_slot) * cfg.frame_tokens


def attention_plan(cfg):
    """The library's kernel and key splits before any fallback."""
    fn = R.load_library()._ZN6reflex14attention_planEiiiiiii
    fn.restype, fn.argtypes = AttnPlan, [ctypes.c_int] * 7
    return fn(cfg.batch, cfg.dyn_tokens, cfg.n_q_heads, cfg.head_dim, slots_rows(cfg), elem(cfg),
              R.ATTN_KERNELS[cfg.attn_kernel])


def pick_splits(cfg, N, K):
    """The library's K splits of an fp32-output GEMM."""
    fn = R.load_library()._ZN6reflex16gemm_pick_splitsEiiiib
    fn.restype, fn.argtypes = ctypes.c_int, [ctypes.c_int] * 4 + [ctypes.c_bool]
    return fn(cfg.batch * cfg.dyn_tokens, N, K, elem(cfg), True)


def plain_key_splits(cfg):
    """Key splits that fill one wave of workgroups: wave pairs where 128-row workgroups would reach one tile per
    split, else 128-row (fp32: 64-row) workgroups; at most 16."""
    rows, eb = cfg.dyn_tokens * cfg.n_q_heads, elem(cfg)
    tiles = ceil(slots_rows(cfg), 64) + 1
    base = cfg.batch * ceil(rows, 128 if eb == 2 else 64)
    groups = base
    if eb == 2 and (cfg.attn_kernel == "pair" or (cfg.attn_kernel == "auto" and 256 // base >= tiles)):
        groups = cfg.batch * ceil(rows, 32)
    return max(1, min(256 // groups, tiles, 16))


def plain_k_splits(cfg, N, K):
    """K splits with streamed weights up to 64 rows and tiles above."""
    M, eb = cfg.batch * cfg.dyn_tokens, elem(cfg)
    if M <= 64:
        return min(max(1, min(ceil(256, ceil(N, 32)), 8)), max(1, K // (64 // eb * 8)))
    base = ceil(N, 128) * ceil(M, 128)
    if eb == 4:
        return 1 if base >= 256 or K < 1024 else min(ceil(256, base), K // 512)

    def power(base):
        s = 1
        while base * s * 2 <= 256 and K % (64 * s * 2) == 0 and K // (s * 2) >= 512:
            s *= 2
        return s

    s, s64 = power(base), power(ceil(N, 128) * ceil(M, 64))
    return s64 if s64 < s and K % (64 * s64) == 0 and K // (64 * s64) in (8, 16) else s


def effective(cfg, K, splits):
    """Splits left after a split's K range is rounded up to the kernels' step."""
    gran = (64 if cfg.batch * cfg.dyn_tokens <= 64 else 128) // elem(cfg)
    return ceil(K, ceil(ceil(K, max(splits, 1)), gran) * gran)


def k_parts(cfg, pick):
    Ko, F = cfg.n_q_heads * cfg.head_dim, cfg.mlp_dim
    return max(effective(cfg, Ko, pick(cfg, cfg.width, Ko)), effective(cfg, F, pick(cfg, cfg.width, F)))


def layout(cfg, part_o, ml_splits, parts):
    """(workspace bytes, bytes of parts 1 .. 16) for the given partial buffers."""
    eb, B, T, L, dh, D = elem(cfg), cfg.batch, cfg.dyn_tokens, cfg.n_layers, cfg.head_dim, cfg.width
    M, S, steps = B * T, 2 * L + 1, max(cfg.num_steps, 1)
    rows_pad, tpad = ceil(T * cfg.n_q_heads, 128) * 128, ceil(T, 64) * 64

    def a256(x):
        return ceil(x, 256) * 256

    sz = [64, T * (dh // 2) * 8, max(cfg.static_len, cfg.frame_tokens) * (dh // 2) * 8,
          steps * B * (D + cfg.state_dim) * eb, steps * B * S * cfg.cond_hidden * eb, S * steps * B * 3 * D * 4,
          M * D * 4, M * D * eb, B * rows_pad * dh * eb, B * T * dh * eb, B * dh * tpad * eb, 0,
          M * cfg.n_q_heads * dh * eb, part_o, B * ml_splits * rows_pad * 8, M * cfg.mlp_dim * eb, parts * M * D * 4, 0]
    tail = [L * a256(sz[9]), L * a256(sz[10]), M * max((cfg.n_q_heads + 2) * dh, 2 * cfg.mlp_dim) * 4,
            M * cfg.action_dim * 4]
    return sum(map(a256, sz + tail)), sum(map(a256, sz[1:17]))


def plans(cfg):
    """What the planner should do: (expected workspace bytes, expected static bytes, plain static bytes, whether
    the plain counts replace the plan's)."""
    eb = elem(cfg)
    part = cfg.batch * ceil(cfg.dyn_tokens * cfg.n_q_heads, 128) * 128 * cfg.head_dim
    few, few_parts = plain_key_splits(cfg), k_parts(cfg, plain_k_splits)
    ap = attention_plan(cfg)
    plain_ws, plain = layout(cfg, few * part * 4, few, few_parts)
    ws, static = layout(cfg, max(ap.splits * part * eb, few * part * 4), max(ap.splits, few),
                        max(few_parts, k_parts(cfg, pick_splits)))
    if static > SCRATCH >= plain:
        return plain_ws, plain, plain, True
    return ws, static, plain, False
