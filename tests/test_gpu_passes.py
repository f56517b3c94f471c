"""The score path's launch shapes on MI355X: row counts on both sides of every
wave and row-block edge, and sequences on both sides of the tile, chunk and
launch-count edges of the two-launch form, against the CPU oracle."""
import numpy as np
import pytest

import cb_workloads as W
from test_gpu_message import check_position, run_position
from test_gpu_parity import cb, check_all_units, gen, orc, run_gpu, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu

# (L, Hq, Hkv, D, T, m, S, dtype)
SHAPES = [
    # rows 1, 16 | 17, 32 | 33, 48 | 49, 64 (one wave, one to four blocks)
    (1, 1, 1, 128, 33, 1, 1, "bf16"), (1, 4, 1, 64, 64, 4, 1, "bf16"),
    (1, 1, 1, 128, 65, 17, 1, "bf16"), (2, 4, 2, 64, 1000, 16, 1, "bf16"),
    (1, 3, 1, 128, 127, 11, 1, "bf16"), (1, 6, 2, 64, 129, 16, 2, "bf16"),
    (1, 7, 1, 128, 256, 7, 1, "bf16"), (1, 8, 2, 64, 257, 16, 1, "bf16"),
    # 65, 96 | 97, 128 (two waves), 129, 192 | 193, 256 | 257, 320 | 321 (four, eight)
    (1, 5, 1, 128, 300, 13, 1, "bf16"), (1, 6, 1, 64, 513, 16, 1, "bf16"),
    (1, 1, 1, 128, 128, 97, 1, "bf16"), (1, 3, 1, 128, 1025, 43, 1, "bf16"),
    (1, 6, 1, 64, 640, 32, 1, "bf16"), (1, 1, 1, 128, 130, 193, 1, "bf16"),
    (1, 1, 1, 64, 129, 257, 1, "bf16"), (1, 3, 1, 128, 200, 107, 1, "bf16"),
    # more than 16 items a unit (the statistics folded by a launch of their
    # own): 65, 313 and 24 of them, the last with two row groups
    (1, 2, 1, 128, 4097, 8, 1, "bf16"), (1, 4, 1, 64, 40000, 4, 1, "bf16"),
    (1, 8, 1, 128, 3000, 65, 1, "bf16"),
    # fp32 in one, two and four blocks a wave
    (1, 3, 1, 64, 97, 5, 1, "f32"), (1, 2, 1, 128, 33, 16, 2, "f32"),
    (1, 3, 1, 128, 1100, 16, 1, "f32"), (1, 5, 1, 64, 700, 13, 1, "f32"),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_launch_shapes(torch, cb, orc, shape):   # noqa: F811
    L, Hq, Hkv, D, T, m, S, dt = shape
    w = W.custom(layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=D, q_len=m, seq_len=T, senders=S,
                 dtype=dt, cfg_id=411)
    say(f"case {shape}")
    q, K, V = gen(w)
    out = run_gpu(torch, cb, w, q, K, V, 0.25)
    check_all_units(orc, w, q, K, V, out, what=str(shape))


@pytest.mark.parametrize("shape", [
    (1, 2, 1, 128, 40, 3, 1, "bf16"), (1, 4, 1, 64, 1100, 8, 1, "bf16"),
    (1, 3, 1, 128, 129, 12, 2, "bf16"), (2, 8, 1, 128, 300, 10, 1, "bf16"),
    (1, 4, 1, 128, 2500, 40, 1, "bf16"), (1, 8, 1, 64, 700, 24, 1, "bf16"),
    (1, 2, 1, 64, 257, 4, 1, "f32")])
@pytest.mark.parametrize("p,alpha", [(2.0, 2.0), (3.0, 1.0)])
def test_position_launch_shapes(torch, cb, orc, shape, p, alpha):   # noqa: F811
    L, Hq, Hkv, D, T, m, S, dt = shape
    w = W.custom(layers=L, q_heads=Hq, kv_heads=Hkv, head_dim=D, q_len=m, seq_len=T, senders=S,
                 dtype=dt, cfg_id=412)
    say(f"case {shape} p={p}")
    q = W.gen_q(w)
    K, _ = W.gen_kv(w, want_v=False)
    check_position(orc, w, q, K, run_position(torch, cb, w, q, K, p, alpha), p, alpha, str(shape))


@pytest.mark.parametrize("q_heads,m", [(3, 40), (7, 20), (8, 5)])   # 160, 160 and 40 rows
@pytest.mark.parametrize("T", [15, 16, 17, 128, 129, 257, 385, 513])
@pytest.mark.parametrize("p,alpha", [(2.0, 2.0), (3.0, 1.0), (float("inf"), 1.0)])
def test_position_pooling_modes(torch, cb, orc, q_heads, m, T, p, alpha):   # noqa: F811
    """Every power mode and head grouping, with one to five tiles in a chunk: a
    block's numerators are stored while the next block is computed, across
    tiles and chunk ends."""
    shape = (1, q_heads, 1, 128, T, m, 1, "bf16")
    w = W.custom(layers=1, q_heads=q_heads, kv_heads=1, head_dim=128, q_len=m, seq_len=T,
                 senders=1, dtype="bf16", cfg_id=413)
    say(f"case {shape} p={p}")
    q = W.gen_q(w)
    K, _ = W.gen_kv(w, want_v=False)
    check_position(orc, w, q, K, run_position(torch, cb, w, q, K, p, alpha), p, alpha, str(shape))


def test_long_rows_of_equal_keys(torch, cb, orc):   # noqa: F811
    """A strong first key and 131071 equal ones, with as many units as workgroups
    are resident: each row's sum adds equal values, whose rounding is the same
    every time, so its error grows with the length of the chain of additions.
    Row r's first logit is v_r, all others are 0: the normaliser is
    log(exp(v_r) + T - 1).  At most 256 additions of tile sums in an item (2^-24
    each, 1.5e-5), as items of 4096 positions in 16-position steps had; in items
    of the whole row the errors reach 2e-4."""
    L, Hkv, G, D, m, S, T = 32, 8, 4, 64, 64, 2, 131072
    lay = cb.layout(L, G * Hkv, Hkv, D, m, T, senders=S, dtype="bf16")
    say(f"case {S * L * Hkv} x {T}")
    v = 5.5 + np.arange(G * m) / 24.0   # 5.5 .. 16.1
    q = torch.zeros((L, Hkv, G * m, D), device="cuda")
    q[..., 0] = torch.from_numpy(v).to(q)
    q = q.to(torch.bfloat16).reshape(L, G * Hkv, m, D)
    v = q[0, :G, :, 0].reshape(-1).double()   # logit v * 8 / sqrt(64)
    k = torch.zeros((S, L, Hkv, T, D), dtype=torch.bfloat16, device="cuda")
    k[..., 0, 0] = 8.0
    imp = torch.empty((S, L, Hkv, T), device="cuda")
    lse = torch.empty((S, L, G * Hkv, m), device="cuda")
    ws = torch.empty(cb.cb_score_workspace_bytes(lay), dtype=torch.uint8, device="cuda")
    cb.cb_score(q, k, lay, imp, lse, ws)
    z = torch.exp(v) + (T - 1)
    err = (lse.reshape(-1, G * m).double() - torch.log(z)).abs().max().item()
    rest = (1.0 / z).sum()
    imp_err = (imp[..., 1:].double().sub_(rest).abs_().max() / rest).item()
    say(f"  lse error {err:.2e}, importance error {imp_err:.2e}")
    # fp32 lse of up to 24 in log2 units (2^-20), then exp2 of it
    assert err < 1.5e-5 + 2e-6 and imp_err < 1.5e-5 + 2e-6
