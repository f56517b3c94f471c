"""The score path's device queue on MI355X: calls that the launch rule sends to
the persistent kernel, in every wave and row-block shape it is built for, against
the definition in 64 bits on every unit; waits that give up; and logits far above
an item's reference maximum, in both forms.  Every test asserts the form that ran."""
import ctypes
import math

import pytest

from parity import FLT_MIN
from test_gpu_parity import cb, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu

DT = {"bf16": "bfloat16", "f32": "float32"}


def form_of(cb, lay, position=False):   # noqa: F811
    out = (ctypes.c_int64 * 6)()
    assert cb._lib.cb_internal_score_form(ctypes.byref(lay), int(position), None, out) == 0
    return dict(zip(("queue", "tokens", "waves", "blocks", "row_groups", "chunks"), out))


def inputs(torch, units, G, m, D, T, dtype, seed=1):   # noqa: F811
    """One sender, `units` layers of one KV head: q [units][G][m][D], K [1][units][1][T][D]."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = getattr(torch, DT[dtype])
    q = torch.randn((units, G, m, D), generator=gen, device="cuda").to(dt)
    k = torch.empty((1, units, 1, T, D), dtype=dt, device="cuda")
    for u in range(units):
        k[0, u, 0] = torch.randn((T, D), generator=gen, device="cuda") * 0.5
    return q, k


def weights64(torch, q, k, u):   # noqa: F811
    """Softmax weights [G*m][T] of one unit and its log normalisers, in 64 bits."""
    qu = q[u].reshape(-1, q.shape[-1]).double()
    x = (qu @ k[0, u, 0].double().t().contiguous()) / math.sqrt(q.shape[-1])
    lse = torch.logsumexp(x, dim=1, keepdim=True)
    return torch.exp(x - lse), lse[:, 0]


def close(torch, got, want, rtol, floor, what):   # noqa: F811
    err = (got.double() - want).abs() - rtol * want.abs() - floor
    assert bool((err <= 0).all()), f"{what}: {err.max().item():.3e} beyond {rtol:.1e}"


# Relative tolerance of importance and row_lse: fp32 logits of about |x| = 10 and
# sums; the test of full-size calls states 1e-5 for fp32 inputs.  bf16 inputs are
# exact in fp32, and so are their products: the same holds for them.
RTOL = 1e-5

# (units, G, m, D, T, dtype, waves, 16-row blocks a wave, items a unit at least)
SHAPES = [
    # one wave: 5 (one block), 12, 20 (two), 40 (three), 64 rows (four)
    (1600, 1, 5, 64, 4200, "bf16", 1, 1, 2), (3200, 4, 3, 128, 300, "bf16", 1, 1, 1),
    (1600, 4, 5, 64, 4097, "bf16", 1, 2, 2), (3200, 4, 8, 128, 257, "bf16", 1, 2, 1),
    (3200, 8, 5, 64, 300, "bf16", 1, 3, 1), (3200, 5, 8, 128, 129, "bf16", 1, 3, 1),
    (360, 4, 16, 64, 33000, "bf16", 1, 4, 9), (3200, 4, 16, 128, 300, "bf16", 1, 4, 1),
    # two waves: 90, 128
    (3200, 3, 30, 64, 300, "bf16", 2, 3, 1), (3200, 3, 30, 128, 200, "bf16", 2, 3, 1),
    (1600, 4, 32, 64, 4200, "bf16", 2, 4, 2), (3200, 4, 32, 128, 300, "bf16", 2, 4, 1),
    # four waves: 160, 256, 300, 384, 512
    (344, 4, 40, 64, 33000, "bf16", 4, 3, 9), (560, 4, 40, 128, 300, "bf16", 4, 3, 1),
    (560, 4, 64, 64, 300, "bf16", 4, 4, 1), (560, 4, 64, 128, 515, "bf16", 4, 4, 1),
    (560, 5, 60, 64, 300, "bf16", 4, 5, 1), (560, 8, 40, 128, 300, "bf16", 4, 5, 1),
    (560, 6, 64, 64, 300, "bf16", 4, 6, 1), (560, 6, 59, 128, 300, "bf16", 4, 6, 1),
    (344, 4, 125, 64, 33000, "bf16", 4, 8, 9), (600, 4, 128, 128, 300, "bf16", 4, 8, 1),
    # eight waves: 500 rows, and two row groups
    (280, 4, 125, 64, 300, "bf16", 8, 4, 1), (280, 4, 128, 128, 300, "bf16", 8, 4, 1),
    (140, 4, 150, 64, 4200, "bf16", 8, 4, 2), (28, 4, 150, 128, 33000, "bf16", 8, 4, 9),
    # fp32
    (2400, 1, 5, 64, 300, "f32", 1, 1, 1), (1080, 4, 3, 128, 300, "f32", 1, 1, 1),
    (2400, 4, 8, 64, 130, "f32", 1, 2, 1), (1080, 4, 8, 128, 300, "f32", 1, 2, 1),
    (2400, 4, 16, 64, 100, "f32", 1, 4, 1), (1080, 8, 5, 128, 300, "f32", 1, 4, 1),
    (1080, 3, 30, 64, 300, "f32", 2, 4, 1), (560, 4, 32, 128, 300, "f32", 2, 4, 1),
    (560, 4, 64, 64, 300, "f32", 4, 4, 1), (280, 4, 64, 128, 300, "f32", 4, 4, 1),
    (560, 5, 60, 64, 300, "f32", 4, 5, 1), (280, 8, 40, 128, 300, "f32", 4, 5, 1),
    (280, 4, 125, 64, 300, "f32", 8, 4, 1), (140, 4, 150, 128, 4200, "f32", 8, 4, 2),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_queue_shapes(torch, cb, shape):   # noqa: F811
    units, G, m, D, T, dtype, waves, blocks, items = shape
    lay = cb.layout(units, G, 1, D, m, T, dtype=dtype)
    f = form_of(cb, lay)
    say(f"case queue {shape} {f}")
    assert (f["queue"], f["waves"], f["blocks"]) == (1, waves, blocks)
    assert -(-T // f["tokens"]) >= items
    q, k = inputs(torch, units, G, m, D, T, dtype)
    imp = torch.full((1, units, 1, T), float("nan"), device="cuda")
    lse = torch.full((1, units, G, m), float("nan"), device="cuda")
    ws = torch.full((cb.cb_score_workspace_bytes(lay),), 0xFF, dtype=torch.uint8, device="cuda")
    for _ in range(2):   # again on a used workspace
        cb.cb_score(q, k, lay, imp, lse, ws)
    assert cb.cb_score_status(lay, ws) == 0
    for u in range(units):
        w, z = weights64(torch, q, k, u)
        close(torch, imp[0, u, 0], w.sum(0), RTOL, G * m * FLT_MIN, f"importance of unit {u}")
        close(torch, lse[0, u].reshape(-1), z, RTOL, RTOL, f"row_lse of unit {u}")


POSITION = [
    # bf16 in one wave (beyond three rounds of the queue's workgroups) and up
    (3200, 4, 3, 64, 200, "bf16", 1, 1), (3200, 3, 16, 128, 100, "bf16", 1, 4),
    (3200, 4, 32, 64, 100, "bf16", 2, 4), (3200, 8, 10, 128, 100, "bf16", 2, 3),
    (560, 4, 40, 64, 300, "bf16", 4, 3), (560, 8, 20, 128, 300, "bf16", 4, 3),
    (560, 3, 60, 64, 300, "bf16", 4, 4), (280, 8, 40, 128, 300, "bf16", 8, 4),
    (140, 4, 150, 64, 4200, "bf16", 8, 4), (28, 4, 150, 128, 9000, "bf16", 8, 4),
    (2400, 4, 3, 64, 100, "f32", 1, 1), (1080, 8, 5, 128, 100, "f32", 1, 4),
    (560, 4, 32, 128, 300, "f32", 2, 4), (280, 4, 64, 128, 300, "f32", 4, 4),
    (140, 4, 150, 64, 4200, "f32", 8, 4),
]


@pytest.mark.parametrize("p,alpha", [(2.0, 2.0), (3.0, 1.0), (float("inf"), 1.0)])
@pytest.mark.parametrize("shape", POSITION)
def test_queue_position_shapes(torch, cb, shape, p, alpha):   # noqa: F811
    units, G, m, D, T, dtype, waves, blocks = shape
    lay = cb.layout(units, G, 1, D, m, T, dtype=dtype)
    f = form_of(cb, lay, True)
    say(f"case queue position {shape} p={p} {f}")
    assert (f["queue"], f["waves"], f["blocks"]) == (1, waves, blocks)
    q, k = inputs(torch, units, G, m, D, T, dtype, seed=2)
    buf = cb.PositionBuffers(lay)
    buf.ws.fill_(0xFF)
    cb.cb_position_score(q, k, lay, buf.score, buf.ws, p=p, alpha=alpha, qscore=buf.qscore,
                         corr=buf.corr, importance=buf.importance)
    assert cb.cb_position_status(lay, buf.ws) == 0

    def pool(x):   # maximum over positions t-3 .. t+3
        return torch.nn.functional.max_pool1d(x.reshape(-1, 1, T), 7, 1, 3).reshape(x.shape)

    Q = torch.zeros(T, dtype=torch.float64, device="cuda")
    num, den = torch.zeros_like(Q), torch.zeros_like(Q)
    for u in range(units):
        w, _ = weights64(torch, q, k, u)
        close(torch, buf.importance.reshape(units, T)[u], w.sum(0), RTOL, G * m * FLT_MIN,
              f"importance of unit {u}")
        Q += w.sum(0) / (m * G)
        b = w.reshape(G, m, T).mean(0)
        if math.isinf(p):
            num = torch.maximum(num, pool(b).amax(0))
            den = torch.maximum(den, pool(b.mean(0)))
        else:
            num += (pool(b) ** p).mean(0)
            den += pool(b.mean(0)) ** p
    corr = num / den if math.isinf(p) else (num / den) ** (1.0 / (p - 1.0))
    Q = pool(Q)
    # a weight's relative error goes into Q once, into the correction p/(p-1) times
    # twice over, and into the score alpha times that
    grow = 2.0 if math.isinf(p) else 2.0 * p / (p - 1.0)
    close(torch, buf.corr.reshape(T), corr, grow * RTOL, 0.0, "correction")
    close(torch, buf.score.reshape(T), buf.qscore.reshape(T).double() * corr ** alpha,
          alpha * grow * RTOL + 1e-6, 0.0, "score")
    close(torch, buf.qscore.reshape(T), Q, RTOL, 0.0, "qscore")


def test_queue_wait_timeout_is_reported(torch, cb):   # noqa: F811
    """With the wait limit at 0 every wait of a second-pass item of the queue gives
    up at once: the kernel still exits, the status says so, and importance,
    row_lse, the selection and the compacted rows are NaN, -1 and zero.  The next
    call on the same workspace is whole again."""
    units, G, m, D, T = 560, 4, 64, 128, 300
    lay = cb.layout(units, G, 1, D, m, T)
    say("case queue wait timeout")
    assert form_of(cb, lay)["queue"] == 1
    q, k = inputs(torch, units, G, m, D, T, "bf16", seed=3)
    v = torch.randn_like(k)
    buf = cb.Buffers(lay, 0.25)
    prev = cb.cb_set_wait_limit(0)
    try:
        buf.k_out.fill_(1)
        cb.run_pipeline(q, k, v, buf)
        assert cb.cb_score_status(lay, buf.ws) == -8
        assert torch.isnan(buf.importance).all().item()
        assert (buf.idx == -1).all().item()
        assert (buf.k_out.view(torch.int16) == 0).all().item()
        cb.cb_score(q, k, lay, buf.importance, buf.row_lse, buf.ws)
        assert cb.cb_score_status(lay, buf.ws) == -8
        assert torch.isnan(buf.row_lse).all().item()
    finally:
        cb.cb_set_wait_limit(prev)
    cb.run_pipeline(q, k, v, buf)
    assert cb.cb_score_status(lay, buf.ws) == 0
    for u in range(0, units, 37):
        w, _ = weights64(torch, q, k, u)
        close(torch, buf.importance[0, u, 0], w.sum(0), RTOL, G * m * FLT_MIN, f"unit {u}")


def test_queue_position_wait_timeout_is_reported(torch, cb):   # noqa: F811
    units, G, m, D, T = 560, 4, 40, 64, 300
    lay = cb.layout(units, G, 1, D, m, T)
    say("case queue position wait timeout")
    assert form_of(cb, lay, True)["queue"] == 1
    q, k = inputs(torch, units, G, m, D, T, "bf16", seed=4)
    buf = cb.PositionBuffers(lay)
    prev = cb.cb_set_wait_limit(0)
    try:
        cb.cb_position_score(q, k, lay, buf.score, buf.ws, importance=buf.importance)
        assert cb.cb_position_status(lay, buf.ws) == -8
        assert torch.isnan(buf.importance).all().item()
        assert torch.isnan(buf.score).all().item()
    finally:
        cb.cb_set_wait_limit(prev)
    cb.cb_position_score(q, k, lay, buf.score, buf.ws, importance=buf.importance)
    assert cb.cb_position_status(lay, buf.ws) == 0
    assert torch.isfinite(buf.score).all().item()
    for u in range(0, units, 37):
        w, _ = weights64(torch, q, k, u)
        close(torch, buf.importance.reshape(units, T)[u], w.sum(0), RTOL, G * m * FLT_MIN,
              f"unit {u}")


# (units, G, m, D, T, dtype, queue): one, two and four waves; 16 x 16 blocks (odd
# block counts, fp32) and 32 x 32
@pytest.mark.parametrize("shape", [
    (8, 4, 4, 128, 131072, "bf16", 0), (8, 4, 8, 128, 131072, "bf16", 0),
    (8, 4, 32, 128, 65536, "bf16", 0), (8, 4, 40, 128, 65536, "bf16", 0),
    (8, 4, 64, 64, 65536, "bf16", 0), (8, 4, 128, 128, 131072, "bf16", 0),
    (8, 4, 16, 128, 65536, "f32", 0),
    # 36 items a unit, folded by every second-pass workgroup (no launch of their own)
    (64, 4, 4, 64, 70000, "bf16", 0),
    (1600, 4, 4, 64, 4200, "bf16", 1), (1600, 4, 8, 64, 4200, "bf16", 1),
    (560, 4, 40, 128, 700, "bf16", 1), (560, 4, 64, 128, 700, "bf16", 1),
    (600, 4, 128, 128, 700, "bf16", 1), (1080, 4, 8, 128, 700, "f32", 1)])
def test_late_large_logits_in_every_form(torch, cb, shape):   # noqa: F811
    """Two positions whose logits lie more than 100 (log2 units) above an item's
    reference maximum: one past the first tile of the first item, with full tiles
    of ordinary logits after it, so that the tile that is redone leaves lanes with
    different maxima to the fast path; and one in the last tile."""
    units, G, m, D, T, dtype, queue = shape
    lay = cb.layout(units, G, 1, D, m, T, dtype=dtype)
    f = form_of(cb, lay)
    say(f"case late logits {shape} {f}")
    assert f["queue"] == queue
    tile = 128   # the longest there is
    assert min(T, f["tokens"]) >= 4 * tile
    q, k = inputs(torch, units, G, m, D, T, dtype, seed=5)
    base = torch.randn(D, generator=torch.Generator().manual_seed(17)).cuda()
    base *= math.sqrt(D) / base.norm()
    q = (base + 0.1 * q.float()).to(q.dtype)
    k *= 0.2
    at = [tile + 5, T - 3]   # logits 100 and 102 in natural units: 144 and 147 in log2
    for i, t in enumerate(at):
        k[0, :, 0, t] = base * ((100 + 2 * i) / math.sqrt(D))
    imp = torch.empty((1, units, 1, T), device="cuda")
    lse = torch.empty((1, units, G, m), device="cuda")
    ws = torch.empty(cb.cb_score_workspace_bytes(lay), dtype=torch.uint8, device="cuda")
    cb.cb_score(q, k, lay, imp, lse, ws)
    assert cb.cb_score_status(lay, ws) == 0
    # an fp32 dot product of D terms whose magnitudes add up to about 105: one
    # rounding unit of that sum moves a weight by as much, relatively
    rtol = RTOL + 2.0 ** -24 * 105 * 2
    for u in range(0, units, max(1, units // 16)):
        w, z = weights64(torch, q, k, u)
        close(torch, imp[0, u, 0], w.sum(0), rtol, G * m * FLT_MIN, f"importance of unit {u}")
        close(torch, lse[0, u].reshape(-1), z, rtol, rtol, f"row_lse of unit {u}")
