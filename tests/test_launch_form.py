"""How the score passes of a call are cut into items and launched (host rule, no
GPU): every form fits the workspace that the call's layout asks for and bounds
the positions of an item, and calls known to run as the device queue or as plain
launches do."""
import ctypes
import random

import pytest


@pytest.fixture(scope="module")
def form():
    import paper_2609_32046_amd as cb

    def ask(lay, position=False, queue_resident=512, resident=512):
        out = (ctypes.c_int64 * 6)()
        st = cb._lib.cb_internal_score_form(ctypes.byref(lay), int(position),
                                            (ctypes.c_int * 2)(queue_resident, resident), out)
        assert st == 0
        return dict(zip(("queue", "tokens", "waves", "blocks", "row_groups", "chunks"), out))

    ask.layout = cb.layout
    return ask


def test_every_form_fits_its_workspace(form):
    rng = random.Random(7)
    for _ in range(4000):
        position = rng.random() < 0.3
        G = rng.randint(1, 8)
        m = rng.randint(1, 1024 // (G if not position else 4 if G <= 4 else 8))
        Hkv, L, S = rng.choice([1, 2, 4, 8]), rng.randint(1, 64), rng.randint(1, 3)
        T = int(2 ** rng.uniform(0, 24))
        if rng.random() < 0.02:
            T = 2**31 - 2**16
        lay = form.layout(L, G * Hkv, Hkv, rng.choice([64, 128]), m, T, senders=S,
                          dtype=rng.choice(["bf16", "f32"]))
        cus = rng.choice([32, 256])
        f = form(lay, position, cus * rng.randint(1, 4), cus * rng.randint(1, 9))
        case = (L, Hkv, G, m, T, S, position, f)
        assert f["tokens"] % 32 == 0 and f["tokens"] <= (4096 if f["queue"] else 8192), case
        assert -(-T // f["tokens"]) <= f["chunks"], case
        rows = (4 if G <= 4 else 8) * m if position else G * m
        assert f["row_groups"] == -(-rows // 512), case
        held = 16 * f["waves"] * f["blocks"]
        assert held >= min(rows, 512), case
        if not f["queue"]:
            assert S * L * Hkv * f["row_groups"] * -(-T // f["tokens"]) <= 1 << 24, case


# units as (layers, kv heads), query heads per KV head, tokens, positions; the
# workgroups resident on 256 compute units
@pytest.mark.parametrize("L,Hkv,G,m,T,resident,queue", [
    (32, 8, 4, 64, 131072, (512, 512), False),    # 256 units: two whole rounds of 8192
    (1, 8, 4, 64, 8192, (512, 512), False),
    (36, 8, 4, 64, 8192, (512, 512), True),
    (40, 8, 4, 64, 4096, (512, 512), False),
    (36, 8, 4, 128, 16384, (512, 512), True),
    (11, 8, 4, 5, 26679, (1024, 2304), False),
    (32, 8, 4, 16, 65536, (1024, 2304), True),
    (8, 8, 1, 1, 131072, (1024, 2304), False),
    (32, 8, 4, 32, 65536, (1024, 1024), True),
    (7, 1, 4, 125, 33329, (256, 256), False),     # one round either way
    (48, 8, 4, 128, 1000, (256, 256), True),
])
def test_known_forms(form, L, Hkv, G, m, T, resident, queue):
    lay = form.layout(L, G * Hkv, Hkv, 128, m, T)
    assert bool(form(lay, False, *resident)["queue"]) == queue


# 512 rows in eight waves of 64 up to 512 items of 1024 positions, then in four of 128
@pytest.mark.parametrize("units,T,waves", [(512, 1000, 8), (513, 1000, 4), (256, 2048, 8),
                                           (256, 2049, 4), (1, 2**19, 8), (1, 2**19 + 1, 4)])
def test_waves_of_512_rows(form, units, T, waves):
    f = form(form.layout(units, 4, 1, 128, 128, T))
    assert (f["waves"], f["blocks"]) == (waves, 32 // waves)
