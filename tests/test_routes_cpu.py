"""The rules that choose a call's kernel, and a decode's split plan, on the host."""
import math
import random

import pytest

import paper_2608_02947_amd as atf
import routes


@pytest.mark.parametrize("batch,group,h_kv,n_k,d,rotate,splits", [
    # (row, KV head) pairs: exactly a round of 256 CUs, just past it, nearly two
    (32, 3, 8, 16000, 128, False, 0), (33, 3, 8, 16000, 128, False, 4), (40, 3, 8, 16000, 128, False, 4),
    (42, 3, 8, 16000, 128, False, 3), (52, 3, 8, 16000, 128, False, 0), (64, 3, 8, 16000, 128, False, 0),
    (33, 3, 8, 16000, 128, True, 4), (42, 3, 8, 4000, 128, True, 3), (56, 3, 8, 4000, 128, True, 0),
    (66, 3, 8, 16000, 128, False, 2), (88, 3, 8, 16000, 128, False, 0), (100, 3, 8, 60000, 128, False, 2),
    # rows too short to pay for the merge, the more so with many heads
    (33, 3, 8, 1000, 128, False, 0), (66, 16, 4, 4000, 128, False, 0), (66, 16, 4, 8000, 128, False, 4),
    (66, 3, 8, 2000, 128, False, 0),
    (17, 1, 16, 16000, 64, False, 4), (24, 1, 16, 4000, 64, True, 2), (40, 1, 16, 4000, 64, True, 2),
    # no room for splits; rotating one or two heads of d = 64 takes the 4-wave kernel
    (132, 3, 8, 16000, 128, False, 0), (132, 1, 16, 4000, 64, True, 1), (264, 2, 8, 1000, 64, True, 1),
    (264, 7, 8, 1000, 64, True, 0), (64, 1, 16, 4000, 64, True, 0), (132, 1, 16, 4000, 64, False, 0),
    # heads of several workgroups: unsplit in small caches only, and splits by eights
    (270, 39, 1, 40029, 128, False, 4), (160, 35, 2, 20121, 128, True, 4), (136, 33, 3, 2783, 64, False, 0),
    (295, 39, 1, 893, 128, True, 0), (16, 64, 1, 123544, 128, False, 64), (10, 64, 1, 14730, 128, True, 58),
])
def test_decode_between_whole_rounds(batch, group, h_kv, n_k, d, rotate, splits):
    direct = routes.decode_direct(batch, group, h_kv, n_k, n_k - 1, d, rotate)
    assert direct == (splits == 0)
    if not direct:
        assert routes.decode_splits(batch, group, h_kv, n_k, n_k - 1, d, rotate)[0] == splits


def test_decode_heads_of_one_kv_head_in_several_workgroups():
    """16x16 tiles up to 16 heads; several workgroups of them only within the last-level cache."""
    tiles = lambda batch, group, h_kv, n_k, **kw: routes.decode_cols16(batch, group, h_kv, n_k, n_k - 1, 128, **kw)
    assert tiles(1, 16, 1, 2 ** 20) and not tiles(1, 17, 1, 1) and not tiles(1, 32, 1, 1)
    assert not tiles(1, 1, 1, 1, cap=2 ** 27 - 64) and tiles(1, 1, 1, 1, cap=2 ** 27 - 65)
    fits = 2 ** 30 // (4 * 128 * 3 * 192)  # 1 GB over three workgroups, 192 rows
    assert tiles(192, 39, 1, fits) and not tiles(192, 39, 1, fits + 1) and tiles(192, 39, 1, fits + 1, ragged=True)
    assert tiles(64, 35, 2, 3276) and not tiles(64, 35, 2, 3277)
    assert tiles(512, 13, 1, 2 ** 16) and tiles(64, 71, 1, 4096) and not tiles(64, 71, 1, 4097)


def test_decode_plans_fit_and_leave_no_split_empty():
    rng = random.Random(3)
    for _ in range(20000):
        batch, h_kv = int(2 ** rng.uniform(0, 10)), rng.choice([1, 2, 3, 4, 8, 16])
        group, rotate = rng.choice([1, 2, 3, 5, 7, 8, 11, 16, 17, 24, 32, 33, 64]), rng.random() < 0.5
        d = rng.choice([64, 128])
        n_k = int(2 ** rng.uniform(0, 19))
        q_pos = rng.choice([n_k - 1, rng.randrange(n_k), n_k + 5])
        splits, room = routes.decode_splits(batch, group, h_kv, n_k, q_pos, d, rotate)
        steps = -(-min(n_k, q_pos + 1) // 128)
        assert 1 <= splits <= room
        if routes.heads_per_block(group) < group and splits % 8 == 0:
            continue  # rounded up
        per = -(-steps // splits)  # steps of every split but the last, which has at least one
        assert (splits - 1) * per < steps, (batch, h_kv, group, n_k, q_pos)


@pytest.mark.parametrize("batch,n_q,n_k,group,h_kv,d,k,rotate,waves", [
    # a chunk against a long cache: few row blocks by 8 waves, more by 4, the chip full
    (1, 64, 65836, 7, 4, 128, 2.0, False, 8), (1, 300, 65836, 7, 4, 128, 2.0, False, 4),
    (1, 1188, 65836, 7, 4, 128, 2.0, False, 4), (1, 1189, 65836, 7, 4, 128, 2.0, False, 0),
    (1, 300, 65836, 7, 4, 128, 2.0, True, 4), (1, 800, 65836, 7, 4, 128, 2.0, True, 0),
    (1, 1024, 1024, 7, 2, 64, 2.0, False, 4), (1, 8191, 8191, 7, 2, 64, 2.0, False, 0),
    # short prompts
    (8, 290, 290, 3, 8, 128, 2.0, False, 0), (1, 290, 290, 3, 8, 128, 2.0, False, 4),
    (32, 48, 48, 7, 4, 128, 2.0, False, 0), (4, 468, 468, 8, 4, 128, math.inf, False, 0),
    (32, 160, 160, 16, 1, 64, 2.0, False, 0), (16, 58, 58, 8, 4, 128, 2.0, True, 0),
    # caches past the last-level cache
    (16, 117, 11166, 1, 16, 64, 2.0, False, 0), (6, 132, 26240, 3, 8, 128, 2.0, False, 4),
    (32, 9, 27936, 8, 4, 128, 2.0, False, 0), (16, 22, 38656, 8, 4, 128, 2.0, False, 4),
])
def test_prefill_kernel(batch, n_q, n_k, group, h_kv, d, k, rotate, waves):
    w = atf.Window(d, 1e6, k)
    assert routes.prefill_waves(w, batch, n_q, n_k, n_k - n_q, group, h_kv, rotate) == waves


def test_prefill_long_streams_take_the_kernel_with_64_bit_offsets():
    w = atf.Window(128, 1e6, 2.0)
    fits = (2 ** 32 - 1) // 256
    assert routes.prefill_waves(w, 1, 16, 1000, 984, 1, 1, cap=fits) == 4
    assert routes.prefill_waves(w, 1, 16, 1000, 984, 1, 1, cap=fits + 1) == 0
    assert routes.prefill_waves(w, 1, 16, 1000, 984, 257, 1) == -1
