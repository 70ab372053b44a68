"""The rules that choose a decode call's kernel and split plan, on the host."""
import random

import pytest

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
])
def test_decode_between_whole_rounds(batch, group, h_kv, n_k, d, rotate, splits):
    direct = routes.decode_direct(batch, group, h_kv, n_k, n_k - 1, d, rotate)
    assert direct == (splits == 0)
    if not direct:
        assert routes.decode_splits(batch, group, h_kv, n_k, n_k - 1, rotate)[0] == splits


def test_decode_plans_fit_and_leave_no_split_empty():
    rng = random.Random(3)
    for _ in range(20000):
        batch, h_kv = int(2 ** rng.uniform(0, 10)), rng.choice([1, 2, 3, 4, 8, 16])
        group, rotate = rng.choice([1, 2, 3, 5, 7, 8, 11, 16, 17, 24, 32, 33, 64]), rng.random() < 0.5
        n_k = int(2 ** rng.uniform(0, 19))
        q_pos = rng.choice([n_k - 1, rng.randrange(n_k), n_k + 5])
        splits, room = routes.decode_splits(batch, group, h_kv, n_k, q_pos, rotate)
        steps = -(-min(n_k, q_pos + 1) // 128)
        assert 1 <= splits <= room
        per = -(-steps // splits)  # steps of every split but the last, which has at least one
        assert (splits - 1) * per < steps, (batch, h_kv, group, n_k, q_pos)
