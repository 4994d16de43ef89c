"""The cut of launches in wide blocks, without a device: how many units a block takes, that no launch has more blocks than
compute units, and that no plan needs more partial results than the workspace holds, over random batches and GPU sizes."""
import numpy as np

import paper_2506_15155_amd as E

DUMMY = 0x1000


def expected(units, n_kv, cus):
    """Units per block by the rule as stated: the fewest that leave no more blocks than CUs; None: no wide launch."""
    room = cus // n_kv
    total = sum(units)
    if len(units) > room or not 12 * room < total <= 32 * room:
        return None
    for b in range(-(-total // room), 33):
        if sum(-(-u // b) for u in units) <= room:
            return b if max(-(-u // b) for u in units) <= 16 else None
    return None


def test_wide_blocks_of_random_batches():
    rng = np.random.default_rng(4)
    wide = many = 0
    for _ in range(600):
        n_kv, group, dim = int(rng.choice([1, 2, 5, 8])), int(rng.choice([1, 3, 4, 8, 16])), int(rng.choice([64, 128]))
        tokens, cus, n = int(rng.choice([16, 24, 102, 512])), int(rng.choice([8, 17, 64, 256])), int(rng.integers(1, 12) if rng.random() < 0.6 else rng.integers(12, 60))
        room = cus // n_kv
        if room == 0:
            continue
        mean = max(1, int(room * rng.uniform(10, 36) * 16 / n))
        lens = [int(rng.integers(max(1, mean // 3), mean * 5 // 3 + 1)) for _ in range(n)]
        need = [-(-x // tokens) for x in lens]
        cb = tokens * 4 * n_kv * dim
        P = E.ellm_pool_create(None, None, cb, n_kv * group, n_kv, dim, n, max(need), flags=1, device_bytes=(sum(need) + 1) * cb)
        ids = []
        for x, s in zip(lens, need):
            ids.append(E.ellm_tensor_create(P, s * tokens))
            E.ellm_tensor_map_chunks(P, ids[-1], 0, s)
        E.ellm_kv_append(P, ids, DUMMY, DUMMY, np.asarray(lens, np.int32), stream=0)
        E.ellm_debug_set_compute_units(P, cus)
        n_split, most = E.ellm_decode_plan(P, ids)
        kernel = E.ellm_debug_decode_kernel(P, ids)
        E.ellm_pool_destroy(P)
        units = [x // tokens * -(-tokens // 16) + -(-(x % tokens) // 16) for x in lens]
        assert n_kv * int(n_split[n_split > 1].sum()) <= 4 * cus + n_kv * (n - 1), (lens, n_kv, cus)
        blocks16 = sum(-(-u // 16) for u in units)
        if blocks16 * n_kv <= cus * (1 if blocks16 > n else 2):
            continue                                     # a small launch: its own rule
        b = expected(units, n_kv, cus)
        if b is None:
            assert kernel != "decode_block_kernel", (lens, n_kv, cus)
            continue
        wide += 1
        many += len(lens) > 16 or int(n_split.sum()) > 64      # more than the small argument table takes
        assert 16 < b <= 32 and kernel == "decode_block_kernel"
        assert list(n_split) == [-(-u // b) for u in units] and most == -(-b // 4) * 64
        assert n_kv * int(n_split.sum()) <= cus
    assert wide > 60 and many > 10
