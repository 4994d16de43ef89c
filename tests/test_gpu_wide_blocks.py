"""Launches that take one workgroup per CU of 17 to 32 units of a request: the smallest and the largest of them, last
waves and units that are not full, against the fp64 oracle; the fused call gives the bits of the separate ones."""
import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
import workloads as W
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


# units of 16 rows per workgroup that the library cuts the launch into, with room for so many workgroups per kv head
@pytest.mark.parametrize("n_q,n_kv,dim,tokens,lens,room,units", [
    (4, 1, 128, 512, [16 * 17 * 3 - 1], 3, 17), (8, 2, 128, 512, [400, 17, 900, 630], 9, 19),
    (4, 1, 128, 512, [16 * 17 * 2 - 15], 2, 17), (6, 1, 128, 512, [1000, 337, 300], 5, 22), (1, 1, 128, 40, [1500, 1, 700], 7, 29),
    (16, 1, 128, 64, [512 * 3 - 1, 510], 4, 32), (8, 1, 128, 24, [700, 800, 12], 6, 30), (3, 3, 64, 16, [500, 500, 1], 4, 32),
    (4, 1, 64, 512, [512 * 4 - 1, 496], 5, 32), (16, 1, 64, 64, [900, 2000, 100], 8, 29), (32, 8, 128, 512, [3000, 900], 9, 29),
    # as many requests, and blocks per kv head, as the small argument table takes, and one more of either
    (4, 1, 128, 512, [272] * 16, 20, 17), (4, 1, 128, 512, [272] * 17, 21, 17), (12, 2, 64, 64, [270] * 16, 18, 17), (12, 2, 64, 64, [270] * 17, 19, 17),
    (4, 1, 128, 512, [5120, 5119, 5111, 5105], 64, 20), (4, 1, 128, 512, [4160, 4159, 4151, 4145, 4160], 65, 20),
    (16, 1, 64, 64, [5120, 5119, 5111, 5105], 64, 20), (16, 1, 64, 64, [4160, 4159, 4151, 4145, 4160], 65, 20),
    (6, 3, 128, 128, [400, 420, 350, 117] * 10, 64, 22), (32, 8, 64, 512, [350] * 30, 32, 22)])
def test_wide_blocks(pool_mode, n_q, n_kv, dim, tokens, lens, room, units):
    n = len(lens)
    need = [-(-(x + 1) // tokens) for x in lens]
    cfg = W.Config("w", 9, n, n_q, n_kv, dim, tokens * 4 * n_kv * dim, sum(need) + 2, max(need) * tokens, "uniform", 1, max(lens))
    rng = np.random.default_rng(5)
    B = H.Both(cfg)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    ids = []
    for s in need:
        ids.append(B.create(cfg.max_tokens))
        assert B.map(ids[-1], 0, s) == 0
    assert B.append(ids, bits(sum(lens), n_kv, dim), bits(sum(lens), n_kv, dim), lens) == 0
    E.ellm_debug_set_compute_units(B.pool, room * n_kv)
    assert E.ellm_debug_decode_kernel(B.pool, ids) == "decode_block_kernel"
    n_split, most = E.ellm_decode_plan(B.pool, ids)
    per = [x // tokens * -(-tokens // 16) + -(-(x % tokens) // 16) for x in lens]
    assert list(n_split) == [-(-u // units) for u in per] and sum(n_split) <= room and most == -(-units // 4) * 64
    q = bits(n, n_q, dim)
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, "decode")
    rc, fused, ref = B.append_decode(ids, bits(n, n_kv, dim), bits(n, n_kv, dim), q)
    assert rc == 0
    H.check_close(fused, ref, "append + decode")
    rc, again = B.decode(ids, q)
    assert rc == 0 and torch.equal(fused, again)
    B.close()


@pytest.mark.parametrize("n_q,n_kv,dim,tokens,lens,kernel", [
    (32, 8, 128, 512, [3500, 3400, 3300, 3600], "decode_block_kernel"), (12, 1, 128, 64, [6000, 900], "decode_block_kernel"),
    (8, 2, 64, 64, [3000, 40], "decode_block_kernel"), (32, 8, 128, 512, [1500, 2500, 800] * 16, "decode_tile_kernel"),
    (12, 2, 64, 64, [9000, 900] * 30, "decode_unit_kernel")])
def test_infinite_v_beside_scores_of_minus_infinity(n_q, n_kv, dim, tokens, lens, kernel):
    """The first tokens of a request have scores of -inf only, whole waves of them, and one an infinite V: 0 * inf, as the
    softmax has it, in the column it stands in and nowhere else."""
    n, need = len(lens), [-(-x // tokens) for x in lens]
    cb = tokens * 4 * n_kv * dim
    dev = torch.zeros((sum(need) + 1) * cb, dtype=torch.uint8, device="cuda")
    P = E.ellm_pool_create(dev, None, cb, n_q, n_kv, dim, n, max(need))
    ids = []
    for s in need:
        ids.append(E.ellm_tensor_create(P, s * tokens))
        E.ellm_tensor_map_chunks(P, ids[-1], 0, s)
    g = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn(n, n_q, dim, device="cuda", generator=g).to(torch.bfloat16)
    k, v = (torch.randn(sum(lens), n_kv, dim, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    q[0] = q[0].abs() + 0.1
    k[:700] = -float("inf")
    v[300, 0, 1] = float("inf")
    E.ellm_kv_append(P, ids, k, v, np.asarray(lens, np.int32))
    assert E.ellm_debug_decode_kernel(P, ids) == kernel
    out = torch.empty_like(q)
    E.ellm_decode_attention(P, ids, q, out)
    want = torch.zeros(n_q, dim, dtype=torch.bool, device="cuda")
    want[:n_q // n_kv, 1] = True
    assert torch.equal(out[0].isnan(), want) and out[1:].isfinite().all()
    kk, vv = k[700:lens[0]].double(), v[700:lens[0]].double()
    for h in range(n_q):
        w = torch.softmax((kk[:, h // (n_q // n_kv)] * q[0, h].double()).sum(-1) / dim ** 0.5, 0)
        ref = (w[:, None] * vv[:, h // (n_q // n_kv)]).sum(0)
        assert (out[0, h].double() - ref)[~want[h]].abs().max() <= H.MAX_ABS
    E.ellm_pool_destroy(P)
