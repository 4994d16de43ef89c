"""Every instance of the attention kernels, by name: tiles, units and blocks; both head sizes; the group sizes that
have instances of their own; read through the table and directly; plain and with the fused append. Against the fp64
oracle with the harness's tolerance (weights and results rounded to bf16, relative 2^-9 each)."""
import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
import workloads as W
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

SHORT = [1, 15, 16, 17, 31, 47, 64, 65, 129, 300]      # around units, tiles, chunks


@pytest.mark.parametrize("kernel,n_q,n_kv,dim,tokens,lens,split", [
    ("decode_tile_kernel", 2, 2, 64, 48, SHORT, 64), ("decode_tile_kernel", 2, 2, 64, 64, SHORT, 192),
    ("decode_tile_kernel", 4, 2, 64, 64, SHORT, 64), ("decode_tile_kernel", 4, 2, 64, 128, SHORT, 192),
    ("decode_tile_kernel", 1, 1, 128, 40, SHORT, 64), ("decode_tile_kernel", 2, 1, 128, 64, SHORT, 192),
    ("decode_unit_kernel", 1, 1, 128, 32, SHORT, 192), ("decode_unit_kernel", 3, 3, 128, 72, SHORT, 64),
    ("decode_tile_kernel", 4, 1, 128, 80, SHORT, 64), ("decode_tile_kernel", 16, 2, 128, 40, SHORT, 192),
    ("decode_unit_kernel", 3, 1, 128, 24, SHORT, 64), ("decode_unit_kernel", 34, 2, 128, 16, SHORT, 192),
    ("decode_unit_kernel", 4, 1, 128, 8, SHORT, 64), ("decode_unit_kernel", 8, 1, 64, 64, SHORT, 192),
    ("decode_unit_kernel", 5, 1, 64, 16, SHORT, 64), ("decode_unit_kernel", 33, 1, 64, 80, SHORT, 192),
    ("decode_unit_kernel", 6, 2, 128, 512, [1500, 3000] * 20, 0), ("decode_unit_kernel", 8, 2, 64, 512, [2500] * 40, 0),
    ("decode_tile_kernel", 8, 8, 128, 64, [63] * 70, 0), ("decode_tile_kernel", 8, 2, 128, 512, [300] * 70, 0),
    ("decode_unit_kernel", 8, 8, 128, 64, [40] * 40, 0), ("decode_unit_kernel", 8, 2, 128, 512, [300, 700, 2000], 0),
    ("decode_block_kernel", 8, 8, 128, 512, [70, 200, 255], 0), ("decode_block_kernel", 8, 2, 128, 512, [3100, 6000], 0),
    ("decode_block_kernel", 8, 1, 128, 64, SHORT[:-1] + [255], 0), ("decode_block_kernel", 16, 1, 128, 24, SHORT, 0),
    ("decode_block_kernel", 3, 1, 64, 16, SHORT, 0), ("decode_block_kernel", 4, 2, 64, 64, SHORT, 0)])
def test_instance(pool_mode, kernel, n_q, n_kv, dim, tokens, lens, split):
    """Append and decode, then the fused call for the next token: the oracle's output, the bits that the separate calls
    give, and the chunks byte for byte (memory that nothing was written to holds bf16 NaN)."""
    n = len(lens)
    need = [-(-(x + 1) // tokens) for x in lens]
    cfg = W.Config("i", 9, n, n_q, n_kv, dim, tokens * 4 * n_kv * dim, sum(need) + 3, max(need) * tokens, "uniform", 1, max(lens))
    assert cfg.chunk_bytes % 4096 == 0 and cfg.group * n_kv == n_q
    rng = np.random.default_rng(6)
    B = H.Both(cfg)
    poison = np.full(cfg.chunk_bytes // 2, H.POISON, np.uint16).view(np.uint8)
    for c in range(cfg.n_chunks):
        B.orc.chunk_set_bytes(c, poison)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    free = rng.permutation(cfg.n_chunks).astype(np.int32)
    ids, at = [], 0
    for s in need:
        ids.append(B.create(cfg.max_tokens))
        assert B.map(ids[-1], 0, s, free[at:at + s]) == 0
        at += s
    for b0 in range(0, n, 16):
        part = lens[b0:b0 + 16]
        assert B.append(ids[b0:b0 + 16], bits(sum(part), n_kv, dim), bits(sum(part), n_kv, dim), part) == 0
    E.ellm_pool_set_split_tokens(B.pool, split)
    q = bits(n, n_q, dim)
    assert E.ellm_debug_decode_kernel(B.pool, ids) == kernel
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, "decode")
    assert E.ellm_debug_decode_kernel(B.pool, ids, 1) == kernel
    rc, fused, ref = B.append_decode(ids, bits(n, n_kv, dim), bits(n, n_kv, dim), q)
    assert rc == 0
    H.check_close(fused, ref, "append + decode")
    rc, again = B.decode(ids, q)
    assert rc == 0 and torch.equal(fused, again)
    B.compare_state()
    for c in range(cfg.n_chunks):
        assert np.array_equal(B.chunk_bytes_dev(c), B.orc.chunk_bytes_of(c)), c
    B.close()
