"""Batches of 129 to 256 requests are one launch where its partial results fit, larger ones launches of 128."""
import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
from tests import gpu_harness as H
from tests.test_gpu_one_way import load

pytestmark = pytest.mark.gpu


def launches(B, ids, q):
    """Of a decode over ids: the hook refuses the second one, if there is a second one."""
    out = torch.empty(q.shape, dtype=torch.bfloat16, device="cuda")
    E.ellm_debug_fail_launch(B.pool, 2)
    rc = E.ellm_decode_attention(B.pool, ids, H.dev_bits(q), out, check=False)
    E.ellm_debug_fail_launch(B.pool, 0)
    torch.cuda.synchronize()
    return 1 if rc == 0 else 2


# the kernel, whether it is one launch, the lengths: short ones, ones that end in a wave, and some of many waves
@pytest.mark.parametrize("kernel,n_kv,group,dim,tokens,n,lo,hi,one", [
    ("decode_tile_kernel", 3, 4, 128, 64, 129, 30, 900, True), ("decode_tile_kernel", 2, 8, 128, 64, 256, 30, 500, True),
    ("decode_tile_kernel", 1, 1, 128, 64, 200, 200, 900, True), ("decode_tile_kernel", 5, 2, 64, 64, 193, 30, 500, True),
    ("decode_unit_kernel", 3, 6, 128, 24, 129, 30, 500, True), ("decode_unit_kernel", 2, 12, 64, 64, 256, 30, 600, True),
    ("decode_unit_kernel", 7, 3, 64, 16, 150, 1, 300, True), ("decode_block_kernel", 1, 3, 128, 64, 136, 3, 156, True),
    ("decode_block_kernel", 2, 4, 64, 64, 256, 1, 200, True), ("decode_block_kernel", 1, 8, 128, 64, 150, 200, 300, True),
    ("decode_tile_kernel", 2, 4, 128, 64, 257, 30, 500, False), ("decode_unit_kernel", 2, 34, 64, 64, 140, 30, 300, False)])
def test_one_launch(pool_mode, kernel, n_kv, group, dim, tokens, n, lo, hi, one):
    rng = np.random.default_rng(n)
    lens = [int(x) for x in rng.integers(lo, hi + 1, size=n)]
    if kernel != "decode_block_kernel":
        lens[n // 3], lens[-1] = 3000, 2100
    B, ids, q = load(n_kv, group, dim, tokens, lens, 31)
    if kernel == "decode_block_kernel" and n == 150:
        E.ellm_debug_set_compute_units(B.pool, 160)             # wide blocks, one for every CU
    assert E.ellm_debug_decode_kernel(B.pool, ids) == kernel
    assert launches(B, ids, q) == (1 if one else 2)
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, kernel)
    E.ellm_pool_prepare(B.pool)
    same = torch.empty_like(out)
    assert E.ellm_decode_attention_noalloc(B.pool, ids, H.dev_bits(q), same, check=False) == 0
    torch.cuda.synchronize()
    assert torch.equal(same, out)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    rc, fused, ref = B.append_decode(ids, bits(n, n_kv, dim), bits(n, n_kv, dim), q)
    assert rc == 0
    H.check_close(fused, ref, "append + decode")
    rc, again = B.decode(ids, q)
    assert rc == 0 and torch.equal(fused, again)
    B.close()



@pytest.mark.parametrize("n,dim,group", [(200, 128, 4), (256, 64, 3)])
def test_replays(n, dim, group):
    """Captured, with the longest arguments that a launch has: every replay gives the eager call's bits, with other calls between."""
    rng = np.random.default_rng(n)
    lens = [int(x) for x in rng.integers(30, 700, size=n)]
    B, ids, q = load(2, group, dim, 64, lens, 32)
    assert launches(B, ids, q) == 1
    rc, want = B.decode(ids, q)
    assert rc == 0
    dq, out = H.dev_bits(q), torch.empty_like(want)
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        assert E.ellm_decode_attention(B.pool, ids, dq, out, check=False) == 0
        assert E.ellm_decode_attention_noalloc(B.pool, ids, dq, out, check=False) == 0
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        rc, eager = B.decode(ids[: n // 2], q[: n // 2])
        assert rc == 0
    B.close()
