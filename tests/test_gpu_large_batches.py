"""Batches of 129 to 256 requests are one launch where its two groups of 128 run the same kernel and their partial results fit; larger
ones are launches of 128. The outputs are those of the groups in calls of their own, bit for bit."""
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
    assert rc in (0, E.ERR.HIP)
    return 1 if rc == 0 else 2


def in_groups(B, ids, q):
    """The groups of 128 in calls of their own."""
    outs = [B.decode(ids[i:i + 128], q[i:i + 128]) for i in range(0, len(ids), 128)]
    assert all(rc == 0 for rc, _ in outs)
    return torch.cat([out for _, out in outs])


# the kernels of the two groups, whether they share a launch, the lengths, and longer requests (at, tokens)
@pytest.mark.parametrize("kernels,n_kv,group,dim,tokens,n,lo,hi,long,one", [
    ("tile tile", 3, 4, 128, 64, 200, 300, 900, [], True), ("tile tile", 2, 8, 128, 64, 256, 200, 600, [(127, 3000), (128, 2100)], True),
    ("tile tile", 1, 1, 128, 64, 250, 600, 1500, [], True), ("tile tile", 7, 4, 128, 64, 147, 1000, 1300, [], True), ("tile tile", 5, 2, 64, 64, 193, 300, 900, [], True),
    ("tile tile", 8, 1, 64, 64, 200, 300, 700, [], True), ("tile tile", 8, 2, 128, 64, 192, 200, 600, [], True),
    ("unit unit", 2, 12, 64, 64, 256, 300, 900, [(40, 3000)], True), ("unit unit", 8, 3, 64, 16, 220, 1, 300, [], True),
    ("unit unit", 1, 8, 128, 64, 256, 200, 300, [], True), ("unit unit", 8, 3, 64, 64, 200, 5, 40, [], True),
    ("block block", 1, 3, 128, 64, 136, 3, 156, [], True), ("block block", 2, 4, 64, 64, 256, 1, 200, [], True),
    ("block block", 2, 8, 128, 64, 200, 300, 500, [], True),                                            # (of up to 32 units)
    ("block block", 1, 3, 128, 64, 136, 3, 100, [(130, 3000)], True),                                   # split ones in the second
    ("tile tile", 2, 8, 128, 64, 200, 100, 300, [(3, 9000), (140, 20000)], True),                       # by combine passes
    ("unit unit", 2, 12, 64, 64, 256, 300, 900, [(140, 30000)], True),                                  # the second only
    ("tile unit", 3, 4, 128, 64, 129, 30, 900, [(43, 3000), (128, 2100)], False), ("unit block", 3, 6, 128, 24, 190, 100, 500, [], False),
    ("tile block", 4, 4, 128, 64, 160, 480, 520, [], False), ("tile tile", 3, 4, 128, 64, 256, 300, 900, [], False),
    ("block block", 2, 4, 128, 64, 257, 30, 500, [], False), ("unit unit", 2, 34, 64, 64, 140, 30, 300, [], False)])
def test_one_launch(pool_mode, kernels, n_kv, group, dim, tokens, n, lo, hi, long, one):
    """One launch where both groups run the same kernel and their partial results fit (3 and 7 kv heads: 341 and 146 waves a
    head, which straddle workgroups), and the same bits either way."""
    rng = np.random.default_rng(n)
    lens = [int(x) for x in rng.integers(lo, hi + 1, size=n)]
    for at, length in long:
        lens[at] = length
    B, ids, q = load(n_kv, group, dim, tokens, lens, 31)
    assert [E.ellm_debug_decode_kernel(B.pool, x) for x in (ids[:128], ids[128:256])] == [f"decode_{k}_kernel" for k in kernels.split()]
    assert launches(B, ids, q) == (1 if one else 2)
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, kernels)
    assert torch.equal(out, in_groups(B, ids, q))
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
    assert rc == 0 and torch.equal(fused, again) and torch.equal(again, in_groups(B, ids, q))
    B.close()


@pytest.mark.parametrize("n,dim,group", [(200, 128, 4), (256, 64, 3)])
def test_replays(n, dim, group):
    """Captured, with the longest arguments that a launch has: every replay gives the eager call's bits, with other calls between."""
    rng = np.random.default_rng(n)
    lens = [int(x) for x in rng.integers(700, 1200, size=n)]
    B, ids, q = load(2, group, dim, 64, lens, 32)
    assert launches(B, ids, q) == 1
    rc, want = B.decode(ids, q)
    assert rc == 0
    dq, outs = H.dev_bits(q), torch.empty(2, *want.shape, dtype=want.dtype, device="cuda")
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        assert E.ellm_decode_attention(B.pool, ids, dq, outs[0], check=False) == 0
        assert E.ellm_decode_attention_noalloc(B.pool, ids, dq, outs[1], check=False) == 0
    for _ in range(4):
        outs.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(outs[0], want) and torch.equal(outs[1], want)
        rc, eager = B.decode(ids[: n // 2], q[: n // 2])
        assert rc == 0
    B.close()


@pytest.mark.parametrize("seed,refused", [(0, False), (14, True)])
def test_the_fixed_workspace_refuses_what_it_refuses_by_groups(seed, refused):
    """16 q heads of 128 for each of 8 kv heads: it holds 252 partial results per kv head. The first group's plan reserves 228 or
    254; their workgroups leave half as many, which would fit either way."""
    n_kv, group, dim, tokens, n = 8, 16, 128, 64, 140
    rng = np.random.default_rng(seed)
    lens = np.asarray([1088 + 64 * int(x) for x in rng.integers(0, 3, size=n)], np.int32)
    need = [-(-int(x) // tokens) for x in lens]
    cb = tokens * 4 * n_kv * dim
    dev = torch.empty(sum(need) * cb, dtype=torch.uint8, device="cuda")
    pool = E.ellm_pool_create(dev, None, cb, n_kv * group, n_kv, dim, n, max(need))
    ids = []
    for x, s in zip(lens, need):
        ids.append(E.ellm_tensor_create(pool, int(x)))
        E.ellm_tensor_map_chunks(pool, ids[-1], 0, s)
    rows = torch.randn(int(lens.sum()), n_kv, dim, device="cuda").to(torch.bfloat16)
    E.ellm_kv_append(pool, ids, rows, rows, lens)
    n_split = E.ellm_decode_plan(pool, ids)[0][:128]
    assert (int(n_split[n_split > 1].sum()) > 252) == refused
    q = torch.randn(n, n_kv * group, dim, device="cuda").to(torch.bfloat16)
    out, want = torch.full_like(q, 5.0), torch.empty_like(q)
    for m in (128, n):
        rc = E.ellm_decode_attention_noalloc(pool, ids[:m], q, out, check=False)
        torch.cuda.synchronize()
        assert rc == (E.ERR.RANGE if refused else 0)
        assert bool((out == 5.0).all()) == refused
    assert E.ellm_decode_attention(pool, ids, q, want, check=False) == 0
    torch.cuda.synchronize()
    assert refused or torch.equal(out, want)
    E.ellm_pool_destroy(pool)
