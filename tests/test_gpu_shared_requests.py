"""Requests that several waves share: their results meet in LDS where the waves are of one workgroup, partial results of
several workgroups are added up by the one that ends last, or by the combine pass where there are many."""
import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
import workloads as W
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


def merge_parts(dim, group, kernel):
    """The library's line between the two, as its sources state it."""
    kb = {"decode_block_kernel": 192, "decode_tile_kernel": 64 * 4, "decode_unit_kernel": 32 * 4}[kernel]
    return min((kb << 10) // (min(group, 16) * dim * 4), 16 if group > 16 else 1 << 30)


# n_kv: workgroups that begin in one kv head and end in the next (3, 5); waves that are no whole number of workgroups (1)
@pytest.mark.parametrize("kernel,n_kv,group,dim,tokens,most", [
    ("decode_tile_kernel", 3, 1, 128, 128, 9), ("decode_tile_kernel", 1, 4, 128, 128, 129), ("decode_tile_kernel", 5, 4, 128, 64, 9),
    ("decode_tile_kernel", 3, 8, 128, 128, 65), ("decode_tile_kernel", 1, 2, 64, 128, 9), ("decode_unit_kernel", 3, 16, 128, 48, 17),
    ("decode_unit_kernel", 1, 6, 128, 24, 43), ("decode_unit_kernel", 5, 3, 64, 64, 9), ("decode_unit_kernel", 1, 34, 64, 64, 17),
    ("decode_block_kernel", 1, 4, 128, 128, 97), ("decode_block_kernel", 2, 8, 128, 128, 49), ("decode_block_kernel", 3, 16, 128, 48, 25),
    ("decode_block_kernel", 1, 6, 128, 64, 65), ("decode_block_kernel", 2, 16, 64, 64, 49)])
def test_sums_of_shared_requests(kernel, n_kv, group, dim, tokens, most):
    """Requests of 1 to 9 waves, in an order that puts their ends at every place in a workgroup, with or without one of
    just too many to be added up without the combine pass, which then adds up all of them. The oracle's output; the same bits from every replay of a graph, with
    other batches decoded in between (counters that did not go back to 0 would give the sums to the wrong workgroup)."""
    blocks = kernel == "decode_block_kernel"
    line = merge_parts(dim, group, kernel)
    at_line = most == line + 1
    assert at_line or most == 9 and line > 9
    step = 256 if blocks else 64
    parts = [most, most - 1] if blocks else [1, 2, 3, 1, 4, 5, 1, 1, 7, 8, 9, 2, 6] + ([most - 1, most] if at_line else [])
    lens = [step * n - (5 * i) % 11 for i, n in enumerate(parts)]
    need = [-(-n // tokens) for n in lens]
    cfg = W.Config("s", 9, len(lens), n_kv * group, n_kv, dim, tokens * 4 * n_kv * dim, sum(need) + 2, max(need) * tokens, "uniform", 1, max(lens))
    rng = np.random.default_rng(11)
    B = H.Both(cfg)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    ids = []
    for n, s in zip(lens, need):
        ids.append(B.create(n))
        assert B.map(ids[-1], 0, s) == 0
    assert B.append(ids, bits(sum(lens), n_kv, dim), bits(sum(lens), n_kv, dim), lens) == 0
    if not blocks:
        E.ellm_pool_set_split_tokens(B.pool, 64)
    assert E.ellm_debug_decode_kernel(B.pool, ids) == kernel
    n_split, _ = E.ellm_decode_plan(B.pool, ids)
    if dim == 128 and tokens in (64, 128):
        assert list(n_split) == parts
    assert not at_line or (n_split.max() > line and (n_split > 1).sum() > (n_split > line).sum())
    assert E.ellm_debug_combined_requests(B.pool, ids) == ((n_split > 1).sum() if at_line or group > 16 else 0)
    q = bits(len(lens), cfg.n_q_heads, dim)
    rc, want = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(want, ref, f"{parts}")
    qd, out, other = H.dev_bits(q), torch.empty_like(want), torch.empty_like(want)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            E.ellm_decode_attention(B.pool, ids, qd, out)
            E.ellm_decode_attention(B.pool, ids[::-1], qd, other)
    torch.cuda.synchronize()
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        rc, again = B.decode(ids, q)
        assert rc == 0 and torch.equal(again, want)
    B.close()
