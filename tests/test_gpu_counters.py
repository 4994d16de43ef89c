"""Partial results of shared requests are counted in memory that outlives a call: the entry point with the fixed workspace has
counters of its own, so that a captured call of it can be replayed beside calls of the other; and counters that are off 0
are put back by ellm_pool_reset_counters."""
import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
import workloads as W
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


def shared(lens, n_q, n_kv, dim, tokens):
    need = [-(-n // tokens) for n in lens]
    cfg = W.Config("c", 9, len(lens), n_q, n_kv, dim, tokens * 4 * n_kv * dim, sum(need) + 1, max(need) * tokens, "uniform", 1, max(lens))
    rng = np.random.default_rng(3)
    B = H.Both(cfg)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    ids = []
    for n, s in zip(lens, need):
        ids.append(B.create(n))
        assert B.map(ids[-1], 0, s) == 0
    assert B.append(ids, bits(sum(lens), n_kv, dim), bits(sum(lens), n_kv, dim), lens) == 0
    return B, ids, bits(len(lens), n_q, dim)


# blocks, shares of tiles and of units, as the kernel's name tells
CASES = [("decode_block_kernel", [3000], 8, 2, 128, 128), ("decode_tile_kernel", [9000, 9100, 17, 9200] * 3, 8, 2, 128, 128),
         ("decode_unit_kernel", [700, 5000, 900] * 4, 12, 1, 64, 24)]


@pytest.mark.parametrize("kernel,lens,n_q,n_kv,dim,tokens", CASES)
def test_replays_with_the_fixed_workspace_beside_other_calls(kernel, lens, n_q, n_kv, dim, tokens):
    """A captured call of one entry point on one stream, calls of the other, over the same requests in another order (so
    that a request's line of counters is another's there), on a second stream: nothing orders them, and all outputs are
    bit for bit those of the calls alone."""
    B, ids, q = shared(lens, n_q, n_kv, dim, tokens)
    if kernel != "decode_block_kernel":
        E.ellm_debug_set_compute_units(B.pool, 64)
    assert E.ellm_debug_decode_kernel(B.pool, ids) == kernel
    assert E.ellm_decode_plan(B.pool, ids)[0].max() > 2
    rc, want = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(want, ref, kernel)
    other = ids[::-1]
    rc, want_other = B.decode(other, q)
    assert rc == 0
    n = 24
    qd = H.dev_bits(q)
    outs = torch.zeros((n, *qd.shape), dtype=qd.dtype, device="cuda")
    outs_other = torch.zeros_like(outs)
    a, b, graph = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    a.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(a):
        with torch.cuda.graph(graph, stream=a):
            for i in range(n):
                E.ellm_decode_attention_noalloc(B.pool, ids, qd, outs[i])
    with torch.cuda.stream(b):         # (the first call here is put behind the stream of the calls before it)
        E.ellm_decode_attention(B.pool, other, qd, outs_other[0])
    torch.cuda.synchronize()
    for _ in range(5):
        outs.zero_()
        outs_other.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(a):
            graph.replay()
        with torch.cuda.stream(b):
            for i in range(n):
                E.ellm_decode_attention(B.pool, other, qd, outs_other[i])
        torch.cuda.synchronize()
        for i in range(n):
            assert torch.equal(outs[i], want), i
            assert torch.equal(outs_other[i], want_other), i
    B.close()


@pytest.mark.parametrize("kernel,lens,n_q,n_kv,dim,tokens", CASES)
def test_counters_are_put_back(kernel, lens, n_q, n_kv, dim, tokens):
    """As calls that overlapped would leave them: off 0. After the reset every later call of either entry point is right,
    whichever stream the reset ran on (calls in turn over another batch, whose partial results lie in the same places)."""
    B, ids, q = shared(lens, n_q, n_kv, dim, tokens)
    if kernel != "decode_block_kernel":
        E.ellm_debug_set_compute_units(B.pool, 64)
    q2 = q[::-1].copy() if len(ids) > 1 else q ^ 0x8000
    want = {}
    for what, values in ((1, q), (2, q2)):
        rc, want[what] = B.decode(ids, values)
        assert rc == 0
    assert not torch.equal(want[1], want[2])
    qd, out, side = {1: H.dev_bits(q), 2: H.dev_bits(q2)}, torch.zeros_like(want[1]), torch.cuda.Stream()
    for value in (1, 2, 5):
        for stream in (side, torch.cuda.current_stream()):
            E.ellm_debug_set_counters(B.pool, value)
            E.ellm_pool_reset_counters(B.pool, stream.cuda_stream)
            for call in (E.ellm_decode_attention, E.ellm_decode_attention_noalloc):
                for what in (1, 2, 1):
                    out.zero_()
                    call(B.pool, ids, qd[what], out)
                    torch.cuda.synchronize()
                    assert torch.equal(out, want[what])
    B.close()


def test_reset_is_not_recorded():
    B, ids, q = shared([3000], 8, 2, 128, 128)
    qd = H.dev_bits(q)
    out = torch.zeros_like(qd)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    E.ellm_decode_attention(B.pool, ids, qd, out)
    torch.cuda.synchronize()
    want = out.clone()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            E.ellm_decode_attention(B.pool, ids, qd, out)
            assert E.ellm_pool_reset_counters(B.pool, stream.cuda_stream, check=False) == E.ERR.INVALID
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    B.close()
