"""The split requests of a launch are added up by the attention kernel, or all of them by the combine pass: either way where one
of them has just as many partial results as the kernel takes, and one more."""
import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
import workloads as W
from tests import gpu_harness as H

DUMMY = 0x1000


def line(dim, group, kernel):
    """Parts of a request that the attention kernel adds up at most, as the library's sources state it."""
    kb = {"decode_block_kernel": 192, "decode_tile_kernel": 64 * 4, "decode_unit_kernel": 32 * 4}[kernel]
    return min((kb << 10) // (min(group, 16) * dim * 4), 16 if group > 16 else 1 << 30)


def test_all_or_none_go_to_the_combine_pass():
    """Without a device: how many requests of a launch the combine pass gets, over random batches."""
    rng = np.random.default_rng(8)
    seen = {True: 0, False: 0}
    for _ in range(300):
        n_kv, group, dim = int(rng.choice([1, 1, 2, 4, 8])), int(rng.choice([1, 4, 8, 12, 16])), int(rng.choice([64, 128]))
        tokens, n = int(rng.choice([16, 24, 102, 512])), int(rng.integers(1, 40))
        mean = float(np.exp(rng.uniform(np.log(50), np.log(12000))))
        lens = [int(x) for x in np.maximum(1, rng.lognormal(np.log(mean), 0.8, n))]
        need = [-(-x // tokens) for x in lens]
        cb = tokens * 4 * n_kv * dim
        P = E.ellm_pool_create(None, None, cb, n_kv * group, n_kv, dim, n, max(need), flags=1, device_bytes=(sum(need) + 1) * cb)
        ids = []
        for x, s in zip(lens, need):
            ids.append(E.ellm_tensor_create(P, s * tokens))
            E.ellm_tensor_map_chunks(P, ids[-1], 0, s)
        E.ellm_kv_append(P, ids, DUMMY, DUMMY, np.asarray(lens, np.int32), stream=0)
        n_split, _ = E.ellm_decode_plan(P, ids)
        kernel = E.ellm_debug_decode_kernel(P, ids)
        got = E.ellm_debug_combined_requests(P, ids)
        E.ellm_pool_destroy(P)
        over = bool(n_split.max() > line(dim, group, kernel))
        seen[over] += 1
        assert got == (int((n_split > 1).sum()) if over else 0), (lens, n_kv, group, dim)
    assert min(seen.values()) > 30


def load(n_kv, group, dim, tokens, lens, seed):
    need = [-(-(n + 1) // tokens) for n in lens]
    cfg = W.Config("o", 9, len(lens), n_kv * group, n_kv, dim, tokens * 4 * n_kv * dim, sum(need) + 2, max(need) * tokens, "uniform", 1, max(lens))
    rng = np.random.default_rng(seed)
    B = H.Both(cfg)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    ids = []
    for n, s in zip(lens, need):
        ids.append(B.create(n + 1))
        assert B.map(ids[-1], 0, s) == 0
    assert B.append(ids, bits(sum(lens), n_kv, dim), bits(sum(lens), n_kv, dim), lens) == 0
    return B, ids, bits(len(lens), n_kv * group, dim)


# (one kv head of 16 or of 34 heads: a request inside one workgroup is on the combine pass's list as well)
@pytest.mark.gpu
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("kernel,n_kv,group,dim,tokens", [
    ("decode_tile_kernel", 3, 8, 128, 128), ("decode_tile_kernel", 1, 4, 128, 128), ("decode_unit_kernel", 3, 16, 128, 48),
    ("decode_unit_kernel", 1, 34, 64, 64), ("decode_block_kernel", 2, 8, 128, 128), ("decode_block_kernel", 1, 12, 128, 64),
    ("decode_block_kernel", 1, 16, 64, 64)])
def test_either_way(kernel, n_kv, group, dim, tokens, over):
    blocks = kernel == "decode_block_kernel"
    most = line(dim, group, kernel) + over
    step = 256 if blocks else 64
    parts = [2, most, 1, 6, 4] if blocks else [1, 2, 3, 1, 4, most, 5, 2]
    lens = [step * n - (5 * i) % 11 for i, n in enumerate(parts)]
    B, ids, q = load(n_kv, group, dim, tokens, lens, 12)
    if not blocks:
        E.ellm_pool_set_split_tokens(B.pool, 64)
    assert E.ellm_debug_decode_kernel(B.pool, ids) == kernel
    n_split, _ = E.ellm_decode_plan(B.pool, ids)
    combined = E.ellm_debug_combined_requests(B.pool, ids)
    if list(n_split) == parts and group <= 16:
        assert combined == (sum(n > 1 for n in parts) if over else 0)
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, f"{parts}")
    for _ in range(3):
        rc, again = B.decode(ids, q)
        assert rc == 0 and torch.equal(again, out)
    if blocks and (group > 8 or dim == 64):
        # (pools whose small launches always go by blocks) what the request that is over the line changes for the others
        # is who adds them up, not the bits
        for b in (0, 2, 3, 4):
            rc, one = B.decode([ids[b]], q[[b]])
            assert rc == 0 and torch.equal(one[0], out[b])
            assert E.ellm_debug_combined_requests(B.pool, [ids[b]]) == 0
    B.close()


@pytest.mark.gpu
@pytest.mark.parametrize("group,dim,n_kv,split,most,combined", [
    (34, 64, 1, 64, 12, True), (20, 128, 3, 64, 9, True),          # a workgroup is one wave
    (34, 64, 3, 128, 16, False), (20, 128, 1, 128, 16, False), (64, 128, 1, 128, 16, False),
    (34, 64, 1, 128, 17, True), (17, 128, 3, 128, 17, True), (64, 128, 2, 128, 17, True),
    (34, 64, 2, 0, 0, True), (48, 128, 1, 0, 0, True)])             # single steps, as cut by the library
def test_groups_of_several_launches(pool_mode, group, dim, n_kv, split, most, combined):
    """More q heads per kv head than one launch handles: few units a wave, with a partial result from each, and shares,
    added up in every launch or by the pass; the same bits from replays of a graph with another batch behind; the fused call gives the bits of the separate ones."""
    parts = [1, 2, most, 3, 1, 5, most - 1, 2] if split else [1, 3, 2, 5, 9, 30]
    per = split or 64
    lens = [per * n - (7 * i) % 13 for i, n in enumerate(parts)]
    B, ids, q = load(n_kv, group, dim, 64, lens, 4)
    if split:
        E.ellm_pool_set_split_tokens(B.pool, split)
    assert E.ellm_debug_decode_kernel(B.pool, ids) == "decode_unit_kernel"
    n_split, _ = E.ellm_decode_plan(B.pool, ids)
    assert E.ellm_debug_combined_requests(B.pool, ids) == (int((n_split > 1).sum()) if combined else 0)
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, f"{parts}")
    qd, got, other = H.dev_bits(q), torch.empty_like(out), torch.empty_like(out)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            E.ellm_decode_attention(B.pool, ids, qd, got)
            E.ellm_decode_attention(B.pool, ids[::-1], qd, other)
    torch.cuda.synchronize()
    for _ in range(3):
        got.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, out)
    rng = np.random.default_rng(6)
    k, v = ((rng.standard_normal((len(lens), n_kv, dim)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16) for _ in range(2))
    rc, fused, ref = B.append_decode(ids, k, v, q)
    assert rc == 0
    H.check_close(fused, ref, "append + decode")
    rc, again = B.decode(ids, q)
    assert rc == 0 and torch.equal(fused, again)
    B.close()
