"""The attention kernels built of 16-row units (one wave per share; one workgroup per block): any group size, any chunk size, at the edges of its units,
tiles, shares and head passes, against the fp64 oracle. Unused memory is bf16 NaN, so a row that does not
belong to a request shows up in the output. Tolerance: the harness's (weights and results are rounded to
bf16, relative 2^-9 each, on outputs of the size of a N(0, 1) average: 2e-2 at most, 2e-3 on average)."""
import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
import workloads as W
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


def config(n_q, n_kv, dim, tokens, batch, most):
    return W.Config("u", 9, batch, n_q, n_kv, dim, tokens * 4 * n_kv * dim, batch * -(-most // tokens) + 4,
                    -(-most // tokens) * tokens, "uniform", 1, most)


@pytest.mark.parametrize("tokens,most", [(1, 40), (8, 70), (16, 200), (24, 300), (40, 700), (72, 1500), (500, 3000)])
@pytest.mark.parametrize("n_q,n_kv,dim", [(3, 1, 128), (16, 1, 64), (17, 1, 64), (14, 2, 128), (4, 2, 64), (33, 1, 128)])
def test_units_and_heads(n_q, n_kv, dim, tokens, most):
    """Chunks below, at and above a unit and a tile; heads below, at and above a pass; the lengths hit one
    token, whole units, whole chunks and one token more or less. Both entry points: append, then decode;
    and the fused call for the next token, which must give the bits that the separate calls give."""
    cfg = config(n_q, n_kv, dim, tokens, 9, most)
    rng = np.random.default_rng(5)
    lens = np.clip([1, 2, 15, 16, 17, 32, 33, tokens, most - 1], 1, most - 1).astype(np.int32)
    B = H.Both(cfg)
    poison = np.full(cfg.chunk_bytes // 2, H.POISON, np.uint16).view(np.uint8)
    for c in range(cfg.n_chunks):
        B.orc.chunk_set_bytes(c, poison)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    ids = []
    for n in lens:
        t = B.create(cfg.max_tokens)
        assert B.map(t, 0, -(-int(n + 1) // tokens)) == 0
        ids.append(t)
    total = int(lens.sum())
    assert B.append(ids, bits(total, n_kv, dim), bits(total, n_kv, dim), list(lens)) == 0
    q, kn, vn = bits(9, n_q, dim), bits(9, n_kv, dim), bits(9, n_kv, dim)
    rco, ref = B.orc.decode(ids, q)
    for split in (0, 192, 64):                # as the library cuts it (mostly a workgroup per block); waves that walk shares of three tiles, of one
        E.ellm_pool_set_split_tokens(B.pool, split)
        rc, out = B.decode(ids, q)
        assert rc == 0 and rco == 0
        H.check_close(out, ref, f"decode, split {split}")
    E.ellm_pool_set_split_tokens(B.pool, 64 * (n_q % 2))
    rc, fused, ref = B.append_decode(ids, kn, vn, q)
    assert rc == 0
    H.check_close(fused, ref, "append + decode")
    rc, again = B.decode(ids, q)
    assert rc == 0 and torch.equal(fused, again)
    B.compare_state()
    for c in range(cfg.n_chunks):
        assert np.array_equal(B.chunk_bytes_dev(c), B.orc.chunk_bytes_of(c)), c
    B.close()


def test_infinite_values_stay_with_their_request():
    """An infinity in V makes its own output infinite and no other; rows that are loaded in place of missing
    ones must not turn it into NaN."""
    cfg = config(6, 1, 128, 24, 3, 60)
    B = H.Both(cfg)
    ids = []
    for n in (5, 24, 50):
        t = B.create(cfg.max_tokens)
        assert B.map(t, 0, -(-n // 24)) == 0
        ids.append(t)
    k = torch.zeros((79, 1, 128), dtype=torch.bfloat16, device="cuda")
    v = torch.ones_like(k)
    v[4, 0, 7] = float("inf")                   # last row of the first request
    E.ellm_kv_append(B.pool, ids, k, v, [5, 24, 50])
    q = torch.randn((3, 6, 128), device="cuda").to(torch.bfloat16)
    for split in (0, 64):
        E.ellm_pool_set_split_tokens(B.pool, split)
        out = torch.empty_like(q)
        E.ellm_decode_attention(B.pool, ids, q, out)
        assert torch.isposinf(out[0, :, 7]).all()
        out[0, :, 7] = 1.0
        assert (out == 1.0).all()
    E.ellm_pool_destroy(B.pool)
    B.orc.close()


@pytest.mark.parametrize("n_q,n_kv,dim,lens", [(4, 1, 128, [256] * 256), (4, 1, 128, [257] * 129), (16, 2, 64, [1, 255, 256, 257, 512, 513]),
                                               (1, 1, 64, [256] * 40), (8, 8, 128, [4096, 4097]),
                                               (8, 8, 64, [257] * 20 + [10] * 30), (8, 8, 64, [10] * 30 + [257] * 20)])
def test_block_limits(n_q, n_kv, dim, lens):
    """Around a block of 256 tokens, and batches on both sides of the limits up to which blocks are taken."""
    cfg = config(n_q, n_kv, dim, 64, len(lens), max(lens))
    rng = np.random.default_rng(3)
    B = H.Both(cfg)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    ids = []
    for n in lens:
        t = B.create(n)
        assert B.map(t, 0, -(-n // 64)) == 0
        ids.append(t)
    assert B.append(ids, bits(sum(lens), n_kv, dim), bits(sum(lens), n_kv, dim), lens) == 0
    q = bits(len(lens), n_q, dim)
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, "decode")
    rc, again = B.decode(ids, q)
    assert rc == 0 and torch.equal(out, again)
    B.close()


def test_small_batches_are_cut_request_by_request():
    """Where every wave gets one step, a request's bits do not depend on its neighbours."""
    cfg = config(12, 2, 128, 24, 6, 500)
    st = W.draw_step(cfg, seed=2)
    B = H.Both(cfg)
    ids = H.load_step(B, st)
    assert B.append(ids, st.k_new, st.v_new) == 0
    rc, out = B.decode(ids, st.q)
    assert rc == 0
    for b in (0, 3, 5):
        rc, one = B.decode([ids[b]], st.q[[b]])
        assert rc == 0 and torch.equal(one[0], out[b])
    B.close()


@pytest.mark.parametrize("parts", [[2, 3, 4], [2, 9, 16, 17, 40], [31, 32, 33, 64, 65, 129, 200]])
@pytest.mark.parametrize("n_q,dim,tokens", [(4, 128, 128), (3, 128, 128), (1, 64, 128), (5, 64, 48)])
def test_combine_widths(n_q, dim, tokens, parts):
    """Few, several and many partial results per request: one, four and sixteen waves add them up, in one
    round of loads or in more; rows in the order of either attention kernel."""
    most = 64 * max(parts)
    cfg = W.Config("c", 9, len(parts), n_q, 1, dim, tokens * 4 * dim, sum(-(-64 * n // tokens) for n in parts) + len(parts) + 2,
                   most + tokens, "uniform", 1, most)
    rng = np.random.default_rng(9)
    B = H.Both(cfg)

    def bits(*shape):
        return (rng.standard_normal(shape).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)

    ids = []
    for n in parts:
        t = B.create(64 * n)
        assert B.map(t, 0, -(-64 * n // tokens)) == 0
        ids.append(t)
    total = 64 * sum(parts)
    assert B.append(ids, bits(total, 1, dim), bits(total, 1, dim), [64 * n for n in parts]) == 0
    q = bits(len(parts), n_q, dim)
    E.ellm_pool_set_split_tokens(B.pool, 64)
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, f"{parts}")
    rc, again = B.decode(ids, q)
    assert rc == 0 and torch.equal(out, again)
    B.close()
