"""Shared requests are stored, counted in and added up in pieces of 1, 2 or 4 q heads, dealt out to the waves of a workgroup by how
many requests meet there: group sizes on both sides of every line, workgroups with one, two and more requests."""
import pytest
import torch

import paper_2506_15155_amd as E
from tests import gpu_harness as H
from tests.test_gpu_one_way import load

pytestmark = pytest.mark.gpu

# (64 tokens a wave, 256 a workgroup) one request over many workgroups; then two, three and more in one; then two long ones
PARTS = [11, 1, 2, 1, 3, 2, 2, 6, 10, 1, 1, 2, 5]


@pytest.mark.parametrize("kernel,n_kv,group,dim,tokens", [
    ("decode_tile_kernel", 3, 1, 128, 64), ("decode_tile_kernel", 2, 2, 64, 64), ("decode_tile_kernel", 3, 4, 128, 64),
    ("decode_tile_kernel", 1, 8, 128, 64), ("decode_unit_kernel", 3, 3, 64, 64), ("decode_unit_kernel", 3, 5, 128, 64),
    ("decode_unit_kernel", 1, 8, 64, 64), ("decode_unit_kernel", 3, 9, 64, 64), ("decode_unit_kernel", 3, 12, 128, 64),
    ("decode_unit_kernel", 1, 13, 64, 64), ("decode_unit_kernel", 3, 16, 128, 64), ("decode_unit_kernel", 2, 16, 64, 64)])
def test_pieces(pool_mode, kernel, n_kv, group, dim, tokens):
    """The oracle's output; the same bits from repeated calls and from calls of the requests in another order between them, which
    would find counters that did not go back to 0."""
    lens = [64 * n - (5 * i) % 11 for i, n in enumerate(PARTS)]
    B, ids, q = load(n_kv, group, dim, tokens, lens, 21)
    E.ellm_pool_set_split_tokens(B.pool, 64)
    assert E.ellm_debug_decode_kernel(B.pool, ids) == kernel
    assert list(E.ellm_decode_plan(B.pool, ids)[0]) == PARTS and E.ellm_debug_combined_requests(B.pool, ids) == 0
    rc, out = B.decode(ids, q)
    rco, ref = B.orc.decode(ids, q)
    assert rc == 0 and rco == 0
    H.check_close(out, ref, f"{kernel} {group}")
    for _ in range(3):
        rc, other = B.decode(ids[::-1], q[::-1].copy())
        assert rc == 0
        H.check_close(other, ref[::-1], "in another order")
        rc, again = B.decode(ids, q)
        assert rc == 0 and torch.equal(again, out)
    B.close()
