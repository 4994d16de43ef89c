"""The copy kernel moves whole chunks, byte for byte, whatever their size and number: fewer pieces than a workgroup has
threads, a last turn that is not full, more chunks than workgroups of a call, more than one launch describes."""
import pytest
import torch

import paper_2506_15155_amd as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,chunks", [(1, 5), (7, 1), (16, 3), (33, 64), (130, 65), (1024, 1), (1024, 2), (1000, 27), (1, 481), (9, 129)])
def test_bytes_of_every_chunk(tokens, chunks):
    kv, dim = 2, 64
    cb = tokens * 4 * kv * dim
    g = torch.Generator(device="cuda").manual_seed(tokens * 1000 + chunks)
    dev = torch.randint(0, 256, ((2 * chunks + 1) * cb,), dtype=torch.uint8, device="cuda", generator=g)
    host = torch.zeros((chunks + 1) * cb, dtype=torch.uint8, pin_memory=True)
    pool = E.ellm_pool_create(dev, host, cb, kv, kv, dim, 1, chunks)
    t = E.ellm_tensor_create(pool, chunks * tokens)
    there = torch.randperm(2 * chunks + 1, generator=torch.Generator().manual_seed(chunks))[:chunks]
    E.ellm_tensor_map_chunks(pool, t, 0, chunks, there.numpy())
    E.ellm_debug_set_copy_kernels(pool, 1)
    before = dev.view(-1, cb).clone()
    E.ellm_chunk_deflate_to_host(pool, t, 0, chunks)
    E.ellm_pool_sync(pool)
    assert torch.equal(dev.view(-1, cb), before)
    table, _ = E.ellm_tensor_get_table(pool, t)
    slots = torch.tensor([-int(e) - 2 for e in table[:chunks]])
    rows = host.view(-1, cb)
    assert torch.equal(rows[slots], before[there.cuda()].cpu())
    unused = sorted(set(range(chunks + 1)) - set(slots.tolist()))
    assert not rows[unused].any()
    back = torch.randperm(2 * chunks + 1, generator=torch.Generator().manual_seed(chunks + 1))[:chunks]
    dev.fill_(0x5A)
    torch.cuda.synchronize()
    E.ellm_chunk_inflate_from_host(pool, t, 0, chunks, back.numpy())
    E.ellm_pool_sync(pool)
    want = torch.full_like(before, 0x5A)
    want[back.cuda()] = before[there.cuda()]
    assert torch.equal(dev.view(-1, cb), want)
    assert E.ellm_pool_get_copy_counts(pool) == (0, 2)
    E.ellm_pool_destroy(pool)


@pytest.mark.parametrize("out_by,in_by", [(1, -1), (-1, 1), (1, 1)])
def test_a_copy_reads_what_the_one_before_it_wrote(out_by, in_by):
    """Offload and fetch of the same chunks in turn, by kernel and by engine, with no wait of the host between: the fetch
    reads the host slots that the offload wrote, the next offload the chunks that the fetch wrote."""
    tokens, chunks, kv, dim = 64, 8, 2, 64
    cb = tokens * 4 * kv * dim
    g = torch.Generator(device="cuda").manual_seed(5)
    dev = torch.randint(0, 256, (chunks * cb,), dtype=torch.uint8, device="cuda", generator=g)
    want = dev.view(-1, cb).clone()
    host = torch.zeros(chunks * cb, dtype=torch.uint8, pin_memory=True)
    pool = E.ellm_pool_create(dev, host, cb, kv, kv, dim, 1, chunks)
    t = E.ellm_tensor_create(pool, chunks * tokens)
    E.ellm_tensor_map_chunks(pool, t, 0, chunks, torch.arange(chunks).numpy())
    torch.cuda.synchronize()
    at = torch.arange(chunks)
    for turn in range(6):
        E.ellm_debug_set_copy_kernels(pool, out_by)
        E.ellm_chunk_deflate_to_host(pool, t, 0, chunks)
        E.ellm_debug_set_copy_kernels(pool, in_by)
        to = torch.randperm(chunks, generator=torch.Generator().manual_seed(turn))
        E.ellm_chunk_inflate_from_host(pool, t, 0, chunks, to.numpy())
        now = torch.empty_like(want)
        now[to.cuda()] = want[at.cuda()]
        want, at = now, to
    E.ellm_pool_sync(pool)
    assert torch.equal(dev.view(-1, cb), want)
    E.ellm_pool_destroy(pool)
