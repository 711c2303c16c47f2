"""The copies behind every emulated or external peer: whole and ragged rounds of a work-group, nothing past the end, every flag up."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROUND = 16 * 1024 * 16   # bytes that one work-group of 1024 threads moves per round


@pytest.mark.parametrize("sizes", [
    [16, 0, ROUND - 16, ROUND, ROUND + 16],
    [3 * ROUND + 16 * 1023, 48],
])
def test_published_chunks_are_whole_and_end_where_they_should(sizes):
    from paper_2605_02953_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(len(sizes))
    src = [torch.randint(0, 256, (n + 64,), dtype=torch.uint8, device="cuda", generator=g) for n in sizes]
    dst = [torch.full((n + 64,), 7, dtype=torch.uint8, device="cuda") for n in sizes]
    signals = torch.zeros(len(sizes), dtype=torch.int32, device="cuda")
    st = B.publish_chunks(dst, src, sizes, list(range(len(sizes))), signals, 5)
    assert st == B.OK, B.status_string(st)
    torch.cuda.synchronize()
    assert signals.tolist() == [5] * len(sizes)
    for n, s, d in zip(sizes, src, dst):
        assert torch.equal(d[:n], s[:n]) and (d[n:] == 7).all()


@pytest.mark.parametrize("op_world,m_per_rank,k", [(2, 1, 16), (2, 33, 520), (8, 17, 1032), (4, 300, 4104)])
def test_gathered_operand_is_whole(op_world, m_per_rank, k):
    """Several work-groups to a shard, shards that end inside a round and inside a cache line."""
    from gpu_util import AgGemmRun
    from paper_2605_02953_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(k)
    shards = [torch.randint(-3, 4, (m_per_rank, k), device="cuda", generator=g).to(torch.bfloat16) for _ in range(op_world)]
    b = torch.randint(-3, 4, (264, k), device="cuda", generator=g).to(torch.bfloat16)
    run = AgGemmRun(B, op_world, m_per_rank, 264, k)
    st = run([s.view(torch.int16) for s in shards], b.view(torch.int16), op_world - 1)
    assert st == B.OK, B.status_string(st)
    torch.cuda.synchronize()
    whole = torch.cat(shards)
    assert torch.equal(run.workspace.view(torch.bfloat16).reshape(-1)[:whole.numel()].view_as(whole), whole)
    # small integers: the fp32 sums are exact
    want = (whole.float() @ b.float().T).to(torch.bfloat16)
    assert torch.equal(run.c.view(torch.bfloat16), want)
