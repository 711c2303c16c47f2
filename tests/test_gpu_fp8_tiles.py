"""fp8 AllGather-GEMM on the 256-row tiles of the tile engine against the CPU oracle, through the C ABI."""
import numpy as np
import pytest
import torch

import synth
from oracle import ag_gemm as oag, formats, schedule as osch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2605_02953_amd import binding
    assert torch.cuda.is_available()
    return binding


from gpu_util import to_dev, bits, nk, AgGemmRun  # noqa: E402


def _case(m_r, n, k, seed):
    """Integers in -2 .. 2 and power-of-two scales: every product, sum and scaled sum is exact in fp32, so the only
    rounding is the final one to bf16 and the bits must be the oracle's."""
    cfg = synth.CONFIGS[5].scaled(world=8, m_per_rank=m_r, n=n, k=k, rank=3)
    rng = synth.rng_for(seed, 5, 77)
    q = lambda shape: synth.quantize_e4m3(rng.integers(-2, 3, size=shape).astype(np.float64), 1.0)   # noqa: E731
    a, b = [q((m_r, k)) for _ in range(8)], q((k, n))
    sa = np.array([2.0 ** (s % 3 - 1) for s in range(8)], dtype=np.float32)
    sb = np.array([2.0 ** (j % 4 - 2) for j in range(n)], dtype=np.float32)
    return cfg, a, sa, b, sb


# one, two, three and five 128-byte K tiles, with and without a ragged last one; all three tile widths; tile rows that
# span two shards and ragged last rows and columns
@pytest.mark.parametrize("k", [16, 112, 128, 144, 256, 400, 640])
@pytest.mark.parametrize("n,block_n", [(4096, 256), (3080, 224), (3072, 192)])
def test_fp8_on_256_row_tiles_is_bit_exact(B, k, n, block_n):
    cfg, a, sa, b, sb = _case(505, n, k, k)
    st, tc = B.tile_config(0, cfg.m, n, k, B.FP8_E4M3)
    assert (st, tc["block_m"], tc["block_n"], tc["splits"]) == (B.OK, 256, block_n, 1)
    run = AgGemmRun(B, 8, cfg.m_per_rank, n, k, esize=1)
    ad, bd = [to_dev(x) for x in a], to_dev(nk(b))
    sched = torch.full((4 * tc["ntiles"],), -1, dtype=torch.int32, device="cuda")
    for scaled in (False, True):
        st = run(ad, bd, cfg.rank, dtype=B.FP8_E4M3, schedule=sched, a_scales=to_dev(sa) if scaled else None,
                 b_scales=to_dev(sb) if scaled else None)
        assert st == B.OK, B.status_string(st)
        torch.cuda.synchronize()
        assert run.status.cpu().tolist()[0] == 0 and not run.signals.cpu().numpy()[8:].any()
        want = oag.ag_gemm(a, b, dtype="e4m3", **(dict(a_scales=sa, b_scales=sb) if scaled else {}))
        assert np.array_equal(bits(run.c), formats.encode_bf16_rne(want.astype(np.float32)))
    assert np.array_equal(run.workspace.cpu().numpy(), oag.gather(a))
    want = [osch.ag_tile(osch.xcd_remap(w, tc["ntiles"], tc["num_xcd"], tc["per_xcd"]), cfg.m, n, 256, block_n, tc["group_m"], cfg.rank, 8)
            for w in range(tc["ntiles"])]
    assert np.array_equal(sched.cpu().numpy().reshape(-1, 4), np.asarray(want, dtype=np.int32))
    assert B.schedule_dump(0, cfg.m, n, k, 8, cfg.rank, B.FP8_E4M3)[1] == want


def test_fp8_epoch_in_memory_on_256_row_tiles(B):
    """The epoch in memory at a size that takes the tile engine: eager, then a recorded launch replayed."""
    cfg, a, sa, b, sb = _case(505, 3080, 256, 1)
    want = formats.encode_bf16_rne(oag.ag_gemm(a, b, dtype="e4m3").astype(np.float32))
    run = AgGemmRun(B, 8, cfg.m_per_rank, cfg.n, cfg.k, esize=1)
    ad, bd = [to_dev(x) for x in a], to_dev(nk(b))
    flags = B.EMULATE_PRODUCER | B.EPOCH_IN_MEMORY

    def check(calls):
        torch.cuda.synchronize()
        sig = run.signals.cpu().numpy()
        assert run.status.cpu().tolist()[0] == 0 and sig[-1] == calls and sig[-2] == 0 and (sig[:8] == calls).all()
        assert np.array_equal(bits(run.c), want)
        run.c.zero_()
        run.workspace.zero_()

    assert run(ad, bd, cfg.rank, flags=flags, dtype=B.FP8_E4M3) == B.OK
    check(1)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        graph.capture_begin()
        try:
            st = run(ad, bd, cfg.rank, flags=flags, dtype=B.FP8_E4M3, stream=side)
        finally:
            graph.capture_end()
    assert st == B.OK
    for i in range(3):
        graph.replay()
        check(2 + i)


# 272 tiles of 128 x 128, the fewest that give way to 256-row tiles, and one row of tiles less; over one node and two
@pytest.mark.parametrize("m_r,rows", [(250, 256), (128, 128)])
def test_fp8_tile_rule_edge(B, m_r, rows):
    cfg, a, sa, b, sb = _case(m_r, 2056, 400, 7)
    st, tc = B.tile_config(0, cfg.m, cfg.n, cfg.k, B.FP8_E4M3)
    assert (st, tc["block_m"]) == (B.OK, rows)
    want = formats.encode_bf16_rne(oag.ag_gemm(a, b, dtype="e4m3", a_scales=sa, b_scales=sb).astype(np.float32))
    for nodes in (1, 2):
        run = AgGemmRun(B, 8, m_r, cfg.n, cfg.k, esize=1)
        st = run([to_dev(x) for x in a], to_dev(nk(b)), cfg.rank, dtype=B.FP8_E4M3, a_scales=to_dev(sa), b_scales=to_dev(sb),
                 tuning=B.tuning(num_nodes=nodes))
        assert st == B.OK, B.status_string(st)
        torch.cuda.synchronize()
        assert run.status.cpu().tolist()[0] == 0
        assert np.array_equal(bits(run.c), want)


# over several nodes fp8 is served where the 128-row listing is complete, also where the problem has 192 large tiles and more
# and their own listing is not (ranks 4 and 6); n is ragged
@pytest.mark.parametrize("m_r,n,nodes,rank", [(70, 16200, 4, 4), (70, 16200, 4, 0), (130, 9736, 8, 6), (130, 9736, 8, 5)])
def test_fp8_of_many_columns_over_several_nodes(B, m_r, n, nodes, rank):
    cfg, a, sa, b, sb = _case(m_r, n, 144, 9)
    run = AgGemmRun(B, 8, m_r, n, cfg.k, esize=1)
    tuning = B.tuning(num_nodes=nodes)
    st, tc = B.tile_config(0, cfg.m, n, cfg.k, B.FP8_E4M3)
    sched = torch.full((4 * tc["ntiles"] * tc["splits"],), -1, dtype=torch.int32, device="cuda")
    st = run([to_dev(x) for x in a], to_dev(nk(b)), rank, dtype=B.FP8_E4M3, schedule=sched, a_scales=to_dev(sa), b_scales=to_dev(sb),
             tuning=tuning)
    assert st == B.OK, B.status_string(st)
    torch.cuda.synchronize()
    assert run.status.cpu().tolist()[0] == 0
    want = formats.encode_bf16_rne(oag.ag_gemm(a, b, dtype="e4m3", a_scales=sa, b_scales=sb).astype(np.float32))
    assert np.array_equal(bits(run.c), want)
    host = B.schedule_dump(0, cfg.m, n, cfg.k, 8, rank, B.FP8_E4M3, tuning=tuning)[1]
    assert [tuple(r) for r in sched.cpu().view(-1, 4).tolist()] == host
