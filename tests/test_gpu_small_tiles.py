"""The 128 x 128 tile of the tile engine at the lengths of its operand ring, and the all-reduce consumer at the rank
counts that have an instance of their own, against the CPU oracle through the C ABI.  Inputs are small integers: every
sum is exact in fp32, so the only rounding is the one to bf16 and the bits must be the oracle's."""
import numpy as np
import pytest
import torch

import synth
from oracle import ag_gemm as oag, formats, gemm_ar as oar

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2605_02953_amd import binding
    assert torch.cuda.is_available()
    return binding


from gpu_util import to_dev, bits, nk, AgGemmRun, GemmArRun, GemmRsRun  # noqa: E402
from test_gpu_moe import _run_and_check  # noqa: E402


def _ok(B, st, run):
    assert st == B.OK, B.status_string(st)
    torch.cuda.synchronize()
    assert run.status.cpu().tolist()[0] == 0


# less than a K tile, up to the three that the ring requests ahead, one more, two turns of the ring's seven pieces; whole
# and ragged last K tiles.  2000 x 2056: 272 tiles, the last row and the last column of tiles ragged
@pytest.mark.parametrize("k", [8, 64, 128, 136, 192, 200, 256, 448, 520])
@pytest.mark.parametrize("kn", [False, True], ids=["b_nk", "b_kn"])
def test_128_row_tiles_are_bit_exact(B, k, kn):
    cfg = synth.CONFIGS[2].scaled(world=8, m_per_rank=250, n=2056, k=k, rank=5)
    st, tc = B.tile_config(4 if kn else 0, cfg.m, cfg.n, k)
    assert (st, tc["block_m"], tc["block_n"], tc["splits"]) == (B.OK, 128, 128, 1)
    shards, b = synth.ag_gemm_inputs(cfg, integer=True)
    run = AgGemmRun(B, 8, cfg.m_per_rank, cfg.n, k)
    st = run([to_dev(s) for s in shards], to_dev(b if kn else nk(b)), cfg.rank, b_layout=B.B_KN if kn else B.B_NK)
    _ok(B, st, run)
    assert np.array_equal(bits(run.workspace), oag.gather(shards))
    assert np.array_equal(bits(run.c), formats.encode_bf16_rne(oag.ag_gemm(shards, b).astype(np.float32)))


# 256-row tiles of B stored [k, n] over the same lengths (its ring has five pieces)
@pytest.mark.parametrize("k", [56, 72, 128, 192, 320, 328])
def test_256_row_tiles_of_a_kn_weight_are_bit_exact(B, k):
    cfg = synth.CONFIGS[2].scaled(world=8, m_per_rank=505, n=3080, k=k, rank=2)
    st, tc = B.tile_config(4, cfg.m, cfg.n, k)
    assert (st, tc["block_m"], tc["block_n"]) == (B.OK, 256, 256)
    shards, b = synth.ag_gemm_inputs(cfg, integer=True)
    run = AgGemmRun(B, 8, cfg.m_per_rank, cfg.n, k)
    _ok(B, run([to_dev(s) for s in shards], to_dev(b), cfg.rank, b_layout=B.B_KN), run)
    assert np.array_equal(bits(run.c), formats.encode_bf16_rne(oag.ag_gemm(shards, b).astype(np.float32)))


# 224 and 192 columns of a [k, n] weight: the last rows and columns ragged
@pytest.mark.parametrize("k", [56, 72, 128, 320, 328])
@pytest.mark.parametrize("m_per_rank,n,block_n", [(2297, 440, 224), (505, 3000, 192)])
def test_narrow_256_row_tiles_of_a_kn_weight_are_bit_exact(B, m_per_rank, n, block_n, k):
    cfg = synth.CONFIGS[2].scaled(world=8, m_per_rank=m_per_rank, n=n, k=k, rank=6)
    st, tc = B.tile_config(4, cfg.m, n, k)
    assert (st, tc["block_m"], tc["block_n"]) == (B.OK, 256, block_n)
    shards, b = synth.ag_gemm_inputs(cfg, integer=True)
    run = AgGemmRun(B, 8, m_per_rank, n, k)
    sched = torch.full((4 * tc["ntiles"],), -1, dtype=torch.int32, device="cuda")
    _ok(B, run([to_dev(s) for s in shards], to_dev(b), cfg.rank, b_layout=B.B_KN, schedule=sched), run)
    assert np.array_equal(bits(run.c), formats.encode_bf16_rne(oag.ag_gemm(shards, b).astype(np.float32)))
    assert [tuple(r) for r in sched.cpu().view(-1, 4).tolist()] == [tuple(r) for r in B.schedule_dump(0, cfg.m, n, k, 8, 6, b_layout=B.B_KN)[1]]


# 128 x 64 tiles, GEMM-ReduceScatter (plain, fused), beside GEMM + AllReduce, which keeps its tiles: from the shortest contraction that takes them, whole
# and ragged last K tiles, at several places of the ring's nine pieces; ragged rows and columns, one tile and 64
@pytest.mark.parametrize("k", [1536, 1544, 1608, 1728])
@pytest.mark.parametrize("m_per_rank,n", [(8, 64), (15, 1000), (32, 4096)])
@pytest.mark.parametrize("kn", [False, True], ids=["b_nk", "b_kn"])
def test_64_column_tiles_reduce_bit_exact(B, m_per_rank, n, k, kn):
    world, d = 8, 3
    cfg = synth.CONFIGS[3].scaled(world=world, m_per_rank=m_per_rank, n=n, k=k)
    layout = B.B_KN if kn else B.B_NK
    for op, block_n in ((1, 64), (3, 128)):   # a two-shot all-reduce deals tiles to ranks: its tiling is fixed
        st, tc = B.tile_config(op, cfg.m, n, k)
        assert (st, tc["block_m"], tc["block_n"]) == (B.OK, 128, block_n)
    a_list, b_list = synth.gemm_rs_inputs(cfg, integer=True)
    parts = [oar.partial_bits(a, b) for a, b in zip(a_list, b_list)]
    full = oar.allreduce_partials_f32_ordered(parts)
    mine = slice(d * m_per_rank, (d + 1) * m_per_rank)
    a_dev, b_dev = to_dev(a_list[d]), to_dev(b_list[d] if kn else nk(b_list[d]))
    ar = GemmArRun(B, world, cfg.m, n, k)
    peers = [None if s == d else to_dev(parts[s]) for s in range(world)]
    st = B.gemm_ar(a_dev, b_dev, layout, ar.gemm_out, peers, ar.out, ar.signals, ar.status, None, cfg.m, n, k, world, d, 1,
                   B.EMULATE_PRODUCER)
    _ok(B, st, ar)
    assert np.array_equal(bits(ar.gemm_out), parts[d]) and np.array_equal(bits(ar.out), full)
    blocks = [None if s == d else to_dev(parts[s][mine]) for s in range(world)]
    signals = torch.zeros(B.signal_words(world, 1), dtype=torch.int32, device="cuda")
    zeros = lambda *shape: torch.zeros(shape, dtype=torch.int16, device="cuda")   # noqa: E731
    gemm_out, scatter, out, status = zeros(cfg.m, n), zeros(world, m_per_rank, n), zeros(m_per_rank, n), ar.status
    assert B.gemm_rs(a_dev, b_dev, layout, gemm_out, blocks, scatter, out, signals, status, None, None, cfg.m, n, k, world, d, 1, 1,
                     B.EMULATE_PRODUCER) == B.OK
    torch.cuda.synchronize()
    assert np.array_equal(bits(gemm_out), parts[d]) and np.array_equal(bits(out), full[mine])
    dsts = [zeros(world, m_per_rank, n) for _ in range(world)]
    assert B.gemm_rs_fuse_scatter(a_dev, b_dev, layout, dsts, blocks, out.fill_(0x7FC0), signals, status, None, None, cfg.m, n, k,
                                  world, d, 1, 2, B.EMULATE_PRODUCER) == B.OK
    torch.cuda.synchronize()
    assert status.cpu().tolist()[0] == 0
    assert np.array_equal(bits(out), full[mine])
    for r in range(world):
        assert np.array_equal(bits(dsts[r][d]), parts[d][r * m_per_rank:(r + 1) * m_per_rank])


# the shortest contractions that take 64 columns beside few and beside many tiles of 128, and the ones just below
@pytest.mark.parametrize("n,k,block_n", [(1000, 504, 128), (1000, 512, 64), (1000, 520, 64), (14272, 1016, 128), (14272, 1024, 64)])
@pytest.mark.parametrize("kn", [False, True], ids=["b_nk", "b_kn"])
def test_64_column_tiles_from_short_contractions_on(B, n, k, block_n, kn):
    world, d, m_r = 4, 2, 5
    st, tc = B.tile_config(1, world * m_r, n, k)
    assert (st, tc["block_m"], tc["block_n"]) == (B.OK, 128, block_n)
    cfg = synth.CONFIGS[3].scaled(world=world, m_per_rank=m_r, n=n, k=k)
    a_list, b_list = synth.gemm_rs_inputs(cfg, integer=True)
    parts = [oar.partial_bits(a, b) for a, b in zip(a_list, b_list)]
    mine = slice(d * m_r, (d + 1) * m_r)
    blocks = [None if s == d else to_dev(parts[s][mine]) for s in range(world)]
    rs = GemmRsRun(B, world, cfg.m, n, k, 5)
    _ok(B, rs(to_dev(a_list[d]), to_dev(b_list[d] if kn else nk(b_list[d])), blocks, d, b_layout=B.B_KN if kn else B.B_NK), rs)
    assert np.array_equal(bits(rs.gemm_out), parts[d]) and np.array_equal(bits(rs.out), oar.allreduce_partials_f32_ordered(parts)[mine])


# 255 tiles of 128 x 128 beside the peers' copies, both layouts of the weight: tiles that share a unit (a ring of two K tiles in
# five pieces); from less than a K tile on, whole and ragged last ones
@pytest.mark.parametrize("k", [8, 72, 128, 192, 200, 328, 512, 584, 1024, 1032, 1096])
@pytest.mark.parametrize("kn", [False, True], ids=["b_nk", "b_kn"])
def test_tiles_that_share_a_unit_reduce_bit_exact(B, k, kn):
    world, d, m_r, n = 8, 5, 240, 2056
    cfg = synth.CONFIGS[3].scaled(world=world, m_per_rank=m_r, n=n, k=k)
    st, tc = B.tile_config(1, cfg.m, n, k)
    assert (st, tc["block_m"], tc["block_n"], tc["ntiles"]) == (B.OK, 128, 128, 255)
    a_list, b_list = synth.gemm_rs_inputs(cfg, integer=True)
    parts = [oar.partial_bits(a, b) for a, b in zip(a_list, b_list)]
    mine = slice(d * m_r, (d + 1) * m_r)
    want = oar.allreduce_partials_f32_ordered(parts)[mine]
    blocks = [None if s == d else to_dev(parts[s][mine]) for s in range(world)]
    rs = GemmRsRun(B, world, cfg.m, n, k, 2)
    for _ in range(2):
        _ok(B, rs(to_dev(a_list[d]), to_dev(b_list[d] if kn else nk(b_list[d])), blocks, d, b_layout=B.B_KN if kn else B.B_NK), rs)
        assert np.array_equal(bits(rs.gemm_out), parts[d]) and np.array_equal(bits(rs.out), want)
        rs.gemm_out.zero_()


# the same tile under AllGather-GEMM of a [k, n] weight, where shorter contractions and up to 128 tiles of 128 columns take it
@pytest.mark.parametrize("k", [512, 520, 584, 640, 1160])
@pytest.mark.parametrize("m_per_rank,n", [(8, 64), (15, 1000), (128, 2048)])
def test_64_column_tiles_gather_bit_exact(B, m_per_rank, n, k):
    cfg = synth.CONFIGS[2].scaled(world=8, m_per_rank=m_per_rank, n=n, k=k, rank=3)
    st, tc = B.tile_config(4, cfg.m, n, k)
    assert (st, tc["block_m"], tc["block_n"]) == (B.OK, 128, 64)
    shards, b = synth.ag_gemm_inputs(cfg, integer=True)
    run = AgGemmRun(B, 8, m_per_rank, n, k)
    _ok(B, run([to_dev(s) for s in shards], to_dev(b), cfg.rank, b_layout=B.B_KN), run)
    assert np.array_equal(bits(run.c), formats.encode_bf16_rne(oag.ag_gemm(shards, b).astype(np.float32)))


# the edge between 128 x 128 and 256-row tiles below three quarters of a round of the latter: GEMM-ReduceScatter of these short
# contractions from 256 tiles of 128 x 128 on, AllGather-GEMM from 384 ([k, n]) and 513 ([n, k]); one to six K tiles; over one node and two; GEMM +
# AllReduce never
@pytest.mark.parametrize("m_per_rank,n,rows", [(240, 2056, (128, 128, 128)), (250, 2440, (256, 128, 128)), (249, 3000, (256, 256, 128)),
                                               (125, 8456, (256, 256, 256))])
@pytest.mark.parametrize("k", [64, 328])
def test_rounds_of_small_tiles_give_way_to_large_ones(B, m_per_rank, n, rows, k):
    world, d = 8, 2
    cfg = synth.CONFIGS[3].scaled(world=world, m_per_rank=m_per_rank, n=n, k=k)
    assert [B.tile_config(op, cfg.m, n, k)[1]["block_m"] for op in (1, 4, 0, 3)] == list(rows) + [128]
    a_list, b_list = synth.gemm_rs_inputs(cfg, integer=True)
    parts = [oar.partial_bits(a, b) for a, b in zip(a_list, b_list)]
    full = oar.allreduce_partials_f32_ordered(parts)
    mine = slice(d * m_per_rank, (d + 1) * m_per_rank)
    a_dev = to_dev(a_list[d])
    peers = [None if s == d else to_dev(parts[s]) for s in range(world)]
    blocks = [None if s == d else to_dev(parts[s][mine]) for s in range(world)]
    shards = [to_dev(a_list[d][r * m_per_rank:(r + 1) * m_per_rank]) for r in range(world)]
    for layout, b_dev in ((B.B_NK, to_dev(nk(b_list[d]))), (B.B_KN, to_dev(b_list[d]))):
        ar = GemmArRun(B, world, cfg.m, n, k)
        _ok(B, ar(a_dev, b_dev, peers, d, b_layout=layout), ar)
        assert np.array_equal(bits(ar.gemm_out), parts[d]) and np.array_equal(bits(ar.out), full)
        for nodes in (1, 2):
            rs = GemmRsRun(B, world, cfg.m, n, k, 1)
            _ok(B, rs(a_dev, b_dev, blocks, d, b_layout=layout, tuning=B.tuning(num_nodes=nodes)), rs)
            assert np.array_equal(bits(rs.gemm_out), parts[d]) and np.array_equal(bits(rs.out), full[mine])
            ag = AgGemmRun(B, world, m_per_rank, n, k)
            _ok(B, ag(shards, b_dev, d, b_layout=layout, tuning=B.tuning(num_nodes=nodes)), ag)
            assert np.array_equal(bits(ag.c), parts[d])


# Over several nodes the dumps write what the size query announces, where 256-row tiles take over from 128 x 128 ones.  1720
# rows as eight nodes of one rank: for rank 6 the listing is complete with tiles of 128 rows and not with 256, so that its
# tiles are visited in the one-node order
@pytest.mark.parametrize("nodes,d", [(2, 2), (8, 5), (8, 6)])
def test_dumps_over_several_nodes_fit_the_size_query(B, nodes, d):
    world, m_r, n, k = 8, 215, 4744, 72
    cfg = synth.CONFIGS[3].scaled(world=world, m_per_rank=m_r, n=n, k=k)
    a_list, b_list = synth.gemm_rs_inputs(cfg, integer=True)
    parts = [oar.partial_bits(a, b) for a, b in zip(a_list, b_list)]
    mine = slice(d * m_r, (d + 1) * m_r)
    want = oar.allreduce_partials_f32_ordered(parts)[mine]
    a_dev = to_dev(a_list[d])
    blocks = [None if s == d else to_dev(parts[s][mine]) for s in range(world)]
    shards = [to_dev(a_list[d][r * m_r:(r + 1) * m_r]) for r in range(world)]
    tuning = B.tuning(num_nodes=nodes)

    def records(query, dtype=B.BF16):
        st, tc = B.tile_config(query, cfg.m, n, k, dtype)
        assert st == B.OK and tc["block_m"] == 256
        assert sorted(B.tile_row_order(0, cfg.m, 128, world, nodes, d)[1]) == list(range(14))
        complete = sorted(B.tile_row_order(0, cfg.m, 256, world, nodes, d)[1]) == list(range(7))
        assert complete == ((nodes, d) != (8, 6))
        return torch.full((4 * tc["ntiles"] + 4 * 2048,), -1, dtype=torch.int32, device="cuda"), 4 * tc["ntiles"]

    def check_records(rec, words, op, layout, dtype=B.BF16):
        r = rec.cpu().tolist()
        assert set(r[words:]) == {-1}
        assert [tuple(r[i:i + 4]) for i in range(0, words, 4)] == B.schedule_dump(op, cfg.m, n, k, world, d, dtype, layout, tuning)[1]

    for layout, b_dev in ((B.B_NK, to_dev(nk(b_list[d]))), (B.B_KN, to_dev(b_list[d]))):
        rec, words = records(1)
        rs = GemmRsRun(B, world, cfg.m, n, k, 1)
        _ok(B, rs(a_dev, b_dev, blocks, d, b_layout=layout, schedule=rec, tuning=tuning), rs)
        assert np.array_equal(bits(rs.gemm_out), parts[d]) and np.array_equal(bits(rs.out), want)
        check_records(rec, words, 1, layout)
        rec, words = records(0 if layout == B.B_NK else 4)
        ag = AgGemmRun(B, world, m_r, n, k)
        _ok(B, ag(shards, b_dev, d, b_layout=layout, schedule=rec, tuning=tuning), ag)
        assert np.array_equal(bits(ag.c), parts[d])
        check_records(rec, words, 0, layout)
    # e4m3 of the same integers; then the time stamps, which go to the same places
    q = lambda x: synth.quantize_e4m3(formats.decode_bf16(x), 1.0)   # noqa: E731
    a8, b8 = q(a_list[d]), q(b_list[d])
    ag = AgGemmRun(B, world, m_r, n, 80, esize=1)
    pad = lambda x: np.concatenate([x, np.zeros((x.shape[0], 8), x.dtype)], axis=1)   # noqa: E731  (k a multiple of 16)
    sh8, b8 = [to_dev(pad(a8[r * m_r:(r + 1) * m_r])) for r in range(world)], to_dev(pad(nk(b8)))
    rec, words = records(0, B.FP8_E4M3)
    _ok(B, ag(sh8, b8, d, dtype=B.FP8_E4M3, schedule=rec, tuning=tuning), ag)
    assert np.array_equal(bits(ag.c), parts[d])
    check_records(rec, words, 0, B.B_NK, B.FP8_E4M3)
    rec.fill_(-1)
    ag.epoch += 1
    st = B.ag_gemm(sh8, b8, B.B_NK, ag.c, None, None, ag.ws_raw, ag.signals, ag.status, rec, None, m_r, n, 80, world, d, B.FP8_E4M3,
                   ag.epoch, B.EMULATE_PRODUCER | B.DUMP_TIMING, tuning=tuning)
    _ok(B, st, ag)
    r = rec.cpu().tolist()
    assert set(r[words:]) == {-1} and -1 not in r[:words]


# the grouped GEMM's 128-column block (ragged last block) with several K tiles, the last one ragged
@pytest.mark.parametrize("t_r,inter,experts", [(128, 264, 64), (128, 1400, 16), (256, 1544, 8)])
@pytest.mark.parametrize("hidden", [200, 456])
@pytest.mark.parametrize("kn", [False, True], ids=["w_nk", "w_kn"])
def test_moe_column_blocks_are_bit_exact(B, t_r, inter, experts, hidden, kn):
    cfg = synth.CONFIGS[4].scaled(world=8, tokens_per_rank=t_r, k=hidden, n=inter, num_experts=experts, top_k=2,
                                  num_local_experts=8, rank=0)
    xs, ids, w = synth.moe_inputs(cfg, integer=True)
    _run_and_check(B, cfg, xs, ids, w, 8 * t_r * 2, integer=True, kn=kn)


# every column block of the 128-row tiles at the lengths of its ring: less than a K tile, up to the four stages ([n, k], 192
# columns) or three K tiles it requests ahead, one more, two turns; whole and ragged last K tiles; the last block ragged
@pytest.mark.parametrize("hidden", [8, 72, 128, 192, 200, 256, 328, 520])
@pytest.mark.parametrize("inter,block_n", [(1528, 128), (1608, 192), (2312, 256)])
@pytest.mark.parametrize("kn", [False, True], ids=["w_nk", "w_kn"])
def test_moe_blocks_at_the_lengths_of_their_rings(B, inter, block_n, hidden, kn):
    cfg = synth.CONFIGS[4].scaled(world=8, tokens_per_rank=128, k=hidden, n=inter, num_experts=8, top_k=2, num_local_experts=8, rank=0)
    assert B.moe_tile_choice(1024, 2, 8, 8, inter) == (B.OK, 128, block_n)
    xs, ids, w = synth.moe_inputs(cfg, integer=True)
    _run_and_check(B, cfg, xs, ids, w, 2048, integer=True, kn=kn)


# many experts of a few rows: [k, n] weights take wider blocks than [n, k] ones (192 and 256 where those take 128), which changes
# nothing in the tile list
@pytest.mark.parametrize("inter,block_n", [(600, 128), (936, 128), (1160, 192)])
@pytest.mark.parametrize("kn", [False, True], ids=["w_nk", "w_kn"])
def test_moe_blocks_of_small_experts(B, inter, block_n, kn):
    cfg = synth.CONFIGS[4].scaled(world=8, tokens_per_rank=6, k=200, n=inter, num_experts=60, top_k=2, num_local_experts=60, rank=0)
    assert B.moe_tile_choice(48, 2, 60, 60, inter) == (B.OK, 128, block_n)
    xs, ids, w = synth.moe_inputs(cfg, integer=True)
    _run_and_check(B, cfg, xs, ids, w, 96, integer=True, kn=kn)


# large experts, [k, n] weights: 256-row tiles of 128 columns where they are one round, of 256 where they are not
@pytest.mark.parametrize("inter", [264, 1032])
@pytest.mark.parametrize("hidden", [72, 128, 328])
def test_moe_large_experts_of_kn_weights(B, inter, hidden):
    cfg = synth.CONFIGS[4].scaled(world=8, tokens_per_rank=512, k=hidden, n=inter, num_experts=8, top_k=2, num_local_experts=8, rank=0)
    assert B.moe_tile_choice(4096, 2, 8, 8, inter) == (B.OK, 256, 256)
    xs, ids, w = synth.moe_inputs(cfg, integer=True)
    _run_and_check(B, cfg, xs, ids, w, 8192, integer=True, block_m=256, kn=True)


# 2, 4 and 8 ranks: every one has its own number of vectors in flight; 5: the loop over any number of ranks.
# 264 columns: a last tile of one vector; 3080 x ~4040: 256-row tiles.  One-shot these sizes are summed by the tiles' own work-groups,
# two-shot by consumers
@pytest.mark.parametrize("world", [2, 4, 5, 8])
@pytest.mark.parametrize("rows,n,k", [(120, 264, 72), (1000, 1288, 64), (4040, 3080, 64)])
def test_all_reduce_consumer_by_rank_count(B, world, rows, n, k):
    cfg = synth.CONFIGS[3].scaled(world=world, m_per_rank=rows // world, n=n, k=k)
    a_list, b_list = synth.gemm_rs_inputs(cfg, integer=True)
    parts = [oar.partial_bits(a, b) for a, b in zip(a_list, b_list)]
    full = oar.allreduce_partials_f32_ordered(parts)
    d = world - 1
    peers = [None if s == d else to_dev(parts[s]) for s in range(world)]
    a_dev, b_dev = to_dev(a_list[d]), to_dev(nk(b_list[d]))
    run = GemmArRun(B, world, cfg.m, n, k)
    run.out.fill_(0x7FC0)
    _ok(B, run(a_dev, b_dev, peers, d), run)
    assert np.array_equal(bits(run.gemm_out), parts[d])
    assert np.array_equal(bits(run.out), full)
    # two-shot, both layouts of the weight: the own output is complete, and every peer's holds exactly the tiles this rank owns
    reduced = [None if s == d else to_dev(full) for s in range(world)]
    bm, bn = run.tc["block_m"], run.tc["block_n"]
    for layout, w_dev in ((B.B_NK, b_dev), (B.B_KN, to_dev(b_list[d]))):
        outs = [torch.full((cfg.m, n), 0x7FC0, dtype=torch.int16, device="cuda") for _ in range(world)]
        sched = torch.full((4 * run.ntiles,), -1, dtype=torch.int32, device="cuda")
        run.epoch += 1
        st = B.gemm_ar_two_shot(a_dev, w_dev, layout, run.gemm_out, peers, outs, reduced, run.signals, run.status, sched, cfg.m, n, k,
                                world, d, run.epoch, B.EMULATE_PRODUCER | B.DUMP_SCHEDULE)
        _ok(B, st, run)
        assert np.array_equal(bits(outs[d]), full)
        want = np.full((cfg.m, n), 0x7FC0, dtype=np.uint16)
        for q, (pm, pn, _, _) in enumerate(sched.cpu().view(-1, 4).tolist()):
            if oar.two_shot_owner(q, world) == d:
                blk = (slice(pm * bm, (pm + 1) * bm), slice(pn * bn, (pn + 1) * bn))
                want[blk] = full[blk]
        assert (want != 0x7FC0).any() == (run.ntiles > d) and not (full == 0x7FC0).any()   # position d is the rank's first tile
        for t in range(world):
            if t != d:
                assert np.array_equal(bits(outs[t]), want), (layout, t)


# Sums by the tiles' own work-groups: one vector per lane and less, two, four and eight of them, the last batch partly empty, a
# last tile of one vector; the queue with 512 tiles, with 272 and with 549
@pytest.mark.parametrize("world,m,n,d", [
    (2, 2, 8, 1), (3, 3, 136, 0), (8, 16, 264, 7), (8, 32, 128, 0), (4, 64, 392, 2), (5, 100, 256, 4), (8, 128, 1024, 5),
    (2, 1024, 8192, 0), (2, 2000, 2056, 1), (2, 1056, 7808, 1),
])
def test_all_reduce_sums_bit_exact(B, world, m, n, d):
    k = 72
    cfg = synth.CONFIGS[3].scaled(world=world, m_per_rank=m // world, n=n, k=k)
    a_list, b_list = synth.gemm_rs_inputs(cfg, integer=True)
    parts = [oar.partial_bits(a, b) for a, b in zip(a_list, b_list)]
    full = oar.allreduce_partials_f32_ordered(parts)
    peers = [None if s == d else to_dev(parts[s]) for s in range(world)]
    a_dev, b_dev = to_dev(a_list[d]), to_dev(nk(b_list[d]))
    ar = GemmArRun(B, world, cfg.m, n, k)
    for flags in (None, B.FLAGS_PRESET):
        ar.out.fill_(0x7FC0)
        _ok(B, ar(a_dev, b_dev, peers, d, flags=flags), ar)
        assert np.array_equal(bits(ar.gemm_out), parts[d]) and np.array_equal(bits(ar.out), full)


# Two rounds of tiles, both sides of each line of the choice between the tiles' own sums and consumers.  2 ranks, K 1200 (t_gemm = 3.02
# t_reduce, X = 64): 448 tiles leave room for the consumers, 456 do not, 513 are three rounds; K 1184 (2.98) is too short.  256-row tiles:
# K 1400 (3.52, X = 56) and 1384; 8 ranks, K 72 (memory-bound), 448 and 464 tiles
@pytest.mark.parametrize("world,m,n,k,block_m,own", [
    (2, 1024, 7168, 1200, 128, False), (2, 1024, 7176, 1200, 128, True), (2, 1032, 7296, 1200, 128, False), (2, 1024, 7176, 1184, 128, False),
    (2, 264, 59272, 1400, 256, True), (2, 264, 59272, 1384, 256, False),
    (8, 264, 57344, 72, 256, False), (8, 264, 59272, 72, 256, True),
])
def test_all_reduce_two_rounds(B, world, m, n, k, block_m, own):
    g = torch.Generator(device="cuda").manual_seed(n + k)
    d = world - 1
    # products and sums of small integers are exact in fp32; every rank's partial is rounded once, and so is their sum in rank order
    a = torch.randint(-3, 4, (m, k), device="cuda", generator=g).to(torch.bfloat16)
    b = torch.randint(-1, 2, (n, k), device="cuda", generator=g).to(torch.bfloat16)
    parts = [torch.randint(-200, 201, (m, n), device="cuda", generator=g).to(torch.bfloat16) for _ in range(world)]
    parts[d] = (a.float() @ b.float().t()).to(torch.bfloat16)
    want = parts[0].float()
    for part in parts[1:]:
        want = want + part.float()
    run = GemmArRun(B, world, m, n, k)
    assert run.tc["block_m"] == block_m
    sched = torch.full((4 * run.ntiles,), -1, dtype=torch.int32, device="cuda")
    peers = [None if s == d else parts[s].view(torch.int16) for s in range(world)]
    _ok(B, run(a.view(torch.int16), b.view(torch.int16), peers, d, schedule=sched), run)
    assert torch.equal(run.gemm_out.view(torch.bfloat16), parts[d]) and torch.equal(run.out.view(torch.bfloat16), want.to(torch.bfloat16))
    # consumers sit behind the first round of tiles; without them the tiles are numbered through
    assert (sched.view(-1, 4)[:, 2].cpu().tolist() == list(range(run.ntiles))) == own


# Rows 16 KiB apart (the tile engine) and 8 KiB (the decode kernel): the chiplets begin the contraction in eight places.  132 tiles
# of 128 x 128; decode tiles of 64 and of 16 rows, split and not.  Integer inputs: any order of the sum gives the same bits
@pytest.mark.parametrize("m_per_rank,n,k", [(64, 4224, 8192), (8, 200, 4096), (2, 72, 12288), (16, 8200, 4096)])
def test_contractions_begun_in_eight_places_are_bit_exact(B, m_per_rank, n, k):
    cfg = synth.CONFIGS[2].scaled(world=8, m_per_rank=m_per_rank, n=n, k=k, rank=3)
    shards, b = synth.ag_gemm_inputs(cfg, integer=True)
    run = AgGemmRun(B, 8, m_per_rank, n, k)
    st = run([to_dev(s) for s in shards], to_dev(nk(b)), cfg.rank)
    _ok(B, st, run)
    assert np.array_equal(bits(run.workspace), oag.gather(shards))
    assert np.array_equal(bits(run.c), formats.encode_bf16_rne(oag.ag_gemm(shards, b).astype(np.float32)))
