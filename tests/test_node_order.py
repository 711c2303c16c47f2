"""The multi-node tile-row order of the library (host evaluation of the function the kernels use)
against the oracle's restatement of the paper's two swizzle listings.  No GPU needed."""
import os

import pytest

from oracle import schedule as S


@pytest.fixture(scope="module")
def B():
    from paper_2605_02953_amd import binding
    return binding


def _rows(name):
    path = os.path.join(os.path.dirname(__file__), "golden", name)
    return [ln.split() for ln in open(path) if ln.strip() and not ln.startswith("#")]


CASES = [(8, 1, 1024, 256), (16, 2, 1024, 256), (8, 2, 997, 256), (16, 2, 997, 256), (32, 4, 997, 256),
         (8, 4, 100, 64), (16, 4, 1000, 128), (8, 2, 16, 128), (32, 8, 300, 256), (12, 3, 77, 32)]


@pytest.mark.parametrize("world,nnodes,m_r,bm", CASES)
def test_library_order_equals_oracle(B, world, nnodes, m_r, bm):
    m = world * m_r
    npm = S.cdiv(m, bm)
    for rank in range(world):
        st, got = B.tile_row_order(0, m, bm, world, nnodes, rank)
        assert st == B.OK
        assert got == [S.ag_swizzle_multinode(t, m, rank, world, nnodes, bm) for t in range(npm)]
        st, got = B.tile_row_order(1, m, bm, world, nnodes, rank)
        assert st == B.OK
        assert got == [S.rs_swizzle_multinode(t, m, rank, world, nnodes, bm) for t in range(npm)]


def test_paper_nonperfect_example_is_visited_once(B):
    # the shapes of the paper's non-perfect tiling example (997 rows per rank; 8, 16, 32 GPUs)
    for world, nnodes, m_r, bm in [tuple(map(int, r)) for r in _rows("nonperfect_tiling_example.txt")]:
        m = world * m_r
        for rank in range(world):
            for op in (0, 1):
                st, got = B.tile_row_order(op, m, bm, world, nnodes, rank)
                assert st == B.OK and sorted(got) == list(range(S.cdiv(m, bm)))


def test_one_node_is_the_plain_rotation(B):
    world, m_r, bm = 8, 505, 256
    m = world * m_r
    npm = S.cdiv(m, bm)
    for rank in range(world):
        assert B.tile_row_order(0, m, bm, world, 1, rank)[1] == [(t + S.cdiv(rank * m_r, bm)) % npm for t in range(npm)]
        assert B.tile_row_order(1, m, bm, world, 1, rank)[1] == [(t + ((rank + 1) * m_r) // bm) % npm for t in range(npm)]


def test_argument_checks(B):
    assert B.tile_row_order(2, 1024, 256, 8, 2, 0)[0] == B.ERR_INVALID_ARG       # unknown order
    assert B.tile_row_order(0, 1024, 256, 8, 3, 0)[0] == B.ERR_INVALID_ARG       # world not a multiple of nnodes
    assert B.tile_row_order(0, 1000, 256, 8, 2, 8)[0] == B.ERR_INVALID_ARG       # rank out of range
    assert B.tile_row_order(0, 1001, 256, 8, 2, 0)[0] == B.ERR_INVALID_ARG       # rows not a multiple of world


# (operator, m_per_rank, n) with world 8, on both sides of every line of the
# tile rule: 256 / 300 / 383 / 512 tiles of 128 x 128, 192 of 256 x 256, and far between them
TILINGS = [(op, m_r, n) for op in ("ag_nk", "ag_kn", "ag_fp8", "rs_nk", "rs_kn")
           for m_r, n in [(16, 512), (128, 4096), (128, 4104), (250, 2048), (250, 2056), (250, 2432), (250, 2440), (249, 3000), (319, 3992), (325, 3472),
                          (119, 11632), (125, 8456), (606, 2336), (505, 3080), (70, 16200), (130, 9736), (33, 16384), (1024, 3584)]]


@pytest.mark.parametrize("nnodes", [1, 2, 4, 8])
def test_the_size_query_holds_for_any_number_of_nodes(B, nnodes):
    """A schedule or timing dump writes one record per work-group into a buffer sized with tile_config, which is not told how
    many nodes there are: tile shape and count must be those of the launch whatever the number of nodes."""
    world, k = 8, 2048
    for kind, m_r, n in TILINGS:
        op, query, dtype, layout = {"ag_nk": (0, 0, B.BF16, B.B_NK), "ag_kn": (0, 4, B.BF16, B.B_KN), "ag_fp8": (0, 0, B.FP8_E4M3, B.B_NK),
                                    "rs_nk": (1, 1, B.BF16, B.B_NK), "rs_kn": (1, 1, B.BF16, B.B_KN)}[kind]
        m = world * m_r
        st, tc = B.tile_config(query, m, n, k, dtype)
        assert st == B.OK
        served = 0
        for rank in range(world):
            st, got = B.schedule_dump(op, m, n, k, world, rank, dtype, layout, B.tuning(num_nodes=nnodes))
            if st == B.ERR_UNSUPPORTED:
                continue
            served += 1
            assert st == B.OK and len(got) == tc["ntiles"] * tc["splits"], (kind, m_r, n, rank)
            # every tile once (its splits after one another), the shards or segments of its rows beside it
            assert sorted({g[:2] for g in got}) == [(i, j) for i in range(S.cdiv(m, tc["block_m"])) for j in range(S.cdiv(n, tc["block_n"]))]
            assert all(g[2:] == (g[0] * tc["block_m"] // m_r, (min((g[0] + 1) * tc["block_m"], m) - 1) // m_r) for g in got)
        assert served or nnodes > 1


# (world, nodes, m_per_rank, n): 256-row tiles whose listing is incomplete for some ranks although the one of 128 rows is
# complete (the first three), incomplete for some ranks at 128 rows, complete everywhere
@pytest.mark.parametrize("world,nnodes,m_r,n", [(8, 4, 70, 16200), (8, 8, 130, 9736), (32, 8, 17, 23568), (8, 4, 37, 16384), (8, 2, 1024, 3584)])
def test_which_shapes_several_nodes_are_served_for(B, world, nnodes, m_r, n):
    """fp8 calls are served where the 128-row listing visits every tile row once, also where they take 256-row tiles; bf16
    calls where the listing at their rule's rows does (256 from 192 tiles of 256 x 256 on)."""
    m, tuning = world * m_r, B.tuning(num_nodes=nnodes)
    large = S.cdiv(m, 256) * S.cdiv(n, 256) >= 192
    for rank in range(world):
        complete = lambda op, bm: sorted(B.tile_row_order(op, m, bm, world, nnodes, rank)[1]) == list(range(S.cdiv(m, bm)))   # noqa: E731
        for op, dtype, layout, bm in ((0, B.FP8_E4M3, B.B_NK, 128), (0, B.BF16, B.B_KN, 256 if large else 128), (1, B.BF16, B.B_NK, 256 if large else 128)):
            st, got = B.schedule_dump(op, m, n, 2048, world, rank, dtype, layout, tuning)
            assert st == (B.OK if complete(op, bm) else B.ERR_UNSUPPORTED), (rank, op, dtype)
