"""Decode-shaped AllGather-GEMM: the tile is cut to the rows there are, whatever the split of the contraction."""
import pytest
import torch

from gpu_util import AgGemmRun

pytestmark = pytest.mark.gpu


def _host_plan(B, m, n, k, dtype):
    st, tc = B.tile_config(0, m, n, k, dtype)
    assert st == B.OK
    return tc["block_m"], tc["block_n"], tc["splits"]


# rows on both sides of every tile height; contractions of one split (less than a 128-byte K tile), two and eight, whole and ragged; one
# ragged column block and several
@pytest.mark.parametrize("world,m_per_rank", [(1, 1), (2, 8), (1, 17), (8, 4), (3, 11), (8, 8), (5, 13)])
@pytest.mark.parametrize("n,k", [(8, 48), (72, 1040), (200, 8192), (1000, 4112)])
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
def test_decode_tiles_are_exact(world, m_per_rank, n, k, fp8):
    from paper_2605_02953_amd import binding as B
    m = world * m_per_rank
    dtype = B.FP8_E4M3 if fp8 else B.BF16
    block_m, block_n, _ = _host_plan(B, m, n, k, dtype)
    assert block_m == (16 if m <= 16 else 32 if m <= 32 else 64 if m <= 64 else 128)
    # 128 x 128 tiles: few of them here, so as many splits as the K tiles (128 bytes each, at least four to a split) allow
    kt = -(-k * (1 if fp8 else 2) // 128)
    assert block_n == (64 if m <= 64 or kt >= 32 else 128)
    g = torch.Generator(device="cuda").manual_seed(m * 10000 + k)
    kind = torch.float8_e4m3fn if fp8 else torch.bfloat16
    store = torch.uint8 if fp8 else torch.int16
    # sums of small integers are exact in fp32, and so is a power of two as a scale
    shards = [torch.randint(-2, 3, (m_per_rank, k), device="cuda", generator=g).to(kind) for _ in range(world)]
    b = torch.randint(-2, 3, (n, k), device="cuda", generator=g).to(kind)
    rows = torch.cat(shards).float() @ b.float().T
    run = AgGemmRun(B, world, m_per_rank, n, k, esize=1 if fp8 else 2)
    a_scales = b_scales = None
    if fp8:
        a_scales = 2.0 ** torch.randint(-2, 3, (world,), device="cuda", generator=g).float()
        b_scales = 2.0 ** torch.randint(-2, 3, (n,), device="cuda", generator=g).float()
        rows = rows * a_scales.repeat_interleave(m_per_rank)[:, None] * b_scales
    for call in range(3):   # the exchanged partials of an earlier call must not be taken for this one's
        run.c.fill_(0x7FC0)
        st = run([s.view(store) for s in shards], b.view(store), (call * 3) % world, dtype=dtype, a_scales=a_scales, b_scales=b_scales)
        assert st == B.OK, B.status_string(st)
        torch.cuda.synchronize()
        assert run.status.cpu().tolist()[0] == 0
        assert torch.equal(run.c.view(torch.bfloat16), rows.to(torch.bfloat16))
        assert torch.equal(run.workspace.view(store), torch.cat(shards).view(store))


def test_narrow_tiles_where_eight_splits_would_meet():
    from paper_2605_02953_amd import binding as B
    assert _host_plan(B, 128, 3584, 8192, B.FP8_E4M3) == (128, 64, 4) and _host_plan(B, 128, 8192, 8192, B.FP8_E4M3) == (128, 128, 4)
    st, tc = B.tile_config(0, 64, 3584, 8192, B.BF16, B.tuning(decode_variant=2))     # asked for by name: as it was
    assert st == B.OK and (tc["block_m"], tc["block_n"], tc["splits"]) == (128, 128, 8)
