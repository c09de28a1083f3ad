"""The attention kernels at the edges of their row blocks, position steps and
position ranges, every stage per element against the oracle (the bounds of
test_gpu_attn.check_block).

The rows of one key/value head are the (token, query head of its group)
pairs: up to 16 rows and 1024 positions take score_kernel, otherwise
flash_kernel in blocks of 64 (up to 64 rows) or 128 rows and steps of 64
positions, in one or several ranges."""
import pytest

import paper_2506_23635_amd as moe
from test_gpu_attn import TINY, Case, check_block, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,G,hd,T,pos0", [
    (16, 2, 64, 2, 1022),      # 16 rows, 1024 positions: the last of score_kernel
    (16, 2, 64, 2, 1023),      # 1025 positions: flash_kernel, the last step one position
    (8, 4, 128, 9, 0),         # 18 rows, one step, one range
    (16, 2, 64, 4, 60),        # 32 rows, positions across a step
    (12, 2, 128, 11, 1500),    # 66 rows: the first size of 128-row blocks
    (16, 2, 64, 8, 2000),      # 64 rows, as many ranges as steps
    (16, 2, 128, 16, 3000),    # 128 rows, the most of the decode path
    (4, 4, 64, 33, 63),        # prefill, one head per group: rows are tokens
    (4, 4, 64, 65, 2000),      # 65 rows: a second wave with one row
    (8, 1, 128, 17, 3500),     # 136 rows over one key/value head: two blocks, many ranges
    (8, 1, 128, 48, 1000),     # 384 rows: whole blocks
])
def test_row_and_range_edges(torch_mod, H, G, hd, T, pos0):  # noqa: F811
    wl = TINY.with_(d=512, n_heads=H, n_kv=G, hd=hd, T=T, pos0=pos0, max_seq=4096)
    case = Case(torch_mod, wl, max_tokens=max(T, 16))
    try:
        x = wl.x()
        y = case.forward(x, pos0)
        kc, vc = case.cache()
        check_block(case, x, pos0, y, case.layer.intermediates(T), kc, vc)
        assert (case.forward(x, pos0) == y).all()
    finally:
        case.close()


# the decode projections take one or two row tiles per workgroup (q|k|v: (H +
# 2G) hd / 16 tiles over d; output: d / 16 tiles over H hd), in batches of 32 K
# tiles of 32 and a shorter one: two from K 2048 (more than 8 tokens: 1024) and
# 384 tiles on, but not between 512 and 1024 tiles, and at K 4096 only below 512
# tiles and for more than 8 tokens
@pytest.mark.parametrize("d,H,G,hd,T,pos0", [
    (512, 60, 15, 64, 16, 0),      # q|k|v 360 tiles: one per workgroup
    (512, 32, 8, 128, 16, 70),     # 384 tiles, half a batch of K: one
    (1280, 32, 8, 128, 5, 1500),   # one batch and a remainder: one; output K 4096
    (6144, 36, 6, 64, 9, 30),      # output 384 tiles, two batches and a remainder: two
    (6144, 4, 4, 64, 1, 3),        # one token: output 384 tiles, less than a batch: one
    (256, 32, 8, 128, 5, 5),       # a remainder of one K tile per wave only
    (1024, 32, 8, 128, 9, 7),      # one batch, nine tokens: two
    (1280, 32, 8, 128, 16, 20),    # ... and a remainder, heads of both halves
    (2304, 48, 8, 128, 5, 30),     # 512 tiles, two batches and a remainder: two
    (2816, 64, 8, 128, 16, 4),     # 640 tiles, a remainder of three: one
    (2048, 64, 32, 128, 7, 9),     # 1024 tiles: two
    (4096, 32, 8, 128, 8, 40),     # K 4096: one
    (4096, 32, 8, 128, 9, 40),     # ... and two
])
def test_projection_tile_pairs(torch_mod, d, H, G, hd, T, pos0):  # noqa: F811
    wl = TINY.with_(d=d, n_heads=H, n_kv=G, hd=hd, T=T, pos0=pos0, max_seq=2048)
    case = Case(torch_mod, wl, max_tokens=16)
    try:
        x = wl.x()
        y = case.forward(x, pos0)
        kc, vc = case.cache()
        check_block(case, x, pos0, y, case.layer.intermediates(T), kc, vc)
        assert (case.forward(x, pos0) == y).all()
    finally:
        case.close()


# several ranges of several steps: at most 1024 workgroups and 128 ranges, so
# these positions leave every range three steps or more, and unevenly many
@pytest.mark.parametrize("H,G,hd,T,pos0", [
    (8, 1, 128, 8, 25000),     # 64 rows: two position groups; at most 128 ranges of 391 steps
    (8, 1, 128, 16, 25000),    # 128 rows: one
    (32, 16, 64, 16, 12600),   # 32 rows; at most 64 ranges of 198 steps
    (96, 16, 64, 16, 12600),   # 96 rows
])
def test_ranges_of_several_steps(torch_mod, H, G, hd, T, pos0):  # noqa: F811
    wl = TINY.with_(d=256, n_heads=H, n_kv=G, hd=hd, T=T, pos0=pos0, max_seq=pos0 + T + 7)
    case = Case(torch_mod, wl, max_tokens=16)
    try:
        x = wl.x()
        moe.attn_profile_enable(case.layer.ctx, 16)
        y = case.forward(x, pos0)
        launches = {k: n for k, (_, n) in moe.attn_profile_read(case.layer.ctx)[0].items()}
        assert launches["combine"] == 1            # several ranges, merged
        moe.attn_profile_enable(case.layer.ctx, 0)
        kc, vc = case.cache()
        check_block(case, x, pos0, y, case.layer.intermediates(T), kc, vc)
        assert (case.forward(x, pos0) == y).all()
    finally:
        case.close()


# the prefill projections on 256 x 256 tiles (from 129 tiles on: 32 feature
# tiles, five token tiles) with a partial last token tile: of one 32-row block,
# of up to 128 rows, and of more
@pytest.mark.parametrize("T", [1044, 1124, 1244])
@pytest.mark.parametrize("d,H,G", [(256, 64, 32), (8192, 4, 4)])   # q|k|v; output
def test_projection_tile_tails(torch_mod, d, H, G, T):  # noqa: F811
    wl = TINY.with_(d=d, n_heads=H, n_kv=G, hd=64, T=T, pos0=3, max_seq=T + 8)
    case = Case(torch_mod, wl, max_tokens=T)
    try:
        x = wl.x()
        moe.attn_profile_enable(case.layer.ctx, 16)
        y = case.forward(x, 3)
        launches = {k: n for k, (_, n) in moe.attn_profile_read(case.layer.ctx)[0].items()}
        assert launches["rope" if d == 256 else "residual"] == 0   # the end is the projection's own
        moe.attn_profile_enable(case.layer.ctx, 0)
        kc, vc = case.cache()
        check_block(case, x, 3, y, case.layer.intermediates(T), kc, vc)
    finally:
        case.close()
