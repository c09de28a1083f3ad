"""The grouped GEMM's two tile sizes (128 x 128 for few rows per expert or few
tiles, 256 x 256 otherwise) at the edges of their token blocks and tiles, with
the experts' loads forced through given logits.

Every element is checked against the oracle with check_chain's bounds; a
recorded timeline runs the same call on the 256 x 256 tiles, whose sums have
the same order, so H, O and y are the same bits.  ffn 128, 384 and 640 give
the down projection 2, 6 and 10 stages of 64 K (whole rounds of four and
remainders), d 256 and 768 the gate/up projection 4 and 12."""
import numpy as np
import pytest

import moe_inputs as mi
import oracle
import paper_2506_23635_amd as moe
from harness import (check_chain, host_experts, load_workload_host, make_layer, read_intermediates,
                     to_np_u16, x_device)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("d,f,loads", [(256, 128, (1, 0, 16)), (256, 384, (31, 33, 0)),
                                       (768, 128, (0, 32, 64)), (256, 640, (65, 96, 97)),
                                       (768, 384, (127, 128, 129)), (256, 384, (0, 255, 257)),
                                       (256, 128, (513, 1, 300))])
def test_loads_at_tile_edges(torch_mod, d, f, loads):
    torch = torch_mod
    wl = mi.WORKLOADS["tiny"].with_(T=sum(loads), d=d, f=f, E=3, k=1, sigma_w=0.05)
    layer = make_layer(wl)
    load_workload_host(layer, wl)
    x_t, x = x_device(wl)
    # token t goes to its expert by a large logit, the experts in a shuffled order
    expert = np.random.default_rng(1).permutation(np.repeat(np.arange(3), loads))
    lg = np.zeros((wl.T, 3), np.float32)
    lg[np.arange(wl.T), expert] = 4.0
    lg_t = torch.from_numpy(lg).cuda()
    outs = []
    for timeline in (False, True):
        buf = torch.zeros(8, dtype=torch.int64, device="cuda")
        moe.moe_profile_gemm_timeline(layer.ctx, buf.data_ptr() if timeline else None, None,
                                      1 if timeline else 0)
        rt_c = layer.route(0, x_t, logits_in=lg_t)
        y = torch.full((wl.T, d), 0x3F80, dtype=torch.int16, device="cuda")
        layer.forward(0, x_t, y, routing=rt_c)
        rt = layer.routing_tensors(rt_c)
        assert tuple(rt["counts"]) == loads
        outs.append((to_np_u16(y),) + read_intermediates(torch, layer, wl.T))
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    y, H, O = outs[0]
    idx, w = oracle.route_from_logits(lg, 1)
    G, U, D = host_experts(wl, range(3))
    y64, y16, hb = oracle.layer_with_routing_ex(x, idx, w, G, U, D, want_hb=True)
    check_chain(x, rt, H, O, y, {"y64": y64, "y16": y16, "hb": hb, "w": w},
                lambda e: (G[e], U[e], D[e]))
    layer.close()


@pytest.mark.parametrize("d,f,loads", [(256, 640, (300, 0, 2600, 257)),      # 5 and 1 feature tiles
                                       (768, 1152, (1, 700, 256, 1024)),     # 9 and 3
                                       (2816, 1408, (513, 40, 255, 300))])   # 11 and 11
def test_tiles_are_dealt_evenly_over_the_xcds(torch_mod, d, f, loads):
    """Whatever the number of feature tiles, every tile is taken once and the
    XCDs (block b runs on XCD b % 8) get the same number of them, one more or
    less."""
    torch = torch_mod
    n_exp = len(loads)
    wl = mi.WORKLOADS["tiny"].with_(T=sum(loads), d=d, f=f, E=n_exp, k=1, sigma_w=0.05)
    layer = make_layer(wl)
    load_workload_host(layer, wl)
    x_t, _ = x_device(wl)
    lg = np.zeros((wl.T, n_exp), np.float32)
    lg[np.arange(wl.T), np.repeat(np.arange(n_exp), loads)] = 4.0
    n = 1024
    bufs = [torch.zeros(n * 8, dtype=torch.int64, device="cuda") for _ in range(2)]
    moe.moe_profile_gemm_timeline(layer.ctx, bufs[0].data_ptr(), bufs[1].data_ptr(), n)
    rt = layer.route(0, x_t, logits_in=torch.from_numpy(lg).cuda())
    layer.forward(0, x_t, torch.empty((wl.T, d), dtype=torch.int16, device="cuda"), routing=rt)
    torch.cuda.synchronize()
    token_tiles = sum((c + 255) // 256 for c in loads)
    for buf, n_ft in ((bufs[0], 2 * f // 256), (bufs[1], d // 256)):
        t = buf.cpu().numpy().view(np.uint64).reshape(n, 8)
        live = t[:, 1] > 0
        what = t[live, 5]
        assert len(what) == len(np.unique(what)) == token_tiles * n_ft
        for e, c in enumerate(loads):
            mine = what[what >> 48 == e]
            assert int(((mine >> 32) & 0xFFFF).sum()) == c * n_ft
        per_xcd = np.bincount(np.nonzero(live)[0] % 8, minlength=8)
        assert per_xcd.max() - per_xcd.min() <= 1, per_xcd
    layer.close()


def test_timeline_token_tiles_count_over_the_experts(torch_mod):
    """The recorded token tile is its index among all local experts' tiles."""
    torch = torch_mod
    d, f, loads = 256, 128, (300, 0, 600, 5)
    wl = mi.WORKLOADS["tiny"].with_(T=sum(loads), d=d, f=f, E=4, k=1, sigma_w=0.05)
    layer = make_layer(wl)
    load_workload_host(layer, wl)
    x_t, _ = x_device(wl)
    lg = np.zeros((wl.T, 4), np.float32)
    lg[np.arange(wl.T), np.repeat(np.arange(4), loads)] = 4.0
    buf = torch.zeros(64 * 8, dtype=torch.int64, device="cuda")
    moe.moe_profile_gemm_timeline(layer.ctx, None, buf.data_ptr(), 64)
    rt = layer.route(0, x_t, logits_in=torch.from_numpy(lg).cuda())
    layer.forward(0, x_t, torch.empty((wl.T, d), dtype=torch.int16, device="cuda"), routing=rt)
    torch.cuda.synchronize()
    t = buf.cpu().numpy().view(np.uint64).reshape(64, 8)
    got = sorted((int(v >> 16) & 0xFFFF, int(v >> 48), int(v >> 32) & 0xFFFF) for v in t[t[:, 1] > 0, 5])
    assert got == [(0, 0, 256), (1, 0, 44), (2, 2, 256), (3, 2, 256), (4, 2, 88), (5, 3, 5)]
    layer.close()
