"""Routing and permutation at the edges of their launch shapes: one workgroup
(with or without the routing), histogram + scan-and-scatter for up to 256
local experts, and the separate launches past that (needs an MI355X)."""
import numpy as np
import pytest
import torch

import moe_inputs as mi
import paper_2606_26607_amd as moe
from tests.util import assert_close_rel, bf16_f64, dev_bf16, host_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    moe.lib()


@pytest.mark.parametrize("T,E,k,e0,El", [
    (100, 65, 4, 0, 65), (300, 256, 8, 0, 256), (2047, 300, 3, 30, 256),   # wide one-workgroup and two launches
    (2100, 128, 8, 0, 128), (5000, 256, 8, 0, 256), (9000, 250, 5, 3, 200),
    (40000, 257, 8, 0, 256), (70000, 128, 8, 0, 128),                      # 1024-pair chunks
    (3000, 257, 8, 0, 257), (300, 1024, 8, 0, 1024),                       # more than 256 local experts
    (150000, 256, 8, 0, 256)])                                             # counts past the two launches' bound
def test_permute_wide(oracle, T, E, k, e0, El):
    ids = mi.random_topk_ids(T, E, k, seed=T + El, hot=None if T > 20000 else e0 + El - 1)
    o = moe.permute(torch.from_numpy(ids).cuda(), E, e0, El)
    torch.cuda.synchronize()
    c, off, r2p, p2r = oracle.permute(ids, e0, El)
    np.testing.assert_array_equal(o["counts"].cpu().numpy(), c)
    np.testing.assert_array_equal(o["offsets"].cpu().numpy(), off)
    np.testing.assert_array_equal(o["row_to_pair"].cpu().numpy()[:len(r2p)], r2p)
    np.testing.assert_array_equal(o["pair_to_row"].cpu().numpy()[:T * k], p2r)


@pytest.mark.parametrize("T,H,E,k,e0,El", [
    (0, 64, 8, 2, 0, 8),                                # no tokens: nothing written
    (1, 8, 16, 16, 0, 16), (300, 8, 8, 2, 2, 2),        # one vector a row; tokens with no row here
    (77, 520, 32, 16, 5, 9), (50, 2040, 8, 3, 0, 8),    # last chunk partly filled; one vector below a whole one
    (33, 2056, 8, 2, 4, 4), (20000, 64, 8, 4, 0, 8),    # second chunk of one vector; several tokens a workgroup
    (1000, 4096, 8, 2, 7, 1), (5000, 264, 96, 5, 12, 12),  # by row: less than a row a token
    (70000, 8, 256, 8, 8, 31), (70000, 8, 256, 8, 8, 32),  # ... several rows a workgroup; one row a token
    (1281, 4096, 16, 8, 0, 16), (1280, 4096, 16, 8, 0, 16)])  # either side of the 80 MiB of cached stores
def test_gather(T, H, E, k, e0, El):
    """The gathered rows are the tokens' own, bit for bit; rows past the last one stay as they were."""
    x = torch.randint(-2 ** 15, 2 ** 15, (T, H), dtype=torch.int16, device="cuda").view(torch.bfloat16)
    ids = torch.from_numpy(mi.random_topk_ids(T, E, k, seed=T + H) if T else np.zeros((0, k), np.int32)).cuda()
    xp = torch.full((max(T * k, 4), H), -7, dtype=torch.int16, device="cuda")
    o = moe.permute(ids, E, e0, El, x=x, out={"x_perm": xp.view(torch.bfloat16)})
    n = int(o["offsets"][-1])
    assert n == int(((ids >= e0) & (ids < e0 + El)).sum())
    rows = o["row_to_pair"][:n].long() // k
    assert torch.equal(xp[:n], x.view(torch.int16)[rows])
    assert bool((xp[n:] == -7).all())


@pytest.mark.parametrize("T,E,k,layout,P", [
    (1, 8, 2, "replicated", 1), (64, 8, 2, "replicated", 1), (128, 16, 1, "ep", 2),   # routed in the workgroup
    (16, 64, 2, "ep", 2), (17, 32, 2, "replicated", 1), (5, 128, 2, "replicated", 1), (3, 256, 4, "replicated", 1),
    (33, 64, 1, "replicated", 1), (20, 128, 1, "replicated", 1), (18, 256, 1, "replicated", 1),
    (64, 256, 8, "ep", 8), (128, 128, 8, "replicated", 1),                            # ... in a launch of its own
    (500, 128, 8, "replicated", 1), (700, 200, 8, "replicated", 1),                   # with the histogram
    (300, 300, 8, "replicated", 1)])                                                  # the separate launches
def test_layer_equals_calls(oracle, T, E, k, layout, P):
    """The whole layer writes what the four calls write, and both what the oracle says."""
    cfg = mi.MoeConfig("prep", T=T, H=64, E=E, k=k, I=64, P=P, layout=layout, rank=P - 1, seed=T + E)
    inp = mi.make_inputs(cfg)
    layer = moe.MoeLayer(T, E, k, cfg.e0, dev_bf16(inp.w13), dev_bf16(inp.w2))
    x, lg = dev_bf16(inp.x), torch.from_numpy(inp.logits).cuda()
    got = []
    for fn in (layer.forward_calls, layer.forward):
        for t in (layer.topk_ids, layer.topk_w, layer.y, layer.out, *layer.bufs.values()):
            t.view(torch.uint8).fill_(0xA5)
        fn(x, lg)
        torch.cuda.synchronize()
        n = int(layer.bufs["offsets"][-1])
        b = {name: t.cpu().numpy() for name, t in layer.bufs.items()}
        got.append([layer.topk_ids.cpu().numpy(), layer.topk_w.cpu().numpy().view(np.uint32), b["counts"],
                    b["offsets"], b["row_to_pair"][:n], b["pair_to_row"][:T * k], host_bf16(layer.y)[:n],
                    host_bf16(layer.out)])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    ids, _ = oracle.route(inp.logits, k)
    np.testing.assert_array_equal(got[1][0], ids)
    np.testing.assert_array_equal(got[1][5], oracle.permute(ids, cfg.e0, cfg.E_l)[3])
    assert_close_rel(bf16_f64(got[1][7]), oracle.layer(inp), what=f"T={T} E={E}")
