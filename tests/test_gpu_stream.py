"""The streaming expert FFN (few rows per expert; needs an MI355X) at the
edges of its row blocks, weight strips and K splits, against the CPU oracle."""
import numpy as np
import pytest
import torch

import moe_inputs as mi
import paper_2606_26607_amd as moe
from tests.util import assert_close_rel, bf16_f64, dev_bf16, host_bf16, ffn_route

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    moe.lib()


# rows per expert; at most 64 rows in all, or (with gathered rows of at most 64 tokens) experts of more
ONE = [1]
B16 = [16, 0, 15, 17, 1]
B64 = [64]
B33 = [33, 31]
MORE = [65, 130, 0, 20, 48]    # passes of 64, 32 and 16 rows, at different points in different waves


@pytest.mark.parametrize("rows,gather,H,Is", [
    (ONE, False, 8, 8),             # one chunk of one slice
    (ONE, True, 4096, 2048),        # K split four ways
    (B16, False, 64, 24),           # one whole slice; a strip past the columns
    (B16, True, 136, 200),          # partial slices, one strip of columns short
    (B16, False, 256, 512),         # K split two ways
    (B64, False, 1000, 328), (B64, False, 2056, 40),
    (B33, True, 768, 1536), (B33, False, 72, 1032),
    (MORE, True, 256, 512), (MORE, True, 200, 120), (MORE, True, 1024, 4096),
])
def test_stream_edges(oracle, rows, gather, H, Is):
    El, k, n = len(rows), 3, sum(rows)
    offs = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    T = 64 if gather else n
    x = mi.random_bf16((T, H), seed=H + Is, tag=80)
    w13 = mi.random_bf16((El, 2 * Is, H), seed=H, tag=81, std=0.05)
    w2 = mi.random_bf16((El, H, Is), seed=H, tag=82, std=0.05)
    r2p = np.random.default_rng(H + n).integers(0, T * k, n).astype(np.int32) if gather else None
    want = oracle.grouped_ffn(x if r2p is None else x[r2p // k], offs, w13, w2)
    runs = []
    for _ in range(2):
        y = torch.full((n + 1, H), 7.0, dtype=torch.bfloat16, device="cuda")
        assert "streaming" == ffn_route(lambda: moe.grouped_ffn(
            dev_bf16(x), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2), y=y, cap_rows=n,
            row_to_pair=None if r2p is None else torch.from_numpy(r2p).cuda(), k=k if gather else 1))
        runs.append(host_bf16(y))
    np.testing.assert_array_equal(runs[0], runs[1])
    assert np.all(bf16_f64(runs[0])[n] == 7.0)  # nothing past the rows
    assert_close_rel(bf16_f64(runs[0])[:n], want, what=f"rows={rows} H={H} Is={Is}")


@pytest.mark.parametrize("T,k,tiles", [(5, 4, False), (40, 4, False), (64, 4, False), (128, 4, True), (400, 2, False)])
def test_stream_shared_and_non_temporal(oracle, T, k, tiles):
    """Weights of more than 64 MiB (loaded with the non-temporal hint), a shared expert beside the routed ones, and
    every row-block width; the last through the mid kernel."""
    El, E, H, Is = 8, 16, 2048, 1088
    ids = mi.random_topk_ids(T, E, k, seed=T)
    _, offs, r2p, _ = oracle.permute(ids, 4, El)
    n, sb, sc = int(offs[-1]), T // 3, T // 2
    x = mi.random_bf16((T, H), seed=T, tag=83)
    w13 = mi.random_bf16((El, 2 * Is, H), seed=1, tag=84, std=0.03)
    w2 = mi.random_bf16((El, H, Is), seed=1, tag=85, std=0.03)
    sw13 = mi.random_bf16((2 * Is, H), seed=1, tag=86, std=0.03)
    sw2 = mi.random_bf16((H, Is), seed=1, tag=87, std=0.03)
    cap = T * k
    full = torch.full((cap,), -1, dtype=torch.int32)
    full[:n] = torch.from_numpy(r2p)
    args = (dev_bf16(x), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2), full.cuda(), k, cap, sb, sc,
            dev_bf16(sw13), dev_bf16(sw2))
    assert ffn_route(lambda: moe.grouped_ffn_shared(*args)) == ("tiled" if tiles else "streaming")
    y, sy = moe.grouped_ffn_shared(*args)
    torch.cuda.synchronize()
    assert_close_rel(bf16_f64(host_bf16(y))[:n], oracle.grouped_ffn(x[r2p // k], offs, w13, w2), what="routed")
    assert_close_rel(bf16_f64(host_bf16(sy))[:sc],
                     oracle.grouped_ffn(x[sb:sb + sc], np.array([0, sc], np.int32), sw13[None], sw2[None]),
                     what="shared")


# rows per expert whose mean takes the mid kernel: runs of 128, 64 and 32 rows, and experts of several runs
MID = [128, 65, 0, 64, 200, 33, 1, 130]


@pytest.mark.parametrize("rows,gather,H,Is", [
    (MID, False, 128, 128), (MID, False, 448, 320), (MID, False, 1024, 192),  # (streaming)
    (MID, True, 128, 2752), (MID, True, 2752, 128),  # two whole slices: fewer than the loads kept in flight
    (MID, True, 1024, 448),
    (MID, False, 200, 72), (MID, False, 56, 264),    # partial last slices; strips past the columns
    (MID, True, 1000, 328),
    ([900, 70, 130, 20], False, 136, 200),
])
def test_mid_edges(oracle, rows, gather, H, Is):
    El, k, n = len(rows), 2, sum(rows)
    offs = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    # (gathered whole-slice widths: the mean of a top-2 layer is 100)
    T = n if not gather else 400 if H % 64 == 0 and Is % 64 == 0 else 700
    x = mi.random_bf16((T, H), seed=H + Is, tag=90)
    w13 = mi.random_bf16((El, 2 * Is, H), seed=H, tag=91, std=0.05)
    w2 = mi.random_bf16((El, H, Is), seed=H, tag=92, std=0.05)
    r2p = np.random.default_rng(H + n).integers(0, T * k, n).astype(np.int32) if gather else None
    want = oracle.grouped_ffn(x if r2p is None else x[r2p // k], offs, w13, w2)
    runs = []
    for _ in range(2):
        y = torch.full((n + 1, H), 7.0, dtype=torch.bfloat16, device="cuda")
        assert "streaming" == ffn_route(lambda: moe.grouped_ffn(
            dev_bf16(x), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2), y=y, cap_rows=n,
            row_to_pair=None if r2p is None else torch.from_numpy(r2p).cuda(), k=k if gather else 1))
        runs.append(host_bf16(y))
    np.testing.assert_array_equal(runs[0], runs[1])
    assert np.all(bf16_f64(runs[0])[n] == 7.0)  # nothing past the rows
    assert_close_rel(bf16_f64(runs[0])[:n], want, what=f"rows={rows} H={H} Is={Is}")


@pytest.mark.parametrize("T,E,k,I,zipf", [(300, 8, 2, 4096, None), (480, 8, 1, 4096, 1.2), (400, 100, 8, 520, 1.2),
                                           (400, 8, 2, 4096, None), (440, 8, 2, 4096, 1.2)])
def test_mid_layer(oracle, T, E, k, I, zipf):
    """A layer call and its four separate calls through the mid kernel (with the non-temporal hint in the first), bit
    for bit and against the oracle."""
    H = 1088
    cfg = mi.MoeConfig("mid", T=T, H=H, E=E, k=k, I=I, P=1, layout="replicated", zipf_s=zipf, seed=T)
    inp = mi.make_inputs(cfg)
    layer = moe.MoeLayer(T, E, k, 0, dev_bf16(inp.w13), dev_bf16(inp.w2))
    x, lg = dev_bf16(inp.x), torch.from_numpy(inp.logits).cuda()
    got = []
    for fn in (layer.forward_calls, layer.forward):
        layer.y.zero_()
        layer.out.zero_()
        fn(x, lg)
        torch.cuda.synchronize()
        got.append([host_bf16(layer.y), host_bf16(layer.out)])
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
    assert_close_rel(bf16_f64(got[1][1]), oracle.layer(inp), what=f"T={T} E={E} k={k}")


@pytest.mark.parametrize("H,Is", [(256, 512), (4096, 1536), (1000, 200)])
def test_no_tokens(H, Is):
    """A gathered call of fixed capacity without tokens writes nothing."""
    El, cap, k = 16, 320, 8
    x = torch.zeros((1, H), dtype=torch.bfloat16, device="cuda")
    w13 = torch.zeros((El, 2 * Is, H), dtype=torch.bfloat16, device="cuda")
    w2 = torch.zeros((El, H, Is), dtype=torch.bfloat16, device="cuda")
    r2p = torch.zeros(cap, dtype=torch.int32, device="cuda")
    y = torch.full((cap, H), 7.0, dtype=torch.bfloat16, device="cuda")
    offs = torch.zeros(El + 1, dtype=torch.int32, device="cuda")
    ws = torch.empty(moe.ffn_workspace_size(cap, El, H, Is), dtype=torch.uint8, device="cuda")
    st = moe.lib().moe_grouped_ffn(x.data_ptr(), 0, r2p.data_ptr(), k, offs.data_ptr(), El, cap, H, Is, w13.data_ptr(),
                                   w2.data_ptr(), y.data_ptr(), ws.data_ptr(), ws.numel(),
                                   torch.cuda.current_stream().cuda_stream or None)
    torch.cuda.synchronize()
    assert st == 0 and bool((y == 7.0).all())


@pytest.mark.parametrize("T,E,k,e0,El,H,Is", [
    (400, 128, 8, 16, 16, 2048, 768),   # by capacities: few rows per expert or many
    (2, 64, 8, 0, 8, 256, 3072),        # ... two waves on a strip's K or one
    (300, 64, 4, 0, 16, 1000, 328)])
def test_capacity_leaves_bits_alone(oracle, T, E, k, e0, El, H, Is):
    """The rows' capacity is a buffer size: gathered calls of the same tokens write the same bits under each."""
    ids = mi.random_topk_ids(T, E, k, seed=T)
    _, offs, r2p, _ = oracle.permute(ids, e0, El)
    n, most = int(offs[-1]), T * min(k, El)
    x = dev_bf16(mi.random_bf16((T, H), seed=T, tag=95))
    w13 = dev_bf16(mi.random_bf16((El, 2 * Is, H), seed=1, tag=96, std=0.03))
    w2 = dev_bf16(mi.random_bf16((El, H, Is), seed=1, tag=97, std=0.03))
    got = []
    for cap in (n, most, 3 * most):
        full = torch.full((cap,), -1, dtype=torch.int32)
        full[:n] = torch.from_numpy(r2p[:n])
        y = moe.grouped_ffn(x, torch.from_numpy(offs).cuda(), w13, w2, row_to_pair=full.cuda(), k=k, cap_rows=cap)
        torch.cuda.synchronize()
        got.append(host_bf16(y)[:n])
    np.testing.assert_array_equal(got[0], got[1])
    np.testing.assert_array_equal(got[1], got[2])


@pytest.mark.parametrize("El,H,Is,rows,k,tiles", [
    # rows not gathered (k = 0): few, or all of them too many for a host that cannot see a hot expert
    (16, 1024, 512, 768, 0, False), (16, 1024, 512, 769, 0, True), (16, 1024, 512, 1500, 0, True),
    (16, 2048, 1024, 256, 0, False), (16, 2048, 1024, 257, 0, True), (16, 5120, 1024, 200, 0, True),
    (72, 1536, 1280, 100, 0, True),
    # gathered: rows is the tokens
    (32, 7168, 256, 64, 8, False), (32, 7168, 256, 65, 8, True), (33, 2048, 1024, 100, 2, True),
    (16, 2048, 1024, 192, 4, False), (16, 2048, 1024, 193, 4, True), (16, 2048, 1024, 256, 2, False),
    (16, 2048, 1024, 257, 2, True), (32, 2048, 1024, 160, 8, False), (32, 2048, 1024, 161, 8, True),
    (32, 2048, 1024, 192, 2, False), (32, 2048, 1024, 193, 2, True), (4, 2048, 1024, 96, 2, False),
    (4, 2048, 1024, 97, 2, True), (8, 2048, 768, 256, 2, False), (8, 2048, 768, 257, 2, True),
    (16, 2048, 512, 448, 1, False), (16, 2048, 512, 449, 1, True),
    (8, 2048, 1024, 348, 2, True), (8, 2048, 1024, 352, 2, False), (8, 2048, 1024, 448, 2, False),
    (8, 2048, 1024, 449, 2, True), (8, 2048, 1024, 400, 3, True),
    (8, 4096, 1280, 284, 2, True), (8, 4096, 1280, 285, 2, False), (8, 4096, 2112, 400, 2, True),
    # widths that are not whole slices
    (8, 1000, 1208, 2048, 0, False), (8, 1000, 1208, 2049, 0, True), (4, 4096, 360, 384, 0, False),
    (4, 4096, 360, 385, 0, True), (4, 328, 808, 4096, 0, False), (4, 328, 808, 4097, 0, True),
    (128, 2048, 96, 2500, 8, False), (128, 2048, 96, 2501, 8, True)])
def test_lines(El, H, Is, rows, k, tiles):
    """Which calls of weights past the caches leave the tiled kernels."""
    assert zeros_route(El, H, Is, rows, k) == ("tiled" if tiles else "streaming")


@pytest.mark.parametrize("El,H,Is,rows,k,general", [
    (2, 208, 32, 3072, 0, False), (2, 208, 32, 3073, 0, True), (16, 208, 32, 4096, 0, False),
    (16, 208, 32, 4097, 0, True), (8, 72, 40, 3072, 2, False), (8, 72, 40, 3073, 2, True)])
def test_narrow_lines(El, H, Is, rows, k, general):
    """Which calls of narrow experts run the general kernel (none runs the tiled ones)."""
    assert zeros_route(El, H, Is, rows, k) == ("general" if general else "streaming")


def zeros_route(El, H, Is, rows, k):
    w13 = torch.zeros((El, 2 * Is, H), dtype=torch.bfloat16, device="cuda")
    w2 = torch.zeros((El, H, Is), dtype=torch.bfloat16, device="cuda")
    x = torch.zeros((rows, H), dtype=torch.bfloat16, device="cuda")
    offs = torch.zeros(El + 1, dtype=torch.int32, device="cuda")
    r2p = torch.zeros(rows * min(k, El), dtype=torch.int32, device="cuda") if k else None
    return ffn_route(lambda: moe.grouped_ffn(x, offs, w13, w2, row_to_pair=r2p, k=max(k, 1)))
