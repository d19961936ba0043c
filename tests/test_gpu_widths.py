"""Widths that are not whole 64-wide K-slices (needs an MI355X): the last
slice of either GEMM is partly past K, and its loads read zeros there, in the
streaming, mid and tiled kernels.  Every case is checked against the CPU
oracle."""
import numpy as np
import pytest
import torch

import moe_inputs as mi
import paper_2606_26607_amd as moe
from tests.util import assert_close_rel, bf16_f64, dev_bf16, ffn_route, host_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    moe.lib()


# rows per expert: several passes of a streaming kernel, whole and partial ones, single rows, none
ROWS = [300, 0, 64, 120, 1, 513, 17]


@pytest.mark.parametrize("H,Is", [(8, 8),         # one slice of one chunk on both sides
                                  (56, 72),       # one slice; one chunk past a slice
                                  (128, 120),     # whole slices; a slice short of one chunk
                                  (136, 96), (1000, 328),
                                  (264, 8248)])   # a split K whose last slice is partial
@pytest.mark.parametrize("gather", [False, True])
def test_partial_last_slice(oracle, H, Is, gather):
    El, k, n = len(ROWS), 2, sum(ROWS)
    offs = np.concatenate([[0], np.cumsum(ROWS)]).astype(np.int32)
    T = n if not gather else 600
    x = mi.random_bf16((T, H), seed=H, tag=70)
    # values past K would be the next row's: make them large, so that one read by mistake shows
    x[:, 0] = mi.f32_to_bf16_bits(np.full(T, 50.0, np.float32))
    w13 = mi.random_bf16((El, 2 * Is, H), seed=H, tag=71, std=0.05)
    w2 = mi.random_bf16((El, H, Is), seed=H, tag=72, std=0.05)
    r2p = np.random.default_rng(H).integers(0, T * k, n).astype(np.int32) if gather else None
    y = moe.grouped_ffn(dev_bf16(x), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2),
                        row_to_pair=None if r2p is None else torch.from_numpy(r2p).cuda(), k=k if gather else 1)
    torch.cuda.synchronize()
    ref = oracle.grouped_ffn(x if r2p is None else x[r2p // k], offs, w13, w2)
    assert_close_rel(bf16_f64(host_bf16(y)), ref, what=f"H={H} Is={Is} gather={gather}")


# ... and with enough rows for the tiled kernels: whole and partial 256-row tiles, 64- and 128-row ones
TILED_ROWS = [3000, 0, 64, 120, 1, 900, 17]


@pytest.mark.parametrize("rows,T,H,Is", [
    (TILED_ROWS, 0, 1000, 328), (TILED_ROWS, 4200, 1000, 328),
    (TILED_ROWS, 0, 136, 352), (TILED_ROWS, 4200, 1032, 72),    # one chunk past a slice, in either GEMM
    (TILED_ROWS, 0, 56, 1016), (TILED_ROWS, 0, 1016, 56),       # one slice; one short of a chunk
    ([300, 64, 0, 57], 0, 264, 8248), ([70, 40], 4200, 8200, 136)])  # split over K, the last piece partial
def test_tiles_mask_the_last_slice(oracle, rows, T, H, Is):
    """What lies past K is the next row's: with infinities there, in the activations and in the down projection's
    weights, a load that is not masked, of either operand, shows in the row before."""
    El, k, n = len(rows), 2, sum(rows)
    offs = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    x = mi.random_bf16((T or n, H), seed=H, tag=110)
    w13 = mi.random_bf16((El, 2 * Is, H), seed=H, tag=111, std=0.05)
    w2 = mi.random_bf16((El, H, Is), seed=H, tag=112, std=0.05)
    r2p = np.random.default_rng(H).integers(0, T * k, n).astype(np.int32) if T else None
    tokens = np.arange(n) if r2p is None else r2p // k
    ref = oracle.grouped_ffn(x[tokens], offs, w13, w2)
    inf = mi.f32_to_bf16_bits(np.array([np.inf], np.float32))[0]
    xi, w2i = x.copy(), w2.copy()
    xi[1::2, :8] = inf
    w2i[:, 1::2, :8] = inf
    y = torch.empty((n, H), dtype=torch.bfloat16, device="cuda")
    args = (dev_bf16(xi), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2i),
            None if r2p is None else torch.from_numpy(r2p).cuda(), k)
    assert ffn_route(lambda: moe.grouped_ffn(*args, cap_rows=n, y=y)) == "tiled"
    even = tokens % 2 == 0
    assert_close_rel(bf16_f64(host_bf16(y))[even][:, 0::2], ref[even][:, 0::2], what=f"H={H} Is={Is} T={T}")


@pytest.mark.parametrize("H,Is,rows", [
    (208, 32, [2500, 0, 300, 1]),                        # mid kernel, more 128-row runs than its grid holds
    (1000, 328, [3000, 72]), (1000, 328, [3000, 73]),
    (1000, 328, [4000, 96]), (1000, 328, [4000, 97]),    # either side of its rows: mid, tiled
    (1000, 352, [500, 300]),                             # weights just above its size: tiled
    (208, 32, [4000, 96]), (208, 32, [4000, 97]),        # the general kernel
    (72, 40, [4100, 0, 5]), (8, 8, [5000])])
def test_small_weights_many_rows(oracle, H, Is, rows):
    n = sum(rows)
    offs = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    x = mi.random_bf16((n, H), seed=H, tag=79)
    w13 = mi.random_bf16((len(rows), 2 * Is, H), seed=H, tag=71, std=0.05)
    w2 = mi.random_bf16((len(rows), H, Is), seed=H, tag=72, std=0.05)
    y = moe.grouped_ffn(dev_bf16(x), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2))
    torch.cuda.synchronize()
    assert_close_rel(bf16_f64(host_bf16(y)), oracle.grouped_ffn(x, offs, w13, w2), what=f"H={H} Is={Is} {rows}")


@pytest.mark.parametrize("T,H,I", [(935, 208, 32), (3072, 72, 40), (4200, 72, 40)])
def test_small_weights_layer(oracle, T, H, I):
    """One call and four calls choose the same kernels: equal bits."""
    cfg = mi.MoeConfig("narrow", T=T, H=H, E=16, k=8, I=I, P=1, layout="replicated", rank=0, seed=T)
    inp = mi.make_inputs(cfg)
    layer = moe.MoeLayer(T, 16, 8, 0, dev_bf16(inp.w13), dev_bf16(inp.w2))
    x, lg = dev_bf16(inp.x), torch.from_numpy(inp.logits).cuda()
    got = []
    for fn in (layer.forward_calls, layer.forward):
        layer.out.view(torch.uint8).fill_(0xA5)
        fn(x, lg)
        torch.cuda.synchronize()
        got.append(host_bf16(layer.out).copy())
    np.testing.assert_array_equal(*got)
    assert_close_rel(bf16_f64(got[0]), oracle.layer(inp), what=f"T={T} H={H} I={I}")


def test_infinite_neighbour(oracle):
    """A row's neighbour in memory holds infinities: they stay out of the row's own result (streaming kernels)."""
    H, Is, n = 200, 72, 300
    x = mi.random_bf16((n, H), seed=5, tag=73)
    x[1::2, :8] = mi.f32_to_bf16_bits(np.array([np.inf], np.float32))[0]
    w13 = mi.random_bf16((1, 2 * Is, H), seed=5, tag=74, std=0.05)
    w2 = mi.random_bf16((1, H, Is), seed=5, tag=75, std=0.05)
    offs = np.array([0, n], np.int32)
    y = moe.grouped_ffn(dev_bf16(x), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2))
    torch.cuda.synchronize()
    got = bf16_f64(host_bf16(y))[0::2]
    ref = oracle.grouped_ffn(x[0::2], np.array([0, len(got)], np.int32), w13, w2)
    assert_close_rel(got, ref, what="rows beside infinite ones")


def test_operand_beyond_4gib(oracle):
    """A token matrix past what 32-bit byte offsets address takes the general kernels; the rows read lie at its
    far end."""
    T, H, Is = (1 << 32) // (2 * 8192) + 600, 8192, 64
    x = torch.empty((T, H), dtype=torch.bfloat16, device="cuda")
    x[-500:] = dev_bf16(mi.random_bf16((500, H), seed=6, tag=76))
    w13 = mi.random_bf16((2, 2 * Is, H), seed=6, tag=77, std=0.02)
    w2 = mi.random_bf16((2, H, Is), seed=6, tag=78, std=0.05)
    r2p = (np.random.default_rng(6).integers(T - 500, T, 130)).astype(np.int32)
    offs = np.array([0, 100, 130], np.int32)
    y = moe.grouped_ffn(x, torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2),
                        row_to_pair=torch.from_numpy(r2p).cuda(), k=1)
    torch.cuda.synchronize()
    rows = host_bf16(x[-500:].contiguous())[r2p - (T - 500)]
    ref = oracle.grouped_ffn(rows, offs, w13, w2)
    assert_close_rel(bf16_f64(host_bf16(y)), ref, what="x above 4 GiB")


@pytest.mark.parametrize("El,H,Is,rows,T,route", [
    (8, 1000, 200, [9, 0, 20, 1, 30, 0, 3, 1], 5000, "tiled"),        # few rows gathered from many tokens
    (4, 264, 8248, [300, 64, 0, 57], 0, "tiled"),                     # split over K in both classes
    (2, 8200, 136, [70, 40], 4200, "tiled"),
    (3, 4096, 1600, [90, 300, 33], 0, "tiled"), (3, 512, 640, [600, 64, 257], 0, "tiled"),   # whole slices
    (8, 72, 40, [1, 0, 700, 3, 2500, 9, 0, 1], 0, "general"), (8, 72, 40, [1, 0, 70, 3, 25, 9, 0, 1], 0, "streaming")])
def test_workspace_is_enough(oracle, El, H, Is, rows, T, route):
    """A call writes inside the workspace it asks for, and its parts do not overlap."""
    n, k = sum(rows), 2
    offs = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    x = mi.random_bf16((T or n, H), seed=H, tag=100)
    w13 = mi.random_bf16((El, 2 * Is, H), seed=H, tag=101, std=0.05)
    w2 = mi.random_bf16((El, H, Is), seed=H, tag=102, std=0.05)
    r2p = np.random.default_rng(H).integers(0, T * k, n).astype(np.int32) if T else None
    need = moe.ffn_workspace_size(n, El, H, Is)
    ws = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    y = torch.empty((n, H), dtype=torch.bfloat16, device="cuda")
    args = (dev_bf16(x), torch.from_numpy(offs).cuda(), dev_bf16(w13), dev_bf16(w2),
            None if r2p is None else torch.from_numpy(r2p).cuda(), k)
    assert ffn_route(lambda: moe.grouped_ffn(*args, cap_rows=n, y=y, workspace=ws[:need])) == route
    assert bool((ws[need:] == 0x5A).all())
    assert_close_rel(bf16_f64(host_bf16(y)), oracle.grouped_ffn(x if r2p is None else x[r2p // k], offs, w13, w2),
                     what=f"H={H} Is={Is} {rows}")
