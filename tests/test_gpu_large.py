"""GPU parity at the benchmark configurations' full sizes, in the launch shapes bench.py
times.  Where the full oracle is affordable it is used in full; above that the product is
checked with an exact Freivalds-style identity over every entry (C r == A (B r) for random
+-1 vectors r, evaluated in float64 where every intermediate is an integer below 2^53) plus
full oracle rows / columns and sampled entries."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_05126_amd as P
import workloads as W
from tests.gpu_util import (FC_TILE_64, FC_TILE_128, FC_TILE_256, DeviceModel, dev, fc_kernel_choice, fill_i32,
                            host_u32, pack_on_gpu, require_gpu)
from tests.helpers import pack_pm1, unpack_words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()
    yield
    torch.cuda.synchronize()


def gemm_on_gpu(a, b):
    m, k = a.shape
    n = b.shape[0]
    ad, bd = pack_on_gpu(a), pack_on_gpu(b)
    c = fill_i32((m, n), 7)
    P.bnn_fc_binary(ad, m, k, bd, n, c_out=c)
    torch.cuda.synchronize()
    return c.cpu().numpy()


def test_gemm_4096_full_oracle():
    m = n = k = 4096
    a = W.draw_bits_pm1(W.rng_for(3, 1, 0), m, k)
    b = W.draw_bits_pm1(W.rng_for(3, 1, 1), n, k)
    print("gemm 4096^3 full oracle", flush=True)
    np.testing.assert_array_equal(gemm_on_gpu(a, b), oracle.fc(a, b))


def test_gemv_m1_8192_full_oracle():
    a = W.draw_bits_pm1(W.rng_for(3, 4, 0), 1, 8192)
    b = W.draw_bits_pm1(W.rng_for(3, 4, 1), 8192, 8192)
    print("gemv 1x8192x8192 full oracle", flush=True)
    np.testing.assert_array_equal(gemm_on_gpu(a, b), oracle.fc(a, b))


def freivalds_check(a, b, c, n_vec=32, seed=99):
    """Exact: (C r) == A (B r) for n_vec random +-1 vectors, blockwise in float64."""
    m, k = a.shape
    n = b.shape[0]
    rng = np.random.default_rng(seed)
    r = (2.0 * rng.integers(0, 2, size=(n, n_vec)) - 1.0)
    br = np.zeros((k, n_vec))
    blk = 1024
    for j0 in range(0, n, blk):                      # B^T r accumulated over row blocks of B
        bb = b[j0:j0 + blk].astype(np.float64)
        br += bb.T @ r[j0:j0 + blk]
    for i0 in range(0, m, blk):
        lhs = c[i0:i0 + blk].astype(np.float64) @ r
        rhs = a[i0:i0 + blk].astype(np.float64) @ br
        if not np.array_equal(lhs, rhs):
            bad = np.argwhere(lhs != rhs)[0]
            raise AssertionError(f"Freivalds mismatch in row {i0 + bad[0]}, vector {bad[1]}")


@pytest.mark.timeout(600)
@pytest.mark.parametrize("size,layer", [(8192, 2), (16384, 3)])
def test_gemm_large_freivalds_rows_cols_samples(size, layer):
    m = n = k = size
    print(f"gemm {size}^3: drawing operands", flush=True)
    a = W.draw_bits_pm1(W.rng_for(3, layer, 0), m, k)
    b = W.draw_bits_pm1(W.rng_for(3, layer, 1), n, k)
    print("  GPU product", flush=True)
    c = gemm_on_gpu(a, b)
    print("  Freivalds over all entries", flush=True)
    freivalds_check(a, b, c)
    print("  64 full rows and 64 full columns from the oracle", flush=True)
    rng = np.random.default_rng(size)
    rows = np.sort(rng.choice(m, 64, replace=False))
    cols = np.sort(rng.choice(n, 64, replace=False))
    rows[0], rows[-1], cols[0], cols[-1] = 0, m - 1, 0, n - 1
    np.testing.assert_array_equal(c[rows], oracle.fc(a[rows], b))
    np.testing.assert_array_equal(c[:, cols], oracle.fc(a, b[cols]))
    print("  2^20 sampled entries (1024 random rows x 1024 random columns)", flush=True)
    ri = rng.choice(m, 1024, replace=False)
    ci = rng.choice(n, 1024, replace=False)
    np.testing.assert_array_equal(c[np.ix_(ri, ci)], oracle.fc(a[ri], b[ci]))
    for _ in range(256):                             # and single dots at unstructured positions
        i, j = int(rng.integers(m)), int(rng.integers(n))
        assert c[i, j] == oracle.dot(a[i], b[j])


def words_of(bits):
    """bool [rows][n] on the GPU -> packed int32 words, in plain torch."""
    rows, n = bits.shape
    b = torch.nn.functional.pad(bits, (0, -n % 32)).reshape(rows, -1, 32).to(torch.int64)
    v = (b << torch.arange(32, device=bits.device)).sum(-1)
    return torch.where(v >= 2 ** 31, v - 2 ** 32, v).to(torch.int32)


# The 256 x 256 tile at its edges: a single round and several, one to five K chunks of 512 bits, 16-byte
# and 4-byte transfers, ragged last tiles; raw sums of one or two chunks run on it only where they are
# larger than 2^26 (streaming stores where n is a multiple of 32).  Reference: the product of the unpacked
# operands in FP32 (integers below 2^24: exact).
@pytest.mark.timeout(300)
@pytest.mark.parametrize("m,n,k,raw,step", [(3600, 3841, 2050, True, True), (4095, 8190, 2100, True, True),
                                            (4096, 8192, 2176, True, True), (3590, 3840, 512, False, True),
                                            (4095, 8190, 520, False, True), (4070, 8160, 1100, False, True),
                                            (8200, 8224, 512, True, False), (8195, 8201, 1000, True, False),
                                            (8193, 8224, 1000, True, False), (8200, 8224, 520, True, False)])
def test_gemm_large_tile_rounds(m, n, k, raw, step):
    print("large tile", m, n, k, raw, step, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + 3 * n + 5 * k)
    a, b = (2 * torch.randint(0, 2, (r, k), dtype=torch.int8, generator=g, device="cuda") - 1 for r in (m, n))
    kw = (k + 31) // 32
    ad, bd = fill_i32((m, kw), 0), fill_i32((n, kw), 0)
    P.bnn_pack_bits(a, m, k, ad)
    P.bnn_pack_bits(b, n, k, bd)
    bt = b.float().t().contiguous()
    want = torch.cat([(a[i:i + 1024].float() @ bt).int() for i in range(0, m, 1024)])
    if raw:
        assert fc_kernel_choice(m, n, k, True, False) == FC_TILE_256
        c = fill_i32((m + 1, n), 123456)
        P.bnn_fc_binary(ad, m, k, bd, n, c_out=c)
        assert torch.equal(c[:m], want)
        assert bool((c[m] == 123456).all())
        del c
    if step:
        assert fc_kernel_choice(m, n, k, False, True) == FC_TILE_256
        thr = want[m // 2].clone()                                          # ties
        thr[::3] = torch.randint(-(k // 4), k // 4 + 1, thr[::3].shape, dtype=torch.int32, generator=g, device="cuda")
        thr[-2:] = torch.tensor([2 ** 31 - 1, -2 ** 31], dtype=torch.int32)
        flip = torch.randint(0, 2, (n,), dtype=torch.uint8, generator=g, device="cuda")
        packed = fill_i32((m + 1, (n + 31) // 32), -1)
        P.bnn_fc_binary(ad, m, k, bd, n, thr=thr, flip=flip, packed_out=packed)
        for i in range(0, m, 1024):
            assert torch.equal(packed[i:min(m, i + 1024)], words_of((want[i:i + 1024] > thr) ^ (flip != 0))), i
        assert bool((packed[m] == -1).all())


# The largest K of the matrix-core path, where T - x of the step no longer fits 24 bits and its sign has to
# decide alone: row i of A is +1 in its first p_i places, row j of B in its first q_j, so that their product
# is K - 2 |p_i - q_j|.
@pytest.mark.timeout(300)
@pytest.mark.parametrize("m,n,tile", [(896, 890, FC_TILE_64), (1700, 1790, FC_TILE_128), (3500, 3584, FC_TILE_256)])
def test_gemm_largest_k(m, n, tile):
    k = (1 << 24) - 2048
    assert fc_kernel_choice(m, n, k, False, True) == tile
    print("largest K", m, n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + n)

    def rows(r):
        ends = torch.randint(0, k + 1, (r,), dtype=torch.int64, generator=g, device="cuda")
        ends[:4] = torch.tensor([0, k, 1, k - 1])
        first = torch.arange(0, k, 32, dtype=torch.int64, device="cuda")
        w = torch.empty((r, k // 32), dtype=torch.int32, device="cuda")
        for i in range(0, r, 32):
            c = (ends[i:i + 32, None] - first).clamp_(0, 32)
            v = (1 << c) - 1
            w[i:i + 32] = torch.where(v >= 2 ** 31, v - 2 ** 32, v).to(torch.int32)
        return ends, w
    (p, a), (q, b) = rows(m), rows(n)
    want = (k - 2 * (p[:, None] - q).abs()).to(torch.int32)
    c = fill_i32((m, n), 7)
    P.bnn_fc_binary(a, m, k, b, n, c_out=c)
    assert torch.equal(c, want)
    lim = torch.tensor([k, k - 1, -k, -k - 1, k + 1, 2 ** 31 - 1, -2 ** 31, 0], dtype=torch.int32, device="cuda")
    thr = torch.cat([lim, lim, lim, lim, lim, lim, lim, lim, want[m // 2, 64:]])            # extremes, then ties
    thr[65::3] -= 1
    packed = fill_i32((m, (n + 31) // 32), -1)
    P.bnn_fc_binary(a, m, k, b, n, thr=thr, packed_out=packed)
    assert torch.equal(packed, words_of(want > thr))


# Raw sums whose rows are so long that 32-bit offsets do not reach over a tile's (from 2^21, 2^22 and 2^23
# columns on for tiles of 256, 128 and 64 rows; over eight rows from 2^26 on), with columns that end inside a quad and on one; the
# reference is the product of the unpacked operands in FP32 (integers below 2^24: exact).
@pytest.mark.timeout(300)
@pytest.mark.parametrize("m,n,k,both,tile", [(200, (1 << 21) + 5, 64, False, FC_TILE_256),
                                             (513, (1 << 21) + 64, 70, False, FC_TILE_256),
                                             (140, (1 << 21) + 36, 1100, False, FC_TILE_256),
                                             (65, (1 << 22) + 7, 1000, False, FC_TILE_128),
                                             (130, (1 << 22) + 8, 32, True, FC_TILE_128),
                                             (9, (1 << 23) + 12, 600, False, FC_TILE_64),
                                             (11, (1 << 23) + 33, 96, True, FC_TILE_64),
                                             (9, (1 << 26) + 36, 32, False, FC_TILE_64),
                                             (66, (1 << 26) + 6, 32, False, FC_TILE_128)])
def test_gemm_raw_with_many_columns(m, n, k, both, tile):
    assert fc_kernel_choice(m, n, k, True, both) == tile
    print("many columns", m, n, k, both, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    a, b = (2 * torch.randint(0, 2, (r, k), dtype=torch.int8, generator=g, device="cuda") - 1 for r in (m, n))
    kw = (k + 31) // 32
    ad, bd = fill_i32((m, kw), 0), fill_i32((n, kw), 0)
    P.bnn_pack_bits(a, m, k, ad)
    P.bnn_pack_bits(b, n, k, bd)
    c = fill_i32((m + 1, n), 123456)
    thr = torch.randint(-9, 10, (n,), dtype=torch.int32, generator=g, device="cuda")
    packed = fill_i32((m, (n + 31) // 32), -1)
    if both:
        P.bnn_fc_binary(ad, m, k, bd, n, thr=thr, packed_out=packed, c_out=c)
    else:
        P.bnn_fc_binary(ad, m, k, bd, n, c_out=c)
    af = a.float()
    for j in range(0, n, 1 << 18):
        want = (af @ b[j:j + (1 << 18)].float().t().contiguous()).int()
        assert torch.equal(c[:m, j:j + (1 << 18)], want), j
        if both:
            bits = (want > thr[j:j + (1 << 18)]).cpu().numpy()
            np.testing.assert_array_equal(host_u32(packed[:, j // 32:(j + (1 << 18)) // 32]), pack_pm1(bits.astype(np.int8)))
    assert bool((c[m] == 123456).all())


@pytest.mark.timeout(300)
def test_vgg_small_batch256_all_logits():
    cid, layers, in_shape = W.model_by_name("vgg_small")
    imgs = W.draw_images(W.rng_for(cid, 0, 0), 256, *in_shape)
    print("vgg_small b256: oracle", flush=True)
    logits, _ = oracle.run_model(layers, imgs)
    dm = DeviceModel(layers, 256, in_shape)
    xd = dev(imgs)
    for mode in (P.RUN_STREAM, P.RUN_GRAPH):
        dm.logits.fill_(-9)
        dm.run(xd, mode)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(dm.logits.cpu().numpy(), logits)


@pytest.mark.timeout(600)
def test_vgg_small_batch4096_sampled_images():
    # images are independent: the logits of image i in the big batch equal those of a batch
    # holding only the sampled images (256 of them, spread over the batch, both ends included)
    cid, layers, in_shape = W.model_by_name("vgg_small")
    batch = 4096
    imgs = W.draw_images(W.rng_for(cid, 0, 0), batch, *in_shape)
    dm = DeviceModel(layers, batch, in_shape)
    print("vgg_small b4096: GPU", flush=True)
    dm.run(dev(imgs), P.RUN_STREAM)
    torch.cuda.synchronize()
    got = dm.logits.cpu().numpy()
    rng = np.random.default_rng(4096)
    idx = np.unique(np.concatenate([[0, 1, 255, 256, 4095], rng.choice(batch, 251, replace=False)]))
    print("vgg_small b4096: oracle on", len(idx), "images", flush=True)
    want, _ = oracle.run_model(layers, imgs[idx])
    np.testing.assert_array_equal(got[idx], want)
    assert np.all(got % 2 == 0) and np.all(np.abs(got) <= 1024)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("hw,c", W.CONV_SWEEP_SHAPES)
def test_conv_sweep_batch1024(hw, c):
    """The per-layer sweep at its full batch.  The whole output is compared with the oracle where
    that costs at most 155 G MAC (six shapes); the three largest layers are compared on 64 images
    spread over the batch (first, last and every 16th in between)."""
    n = 1024
    cw = c // 32
    rng = W.rng_for(4, hw, c % 1000)
    xw = rng.integers(0, 2**32, size=(n, hw, hw, cw), dtype=np.uint32)
    wt = W.draw_pm1(rng, (c, 3, 3, c))
    thr = W.draw_threshold(rng, c, 9 * c)
    flip = W.draw_flip(rng, c)
    wd = dev(pack_pm1(wt.reshape(c * 9, c)).reshape(c, 3, 3, cw))
    out = fill_i32((n, hw, hw, cw), -1)
    P.bnn_conv_binary(dev(xw), n, hw, hw, c, wd, c, thr=dev(thr), flip=dev(flip), pool=1, packed_out=out)
    torch.cuda.synchronize()
    got = host_u32(out)
    macs = n * hw * hw * c * 9 * c
    full = macs <= 155e9
    idx = np.arange(n) if full else np.unique(np.concatenate([np.arange(0, n, 16), [1, n - 1]]))
    print(f"conv sweep {hw}x{hw} C{c} batch {n}: oracle on {len(idx)} images", flush=True)
    x_s = unpack_words(xw[idx], c)
    want = pack_pm1(oracle.step(oracle.conv2d(x_s, wt, 1, -1), thr, flip))
    np.testing.assert_array_equal(got[idx], want)
    # the other images: bits look random, none of the fill value survives
    assert not np.any(np.all(got.reshape(n, -1) == 0xFFFFFFFF, axis=1))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,hw,ci,co,pool", [(8192, 4, 1024, 128, 2), (2048, 8, 512, 256, 1), (2050, 8, 512, 128, 2),
                                             (4096, 4, 1024, 128, 1), (1030, 8, 512, 128, 2), (3001, 5, 512, 256, 1),
                                             (2100, 7, 1024, 128, 1), (1024, 8, 512, 192, 2), (1500, 6, 608, 160, 1)])
def test_conv_wide_layers_streamed_weights_sampled_images(n, hw, ci, co, pool):
    """C_in >= 512 at a batch that selects the largest block tile (weight chunks streamed through two
    LDS buffers): sampled images against the oracle, first / last / ragged-tail images included."""
    cw = (ci + 31) // 32
    rng = W.rng_for(4, hw + 50, ci % 1000 + co)
    print(f"conv wide {hw}x{hw} {ci}->{co} batch {n} pool {pool}", flush=True)
    xw = rng.integers(0, 2**32, size=(n, hw, hw, cw), dtype=np.uint32)
    if ci % 32:
        xw[..., -1] &= np.uint32((1 << (ci % 32)) - 1)       # tail bits of the last word are zero
    wt = W.draw_pm1(rng, (co, 3, 3, ci))
    thr = W.draw_threshold(rng, co, 9 * ci)
    flip = W.draw_flip(rng, co)
    wd = dev(pack_pm1(wt.reshape(co * 9, ci)).reshape(co, 3, 3, cw))
    out = fill_i32((n, hw // pool, hw // pool, (co + 31) // 32), -1)
    P.bnn_conv_binary(dev(xw), n, hw, hw, ci, wd, co, thr=dev(thr), flip=dev(flip), pool=pool, packed_out=out)
    torch.cuda.synchronize()
    got = host_u32(out)
    idx = np.array([0, 1, 15, 16, n // 2 + 3, n - 17, n - 2, n - 1])
    x_s = unpack_words(xw[idx], ci)
    s = oracle.step(oracle.conv2d(x_s, wt, 1, -1), thr, flip)
    if pool == 2:
        s = oracle.maxpool2(s)
    np.testing.assert_array_equal(got[idx], pack_pm1(s))
    assert not np.any(np.all(got.reshape(n, -1) == 0xFFFFFFFF, axis=1))
