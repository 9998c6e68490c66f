"""Parity of the per-order channel-mixing linear (el_forward / el_backward through the C ABI,
MFMA kernels and the plain fallback) with the fp64 CPU oracle.  Tolerances as everywhere: fp32
max|err|/rms(ref) <= 1e-5 per output tensor, fp64 max(|err| / max(|ref|, rms(ref))) <= 1e-12."""
import sys

import numpy as np
import pytest

from oracle import equivariant_linear as oel
from paper_2504_10700_amd import workloads
from gpu_util import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def el():
    import torch
    assert torch.cuda.is_available()
    from paper_2504_10700_amd import el_binding
    return el_binding


def run_case(el, N, k_in, k_out, l_max, dtype, seed):
    import torch
    print(f"case N={N} k_in={k_in} k_out={k_out} l_max={l_max} {dtype}", flush=True)
    sys.stdout.flush()
    dev = torch.device("cuda:0")
    tdt = torch.float32 if dtype == "f32" else torch.float64
    X, W, dY = workloads.make_linear_inputs(N, k_in, k_out, l_max, seed)
    Xd, Wd, dYd = (torch.tensor(x, dtype=tdt, device=dev) for x in (X, W, dY))
    cfg = el.make_config(k_in, k_out, l_max, el.SC_F32 if dtype == "f32" else el.SC_F64)
    Y = torch.full((N, k_out, (l_max + 1) ** 2), float("nan"), dtype=tdt, device=dev)
    dX, dW = torch.full_like(Xd, float("nan")), torch.full_like(Wd, float("nan"))
    nbytes = el.el_workspace_bytes(cfg, N)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    el.el_forward(cfg, N, Xd, Wd, Y)
    el.el_backward(cfg, N, Xd, Wd, dYd, dX, dW, ws, nbytes)
    torch.cuda.synchronize()
    X64, W64, dY64 = (x.double().cpu().numpy() for x in (Xd, Wd, dYd))
    errs = [check("Y", Y.cpu().numpy(), oel.forward(X64, W64), dtype)]
    dX_ref, dW_ref = oel.backward(X64, W64, dY64)
    errs.append(check("dX", dX.cpu().numpy(), dX_ref, dtype))
    errs.append(check("dW", dW.cpu().numpy(), dW_ref, dtype))
    print("  errors Y, dX, dW: " + ", ".join(f"{e:.2e}" for e in errs), flush=True)
    Y2, dX2, dW2 = torch.empty_like(Y), torch.empty_like(dX), torch.empty_like(dW)
    el.el_forward(cfg, N, Xd, Wd, Y2)
    el.el_backward(cfg, N, Xd, Wd, dYd, dX2, dW2, ws, nbytes)
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2) and torch.equal(dX, dX2) and torch.equal(dW, dW2), "not reproducible"


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("l_max", [0, 1, 2, 3])
def test_mfma_kernels_small(el, dtype, l_max):
    # 333 atoms: 20 full row tiles and a ragged one, several ranges in the dW kernel
    run_case(el, 333, 128, 128, l_max, dtype, 8000 + l_max)


@pytest.mark.parametrize("k_in,k_out", [(64, 192), (256, 64), (128, 256), (4, 64)])
def test_mfma_kernels_other_channel_counts(el, k_in, k_out):
    run_case(el, 90, k_in, k_out, 3, "f32", 8100 + k_in)
    run_case(el, 50, k_in, k_out, 1, "f64", 8200 + k_out)


@pytest.mark.parametrize("k_in,k_out", [(96, 40), (7, 5), (128, 100)])
def test_plain_fallback(el, k_in, k_out):
    run_case(el, 70, k_in, k_out, 3, "f32", 8300 + k_in)
    run_case(el, 33, k_in, k_out, 2, "f64", 8400 + k_out)


# Products cut along the reduction.  Any channel count (fewer reduction steps than waves, a reduction
# and columns that are no multiple of 4 and 16), atoms around a row tile; and the batch size up to which they serve
# the tiled channel counts too (4 x 256 tiles of 16 atoms x 16 columns in fp32, 8 x 256 in fp64; dX reads W as it
# is up to 256 tiles).
@pytest.mark.parametrize("N,k_in,k_out,l_max,dtype", [
    (1, 3, 1, 3, "f32"), (15, 100, 128, 3, "f32"), (17, 1, 17, 2, "f64"), (65, 13, 33, 1, "f32"), (67, 33, 31, 0, "f64"),
    (263, 100, 50, 2, "f32"), (259, 90, 70, 3, "f64"),
    (512, 128, 128, 3, "f32"), (513, 128, 128, 3, "f32"), (2048, 64, 128, 3, "f32"), (2049, 64, 128, 3, "f32"), (4096, 16, 64, 1, "f32"), (4097, 16, 64, 1, "f32"),
    (4096, 64, 128, 1, "f64"), (4097, 64, 128, 1, "f64")])
def test_products_cut_along_the_reduction(el, N, k_in, k_out, l_max, dtype):
    run_case(el, N, k_in, k_out, l_max, dtype, 8700 + N)


# Channel counts for which a tile would be mostly padding (a thread per result) and their neighbours on the other side of
# the rule; dX takes it with the counts exchanged.
@pytest.mark.parametrize("N,k_in,k_out,l_max,dtype", [
    (300, 5, 8, 0, "f32"), (300, 6, 8, 0, "f32"), (257, 4, 8, 1, "f64"), (257, 2, 33, 1, "f32"), (255, 2, 8, 2, "f32"),
    (256, 3, 8, 2, "f64"), (300, 1, 1, 3, "f32"), (100, 4, 4, 3, "f64"), (100, 5, 4, 3, "f32")])
def test_few_channels(el, N, k_in, k_out, l_max, dtype):
    run_case(el, N, k_in, k_out, l_max, dtype, 8750 + N)


def test_more_tiles_than_a_grid_holds(el):
    """2^28 atoms with one channel in and one or nine out (2^24 tiles of 16 atoms), and one atom with 32 770 channels (2049^2
    tiles of dW): more threads than the 2^32 of a grid.  One term per result: a product rounded once."""
    import torch
    n = 2 ** 28 + 17
    X = torch.randn((n, 1, 1), device="cuda")
    for k_out in (1, 9):
        W = torch.randn((1, 1, k_out), device="cuda")
        Y = torch.full((n, k_out, 1), float("nan"), device="cuda")
        el.el_forward(el.make_config(1, k_out, 0), n, X, W, Y)
        for j in range(k_out):
            assert torch.equal(Y[:, j], X[:, 0] * W[0, 0, j]), (k_out, j)
        del Y
    del X
    k = 32770
    X, dY, dX = torch.randn((1, k, 1), device="cuda"), torch.randn((1, k, 1), device="cuda"), torch.full((1, k, 1), float("nan"), device="cuda")
    W, dW = torch.ones((1, k, k), device="cuda"), torch.full((1, k, k), float("nan"), device="cuda")
    cfg = el.make_config(k, k, 0)
    nbytes = el.el_workspace_bytes(cfg, 1)
    el.el_backward(cfg, 1, X, W, dY, dX, dW, torch.empty(nbytes, dtype=torch.uint8, device="cuda"), nbytes)
    assert torch.equal(dW[0], X[0] * dY[0].T)
    want = dY.double().sum().item()
    assert abs(dX.double() - want).max().item() <= 2.0 ** -23 * abs(want) + 1e-9 * k ** 0.5
    del X, dY, dX, W, dW
    torch.cuda.empty_cache()


# The products on the bfloat16 matrix cores: one chunk of the reduction and several, a ragged last row tile, two
# groups of columns; and the kernel of reductions that are no multiple of 32.
@pytest.mark.parametrize("N,k_in,k_out", [(2065, 32, 128), (2100, 96, 256), (2049, 160, 128), (2070, 48, 128)])
def test_products_of_split_values(el, N, k_in, k_out):
    run_case(el, N, k_in, k_out, 3, "f32", 8800 + k_in)


# ... and the sides of the rule that takes units of 16 atoms x 128 columns to them (512, 640 and 1280 units with 64 channels
# summed, 512 with 32), against torch in fp64: forward and, with the channel counts exchanged, dX.
@pytest.mark.parametrize("N,k_red", [(8192, 64), (8193, 64), (10240, 64), (10241, 64), (20480, 64), (20481, 64), (8193, 32)])
def test_batches_on_both_sides_of_the_rule(el, N, k_red):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(8850)
    X = torch.randn((N, k_red, 16), generator=gen, device="cuda")
    W = torch.randn((4, k_red, 128), generator=gen, device="cuda") / k_red ** 0.5
    Y, dX, dW = torch.empty((N, 128, 16), device="cuda"), torch.empty((N, 128, 16), device="cuda"), torch.empty((4, 128, k_red), device="cuda")
    el.el_forward(el.make_config(k_red, 128, 3), N, X, W, Y)
    cfg = el.make_config(128, k_red, 3)
    nbytes = el.el_workspace_bytes(cfg, N)
    el.el_backward(cfg, N, torch.zeros_like(dX), W.transpose(1, 2).contiguous(), X, dX, dW,
                   torch.empty(nbytes, dtype=torch.uint8, device="cuda"), nbytes)
    for c in range(16):
        ref = X[:, :, c].double() @ W[int(c ** 0.5)].double()
        for what, got in (("Y", Y), ("dX", dX)):
            err = ((got[:, :, c].double() - ref).abs().max() / ref.square().mean().sqrt()).item()
            assert err <= 1e-5, (what, c, err)


# ... and of the rule that gives a row tile a workgroup of its own, two on a compute unit (256 units; the first and the last of its
# units with 128 channels summed, 96, 64 and 32, one more, and two groups of columns).
@pytest.mark.parametrize("N,k_red,k_cols", [(4096, 128, 128), (4097, 128, 128), (5120, 128, 128), (5121, 128, 128), (6656, 96, 128), (6657, 96, 128),
                                            (4111, 64, 128), (6650, 64, 128), (20497, 64, 128), (4105, 32, 128), (8192, 32, 128), (2049, 160, 256)])
def test_a_workgroup_for_every_row_tile(el, N, k_red, k_cols):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(8870 + k_red)
    X = torch.randn((N, k_red, 16), generator=gen, device="cuda")
    W = torch.randn((4, k_red, k_cols), generator=gen, device="cuda") / k_red ** 0.5
    Y = torch.full((N + 1, k_cols, 16), 7.0, device="cuda")
    el.el_forward(el.make_config(k_red, k_cols, 3), N, X, W, Y)
    assert (Y[N] == 7).all()
    for c in range(16):
        ref = X[:, :, c].double() @ W[int(c ** 0.5)].double()
        err = ((Y[:N, :, c].double() - ref).abs().max() / ref.square().mean().sqrt()).item()
        assert err <= 1e-5, (c, err)


# dX of these products reads W as it is: the same sums in the same order as el_forward on W transposed, also in tiles
# that are computed again.  One chunk of the reduction and several, two groups of columns, a reduction that is no multiple of
# 32, a ragged last row tile and none.
@pytest.mark.parametrize("N,k_in,k_out", [(2065, 128, 32), (2049, 128, 160), (1100, 256, 96), (2070, 128, 48),
                                          (3072, 128, 512), (3073, 128, 512),
                                          (4300, 128, 128), (4150, 128, 96), (5500, 128, 64)])   # (the forward's tiles in workgroups of their own)
def test_dx_is_the_product_with_w_transposed(el, N, k_in, k_out):
    import torch
    X, W, dY = (torch.tensor(x, dtype=torch.float32, device="cuda:0") for x in workloads.make_linear_inputs(N, k_in, k_out, 3, 8960))
    dY[5, 7, 2], dY[700, 3, 0], dY[1000, 1, 12], dY[N - 1, k_out - 1, 15] = np.inf, 3.4e38, np.nan, -3.4e38
    cfg = el.make_config(k_in, k_out, 3)
    nbytes = el.el_workspace_bytes(cfg, N)
    dX, ref, dW = torch.empty_like(X), torch.empty_like(X), torch.empty_like(W)
    el.el_backward(cfg, N, X, W, dY, dX, dW, torch.empty(nbytes, dtype=torch.uint8, device="cuda:0"), nbytes)
    el.el_forward(el.make_config(k_out, k_in, 3), N, dY, W.transpose(1, 2).contiguous(), ref)
    torch.cuda.synchronize()
    assert ref.isnan().any() and torch.equal(dX.isnan(), ref.isnan())
    assert torch.equal(dX.nan_to_num(nan=0.0), ref.nan_to_num(nan=0.0))


def test_values_that_do_not_split(el):
    """Infinities, NaN and values that round to a bfloat16 infinity: the results of the tiles they are in are those of the
    products in fp32, the others are untouched."""
    import torch
    N, K = 2080, 128
    X, W, _ = workloads.make_linear_inputs(N, K, K, 3, 8900)
    W *= 1e-3
    X[5, 7, 2], X[700, 3, 0], X[1300, 100, 12], X[2079, 127, 15] = np.inf, 3.4e38, np.nan, -3.4e38
    Xd, Wd = (torch.tensor(x, dtype=torch.float32, device="cuda:0") for x in (X, W))
    Y = torch.empty((N, K, 16), device="cuda:0")
    el.el_forward(el.make_config(K, K, 3), N, Xd, Wd, Y)
    torch.cuda.synchronize()
    got = Y.double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = oel.forward(Xd.double().cpu().numpy(), Wd.double().cpu().numpy())
    assert np.isposinf(ref).any() and np.isneginf(ref).any() and np.isnan(ref).any()
    assert (np.isnan(got) == np.isnan(ref)).all()
    inf = np.isinf(ref)
    assert (got[inf] == ref[inf]).all()
    for where in (np.isfinite(ref) & (np.abs(ref) > 1e25), np.isfinite(ref) & (np.abs(ref) < 1e25)):
        err = np.abs(got[where] - ref[where]).max() / np.sqrt((ref[where] ** 2).mean())
        assert err <= 1e-5, err


@pytest.mark.parametrize("x_scale,w_scale", [(s, 1.0) for s in (1e-30, 1e-34, 1e-36, 1e-38)] +
                         [(1.0, s) for s in (1e-30, 1e-34, 1e-36, 1e-38)] + [(1e-17, 1e-17), (1e-19, 1e-18), (1e36, 1e-36)])
def test_small_values(el, x_scale, w_scale):
    """Products of values whose last bits no bfloat16 part holds (below 2^-110, 8e-34), or whose products are near the
    smallest fp32 value: forward and dX keep the bound of all others."""
    import torch
    N, K = 2065, 128
    X, W, _ = workloads.make_linear_inputs(N, K, K, 3, 8970)
    X, W = (torch.tensor(v * s, dtype=torch.float32) for v, s in ((X, x_scale), (W, w_scale)))
    ref = oel.forward(X.double().numpy(), W.double().numpy())
    Xd, Wd = X.cuda(), W.cuda()
    Y, dX, dW = torch.empty_like(Xd), torch.empty_like(Xd), torch.empty_like(Wd)
    cfg = el.make_config(K, K, 3)
    el.el_forward(cfg, N, Xd, Wd, Y)
    nbytes = el.el_workspace_bytes(cfg, N)   # dX of (Wt, dY = X) is the forward of (X, W)
    el.el_backward(cfg, N, torch.zeros_like(Xd), Wd.transpose(1, 2).contiguous(), Xd, dX, dW,
                   torch.empty(nbytes, dtype=torch.uint8, device="cuda:0"), nbytes)
    for what, got in (("Y", Y), ("dX", dX)):
        err = np.abs(got.double().cpu().numpy() - ref).max() / np.sqrt((ref ** 2).mean())
        print(f"  X {x_scale:g} W {w_scale:g} {what}: {err:.2e}", flush=True)
        assert err <= 1e-5, (what, err)


def test_values_of_every_exponent_keep_their_bits(el):
    """W a permutation of the channels: the result is the permuted input, bit for bit, whatever the exponent: a row tile of
    16 atoms per exponent from the smallest subnormal value to the largest finite one, and one with all of them."""
    import torch
    K, tiles = 128, 278
    rng = np.random.default_rng(8980)
    e = np.repeat(np.arange(-149, 129), 16)[:, None, None] * np.ones((1, K, 16))
    e[-16:] = rng.integers(-149, 128, (16, K, 16))
    with np.errstate(over="ignore"):
        X = np.ldexp(rng.choice([-1.0, 1.0], e.shape) * rng.uniform(1, 2, e.shape), e.astype(np.int64)).astype(np.float32)
    X = np.clip(X, -np.finfo(np.float32).max, np.finfo(np.float32).max)
    N = 16 * tiles
    W = np.zeros((4, K, K), dtype=np.float32)
    want = np.empty_like(X)
    for l in range(4):
        perm = rng.permutation(K)
        W[l, perm, np.arange(K)] = 1.0
        want[:, :, l * l:(l + 1) ** 2] = X[:, perm, l * l:(l + 1) ** 2]
    Xd, Wd, want = (torch.tensor(v, device="cuda:0") for v in (X, W, want))
    Y, dX, dW = torch.empty_like(Xd), torch.empty_like(Xd), torch.empty_like(Wd)
    cfg = el.make_config(K, K, 3)
    el.el_forward(cfg, N, Xd, Wd, Y)
    nbytes = el.el_workspace_bytes(cfg, N)
    el.el_backward(cfg, N, torch.zeros_like(Xd), Wd.transpose(1, 2).contiguous(), Xd, dX, dW,
                   torch.empty(nbytes, dtype=torch.uint8, device="cuda:0"), nbytes)
    for what, got in (("Y", Y), ("dX", dX)):
        wrong = (got != want).flatten(1).any(1).nonzero().flatten()
        assert wrong.numel() == 0, (what, wrong[:20].tolist())


# Such values where a workgroup makes several passes over its row tiles (625 tiles on a workgroup per CU: passes of two and of one), in the
# first tile of a pair, the second, the single one behind them and the last, ragged one: the rows of those tiles are the products in
# fp32, and those of every other tile, the other one of the pair included, keep their bits.  Columns 64 to 127 of W have one nonzero value, 1:
# there a small value comes back as it is.
@pytest.mark.parametrize("value", [1.2345e-36, float("inf"), 3.4e38])
def test_values_that_do_not_split_in_several_passes(el, value):
    import torch
    N, K = 9990, 128
    cus, tiles = torch.cuda.get_device_properties(0).multi_processor_count, -(-N // 16)
    starts = [tiles * r // cus for r in range(cus + 1)]
    threes = [a for a, b in zip(starts, starts[1:]) if b - a == 3]
    bad = [threes[0], threes[len(threes) // 3] + 1, threes[len(threes) // 2] + 2, tiles - 1]
    gen = torch.Generator(device="cuda").manual_seed(8910)
    X0 = torch.randn((N, K, 16), generator=gen, device="cuda")
    W = torch.randn((4, K, K), generator=gen, device="cuda") / K ** 0.5
    W[:, :, 64:] = 0
    for l in range(4):
        W[l, torch.randperm(K, generator=gen, device="cuda")[:64], torch.arange(64, 128, device="cuda")] = 1
    X = X0.clone()
    for t in bad:
        X[16 * t + 3, 7, 2] = value
    cfg = el.make_config(K, K, 3)
    nbytes = el.el_workspace_bytes(cfg, N)
    ws, dW, Wt = torch.empty(nbytes, dtype=torch.uint8, device="cuda"), torch.empty_like(W), W.transpose(1, 2).contiguous()

    def forward(x):
        Y = torch.empty_like(x)
        el.el_forward(cfg, N, x, W, Y)
        return Y

    def dx(x):                                   # dX of (Wt, dY = x) is the forward of (x, W)
        dX = torch.empty_like(x)
        el.el_backward(cfg, N, torch.zeros_like(x), Wt, x, dX, dW, ws, nbytes)
        return dX

    touched = torch.zeros(N, dtype=torch.bool, device="cuda")
    for t in bad:
        touched[16 * t:16 * t + 16] = True
    order = torch.tensor([int(c ** 0.5) for c in range(16)], device="cuda")
    rows = X[touched].double()
    ref = torch.stack([rows[:, :, c] @ W[order[c]].double() for c in range(16)], dim=2)
    for run in (forward, dx):
        clean, got = run(X0), run(X)
        assert torch.equal(got[~touched], clean[~touched]), run.__name__
        g = got[touched].double()
        assert torch.equal(g.isnan(), ref.isnan()) and torch.equal(g.isinf(), ref.isinf()), run.__name__
        fine = ref.isfinite() & (ref.abs() < 1e25)
        assert ((g - ref)[fine].abs().max() / ref[fine].square().mean().sqrt()).item() <= 1e-5
        if value < 1:
            assert torch.equal(g[:, 64:], ref[:, 64:]), run.__name__


# dW: ranges of atoms that end inside a chunk of four (the copies that fill it count nothing), and every launch that adds the ranges up: the
# product that reads W as it is and the one that reads it transposed, the workgroups of the products of split values that have
# a tile less than others (282 tiles on 256), all of them (257 and 511 on 256 within one tile of even), and a launch of its own.
@pytest.mark.parametrize("N,k_in,k_out,l_max,dtype", [
    (2, 128, 64, 3, "f32"), (17, 128, 128, 3, "f32"), (19, 256, 64, 3, "f32"), (1000, 128, 128, 3, "f32"), (1001, 64, 64, 2, "f64"),
    (4097, 128, 128, 3, "f32"), (4499, 128, 128, 3, "f32"), (8171, 128, 128, 3, "f32"), (2070, 64, 64, 1, "f32"), (1030, 192, 64, 0, "f64")])
def test_ranges_of_dw(el, N, k_in, k_out, l_max, dtype):
    assert not adds_ranges_in_a_launch_of_its_own(N, k_in, k_out, l_max, dtype)
    run_case(el, N, k_in, k_out, l_max, dtype, 8990 + N)


def adds_ranges_in_a_launch_of_its_own(N, k_in, k_out, l_max, dtype):
    """The library's choice of kernel for dX (columns: the input channels): on a tiled kernel the sum of the ranges cannot ride."""
    import torch
    cus, tiles = torch.cuda.get_device_properties(0).multi_processor_count, -(-N // 16)
    long_other = dtype == "f64" or (k_in > 64 and k_in % 128 != 0)
    small = tiles * (k_in // 16) <= (8 if long_other else 4) * cus
    units = tiles * (k_in // 128)
    parts = dtype == "f32" and l_max == 3 and k_in % 128 == 0 and k_out % 32 == 0 and (
        units <= 2 * cus or k_out > 64 or (k_out == 64 and (units > 5 * cus or units % cus == 0 or units % cus > cus // 2)))
    return not small and not parts


# ... whose workgroups take slices of 256 (fp64 128) values of dW in turn: one column group and several, more slices than one range has.
@pytest.mark.parametrize("N,k_in,k_out,l_max,dtype", [
    (8193, 128, 64, 3, "f32"), (4113, 64, 64, 3, "f32"), (2065, 128, 128, 2, "f32"), (4113, 128, 128, 3, "f64"), (8209, 64, 64, 1, "f64"),
    (4110, 64, 192, 0, "f32")])
def test_ranges_of_dw_added_in_a_launch_of_their_own(el, N, k_in, k_out, l_max, dtype):
    assert adds_ranges_in_a_launch_of_its_own(N, k_in, k_out, l_max, dtype)
    run_case(el, N, k_in, k_out, l_max, dtype, 8990 + N)


@pytest.mark.parametrize("N,k_in,k_out,l_max,dtype", [
    (1, 128, 128, 3, "f32"), (17, 64, 64, 0, "f32"), (63, 128, 64, 1, "f32"), (448, 128, 128, 3, "f32"), (449, 128, 128, 3, "f32"),
    (187, 256, 256, 3, "f32"), (188, 256, 256, 3, "f32"), (320, 64, 128, 2, "f64"), (321, 64, 128, 2, "f64"), (93, 256, 256, 1, "f64"),
    (5, 100, 128, 2, "f32"), (1024, 96, 96, 3, "f32"), (1025, 96, 96, 3, "f32"), (66, 7, 9, 3, "f64"), (34, 64, 96, 3, "f32"),
    (130, 300, 300, 0, "f32"), (16, 6, 20, 1, "f64"), (3, 33, 1, 3, "f32")])
def test_backward_of_small_batches_in_one_launch(el, N, k_in, k_out, l_max, dtype):
    run_case(el, N, k_in, k_out, l_max, dtype, 8700 + N + k_in)


# dX in the buffer of X, around the batches that have dX and dW in one launch otherwise; W's buffer as that of dW where the launch of
# dX reads W transposed (more than a workgroup of 16 atoms x 16 columns per compute unit).
@pytest.mark.parametrize("N,k_in,k_out,l_max,dtype,over_w", [
    (1, 64, 64, 3, "f32", False), (40, 128, 128, 3, "f32", False), (333, 128, 64, 3, "f32", False), (449, 128, 128, 3, "f32", False),
    (300, 64, 128, 1, "f64", False), (440, 256, 64, 3, "f32", True), (310, 256, 64, 2, "f64", True)])
def test_backward_in_place(el, N, k_in, k_out, l_max, dtype, over_w):
    import torch
    print(f"case N={N} k_in={k_in} k_out={k_out} l_max={l_max} {dtype} in place", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.float64
    X, W, dY = (torch.tensor(x, dtype=tdt, device="cuda:0") for x in workloads.make_linear_inputs(N, k_in, k_out, l_max, 8990 + N))
    dX_ref, dW_ref = oel.backward(*(x.double().cpu().numpy() for x in (X, W, dY)))
    cfg = el.make_config(k_in, k_out, l_max, el.SC_F32 if dtype == "f32" else el.SC_F64)
    nbytes = el.el_workspace_bytes(cfg, N)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
    dW = W if over_w else torch.full_like(W, float("nan"))
    el.el_backward(cfg, N, X, W, dY, X, dW, ws, nbytes)
    torch.cuda.synchronize()
    check("dX", X.cpu().numpy(), dX_ref, dtype)
    check("dW", dW.cpu().numpy(), dW_ref, dtype)


def test_infinite_row_at_the_end_of_a_range(el):
    import torch
    N, K = 5, 128
    X, _, dY = workloads.make_linear_inputs(N, K, K, 3, 8995)
    dY[N - 1, 3, 2], X[N - 1, 9, 5] = np.inf, -np.inf
    Xd, dYd = (torch.tensor(x, dtype=torch.float32, device="cuda:0") for x in (X, dY))
    Wd, dX, dW = torch.zeros((4, K, K), device="cuda:0"), torch.empty_like(Xd), torch.empty((4, K, K), device="cuda:0")
    cfg = el.make_config(K, K, 3)
    nbytes = el.el_workspace_bytes(cfg, N)
    el.el_backward(cfg, N, Xd, Wd, dYd, dX, dW, torch.empty(nbytes, dtype=torch.uint8, device="cuda:0"), nbytes)
    got = dW.double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = oel.backward(Xd.double().cpu().numpy(), Wd.double().cpu().numpy(), dYd.double().cpu().numpy())[1]
    assert np.isinf(ref).any() and not np.isnan(ref).any()
    assert (np.isinf(got) == np.isinf(ref)).all() and (got[np.isinf(ref)] == ref[np.isinf(ref)]).all()


def test_degenerate_sizes_and_errors(el):
    import torch
    run_case(el, 1, 128, 128, 3, "f32", 8501)
    run_case(el, 16, 128, 128, 3, "f32", 8502)
    cfg = el.make_config(128, 128, 3)
    dW = torch.full((4, 128, 128), float("nan"), device="cuda:0")
    el.el_forward(cfg, 0, None, None, None)
    el.el_backward(cfg, 0, None, None, None, None, dW, None, 0)
    torch.cuda.synchronize()
    assert not dW.cpu().numpy().any()
    X = torch.zeros((8, 128, 16), device="cuda:0")
    W = torch.zeros((4, 128, 128), device="cuda:0")
    with pytest.raises(el.ScError) as e:
        el.el_backward(cfg, 8, X, W, X, X.clone(), dW, None, 0)
    assert e.value.status == 3
    with pytest.raises(el.ScError) as e:
        el.el_forward(cfg, 8, X.data_ptr() + 4, W, X.clone())
    assert e.value.status == 1


def test_full_size(el):
    # the shape bench.py times: 10 000 atoms, 128 -> 128 channels, l <= 3
    run_case(el, 10_000, 128, 128, 3, "f32", 8601)
