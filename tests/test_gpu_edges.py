"""Edges of the output tiles and K-steps: token and feature counts that leave a
part of a 256 x 256 tile, of a thin tile or of a 64-wide K-step empty.

Rows and columns past the tensors are copied from the last one that exists, so
every output at an edge is compared with the oracle on its own tile (2e-2, the
bar of the bf16 parity tests), W is unpruned with Inf and NaN at dropped
positions, and the outputs sit between poisoned guards.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import lors as olors  # noqa: E402
from paper_2501_08582_amd import ops, synth  # noqa: E402
from gpu_helpers import TOL, dev_to_f64, to_dev, to_f64, unprune, worst_tile  # noqa: E402
import split_rule  # noqa: E402

pytestmark = pytest.mark.gpu

FMT = {"magnitude": ops.BITMAP, "2:4": ops.TWO_FOUR}
GUARD = 4096


def _guarded(shape, dtype):
    n = int(np.prod(shape)) * torch.tensor([], dtype=dtype).element_size()
    buf = torch.full((2 * GUARD + n,), 0xA5, dtype=torch.uint8, device="cuda")
    buf[GUARD:GUARD + n] = 0xFF  # NaN
    return buf, buf[GUARD:GUARD + n].view(dtype).view(shape)


# R a multiple of 64: fixed copies in dX; R % 64 = 8: its last K-step checks its
# lanes.  The forward has few tokens but where noted.
@pytest.mark.parametrize("R,C,L,r,mask,scale", [
    (64, 64, 1, 16, "magnitude", 2.0),        # one token, one K-step, a quarter of a tile
    (320, 192, 63, 5, "2:4", 2.0),            # below one token K-step of the weight gradient
    (192, 448, 65, 16, "magnitude", 0.3),     # two token K-steps, 63 rows shared
    (448, 576, 129, 40, "2:4", 0.5),
    (264, 192, 200, 8, "magnitude", 2.0),     # dX: checked copies, thin
    (192, 264, 321, 64, "magnitude", 1.5),
    (1032, 1096, 130, 24, "2:4", 2.0),        # the same, odd feature halves
    (4160, 4224, 513, 16, "magnitude", 2.0),  # forward and dX: 128-token thin tiles, the last of one token
    (256, 256, 300, 100, "magnitude", 2.0),   # ranks above 64
    (264, 328, 193, 72, "2:4", 0.3),
    (4096, 192, 1100, 24, "magnitude", 2.0),  # forward: a grid of 192-token thin tiles
    (192, 4160, 1090, 24, "2:4", 1.5),        # dX: the same
    (200, 4096, 1100, 128, "2:4", 2.0),       # dX: the same above rank 64, checked copies
    (320, 4160, 2300, 128, "magnitude", 1.0), # dX: a wave of feature halves, then thinner tiles; forward: thin
])
def test_edges(R, C, L, r, mask, scale):
    name = "llama2_7b_up_proj_2_4" if mask == "2:4" else "llama2_7b_q_proj"
    inp = synth.make(synth.workload(name).with_(R=R, C=C, r=r, scale=scale, seed=4000 + L), L=L)
    inp.W = unprune(inp.W, inp.M, "bf16", seed=L)
    X, W, B, A, dY = (to_dev(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A, inp.dY))
    M = ops.mask_pack(torch.from_numpy(inp.M).cuda(), FMT[mask])
    print("edges", (R, C, L, r, mask, scale), flush=True)
    bufs = {"Y": _guarded((L, R), torch.bfloat16), "dX": _guarded((L, C), torch.bfloat16),
            "dB": _guarded((R, r), torch.float32), "dA": _guarded((r, C), torch.float32)}
    out = {k: v[1] for k, v in bufs.items()}
    ops.forward(X, W, M, B, A, scale, FMT[mask], out=out["Y"])
    ops.backward(dY, X, W, M, B, A, scale, FMT[mask], out=(out["dX"], out["dB"], out["dA"], None))
    torch.cuda.synchronize()
    x, w, b, a, dy = (to_f64(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A, inp.dY))
    rdX, rdB, rdA, _ = olors.backward(dy, x, w, inp.M, b, a, scale)
    want = {"Y": olors.forward(x, w, inp.M, b, a, scale), "dX": rdX, "dB": rdB, "dA": rdA}
    for k, (buf, view) in bufs.items():
        n = view.numel() * view.element_size()
        assert torch.all(buf[:GUARD] == 0xA5) and torch.all(buf[GUARD + n:] == 0xA5), f"{k}: a guard byte changed"
        got = dev_to_f64(view)
        assert np.all(np.isfinite(got)), f"{k}: not finite"
        err, at = worst_tile(got, want[k], (64, 64))
        assert err <= TOL["bf16"], f"{k} block {at}: rel err {err:.3e}"


# the kernel for few tokens: 16- and 32-feature workgroups, each token block,
# each rank bucket, contractions below, at and past one block per wave, with
# and without a ragged last block; the last row of a case is past the rule
# (its 65 tokens run as thin tiles)
@pytest.mark.parametrize("R,C,L,r,mask,scale", [
    (8, 8, 1, 1, "magnitude", 2.0),
    (40, 64, 16, 16, "2:4", 0.5),
    (4096, 1024, 17, 32, "magnitude", 1.5),
    (264, 2120, 33, 48, "2:4", 2.0),
    (1024, 584, 64, 64, "magnitude", 2.0),
    (520, 1096, 65, 90, "2:4", 0.1),
    (256, 1096, 130, 128, "magnitude", 2.0),
    (8200, 328, 9, 12, "2:4", 2.0),
    (8232, 640, 31, 64, "magnitude", 1.0),
    (8264, 1152, 20, 32, "magnitude", 2.0),
    (8192, 72, 32, 128, "magnitude", 2.0),
    (8192, 192, 65, 16, "magnitude", 2.0),
])
def test_few_tokens_forward(R, C, L, r, mask, scale):
    name = "llama2_7b_up_proj_2_4" if mask == "2:4" else "llama2_7b_q_proj"
    inp = synth.make(synth.workload(name).with_(R=R, C=C, r=r, scale=scale, seed=5000 + R + L), L=L)
    inp.W = unprune(inp.W, inp.M, "bf16", seed=L)
    bias = synth.f32_to_bf16_bits(np.random.default_rng(L).standard_normal(R).astype(np.float32) * 0.1)
    X, W, B, A, bt = (to_dev(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A, bias))
    M = ops.mask_pack(torch.from_numpy(inp.M).cuda(), FMT[mask])
    print("few tokens", (R, C, L, r, mask, scale), flush=True)
    buf, Y = _guarded((L, R), torch.bfloat16)
    ops.forward(X, W, M, B, A, scale, FMT[mask], bias=bt, out=Y)
    again = ops.forward(X, W, M, B, A, scale, FMT[mask], bias=bt)
    torch.cuda.synchronize()
    n = Y.numel() * 2
    assert torch.all(buf[:GUARD] == 0xA5) and torch.all(buf[GUARD + n:] == 0xA5), "a guard byte changed"
    assert torch.equal(Y, again)  # the waves' partial sums are added in a fixed order
    x, w, b, a = (to_f64(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A))
    err, at = worst_tile(dev_to_f64(Y), olors.forward(x, w, inp.M, b, a, scale, to_f64(bias, "bf16")), (32, 32))
    assert err <= TOL["bf16"], f"block {at}: rel err {err:.3e}"


def test_two_four_rows_past_the_output_features_are_dropped():
    """R is no multiple of 32: the weight gradient's tile has rows past R,
    computed from repeated columns of dY.  An infinity in the last column of
    dY may reach dA only where the last row's mask keeps an entry."""
    R, C, L, r = 264, 256, 128, 16
    inp = synth.make(synth.workload("llama2_7b_up_proj_2_4").with_(R=R, C=C, r=r, seed=6000), L=L)
    X, W, B, A, dY = (to_dev(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A, inp.dY))
    dY[5, R - 1] = float("inf")
    M = ops.mask_pack(torch.from_numpy(inp.M).cuda(), ops.TWO_FOUR)
    dA = ops.backward(dY, X, W, M, B, A, 2.0, ops.TWO_FOUR, need_dx=False)[2]
    dropped = torch.from_numpy(inp.M[R - 1] == 0).cuda()
    assert torch.isfinite(dA[:, dropped]).all()
    assert not torch.isfinite(dA[:, ~dropped]).any()


# fp32: 32 x 32 tiles and 32-wide k blocks, each rank-pair bucket, more blocks
# than waves; sums of up to 600 products in another order stay within 1e-5
@pytest.mark.parametrize("R,C,L,r,mask,scale", [
    (4, 4, 1, 1, "random", 2.0), (32, 36, 31, 8, "2:4", 1.5), (100, 300, 33, 9, "random", 0.3),
    (36, 600, 97, 32, "2:4", 2.0), (132, 68, 300, 64, "random", 1.0), (68, 132, 65, 101, "2:4", 0.5),
])
def test_fp32_edges(R, C, L, r, mask, scale):
    wl = synth.workload("fp32_256x256_r8").with_(R=R, C=C, r=r, mask=mask, scale=scale, seed=7000 + R)
    inp = synth.make(wl, L=L)
    inp.W = unprune(inp.W, inp.M, "f32", seed=R)
    fmt = ops.TWO_FOUR if mask == "2:4" else ops.BITMAP
    X, W, B, A, dY = (to_dev(t, "f32") for t in (inp.X, inp.W, inp.B, inp.A, inp.dY))
    M = ops.mask_pack(torch.from_numpy(inp.M).cuda(), fmt)
    bias = np.random.default_rng(R).standard_normal(R).astype(np.float32)
    Y = ops.forward(X, W, M, B, A, scale, fmt, bias=to_dev(bias, "f32"))
    dX, dB, dA, dbias = ops.backward(dY, X, W, M, B, A, scale, fmt, need_dbias=True)
    x, w, b, a, dy = (np.asarray(t, np.float64) for t in (inp.X, inp.W, inp.B, inp.A, inp.dY))
    ref = olors.backward(dy, x, w, inp.M, b, a, scale, with_bias=True)
    for k, got, want in zip(("Y", "dX", "dB", "dA", "dbias"), (Y, dX, dB, dA, dbias),
                            (olors.forward(x, w, inp.M, b, a, scale, np.asarray(bias, np.float64)), *ref)):
        err, at = worst_tile(dev_to_f64(got), want, (32, 32))
        assert err <= TOL["f32"], f"{k} block {at}: rel err {err:.3e}"


# mask derivation and packing: whole-word rows (vector loads, a last wave of
# words that is not full) and rows that end inside a word, of which all, some
# or one in sixteen start on a 16-byte vector
@pytest.mark.parametrize("dtype", [torch.uint8, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("R,C,fmt", [(1, 32, ops.BITMAP), (3, 352, ops.TWO_FOUR), (67, 96, ops.BITMAP),
                                     (65, 1024, ops.TWO_FOUR), (5, 36, ops.TWO_FOUR), (9, 1000, ops.BITMAP),
                                     (35, 112, ops.TWO_FOUR), (7, 85, ops.BITMAP)])
def test_mask_words(dtype, R, C, fmt):
    from oracle import masks as omasks
    rng = np.random.default_rng(R + C)
    keep = rng.random((R, C)) < 0.5
    if fmt == ops.TWO_FOUR:
        keep = (rng.random((R, C // 4, 4)).argsort(2) < 2).reshape(R, C)
    val = torch.from_numpy(rng.integers(1, 200, (R, C))).to(dtype) * torch.from_numpy(keep).to(dtype)
    if dtype != torch.uint8:
        val = torch.where(torch.from_numpy(rng.random((R, C)) < 0.5), -val, val)  # -0 counts as zero
    M = ops.mask_pack(val.cuda(), fmt) if dtype == torch.uint8 else ops.mask_from_weight(val.cuda(), fmt)
    pack = omasks.pack_2_4 if fmt == ops.TWO_FOUR else omasks.pack_bitmap
    assert np.array_equal(M.cpu().numpy().view(np.uint32).reshape(-1), np.asarray(pack(keep.astype(np.uint8))).reshape(-1))
    if fmt == ops.TWO_FOUR:  # the first bad group, wherever it lies
        g = int(rng.integers(R * (C // 4)))
        val.view(R * C // 4, 4)[g] = 0
        with pytest.raises(ValueError, match=f"row {g // (C // 4)}, group {g % (C // 4)}"):
            ops.mask_pack(val.cuda(), fmt) if dtype == torch.uint8 else ops.mask_from_weight(val.cuda(), fmt)


@pytest.mark.parametrize("na,nb", [(0, 5), (1, 0), (3, 4), (4096, 257), (1 << 20, 1 << 21)])
def test_round_bf16(na, nb):
    from paper_2501_08582_amd import _lib
    g = torch.Generator(device="cuda").manual_seed(na + nb)
    a, b = (torch.randn(n, generator=g, device="cuda") for n in (na, nb))
    if na > 2:
        a[:3] = torch.tensor([float("inf"), 2.0 ** -140, 1.00390625], device="cuda")  # the last one a tie
    (ba, oa), (bb, ob) = (_guarded((n,), torch.bfloat16) for n in (na, nb))
    _lib.check(_lib.round_bf16(a.data_ptr() if na else None, na, oa.data_ptr() if na else None,
                               b.data_ptr() if nb else None, nb, ob.data_ptr() if nb else None,
                               torch.cuda.current_stream().cuda_stream), "lors_round_bf16")
    for buf, out, want in ((ba, oa, a), (bb, ob, b)):
        assert torch.equal(out, want.to(torch.bfloat16))
        assert torch.all(buf[:GUARD] == 0xA5) and torch.all(buf[GUARD + 2 * out.numel():] == 0xA5)


# the transposed mask, through the weight gradient it masks: rows and columns
# that end inside a word, a pair of words and a workgroup's 16 words
@pytest.mark.parametrize("R,C,mask", [(8, 8, "magnitude"), (72, 520, "2:4"), (96, 48, "magnitude"), (136, 1032, "2:4"),
                                      (64, 2048, "2:4"), (1000, 40, "magnitude")])
def test_transposed_mask(R, C, mask):
    name = "llama2_7b_up_proj_2_4" if mask == "2:4" else "llama2_7b_q_proj"
    inp = synth.make(synth.workload(name).with_(R=R, C=C, r=8, seed=8000 + R), L=32)
    X, W, B, A, dY = (to_dev(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A, inp.dY))
    M = ops.mask_pack(torch.from_numpy(inp.M).cuda(), FMT[mask])
    _, dB, dA, _ = ops.backward(dY, X, W, M, B, A, 2.0, FMT[mask], need_dx=False)
    x, w, b, a, dy = (to_f64(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A, inp.dY))
    _, rdB, rdA, _ = olors.backward(dy, x, w, inp.M, b, a, 2.0)
    for k, got, want in (("dB", dB, rdB), ("dA", dA, rdA)):
        err, at = worst_tile(dev_to_f64(got), want, (8, 8))
        assert err <= TOL["bf16"], f"{k} block {at}: rel err {err:.3e}"


# Shapes with an edge form W + s.B.A with s outside the bf16 operands, whatever
# the scale: here s.B (or s.A) is past bf16's largest number, s.B.A is not.
# Thin tiles in both directions, then whole tiles of the forward and of dX.
@pytest.mark.parametrize("R,C,L", [(576, 576, 2056), (2112, 64, 4168), (64, 2112, 4168)])
@pytest.mark.parametrize("large", ["B", "A"])
def test_edge_tiles_keep_the_scale_out_of_bf16(R, C, L, large):
    s, r, rng = 4.0, 8, np.random.default_rng(L + R)
    f = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    u = lambda *shape: (rng.uniform(1, 1.9, shape) * rng.choice([-1, 1], shape)).astype(np.float32)
    up, down = np.float32(2.0 ** 126), np.float32(2.0 ** -126)
    Bv, Av = u(R, r) * (up if large == "B" else down), u(r, C) * (down if large == "B" else up)
    Mk = (rng.random((R, C)) < 0.5).astype(np.uint8)
    X, W, B, A, dY = (synth.f32_to_bf16_bits(v) for v in (f(L, C), f(R, C) * Mk, Bv, Av, f(L, R)))
    Xt, Wt, Bt, At, dYt = (to_dev(t, "bf16") for t in (X, W, B, A, dY))
    M = ops.mask_pack(torch.from_numpy(Mk).cuda(), ops.BITMAP)
    print("scale outside", (R, C, L, large), flush=True)
    Y = ops.forward(Xt, Wt, M, Bt, At, s)
    dX = ops.backward(dYt, Xt, Wt, M, Bt, At, s)[0]  # (dB and dA do leave their range)
    x, w, b, a, dy = (to_f64(t, "bf16") for t in (X, W, B, A, dY))
    Wm = np.where(Mk, w + s * (b @ a), 0.0)
    for k, got, want in (("Y", Y, x @ Wm.T), ("dX", dX, dy @ Wm)):
        got = dev_to_f64(got)
        assert np.all(np.isfinite(got)), f"{k}: not finite"
        err, at = worst_tile(got, want, (64, 64))
        assert err <= TOL["bf16"], f"{k} block {at}: rel err {err:.3e}"


@pytest.mark.parametrize("fmt", [ops.BITMAP, ops.TWO_FOUR])
@pytest.mark.parametrize("R,C", [(36, 36), (100, 68), (68, 300)])
def test_fp32_blocks_past_the_tensors_keep_nothing(R, C, fmt):
    """R and C end inside a 32-wide k block.  A column of A that is not finite
    and that the mask drops from every row leaves dX exactly 0 there, and an
    infinite row of B gives Y an infinity: no NaN comes from the block's end."""
    L, r = 40, 8
    rng = np.random.default_rng(R + C)
    Mk = np.tile(np.array([0, 1, 1, 0], np.uint8), (R, C // 4))  # drops every column n with n % 4 in (0, 3)
    f = lambda *shape: np.abs(rng.standard_normal(shape)).astype(np.float32) + np.float32(0.1)
    X, W, B, A, dY = f(L, C), f(R, C) * Mk, f(R, r), f(r, C), f(L, R)
    M = ops.mask_pack(torch.from_numpy(Mk).cuda(), fmt)
    Xt, Wt, dYt = (to_dev(t, "f32") for t in (X, W, dY))
    Ainf = A.copy()
    Ainf[0, 0::4], Ainf[1, 3::4] = np.inf, np.nan
    dX = dev_to_f64(ops.backward(dYt, Xt, Wt, M, to_dev(B, "f32"), to_dev(Ainf, "f32"), 1.5, fmt)[0])
    assert np.all(dX[:, 0::4] == 0) and np.all(dX[:, 3::4] == 0)
    ref = olors.backward(*(np.asarray(t, np.float64) for t in (dY, X, W)), Mk, B.astype(np.float64),
                         A.astype(np.float64), 1.5)[0]
    assert worst_tile(dX, ref, (32, 32))[0] <= TOL["f32"]
    Binf = B.copy()
    Binf[R - 1, 2] = np.inf
    Y = dev_to_f64(ops.forward(Xt, Wt, M, to_dev(Binf, "f32"), to_dev(A, "f32"), 1.5, fmt))
    assert np.all(Y[:, R - 1] == np.inf) and np.all(np.isfinite(Y[:, :R - 1]))


# tile forward: a last K-step that ends past C, as thin tiles and as whole ones;
# few tokens
@pytest.mark.parametrize("R,L", [(520, 2056), (2112, 4168), (520, 40)])
@pytest.mark.parametrize("fmt", [ops.BITMAP, ops.TWO_FOUR])
def test_columns_past_the_contraction_keep_nothing(R, L, fmt):
    """An infinite row of B gives Y an infinity: no NaN comes from the columns
    past C of the last K-step."""
    C, r = 72, 8
    rng = np.random.default_rng(R + L)
    Mk = np.tile(np.array([0, 1, 1, 0], np.uint8), (R, C // 4))
    f = lambda *shape: np.abs(rng.standard_normal(shape)).astype(np.float32) + np.float32(0.1)
    B = f(R, r)
    B[R - 1, 2] = np.inf
    X, W, B, A = (to_dev(synth.f32_to_bf16_bits(v), "bf16") for v in (f(L, C), f(R, C) * Mk, B, f(r, C)))
    Y = ops.forward(X, W, ops.mask_pack(torch.from_numpy(Mk).cuda(), fmt), B, A, 1.5, fmt)
    assert torch.all(Y[:, R - 1] == float("inf")) and torch.isfinite(Y[:, :R - 1]).all()


# Every instance of the tile kernels of Y and dX: whole tiles and each thin one,
# each kind of copy and merge, at a rank of each 16-wide rank block (5 and 100
# also fill up an 8-rank chunk).  Sizes as (tokens, output features) with the
# kernels they are meant to run (up to rank 64 and above), on whole tiles and
# with edges; 320 or 328 features are contracted (5 K-steps, or 6 of which the
# last one holds 8 and checks its lanes).
TILE_SIZES = {
    "64": ((1024, 2048), (1000, 2040), {64}, {64}),
    "128": ((1024, 4096), (520, 4168), {128}, {128}),
    "192": ((1536, 4096), (1531, 4088), {192}, {192}),
    "256": ((2048, 4096), (2040, 4088), {256}, {256}),
    "whole": ((2304, 4096), (2060, 4168), {"whole"}, {256, 64}),
}


@pytest.mark.parametrize("copies", ["folded", "unfolded", "edges", "checked"])
@pytest.mark.parametrize("tile", list(TILE_SIZES))
@pytest.mark.parametrize("kind", ["fwd", "dx"])
def test_tile_kernels(kind, tile, copies):
    whole, edges, low, high = TILE_SIZES[tile]
    L, N = whole if copies in ("folded", "unfolded") else edges
    K, s = (328 if copies == "checked" else 320), (0.3 if copies == "unfolded" else 2.0)
    R, C = (N, K) if kind == "fwd" else (K, N)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    mask = "2:4" if copies in ("unfolded", "checked") else "magnitude"
    name = "llama2_7b_up_proj_2_4" if mask == "2:4" else "llama2_7b_q_proj"
    inp = synth.make(synth.workload(name).with_(R=R, C=C, r=128, scale=s, seed=9000 + L + K), L=L)
    inp.W = unprune(inp.W, inp.M, "bf16", seed=N)
    bias = synth.f32_to_bf16_bits(np.random.default_rng(L).standard_normal(R).astype(np.float32) * 0.1)
    X, W, bt, dY = (to_dev(t, "bf16") for t in (inp.X, inp.W, bias, inp.dY))
    M = ops.mask_pack(torch.from_numpy(inp.M).cuda(), FMT[mask])
    x, w, bb, dy = (to_f64(t, "bf16") for t in (inp.X, inp.W, bias, inp.dY))
    for r in (5, 24, 48, 64, 72, 96, 100, 128):
        print("tile kernels", kind, (R, C, L, r), tile, copies, flush=True)
        if cus == 256:
            assert split_rule.kernels(kind, L, R, C, r) == (low if r <= 64 else high, copies == "checked")
        assert (split_rule.fwd_whole_tiles if kind == "fwd" else split_rule.dx_whole_tiles)(L, R, C) == (
            copies in ("folded", "unfolded"))
        Bh, Ah = np.ascontiguousarray(inp.B[:, :r]), inp.A[:r]
        B, A = to_dev(Bh, "bf16"), to_dev(Ah, "bf16")
        buf, out = _guarded((L, N), torch.bfloat16)
        if kind == "fwd":
            ops.forward(X, W, M, B, A, s, FMT[mask], bias=bt, out=out)
        else:
            dB, dA = (torch.empty(shape, device="cuda") for shape in ((R, r), (r, C)))
            ops.backward(dY, X, W, M, B, A, s, FMT[mask], out=(out, dB, dA, None))
        torch.cuda.synchronize()
        assert torch.all(buf[:GUARD] == 0xA5) and torch.all(buf[GUARD + 2 * L * N:] == 0xA5), "a guard byte changed"
        Wm = olors.merged_weight(w, inp.M, to_f64(Bh, "bf16"), to_f64(Ah, "bf16"), s)
        want = x @ Wm.T + bb if kind == "fwd" else dy @ Wm
        got = dev_to_f64(out)
        assert np.all(np.isfinite(got)), f"rank {r}: not finite"
        err, at = worst_tile(got, want, (64, 64))
        assert err <= TOL["bf16"], f"rank {r}, block {at}: rel err {err:.3e}"


@pytest.mark.parametrize("R,C,L,r", [(256, 64, 768, 1), (264, 64, 200, 5), (512, 128, 256, 24), (72, 40, 33, 64), (256, 64, 256, 16)])
def test_sparse_mfma_first_k_steps(R, C, L, r):
    """The structured-sparse forward with one or two K-steps, where the first
    operands and accumulators are a large part of the result: the same bits on
    every call, whatever ran before, and the oracle's values."""
    inp = synth.make(synth.workload("llama2_7b_up_proj_2_4").with_(R=R, C=C, r=r, seed=6100 + R + r), L=L)
    inp.W = unprune(inp.W, inp.M, "bf16", seed=r)
    X, W, B, A = (to_dev(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A))
    M = ops.mask_pack(torch.from_numpy(inp.M).cuda(), ops.TWO_FOUR)
    first = ops.forward(X, W, M, B, A, 2.0, ops.TWO_FOUR, sparse_mfma=True)
    x, w, b, a = (to_f64(t, "bf16") for t in (inp.X, inp.W, inp.B, inp.A))
    err, at = worst_tile(dev_to_f64(first), olors.forward(x, w, inp.M, b, a, 2.0), (32, 32))
    assert err <= TOL["bf16"], f"block {at}: rel err {err:.3e}"
    for _ in range(8):
        ops.backward(first, X, W, M, B, A, 2.0, ops.TWO_FOUR)
        assert torch.equal(ops.forward(X, W, M, B, A, 2.0, ops.TWO_FOUR, sparse_mfma=True), first)
