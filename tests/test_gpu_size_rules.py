"""The sizes at which a launch rule changes kernels, or at which a kernel's own tiling leaves remainders, each against
the CPU oracle (or, where the oracle would take too long, an fp64 computation on the device)."""
import math

import numpy as np
import pytest
import torch

import oracle
from conftest import assert_rel_l2, to_np
from paper_2506_05096_amd import binding as ab

pytestmark = pytest.mark.gpu
DEV = "cuda"


# score: 16 tokens per workgroup below 28672 tokens (fp32 20480; 49152 where the arrays hold more than 256 MB), 64 per wave from
# there on; streaming loads above 256 MB, up to 24576 tokens above 200; slabs of 128 channels, four in flight, in fp32 two, or four of 64;
# a width that is no multiple of the 16-byte vector ends on single channels.  Bit-exact.
@pytest.mark.parametrize("n,c,stride,dtype", [
    (15, 128, 128, torch.bfloat16), (16, 256, 256, torch.bfloat16), (17, 384, 384, torch.bfloat16),      # 1 - 3 slabs
    (33, 512, 512, torch.bfloat16), (40, 640, 648, torch.bfloat16), (31, 1152, 1152, torch.bfloat16),    # 4, 5, 9 slabs
    (50, 515, 520, torch.bfloat16), (50, 1, 8, torch.bfloat16), (50, 130, 131, torch.bfloat16),          # ragged widths, element path
    (47, 63, 64, torch.float32), (48, 64, 64, torch.float32), (49, 321, 324, torch.float32), (20, 3, 4, torch.float32),
    (49151, 24, 24, torch.bfloat16), (49152, 24, 24, torch.bfloat16), (49153, 40, 40, torch.float32),
    (28671, 24, 24, torch.bfloat16), (28672, 24, 24, torch.bfloat16), (20479, 20, 20, torch.float32), (20480, 40, 40, torch.float32),
    (49151, 1371, 1376, torch.bfloat16), (49152, 1371, 1376, torch.bfloat16), (24576, 2136, 2136, torch.bfloat16),   # streaming
])
@pytest.mark.parametrize("mode", [ab.DELTA_L2, ab.DELTA_MEAN_ABS])
def test_score_sizes(n, c, stride, dtype, mode):
    g = torch.Generator().manual_seed(n + c)
    prev, cur = torch.randn(n, stride, generator=g).to(dtype), torch.randn(n, stride, generator=g).to(dtype)
    exp = oracle.score(to_np(cur)[:, :c], to_np(prev)[:, :c], mode)
    out = torch.full((n,), -1.0, device=DEV)
    ab.astraea_score(cur.to(DEV)[:, :c], prev.to(DEV)[:, :c], out, mode)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), exp.view(np.uint32))


# The chains run half a slab of 128 channels behind two tiles and four slabs in flight, in fp32 two: every pair of remainders, and a
# ragged last slab.
@pytest.mark.parametrize("slabs", range(6, 18))
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_score_ring(slabs, dtype):
    test_score_sizes(35, slabs * 128 - 5 * (slabs % 2), slabs * 128, dtype, ab.DELTA_L2)


# fp32 slabs of 64 channels, four in flight, above 8192 tokens, and of 128 up to there; the element path, whose chains read a quarter of a slab ahead.
@pytest.mark.parametrize("n,c,stride,dtype", [(8193, slabs * 64 - 4 * (slabs % 2), slabs * 64, torch.float32) for slabs in range(1, 10)] + [
    (8192, 512, 512, torch.float32), (8195, 321, 324, torch.float32)] + [
    (n, c, c + 1, dtype) for n, c in ((35, 1), (35, 127), (35, 128), (35, 255), (35, 300), (8193, 449)) for dtype in (torch.bfloat16, torch.float32)])
def test_score_slabs_by_tokens(n, c, stride, dtype):
    test_score_sizes(n, c, stride, dtype, ab.DELTA_MEAN_ABS)


# fp32 linear: 128-, 64- or 32-wide tiles by an estimate of the rounds they leave (32: the four waves split the contraction, and
# a 64-wide contraction leaves two of them without a stage); stages of 32 indices, four in flight, 128: of 16 in pairs.  `tile` is what the
# launch says it takes; each tile meets ragged rows and features and contractions that end inside the ring.  Bound: sums of c_in
# products of size ~1/sqrt(c_in) in fp32, error below c_in * 2^-24 / sqrt(c_in) * 4 <= 1e-4 absolute at c_in <= 4096.
@pytest.mark.parametrize("n,k,c_in,c_out,gather,scatter,bias,act,tile", [
    (40, 33, 64, 40, True, True, True, ab.ACT_NONE, 32),             # two stages for four waves
    (300, 31, 192, 104, True, False, False, ab.ACT_GELU_TANH, 32),   # six stages
    (300, 257, 448, 264, False, True, True, ab.ACT_NONE, 32),        # fourteen stages
    (1100, 1001, 512, 264, True, True, True, ab.ACT_NONE, 32),       # sixteen stages
    (2100, 2049, 128, 512, True, True, True, ab.ACT_NONE, 64),       # four stages, one row in the last tile
    (2100, 2016, 320, 520, True, False, True, ab.ACT_GELU_TANH, 64), # ten stages, eight features in the last tile
    (2100, 2047, 192, 2056, False, True, True, ab.ACT_NONE, 64),     # at the edge of a round of the 128 tile
    (4100, 4095, 64, 1032, True, True, True, ab.ACT_NONE, 64),       # two stages
    (2100, 2000, 320, 504, True, False, True, ab.ACT_GELU_TANH, 64), # ten stages
    (2100, 1985, 256, 456, False, True, False, ab.ACT_NONE, 64),     # eight stages, one row in the last tile
    (2100, 2048, 128, 2048, True, True, False, ab.ACT_NONE, 128),    # whole tiles, the ring once round
    (4100, 4000, 64, 1000, True, True, True, ab.ACT_GELU_TANH, 128), # two stages
    (4100, 4000, 192, 1000, False, True, True, ab.ACT_NONE, 128),    # six stages
    (4100, 3969, 448, 904, True, False, False, ab.ACT_NONE, 128),    # fourteen stages, one row and eight features in the last tile
])
def test_linear_f32_tiles(n, k, c_in, c_out, gather, scatter, bias, act, tile):
    assert ab.astraea_linear_plan(ab.F32, k, c_in, c_out)["tile_tokens"] == tile
    g = torch.Generator(device=DEV).manual_seed(n + k + c_in)
    idx = torch.randperm(n, device=DEV, generator=g)[:k].sort().values.to(torch.int32)
    x = torch.randn(n if gather else k, c_in, device=DEV, generator=g)
    w = torch.randn(c_out, c_in, device=DEV, generator=g) * c_in ** -0.5
    b = torch.randn(c_out, device=DEV, generator=g) if bias else None
    y = torch.randn(n if scatter else k, c_out + 8, device=DEV, generator=g)
    exp = y.double()
    ref = (x[idx.long()] if gather else x).double() @ w.double().T + (b.double() if bias else 0.0)
    if act == ab.ACT_GELU_TANH:
        ref = torch.nn.functional.gelu(ref, approximate="tanh")
    exp[idx.long() if scatter else slice(None), :c_out] = ref
    ab.astraea_sparse_linear(x, w, b, idx, k, y[:, :c_out], act=act, x_is_compact=not gather, y_is_compact=not scatter, N=n)
    torch.cuda.synchronize()
    assert (y.double() - exp).abs().max().item() <= 1e-4
    keep = torch.ones(y.shape, dtype=torch.bool, device=DEV)
    keep[idx.long() if scatter else slice(None), :c_out] = False
    assert torch.equal(y[keep].double(), exp[keep])


# Eight waves on 128 x 128 tiles (one round of them, and more where the contraction is deep) and on 64 features x 128 tokens: ragged rows and features, a feature tile of eight, a row
# in the last tile, stages that are no multiple of the register sets; the values that send a workgroup to fp32 products.  Bounds as above and below.
@pytest.mark.parametrize("n,k,c_in,c_out,gather,scatter,bias,act,features", [
    (3100, 3001, 512, 648, True, True, True, ab.ACT_GELU_TANH, 128), (3100, 2945, 576, 776, False, True, True, ab.ACT_NONE, 128),
    (3100, 3072, 1088, 768, True, False, False, ab.ACT_NONE, 128),
    (2100, 2000, 4160, 4104, True, True, True, ab.ACT_NONE, 128),                  # 528 tiles
    (1300, 1250, 512, 776, True, True, True, ab.ACT_NONE, 64), (1300, 1281, 576, 776, True, False, True, ab.ACT_GELU_TANH, 64),
    (1300, 1250, 640, 776, False, True, False, ab.ACT_NONE, 64), (3100, 3001, 512, 1288, True, True, True, ab.ACT_NONE, 64),
])
def test_linear_f32_halves(n, k, c_in, c_out, gather, scatter, bias, act, features):
    assert ab.astraea_linear_plan(ab.F32, k, c_in, c_out)["tile_features"] == features and ab.astraea_linear_waves(ab.F32, k, c_in, c_out) == 8
    test_linear_f32_tiles(n, k, c_in, c_out, gather, scatter, bias, act, 128)


@pytest.mark.parametrize("k,c_out,tile", [(100, 72, 32), (2000, 504, 64), (4000, 1000, 128)])
def test_linear_f32_operand_past_4_gib(k, c_out, tile):
    """Rows beyond the reach of a 32-bit byte offset: 4110 rows of 2 MiB pitch."""
    n, c_in = 4110, 64
    assert ab.astraea_linear_plan(ab.F32, k, c_in, c_out)["tile_tokens"] == tile
    g = torch.Generator(device=DEV).manual_seed(3)
    x = torch.empty(n, 1 << 19, device=DEV)[:, :c_in]
    x.copy_(torch.randn(n, c_in, device=DEV, generator=g))
    w = torch.randn(c_out, c_in, device=DEV, generator=g) * c_in ** -0.5
    idx = torch.arange(n - k, n, dtype=torch.int32, device=DEV)
    y = torch.empty(k, c_out, device=DEV)
    ab.astraea_sparse_linear(x, w, None, idx, k, y)
    torch.cuda.synchronize()
    assert (y.double() - x[n - k:].double() @ w.double().T).abs().max().item() <= 1e-4


# ... and contractions of 512 and more there, which keep the tiles that 32-bit offsets had before they took other kernels: 32 x 32 in four parts of the
# contraction, stages of 32 indices in turn.  A first product of 2^26 swallows every later one of 1 in its own part: 2^26 has a unit of 8.  So one part
# loses c_in - 1 and four lose a quarter, and 8 more by the last sums; then random terms, bound as above.
@pytest.mark.parametrize("k,c_in,c_out", [(1250, 512, 776), (1323, 4096, 1000)])
def test_linear_f32_parts_past_4_gib(k, c_in, c_out):
    n = 4110
    x = torch.empty(n, 1 << 19, device=DEV)[:, :c_in]
    x.fill_(1.0)
    x[:, 0] = 2.0 ** 26
    idx = torch.arange(n - k, n, dtype=torch.int32, device=DEV)
    y = torch.empty(k, c_out, device=DEV)
    ab.astraea_sparse_linear(x, torch.ones(c_out, c_in, device=DEV), None, idx, k, y)
    torch.cuda.synchronize()
    assert (y.double() - (2.0 ** 26 + c_in - 1)).abs().max().item() <= c_in / 4 + 8
    g = torch.Generator(device=DEV).manual_seed(k)
    x.copy_(torch.randn(n, c_in, device=DEV, generator=g))
    w = torch.randn(c_out, c_in, device=DEV, generator=g) * c_in ** -0.5
    ab.astraea_sparse_linear(x, w, None, idx, k, y)
    torch.cuda.synchronize()
    assert (y.double() - x[n - k:].double() @ w.double().T).abs().max().item() <= 1e-4


# fp32 linear, magnitudes of a whole operand or of part of the contraction: zeros at its start, growth and fall along it, the ends of the
# range, infinities, in the tiles that form products of bf16 parts.  Bound, of the sum of magnitudes: 2^-21 for
# the products and 2^-24 for each rounding of the sum, of which three per 16 indices are allowed here; either form stays below.
@pytest.mark.parametrize("k,c_in,c_out,tile", [(705, 1088, 1096, 64), (2049, 128, 512, 64), (1000, 64, 4096, 128), (1001, 320, 3976, 128)])
@pytest.mark.parametrize("values", ["plain", "w tiny", "x huge", "x grows", "x falls", "w starts at 0", "x is 0", "x inf"])
def test_linear_f32_split_range(k, c_in, c_out, tile, values):
    assert ab.astraea_linear_plan(ab.F32, k, c_in, c_out)["tile_tokens"] == tile
    g = torch.Generator(device=DEV).manual_seed(k + c_in)
    x, w = torch.randn(k, c_in, device=DEV, generator=g), torch.randn(c_out, c_in, device=DEV, generator=g)
    if values == "w tiny":
        w *= 2.0 ** -105
    elif values == "x huge":
        x *= 2.0 ** 90
    elif values == "x grows":
        x[:, 2 * c_in // 3:] *= 2.0 ** 20
    elif values == "x falls":
        x[:, 2 * c_in // 3:] *= 2.0 ** -20
    elif values == "w starts at 0":
        w[:, :c_in - 8] = 0.0
    elif values == "x is 0":
        x.zero_()
    elif values == "x inf":
        x[k // 2, 5] = math.inf
    y = torch.full((k, c_out), math.nan, device=DEV)
    ab.astraea_sparse_linear(x, w, None, None, k, y, x_is_compact=True, y_is_compact=True, N=k)
    torch.cuda.synchronize()
    if values == "x inf":
        assert torch.equal(y[k // 2], torch.copysign(torch.full_like(y[0], math.inf), w[:, 5]))
        x[k // 2], y[k // 2] = 0.0, 0.0
    ref, size = x.double() @ w.double().T, x.double().abs() @ w.double().abs().T
    bound = (2.0 ** -21 + c_in * 3 / 16 * 2.0 ** -24) * size + 2.0 ** -140
    assert bool(((y.double() - ref).abs() <= bound).all()), ((y.double() - ref).abs() / bound).max().item()


@pytest.mark.parametrize("k,c_in,c_out", [(3001, 512, 648), (1281, 576, 776)])
@pytest.mark.parametrize("values", ["plain", "w tiny", "x huge", "x grows", "x falls", "w starts at 0", "x is 0", "x inf"])
def test_linear_f32_halves_range(k, c_in, c_out, values):
    test_linear_f32_split_range(k, c_in, c_out, 128, values)


# fp32 linear in 64-wide tiles, whose waves hold half of every 32 contraction indices each: infinities that one half or both halves meet, and
# halves that cancel, of the smallest and of ragged contractions.  Bound as above: cancelling halves are exact to the sum of magnitudes.
@pytest.mark.parametrize("k,c_in,c_out", [(4095, 64, 1032), (2049, 128, 512), (2000, 320, 504)])
@pytest.mark.parametrize("channels,cancel", [((), True), ((3,), False), ((17,), False), ((0, 31), False), ((-1,), False)])
def test_linear_f32_halves_of_the_contraction(k, c_in, c_out, channels, cancel):
    assert ab.astraea_linear_plan(ab.F32, k, c_in, c_out)["tile_tokens"] == 64
    g = torch.Generator(device=DEV).manual_seed(k + c_in)
    x, w = torch.randn(k, c_in, device=DEV, generator=g), torch.randn(c_out, c_in, device=DEV, generator=g).abs() + 0.5
    if cancel:
        x = x.view(k, c_in // 32, 2, 16)
        x[:, :, 1] = -x[:, :, 0]
        x = x.reshape(k, c_in)
        w = w.view(c_out, c_in // 32, 2, 16)[:, :, :1].expand(-1, -1, 2, -1).reshape(c_out, c_in).contiguous()
    for c in channels:
        x[k // 2, c] = math.inf
    y = torch.full((k, c_out), math.nan, device=DEV)
    ab.astraea_sparse_linear(x, w, None, None, k, y, x_is_compact=True)
    torch.cuda.synchronize()
    if channels:
        assert bool((y[k // 2] == math.inf).all())
        x[k // 2], y[k // 2] = 0.0, 0.0
    bound = (2.0 ** -21 + c_in * 3 / 16 * 2.0 ** -24) * (x.double().abs() @ w.double().abs().T) + 2.0 ** -140
    assert bool(((y.double() - x.double() @ w.double().T).abs() <= bound).all())


# fp32 linear, magnitudes that differ between rows, between channels and inside a row: each result stands on its own row and feature
# alone.  Bound, elementwise, of the sum of magnitudes: 2^-22 for the products and 2^-24 for each rounding of the sum, eight per 16 indices.
@pytest.mark.parametrize("k,c_in,c_out,tile", [(300, 128, 264, 32), (705, 1088, 1096, 64), (2049, 128, 512, 64), (1000, 64, 4096, 128), (1001, 320, 3976, 128)])
@pytest.mark.parametrize("values", ["x rows", "w rows", "opposed", "outlier", "tiny x huge", "nan"])
def test_linear_f32_spread_magnitudes(k, c_in, c_out, tile, values):
    assert ab.astraea_linear_plan(ab.F32, k, c_in, c_out)["tile_tokens"] == tile
    g = torch.Generator(device=DEV).manual_seed(k + c_in)
    x, w = torch.randn(k, c_in, device=DEV, generator=g), torch.randn(c_out, c_in, device=DEV, generator=g)
    fall = {m: 2.0 ** -(torch.arange(m, device=DEV) % 24).float() for m in (k, c_in, c_out)}
    if values == "x rows":
        x *= fall[k][:, None]
    elif values == "w rows":
        w *= fall[c_out][:, None]
    elif values == "opposed":
        x, w = x * fall[c_in], w / fall[c_in]
    elif values == "outlier":
        x[5] *= 2.0 ** 40
        x[9, c_in - 1] = 2.0 ** 20
        w[7, 3] = -2.0 ** 30
    elif values == "tiny x huge":              # magnitudes near fp32's lowest, which lose bits in narrower parts
        x, w = x * 2.0 ** -(100 + torch.arange(k, device=DEV) % 24).float()[:, None], w * 2.0 ** 100
    elif values == "nan":
        x[k // 2, c_in - 1] = math.nan
    y = torch.full((k, c_out), math.inf, device=DEV)
    ab.astraea_sparse_linear(x, w, None, None, k, y, x_is_compact=True, y_is_compact=True, N=k)
    torch.cuda.synchronize()
    if values == "nan":
        assert bool(y[k // 2].isnan().all())
        x[k // 2], y[k // 2] = 0.0, 0.0
    ref, size = x.double() @ w.double().T, x.double().abs() @ w.double().abs().T
    bound = (2.0 ** -22 + c_in / 2 * 2.0 ** -24) * size + 2.0 ** -140
    assert bool(((y.double() - ref).abs() <= bound).all()), ((y.double() - ref).abs() / bound).max().item()
    if values == "x rows":                     # ... and not on the rows that share its tile
        grown = x * 2.0 ** 20
        grown[3] = x[3]
        z = torch.full_like(y, math.inf)
        ab.astraea_sparse_linear(grown, w, None, None, k, z, x_is_compact=True, y_is_compact=True, N=k)
        torch.cuda.synchronize()
        assert torch.equal(z[3], y[3])


@pytest.mark.parametrize("k,c_in,c_out", [(3001, 512, 648), (1281, 576, 776)])
@pytest.mark.parametrize("values", ["x rows", "w rows", "opposed", "outlier", "tiny x huge", "nan"])
def test_linear_f32_halves_magnitudes(k, c_in, c_out, values):
    test_linear_f32_spread_magnitudes(k, c_in, c_out, 128, values)


# bf16 attention: 256 queries per workgroup, 32 per wave (rows pass through LDS whole, four at a time), 64 keys per tile; the
# items of a partly filled round are cut into key shares where the launch's estimate says so, and `groups` is 1 where none of the launches in
# key groups takes the call.  `hot` plants one key whose logit overflows the first tile's offset, so that the workgroup repeats its
# sweep; compact queries may outnumber the keys.  Oracle: fp64 softmax; bar: relative L2 1e-2 per row and head.
@pytest.mark.parametrize("n,h,k,hot,scatter,splits", [
    (1, 1, 1, False, True, 1), (63, 2, 31, False, True, 1), (64, 1, 33, True, False, 1), (65, 3, 65, True, True, 1),
    (96, 3, 89, True, True, 1), (129, 4, 5000, True, False, 1), (300, 60, 300, False, True, 1), (512, 24, 2900, True, False, 1),
    (100, 2, 16384, True, False, 1), (100, 2, 16385, True, False, 1), (128, 1, 16385, False, False, 1),      # V direct, retiled
    (4000, 1, 30, True, True, 8), (4000, 3, 3000, True, True, 5), (4100, 24, 4000, False, False, 2), (4000, 12, 1400, True, True, 3),
    (1500, 8, 8449, True, False, 6), (2025, 12, 5700, True, False, 4), (3000, 24, 2800, True, True, None),                                # whole items and shares
])
def test_attn_bf16_tiles(n, h, k, hot, scatter, splits, groups=1):
    assert ab.astraea_attn_key_groups(n, h, k) == groups
    if splits is not None:
        assert ab.astraea_attn_plan(n, h, k)["splits"] == splits
    g = torch.Generator(device=DEV).manual_seed(n + h + k)
    q, kc, vc = (torch.randn(m, h, 128, device=DEV, generator=g).bfloat16() for m in (k, n, n))
    if hot:
        q[[0, k // 2, k - 1], :, 0] = 64.0
        kc[n - 1, :, 0] = 64.0                               # 362 nats above the rest for those rows
    idx = torch.randperm(max(n, k), device=DEV, generator=g)[:k].sort().values.to(torch.int32)
    scale = 1.0 / math.sqrt(128)
    lse = torch.full((k, h), math.nan, device=DEV)
    ws = torch.full((ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, 128),), 255, dtype=torch.uint8, device=DEV)
    out = torch.randn(n if scatter else k, h * 128 + 8, device=DEV, generator=g).bfloat16()
    before = out.clone()
    if scatter:
        ab.astraea_sparse_attn_update_fwd(q, kc, vc, idx, k, out[:, :h * 128], scale, q_is_compact=True, lse_sel=lse, workspace=ws)
        got = out[idx.long(), :h * 128]
    else:
        out = torch.empty(k, h, 128, dtype=torch.bfloat16, device=DEV)
        ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, out, scale, q_is_compact=True, lse_sel=lse, workspace=ws)
        got = out
    torch.cuda.synchronize()
    for i in range(h):
        logits = (q[:, i].double() @ kc[:, i].double().T.contiguous()) * scale
        ref = torch.softmax(logits, 1) @ vc[:, i].double()
        assert_rel_l2(got.view(k, h, 128)[:, i].double().cpu().numpy(), ref.cpu().numpy(), tag=f"head {i}")
        want = torch.logsumexp(logits, 1)
        # bf16 rounding of P averages out over the keys of a flat row and is absent where one key carries the row; single
        # tiles of a handful of keys can show all of it, 2^-9
        assert ((lse[:, i].double() - want).abs() / want.abs().clamp(min=1.0)).max().item() <= 2.0 ** -9
    if scatter:
        keep = torch.ones(out.shape, dtype=torch.bool, device=DEV)
        keep[idx.long(), :h * 128] = False
        assert torch.equal(out[keep], before[keep])


# Workgroups of four waves, 128 queries: where every half of an item gets a CU of its own (up to 256 halves), and in sweeps of up to 24 key
# tiles of more than 32 items per XCD, none of them cut.  Both sides of each line (`queries` is what the launch says), with rows that send a
# workgroup through its sweep again, a second half without queries, shares of halves, and one key tile; V direct and retiled.
@pytest.mark.parametrize("n,h,k,hot,scatter,queries,splits", [
    (300, 16, 2048, True, False, 128, 1), (2100, 16, 2049, True, True, 256, 1),
    (1536, 8, 10000, True, False, 128, 1), (1537, 8, 10000, True, False, 256, 1), (1536, 8, 8300, True, False, 256, 8),
    (60, 24, 3000, False, False, 128, 1), (65, 24, 2900, True, False, 128, 1), (64, 40, 1800, True, False, 128, 1),
    (96, 8, 128, True, False, 128, 1), (96, 8, 129, True, False, 128, 1), (300, 24, 1025, True, False, 128, 1), (300, 60, 300, True, True, 128, 1), (4000, 2, 300, True, True, 128, 8), (4200, 4, 4200, True, True, 256, 3),
    (1536, 4, 20000, True, False, 128, 1), (1537, 4, 20000, True, False, 256, 1), (77, 8, 17000, True, False, 128, 1),
])
def test_attn_bf16_half_workgroups(n, h, k, hot, scatter, queries, splits):
    assert ab.astraea_attn_plan(n, h, k)["queries_per_workgroup"] == queries
    test_attn_bf16_tiles(n, h, k, hot, scatter, splits)          # one key group


# Four-wave workgroups whose output rows lie over the second V buffer, all of them sweeping again (logits 90 nats above the first key tile's) with
# their last key tile in that buffer (even numbers of tiles) or in the first: values 2^10 times larger in the last tile show a wave
# that read anything else there.  V direct and retiled.  Bars as above.
@pytest.mark.parametrize("n,h,k", [(128, 8, 2000), (192, 16, 1024), (256, 16, 2048), (300, 24, 1000), (1472, 8, 10000), (1536, 8, 10000), (128, 4, 16500), (192, 4, 16500)])
def test_attn_bf16_half_workgroups_that_sweep_again(n, h, k):
    plan = ab.astraea_attn_plan(n, h, k)
    assert plan["queries_per_workgroup"] == 128 and plan["splits"] == 1 and ab.astraea_attn_key_groups(n, h, k) == 1
    q, kc, vc = _attn_rise_case(n, h, k, 128, 90.0, torch.bfloat16, 64)
    vc[n - 64:] *= 2.0 ** 10
    lse = torch.full((k, h), math.nan, device=DEV)
    out = torch.empty(k, h, 128, dtype=torch.bfloat16, device=DEV)
    ws = torch.full((ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, 128),), 255, dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, out, 1.0 / math.sqrt(128), q_is_compact=True, lse_sel=lse, workspace=ws)
    torch.cuda.synchronize()
    for i in range(h):
        logits = q[:, i].double() @ kc[:, i].double().T.contiguous() / math.sqrt(128)
        ref = torch.softmax(logits, 1) @ vc[:, i].double()
        assert_rel_l2(out[:, i].double().cpu().numpy(), ref.cpu().numpy(), tag=f"head {i}")
        want = torch.logsumexp(logits, 1)
        assert ((lse[:, i].double() - want).abs() / want.abs().clamp(min=1.0)).max().item() <= 2.0 ** -9


# Eight waves as two or four key groups (`groups` is what the launch says): one key block per group, uneven shares of the keys, ragged last tiles of
# keys and queries, query waves without rows, a full round, and rows that send the workgroup through its sweep again.  Next to them
# the shares that key groups leave to the merging launch, each number of them.  Bars as above.
@pytest.mark.parametrize("n,h,k,hot,scatter,groups,splits", [
    (97, 1, 1, False, True, 4, 1), (128, 3, 40, True, True, 4, 1), (129, 2, 65, True, True, 4, 1), (161, 5, 64, False, False, 4, 1),
    (223, 24, 255, True, False, 4, 1), (255, 16, 129, True, True, 4, 1), (1500, 24, 610, True, True, 4, None),
    (1028, 4, 4102, False, False, 2, 1), (1460, 16, 1460, True, True, 2, 1), (1089, 8, 3969, True, False, 2, 1), (1500, 2, 16384, False, False, 2, 1),
    (129, 2, 5000, True, False, 4, 1), (300, 1, 255, False, True, 4, 1), (512, 9, 257, True, True, 4, 1), (2025, 24, 608, True, True, 4, 3),
    (4100, 24, 1100, False, False, 2, 2), (900, 24, 450, True, True, 4, 1), (2048, 16, 2048, True, True, 2, 1), (500, 8, 128, True, True, 4, 1), (500, 8, 129, True, True, 4, 1),
    (130, 16, 2000, True, False, 1, 1), (3716, 12, 1400, True, True, 1, 3), (1762, 2, 2470, False, False, 1, 4), (957, 1, 41, True, True, 1, 5),
    (762, 1, 167, False, True, 1, 6), (2080, 1, 37, True, True, 1, 7), (1398, 1, 20, False, True, 1, 8),
])
def test_attn_bf16_key_groups(n, h, k, hot, scatter, groups, splits):
    test_attn_bf16_tiles(n, h, k, hot, scatter, splits, groups)


# Key groups that all sweep again, the first of them with logits 90 nats below the others' and its own later ones, or none but the first one's
# rows above its offset; queries by index, the compact result and the cached rows written at once.
@pytest.mark.parametrize("n,h,k", [(700, 8, 600), (161, 4, 161), (1460, 16, 1460), (1411, 16, 1400), (128, 8, 128), (192, 8, 190), (2048, 16, 2048)])
@pytest.mark.parametrize("rise_nats", [30.0, 90.0])
def test_attn_bf16_key_groups_that_sweep_again(n, h, k, rise_nats):
    assert ab.astraea_attn_key_groups(n, h, k) > 1
    q, kc, vc = _attn_rise_case(n, h, n, 128, rise_nats, torch.bfloat16, 32)
    vc[n - 32:] *= 2.0 ** 10
    g = torch.Generator(device=DEV).manual_seed(k)
    idx = torch.randperm(n, device=DEV, generator=g)[:k].sort().values.to(torch.int32)
    lse = torch.full((k, h), math.nan, device=DEV)
    out = torch.empty(k, h, 128, dtype=torch.bfloat16, device=DEV)
    cache = torch.randn(n, h * 128, device=DEV, generator=g).bfloat16()
    want_cache = cache.clone()
    ws = torch.full((ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, 128),), 255, dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_scatter_fwd(q, kc, vc, idx, k, out, cache, 1.0 / math.sqrt(128), lse_sel=lse, workspace=ws)
    torch.cuda.synchronize()
    want_cache[idx.long()] = out.view(k, -1)
    assert torch.equal(cache, want_cache)
    for i in range(h):
        logits = q[idx.long(), i].double() @ kc[:, i].double().T.contiguous() / math.sqrt(128)
        ref = torch.softmax(logits, 1) @ vc[:, i].double()
        assert_rel_l2(out[:, i].double().cpu().numpy(), ref.cpu().numpy(), tag=f"head {i}")
        want = torch.logsumexp(logits, 1)
        assert ((lse[:, i].double() - want).abs() / want.abs().clamp(min=1.0)).max().item() <= 2.0 ** -9


# Keys whose logits are minus infinity for some rows: all of a key group's or a key share's first tile, of the whole of it, of the first tile of all
# keys, of every key but the last.  They weigh nothing, as in softmax; the other rows see plain logits.  Four key groups, two, shares that a
# launch merges, four and eight waves on whole items, V retiled (`groups`, `splits`: what the launch says).  Bars as above.
@pytest.mark.parametrize("n,h,k,groups,splits", [(700, 8, 600, 4, 1), (1460, 16, 1460, 2, 1), (3716, 12, 1400, 1, 3), (130, 16, 2000, 1, 1),
                                                 (2100, 24, 4100, 1, 1), (300, 2, 16400, 1, 1)])
@pytest.mark.parametrize("where", ["first tile", "share's first tile", "share", "all but the last"])
def test_attn_bf16_logits_of_minus_infinity(n, h, k, groups, splits, where):
    plan = ab.astraea_attn_plan(n, h, k)
    assert ab.astraea_attn_key_groups(n, h, k) == groups and (groups > 1 or plan["splits"] == splits)
    unit = 32 if groups == 4 else 64
    tiles, parts = -(-n // unit), max(groups, splits)
    begin = tiles // parts * unit if groups > 1 else plan["tiles_per_split"] * unit % (n // 64 * 64)     # of the second group or share
    lo, hi = {"first tile": (0, 64), "share's first tile": (begin, begin + 64), "share": (begin, begin + max(tiles // parts, 1) * unit + unit),
              "all but the last": (0, n - 1)}[where]
    hi = min(hi, n - 1)
    g = torch.Generator(device=DEV).manual_seed(n + k)
    q, kc, vc = (torch.randn(m, h, 128, device=DEV, generator=g).bfloat16() for m in (k, n, n))
    q[:, :, 0], kc[:, :, 0] = 2.0 ** -126, 0.0
    q[::3, :, 0], kc[lo:hi, :, 0] = 64.0, -3e38
    lse = torch.full((k, h), math.nan, device=DEV)
    out = torch.empty(k, h, 128, dtype=torch.bfloat16, device=DEV)
    ws = torch.full((ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, 128),), 255, dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, out, 1.0 / math.sqrt(128), q_is_compact=True, lse_sel=lse, workspace=ws)
    torch.cuda.synchronize()
    for i in range(h):
        logits = q[:, i].double() @ kc[:, i].double().T.contiguous()
        logits = torch.where(logits < -3.4e38, -math.inf, logits) / math.sqrt(128)
        ref = torch.softmax(logits, 1) @ vc[:, i].double()
        assert_rel_l2(out[:, i].double().cpu().numpy(), ref.cpu().numpy(), tag=f"head {i}")
        want = torch.logsumexp(logits, 1)
        assert ((lse[:, i].double() - want).abs() / want.abs().clamp(min=1.0)).max().item() <= 2.0 ** -9


# The compact result and the cached rows from one call, against the two calls it stands for: whole and cut work items, both workgroup
# sizes, key groups (`groups`), cached buffers that the kernel writes itself and those that get a launch of their own (stride, alignment, memory shared with q).
@pytest.mark.parametrize("dtype,n,h,d,k,queries,splits,groups", [
    (torch.bfloat16, 2025, 24, 128, 608, 256, 3, 4), (torch.bfloat16, 2100, 16, 128, 2049, 256, 1, 1), (torch.bfloat16, 300, 3, 128, 77, 128, 1, 4),
    (torch.bfloat16, 300, 30, 128, 300, 128, 1, 4), (torch.bfloat16, 4000, 2, 128, 300, 128, 8, 1), (torch.bfloat16, 1460, 16, 128, 1460, 128, 1, 2),
    (torch.bfloat16, 3716, 12, 128, 1400, 256, 3, 1), (torch.bfloat16, 90, 3, 128, 77, 128, 1, 1), (torch.bfloat16, 300, 60, 128, 300, 128, 1, 1),
    (torch.float32, 700, 8, 64, 60, 128, 2, 0), (torch.float32, 97, 2, 128, 97, 128, 1, 0), (torch.float32, 2500, 8, 128, 2500, 256, 3, 0),
    (torch.float32, 2700, 24, 64, 2700, 256, 8, 0),
])
@pytest.mark.parametrize("cache", ["plain", "padded", "odd stride", "misaligned", "shares q"])
def test_attn_result_and_cached_rows(dtype, n, h, d, k, queries, splits, groups, cache):
    room = max(ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d), 256)
    plan = ab.astraea_attn_plan(n, h, k) if dtype == torch.bfloat16 else ab.astraea_attn_plan_f32(n, h, d, k, room)
    assert (plan["queries_per_workgroup"], plan["splits"]) == (queries, splits)
    assert dtype == torch.float32 or ab.astraea_attn_key_groups(n, h, k) == groups
    g = torch.Generator(device=DEV).manual_seed(n + k)
    e = h * d
    both = torch.randn(n, 2, e, device=DEV, generator=g).to(dtype)
    q = both[:, 0].view(n, h, d)
    kc, vc = (torch.randn(n, h, d, device=DEV, generator=g).to(dtype) for _ in range(2))
    base = both if cache == "shares q" else torch.randn((n + 3) * (e + 16), device=DEV, generator=g).to(dtype)

    def view(b):
        return {"plain": lambda: b[:n * e].view(n, e), "padded": lambda: b.view(n + 3, e + 16)[:, 8:8 + e],
                "odd stride": lambda: b[:n * (e + 3)].view(n, e + 3)[:, :e], "misaligned": lambda: b[1:1 + n * e].view(n, e),
                "shares q": lambda: b[:, 1]}[cache]()
    idx = torch.randperm(n, device=DEV, generator=g)[:k].sort().values.to(torch.int32)
    if cache == "padded":
        idx[-1] = n + 7                                      # outside the keys and the cached buffer: writes nothing there
    ws = torch.empty(room, dtype=torch.uint8, device=DEV)
    o0, lse0 = torch.empty(k, h, d, dtype=dtype, device=DEV), torch.empty(k, h, device=DEV)
    o1, lse1 = torch.empty_like(o0), torch.empty_like(lse0)
    want = base.clone()
    ab.astraea_sparse_attn_fwd(q, kc, vc, idx, k, o0, d ** -0.5, lse_sel=lse0, workspace=ws)
    ab.astraea_scatter_update(view(want), o0.view(k, e), idx, k)
    ab.astraea_sparse_attn_scatter_fwd(q, kc, vc, idx, k, o1, view(base), d ** -0.5, lse_sel=lse1, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(o0, o1) and torch.equal(lse0, lse1) and torch.equal(base, want)


def _attn_rise_case(n, h, k, d, rise_nats, dtype, first_tile):
    """Logits near zero, except that those of the first key tile lie `rise_nats` lower."""
    g = torch.Generator(device=DEV).manual_seed(n + k + d)
    q, kc = (0.05 * torch.randn(m, h, d, device=DEV, generator=g) for m in (k, n))
    q[:, :, 0], kc[:, :, 0] = 8.0, 0.0
    kc[:first_tile, :, 0] = -rise_nats * math.sqrt(d) / 8.0
    return q.to(dtype), kc.to(dtype), torch.randn(n, h, d, device=DEV, generator=g).to(dtype)


# V retiled (more than 16384 queries): packed cache and head-major strides, queries gathered by index, flat logits and logits
# that rise above the first key tile's inside and past the margin of the row sums.  Bars as above.
@pytest.mark.parametrize("layout,rise_nats", [("packed", 0.0), ("head", 0.0), ("packed", 20.0), ("head", 45.0), ("packed", 90.0)])
def test_attn_bf16_retiled_layouts_and_rises(layout, rise_nats):
    n, h, k = 16500, 2, 16400
    q, kc, vc = _attn_rise_case(n, h, n, 128, rise_nats, torch.bfloat16, 64)
    if layout == "packed":
        q, kc, vc = torch.stack((q, kc, vc), 1).unbind(1)
    else:
        q, kc, vc = (t.transpose(0, 1).contiguous().transpose(0, 1) for t in (q, kc, vc))
    assert kc.stride(0 if layout == "packed" else 1) == (3 * h * 128 if layout == "packed" else n * 128)
    g = torch.Generator(device=DEV).manual_seed(k)
    idx = torch.randperm(n, device=DEV, generator=g)[:k].sort().values.to(torch.int32)
    lse = torch.full((k, h), math.nan, device=DEV)
    ws = torch.full((ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, 128),), 255, dtype=torch.uint8, device=DEV)
    out = torch.empty(k, h, 128, dtype=torch.bfloat16, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, idx, k, out, 1.0 / math.sqrt(128), lse_sel=lse, workspace=ws)
    torch.cuda.synchronize()
    for i in range(h):
        logits = q[idx.long(), i].double() @ kc[:, i].double().T.contiguous() / math.sqrt(128)
        ref = torch.softmax(logits, 1) @ vc[:, i].double()
        assert_rel_l2(out[:, i].double().cpu().numpy(), ref.cpu().numpy(), tag=f"head {i}")
        want = torch.logsumexp(logits, 1)
        assert ((lse[:, i].double() - want).abs() / want.abs().clamp(min=1.0)).max().item() <= 2.0 ** -9


# Logits 45 nats above those of the first key tile, inside the margin of the row sums, over values of 2^66: the accumulators
# of the first sweep overflow.  Compact queries fewer and more than the keys, in shares of four and of eight waves, in key groups, and whole, V direct and
# retiled.  Bar: relative L2 1e-2 per row (bf16 probabilities and results).
@pytest.mark.parametrize("n,h,k,groups,splits", [(1300, 2, 100, 1, 7), (3716, 12, 1400, 1, 3), (4100, 24, 1100, 2, 2), (1300, 2, 5000, 4, 3), (300, 24, 1000, 1, 1),
                                                 (300, 1, 16385, 1, 1)])
def test_attn_bf16_large_values_in_rows_that_rise(n, h, k, groups, splits):
    assert ab.astraea_attn_key_groups(n, h, k) == groups and ab.astraea_attn_plan(n, h, k)["splits"] == splits
    q, kc, vc = _attn_rise_case(n, h, k, 128, 45.0, torch.bfloat16, 64)
    vc *= 2.0 ** 66
    out = torch.empty(k, h, 128, dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, 128), dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, out, 1.0 / math.sqrt(128), q_is_compact=True, workspace=ws)
    torch.cuda.synchronize()
    for i in range(h):
        ref = torch.softmax((q[:, i].double() @ kc[:, i].double().T.contiguous()) / math.sqrt(128), 1) @ vc[:, i].double()
        assert_rel_l2(out[:, i].double().cpu().numpy(), ref.cpu().numpy(), tag=f"head {i}")


# fp32 attention: 128 queries per workgroup, tiles of 32 keys in two LDS stages, key ranges shared out when the selection is
# small; `hot` raises a row's exponent offset in the last tile; `pitch`: keys 2^25 floats apart, past 32-bit offsets.
# Bounds: a logit L is a sum of d products, off by up to d * 2^-24 * |L|.  Without the hot key |L| is a few nats and the
# errors of its terms average out: 1e-5.  The hot key gives logits of up to 25 nats to the other rows (128 * 2^-24 * 25 =
# 2e-4 of a probability, times values of size 3) and 362 nats to the hot rows, whose log-sum-exp is that logit.
@pytest.mark.parametrize("n,h,k,d,hot,scatter,pitch", [
    (1, 1, 1, 64, False, True, None), (31, 2, 31, 128, False, False, None), (32, 1, 5, 64, True, True, None),
    (33, 3, 33, 64, True, True, None), (65, 2, 127, 128, True, False, None), (300, 2, 129, 64, False, True, None),
    (1000, 3, 257, 128, True, True, None), (2085, 8, 300, 64, True, True, None), (700, 2, 5000, 64, True, False, None),
    (40, 1, 33, 64, True, False, 1 << 25), (70, 1, 33, 128, False, False, 1 << 25),
])
def test_attn_f32_tiles(n, h, k, d, hot, scatter, pitch):
    g = torch.Generator(device=DEV).manual_seed(n + h + k)
    q, kc, vc = (torch.randn(m, h, d, device=DEV, generator=g) for m in (k, n, n))
    if hot:
        q[[0, k // 2, k - 1], :, 0] = 64.0
        kc[n - 1, :, 0] = 64.0 * math.sqrt(d / 128)          # 362 nats above the rest for those rows
    if pitch:
        wide = [torch.empty(n, pitch, device=DEV)[:, :h * d].view(n, h, d) for _ in range(2)]
        for dst, src in zip(wide, (kc, vc)):
            dst.copy_(src)
    idx = torch.randperm(max(n, k), device=DEV, generator=g)[:k].sort().values.to(torch.int32)
    scale = 1.0 / math.sqrt(d)
    lse = torch.full((k, h), math.nan, device=DEV)
    ws = torch.full((max(256, ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)),), 255, dtype=torch.uint8, device=DEV)
    out = torch.randn(n if scatter else k, h * d + 8, device=DEV, generator=g)
    before = out.clone()
    kv = wide if pitch else (kc, vc)
    if scatter:
        ab.astraea_sparse_attn_update_fwd(q, *kv, idx, k, out[:, :h * d], scale, q_is_compact=True, lse_sel=lse, workspace=ws)
        got = out[idx.long(), :h * d].view(k, h, d)
    else:
        got = torch.empty(k, h, d, device=DEV)
        ab.astraea_sparse_attn_fwd(q, *kv, None, k, got, scale, q_is_compact=True, lse_sel=lse, workspace=ws)
    torch.cuda.synchronize()
    tol, tol_lse = (6e-4, d * 2.0 ** -24 * 362) if hot else (1e-5, 1e-5)
    for i in range(h):
        logits = (q[:, i].double() @ kc[:, i].double().T.contiguous()) * scale
        ref = torch.softmax(logits, 1) @ vc[:, i].double()
        assert (got[:, i].double() - ref).abs().max().item() <= tol
        assert (lse[:, i].double() - torch.logsumexp(logits, 1)).abs().max().item() <= tol_lse
    if scatter:
        keep = torch.ones(out.shape, dtype=torch.bool, device=DEV)
        keep[idx.long(), :h * d] = False
        assert torch.equal(out[keep], before[keep])


# Workgroups of eight waves (256 queries, tiles staged a whole tile ahead) and of four: items whole, all cut along the keys, and cut only past the
# last whole round (24 heads x 11 tiles of queries are 33 items per XCD); both sides of four key tiles, from which eight waves are taken, shares of one tile,
# ragged last tiles of keys and queries, a workgroup whose last four waves have no queries.  `queries`, `cut`: what the launch says.  A workspace of the size named is not written
# past, and without one the result is the same up to the order of the sums: 1e-5 as above.
@pytest.mark.parametrize("n,h,k,d,hot,scatter,queries,cut", [
    (4097, 8, 2047, 64, True, False, 256, "all"), (600, 24, 2700, 64, True, False, 256, "tail"), (600, 24, 2699, 128, True, False, 256, "tail"),
    (257, 8, 6000, 64, False, False, 256, "none"), (2100, 24, 1401, 64, False, True, 256, "none"), (2500, 8, 2500, 128, True, True, 256, "all"),
    (193, 8, 8192, 64, True, False, 256, "none"), (256, 8, 8065, 64, True, False, 256, "none"), (500, 24, 2700, 64, True, False, 256, "tail"),
    (200, 4, 16300, 128, False, False, 256, "none"), (193, 8, 8100, 128, True, False, 256, "none"),
    (192, 8, 8192, 64, True, False, 128, "none"), (33, 8, 8192, 64, True, False, 128, "none"), (97, 4, 16300, 128, False, False, 128, "none"),
    (33, 24, 2700, 64, True, False, 128, "none"), (65, 24, 2690, 128, False, False, 128, "none"), (150, 24, 5500, 64, True, False, 128, "none"),
    (1100, 16, 900, 128, True, True, 128, "all"), (2100, 2, 2100, 64, True, True, 128, "all"),
])
def test_attn_f32_eight_waves(n, h, k, d, hot, scatter, queries, cut):
    need = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)
    plan = ab.astraea_attn_plan_f32(n, h, d, k, need)
    assert plan["queries_per_workgroup"] == queries
    assert cut == ("none" if plan["splits"] == 1 else "all" if plan["full_items"] == 0 else "tail")
    test_attn_f32_tiles(n, h, k, d, hot, scatter, None)
    g = torch.Generator(device=DEV).manual_seed(n)
    q, kc, vc = (torch.randn(m, h, d, device=DEV, generator=g) for m in (k, n, n))
    ws = torch.full((need + 65536,), 170, dtype=torch.uint8, device=DEV)
    a, b = torch.empty_like(q), torch.empty_like(q)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, a, d ** -0.5, q_is_compact=True, workspace=ws[:need] if need else None)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, b, d ** -0.5, q_is_compact=True)
    torch.cuda.synchronize()
    assert (a - b).abs().max().item() <= 1e-5 and bool((ws[need:] == 170).all())


def _f32_queries(n, h, d, k):
    return ab.astraea_attn_plan_f32(n, h, d, k, max(256, ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)))["queries_per_workgroup"]


F32_EIGHT_WAVES = [(193, 8, 64, 8192), (500, 24, 64, 2700), (200, 4, 128, 16300)]    # four key tiles; eight, and shares of one; seven of 32 keys


def test_f32_eight_wave_sizes():
    assert all(_f32_queries(*s) == 256 for s in F32_EIGHT_WAVES)


# Rows whose first key tile lies 45 nats below the rest: a fixed exponent offset would leave arguments of 65 to the
# exponential (rounded by 2^-18: 1.5e-6 of a probability in the mean square) and 2^65 in the accumulators, which
# values of 2^64 then overflow.  Values of 2^110 leave the accumulators seven bits above the largest sum of 1300.  Expected
# error: arguments of 4 are rounded by 2^-22, 1e-7 in the mean square; an accumulator walks 1300 steps at random, each
# rounded by 0.4 * 2^-24 of its size in the mean square: sqrt(1300 / 2) * 0.4 * 2^-24 = 6.1e-7.  Bound: 1.5 times that,
# since the head-dims of one head are few.  16 queries and more: with and without key shares.
@pytest.mark.parametrize("rise_nats,size", [(45.0, 0), (45.0, 64), (0.0, 110)])
@pytest.mark.parametrize("h,k,d", [(2, 16, 64), (12, 3000, 64), (2, 16, 128), (6, 6000, 128)])
def test_attn_f32_rows_that_rise_from_a_low_first_tile(h, k, d, rise_nats, size):
    n = 1300
    q, kc, vc = _attn_rise_case(n, h, k, d, rise_nats, torch.float32, 32)
    vc *= 2.0 ** size
    out = torch.empty(k, h, d, device=DEV)
    ws = torch.empty(max(256, ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)), dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, out, 1.0 / math.sqrt(d), q_is_compact=True, workspace=ws)
    torch.cuda.synchronize()
    for i in range(h):
        ref = torch.softmax((q[:, i].double() @ kc[:, i].double().T.contiguous()) / math.sqrt(d), 1) @ vc[:, i].double()
        assert ((out[:, i].double() - ref).norm() / ref.norm()).item() <= 9e-7


@pytest.mark.parametrize("d,n,h,k,queries", [(64, 300, 2, 140, 128), (128, 300, 2, 140, 128), (64, 300, 8, 8100, 256), (128, 200, 4, 16300, 256)])
def test_attn_f32_non_finite_inputs_stay_in_their_rows_and_head_dims(d, n, h, k, queries):
    """A NaN or an infinity in a row of Q spoils that row alone, one in V its head-dim alone."""
    assert _f32_queries(n, h, d, k) == queries
    g = torch.Generator(device=DEV).manual_seed(d)
    q, kc, vc = (torch.randn(m, h, d, device=DEV, generator=g) for m in (k, n, n))
    ref = torch.softmax((q[:, 1].double() @ kc[:, 1].double().T.contiguous()) / math.sqrt(d), 1) @ vc[:, 1].double()
    q[3, 1, 5], q[133, 1, 0], vc[50, 1, 7], vc[2, 1, 40] = math.nan, math.inf, math.inf, math.nan
    o = torch.empty(k, h, d, device=DEV)
    ws = torch.empty(max(256, ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)), dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, o, 1.0 / math.sqrt(d), q_is_compact=True, workspace=ws)
    torch.cuda.synchronize()
    rows, dims = torch.ones(k, dtype=torch.bool, device=DEV), torch.ones(d, dtype=torch.bool, device=DEV)
    rows[[3, 133]], dims[[7, 40]] = False, False
    assert torch.isfinite(o[:, 0]).all() and torch.isnan(o[~rows, 1]).all()
    assert torch.isposinf(o[rows, 1][:, 7]).all() and torch.isnan(o[rows, 1][:, 40]).all()
    assert (o[rows, 1][:, dims].double() - ref[rows][:, dims]).abs().max().item() <= 1e-5


# top-k in one workgroup: an even number of elements per thread up to 32768 scores, wave w owning a contiguous range; passes
# over the bits in which the keys differ.  Whole numbers, exact.
@pytest.mark.parametrize("n", [1, 63, 64, 65, 1025, 2047, 2048, 2049, 4096, 4097, 18431, 18432, 18433, 30720, 30721, 32768, 32769])
@pytest.mark.parametrize("kind", ["narrow", "ties", "equal", "extremes", "zeros"])
def test_topk_sizes(n, kind):
    g = torch.Generator().manual_seed(n)
    s = 5.54 + 0.1 * torch.randn(n, generator=g)
    if kind == "ties":
        s = torch.randint(0, 3, (n,), generator=g).float()
    elif kind == "equal":
        s = torch.full((n,), -0.0)
        s[n // 2:] = 0.0                                      # -0 and +0 are the same score
    elif kind == "zeros":                                     # the lowest score shared by most: thresholds above it and at it
        s[torch.rand(n, generator=g) < 0.8] = 0.0
    elif kind == "extremes":
        special = torch.tensor([math.inf, -math.inf, math.nan, 3.4e38, -3.4e38, 1e-45, -1e-45, 0.0, -0.0])
        pick = torch.rand(n, generator=g) < 0.4
        s[pick] = special[torch.randint(0, 9, (int(pick.sum()),), generator=g)]
    skip0 = torch.randint(0, 9, (n,), generator=g).to(torch.int32)
    for k in sorted({0, 1, n // 10, n // 3, n - 1, n}):
        e_idx, e_rest, e_mask = oracle.topk(s.numpy(), k)
        idx, rest, skip = (torch.full((n + 1,), -7, dtype=torch.int32, device=DEV) for _ in range(3))
        mask = torch.full((n + 1,), 9, dtype=torch.uint8, device=DEV)
        skip[:n] = skip0.to(DEV)
        ws = torch.full((ab.workspace_bytes(ab.OP_SELECT_TOPK, n),), 255, dtype=torch.uint8, device=DEV)
        ab.astraea_select_topk(s.to(DEV), k, idx, ws, idx_remain=rest, sel_mask=mask, skip_count=skip)
        torch.cuda.synchronize()
        assert np.array_equal(idx[:k].cpu().numpy(), e_idx) and (idx[k:] == -7).all()
        assert np.array_equal(rest[:n - k].cpu().numpy(), e_rest) and (rest[n - k:] == -7).all()
        assert np.array_equal(mask[:n].cpu().numpy(), e_mask) and mask[n].item() == 9
        e_skip = np.where(e_mask != 0, 0, skip0.numpy() + 1)
        assert np.array_equal(skip[:n].cpu().numpy(), e_skip) and skip[n].item() == -7


# Selection by a launch per digit (12288 scores a workgroup, 32769 to 786432 of them, workspaces that hold its slots) and by
# histograms in one place (more scores, smaller workspaces): edges of the workgroups' runs and of both ranges, against the oracle.
@pytest.mark.parametrize("kind", ["narrow", "ties", "extremes"])
@pytest.mark.parametrize("n,small", [(32769, False), (36863, False), (36864, False), (36865, False), (36865, True), (118800, True),
                                     (135169, False), (196608, False), (196609, False), (786432, False), (786433, False)])
def test_topk_of_several_workgroups(n, small, kind):
    g = torch.Generator().manual_seed(n)
    s = 5.54 + 0.1 * torch.randn(n, generator=g)
    if kind == "ties":
        s = torch.randint(-1, 2, (n,), generator=g).float() * 0.5
    elif kind == "extremes":
        special = torch.tensor([math.inf, -math.inf, math.nan, 3.4e38, -3.4e38, 1e-45, -1e-45, 0.0, -0.0])
        s = special[torch.randint(0, 9, (n,), generator=g)]
    size = ab.workspace_bytes(ab.OP_SELECT_TOPK, n)
    if small:
        assert size > 64 + 8448 + 8 * ((n + 2047) // 2048)
        size = -(-(8448 + 8 * ((n + 2047) // 2048)) // 256) * 256
    for k in (0, 1, n // 3, n - 1, n):
        e_idx, e_rest, e_mask = oracle.topk(s.numpy(), k)
        idx, rest, skip = (torch.full((n + 1,), -7, dtype=torch.int32, device=DEV) for _ in range(3))
        mask = torch.full((n + 1,), 9, dtype=torch.uint8, device=DEV)
        ws = torch.full((size + 256,), 255, dtype=torch.uint8, device=DEV)
        ab.astraea_select_topk(s.to(DEV), k, idx, ws[:size], idx_remain=rest, sel_mask=mask, skip_count=skip)
        torch.cuda.synchronize()
        assert (ws[size:] == 255).all()
        assert np.array_equal(idx[:k].cpu().numpy(), e_idx) and (idx[k:] == -7).all()
        assert np.array_equal(rest[:n - k].cpu().numpy(), e_rest) and (rest[n - k:] == -7).all()
        assert np.array_equal(mask[:n].cpu().numpy(), e_mask) and mask[n].item() == 9
        assert np.array_equal(skip[:n].cpu().numpy(), np.where(e_mask != 0, 0, -6)) and skip[n].item() == -7


# bf16 linear: tiles of 256 features x 256, 192 or 128 tokens by the launch's estimate (the sizes below take each of them), edges
# of the token tiles, ragged features, more and fewer tiles than CUs, one to many contraction steps.  Reference: fp64; bar:
# relative L2 1e-2 per row (bf16 inputs and result).
@pytest.mark.parametrize("n,k,c_in,c_out,gather,scatter,bias,act,tile", [
    (5, 1, 64, 8, True, True, True, ab.ACT_NONE, 128), (300, 127, 64, 264, True, False, False, ab.ACT_GELU_TANH, 128),
    (300, 129, 128, 512, False, True, True, ab.ACT_NONE, 128), (700, 608, 192, 3072, True, True, True, ab.ACT_GELU_TANH, 128),
    (2000, 1755, 512, 12288, True, False, True, ab.ACT_NONE, 192), (3600, 3457, 320, 3072, False, True, True, ab.ACT_NONE, 192),
    (3600, 3456, 256, 3080, True, True, False, ab.ACT_GELU_TANH, 192), (7100, 7020, 320, 3072, True, True, True, ab.ACT_NONE, 192),
    (5100, 5000, 128, 3072, True, True, True, ab.ACT_NONE, 256), (5200, 5121, 192, 3064, False, True, True, ab.ACT_GELU_TANH, 256),
    (9000, 8192, 64, 2048, True, False, True, ab.ACT_NONE, 256),                                   # one whole round
    (9000, 8193, 128, 2048, True, True, True, ab.ACT_NONE, 192), (12100, 12000, 9216, 2048, False, True, True, ab.ACT_NONE, 192),
    (33100, 33000, 3136, 3072, True, True, True, ab.ACT_NONE, 256),
])
def test_linear_bf16_tiles(n, k, c_in, c_out, gather, scatter, bias, act, tile, features=256, few=0):
    assert ab.astraea_linear_few_rows(k, c_in, c_out)["tile_tokens"] == few
    assert ab.astraea_linear_plan(ab.BF16, k, c_in, c_out) == {
        "tile_features": features, "tile_tokens": tile, "tiles": -(-k // tile) * -(-c_out // features)}
    g = torch.Generator(device=DEV).manual_seed(n + k + c_in)
    idx = torch.randperm(n, device=DEV, generator=g)[:k].sort().values.to(torch.int32)
    x = torch.randn(n if gather else k, c_in, device=DEV, generator=g).bfloat16()
    w = (torch.randn(c_out, c_in, device=DEV, generator=g) * c_in ** -0.5).bfloat16()
    b = torch.randn(c_out, device=DEV, generator=g).bfloat16() if bias else None
    y = torch.randn(n if scatter else k, c_out + 8, device=DEV, generator=g).bfloat16()
    before = y.clone()
    ref = (x[idx.long()] if gather else x).double() @ w.double().T.contiguous() + (b.double() if bias else 0.0)
    if act == ab.ACT_GELU_TANH:
        ref = torch.nn.functional.gelu(ref, approximate="tanh")
    ab.astraea_sparse_linear(x, w, b, idx, k, y[:, :c_out], act=act, x_is_compact=not gather, y_is_compact=not scatter, N=n)
    torch.cuda.synchronize()
    got = y[idx.long() if scatter else slice(None), :c_out]
    assert_rel_l2(got.double().cpu().numpy(), ref.cpu().numpy())
    keep = torch.ones(y.shape, dtype=torch.bool, device=DEV)
    keep[idx.long() if scatter else slice(None), :c_out] = False
    assert torch.equal(y[keep], before[keep])


@pytest.mark.parametrize("k", [300, 16385])      # V tiles direct and retiled
def test_attn_bf16_non_finite_values_stay_in_their_head_dims(k):
    """An infinity in the last row of V, which the last, partly filled tile ends on, reaches every result of its head-dim
    and nothing else: rows past the last key count as zero."""
    n, h = 100, 2
    g = torch.Generator(device=DEV).manual_seed(k)
    q, kc, vc = (torch.randn(m, h, 128, device=DEV, generator=g).bfloat16() for m in (k, n, n))
    vc[n - 1, 1, 7], vc[n - 1, 0, 70] = math.inf, math.nan
    o = torch.empty(k, h, 128, dtype=torch.bfloat16, device=DEV)
    ws = torch.full((ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, 128),), 255, dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, o, 1.0 / math.sqrt(128), q_is_compact=True, workspace=ws)
    torch.cuda.synchronize()
    assert torch.isposinf(o[:, 1, 7]).all() and torch.isnan(o[:, 0, 70]).all()
    o[:, 1, 7], o[:, 0, 70] = 0.0, 0.0
    assert torch.isfinite(o).all()


# fp32 attention: tiles of 64 (d = 64) or 32 (d = 128) keys whose operands are split into bf16 parts; where a sum is not finite or K is
# too large the workgroup takes the fp32 products.  Edges of tiles and query blocks,
# then magnitudes: in K (its queries the other way, so that logits stay), in V, from tile to tile, zeros, an infinity.
# fp64 on the device.  Bound: a logit is off by a few 2^-23 of |q| |k| scale, a result by that, relative, and a few 2^-23 of |V|.
@pytest.mark.parametrize("n,h,d,k", [(1, 1, 64, 1), (63, 2, 64, 31), (64, 1, 64, 128), (65, 3, 64, 129), (257, 2, 64, 300),
                                     (31, 1, 128, 5), (32, 2, 128, 32), (33, 1, 128, 128), (225, 2, 128, 130), (700, 8, 64, 60)] + F32_EIGHT_WAVES)
@pytest.mark.parametrize("values", ["plain", "k tiny", "k huge", "v tiny", "v huge", "v grows", "v falls", "v falls far", "zeros", "inf"])
def test_attn_f32_split_range(n, h, d, k, values):
    g = torch.Generator(device=DEV).manual_seed(n + h + d + k)
    q, kc, vc = (torch.randn(m, h, d, device=DEV, generator=g) for m in (k, n, n))
    step = (torch.arange(n, device=DEV) // 64).float()[:, None, None]
    if values in ("k tiny", "k huge"):
        f = 2.0 ** (-70 if values == "k tiny" else 40)               # -70: past the range of the scaling
        q, kc = q / f, kc * f
    elif values.startswith("v "):
        vc = vc * {"v tiny": 2.0 ** -60, "v huge": 2.0 ** 100, "v grows": 2.0 ** (9 * step), "v falls": 2.0 ** (-9 * step),
                   "v falls far": 2.0 ** (-30 * step)}[values]
    elif values == "zeros":
        kc[: n // 2] = 0.0
        vc[n // 2:] = 0.0
        q[0] = 0.0
    elif values == "inf" and n > 1:                    # the last key has a test of its own
        vc[n // 2 - 1, 0, 3] = math.inf
    scale = 1.0 / math.sqrt(d)
    ws = torch.empty(max(1, ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)), dtype=torch.uint8, device=DEV)
    o, lse = torch.full((k, h, d), math.nan, device=DEV), torch.full((k, h), math.nan, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, o, scale, q_is_compact=True, lse_sel=lse, workspace=ws)
    torch.cuda.synchronize()
    logits = torch.stack([q[:, i].double() @ kc[:, i].double().T.contiguous() for i in range(h)]) * scale         # [h, k, n]
    size = (q.double().norm(dim=2).T[:, :, None] * kc.double().norm(dim=2).T[:, None, :] * scale).amax(dim=2)     # [h, k]
    p = torch.softmax(logits, 2)
    finite = torch.where(vc.isinf(), torch.zeros_like(vc), vc).double()
    exp = torch.stack([p[i] @ finite[:, i] for i in range(h)], 1)
    spread = torch.stack([p[i] @ finite[:, i].abs() for i in range(h)], 1)
    if values == "inf" and n > 1:
        assert bool((o[:, 0, 3] == math.inf).all())
        o[:, 0, 3], exp[:, 0, 3] = 0.0, 0.0
    bound = 8 * 2.0 ** -23 * (1.0 + size.T[:, :, None]) * spread + 2.0 ** -140
    assert bool(((o.double() - exp).abs() <= bound).all()), ((o.double() - exp).abs() / bound).max().item()
    assert bool(((lse.double() - torch.logsumexp(logits, 2).T).abs() <= 8 * 2.0 ** -23 * (1.0 + size.T + lse.double().abs())).all())


# fp32 attention, magnitudes that differ between keys, head-dims and tiles: V's head-dims, opposed head-dims of q and K, a huge key
# that half the queries turn away from, huge values behind negligible weights, an outlier of V in another head-dim.
# Bound, to first order: with s_n = scale sum_d |q_d k_nd|, a logit is off by a few 2^-23 s_n and its exponential's argument by a few 2^-23 of
# itself; a result is off by that, weighted, and a few 2^-23 of the weighted |V|.
@pytest.mark.parametrize("n,h,d,k", [(65, 2, 64, 129), (700, 8, 64, 60), (225, 2, 128, 130), (97, 1, 128, 300)] + F32_EIGHT_WAVES)
@pytest.mark.parametrize("values", ["v head-dims", "opposed", "huge key", "hidden values", "v outlier", "q rows", "k past range", "tiny scale", "scale past range", "nan"])
def test_attn_f32_spread_magnitudes(n, h, d, k, values):
    g = torch.Generator(device=DEV).manual_seed(n + h + d + k)
    q, kc, vc = (torch.randn(m, h, d, device=DEV, generator=g) for m in (k, n, n))
    fall = 2.0 ** -(torch.arange(d, device=DEV) % 24).float()
    scale = 1.0 / math.sqrt(d)
    if values == "v head-dims":
        vc *= fall
    elif values == "opposed":
        q, kc = q * fall, kc / fall
    elif values == "huge key":
        kc[n // 3] *= 2.0 ** 40
        q[:, :, :] = torch.where(((q * kc[n // 3]).sum(2, keepdim=True) > 0), -q, q)
        q[0] = 0.0
    elif values == "hidden values":
        q[:, :, 0] = 16.0
        kc[:32, :, 0] = -8.0 / scale            # weights of e^-128 before the other logits, and 2^20 in V
        vc[:32] *= 2.0 ** 20
    elif values == "v outlier":
        vc[n // 2, 0, 5] = 2.0 ** 40
    elif values == "q rows":
        q *= 2.0 ** -(torch.arange(k, device=DEV) % 24).float()[:, None, None]
    elif values == "k past range":             # of the split: the fp32 products serve
        q, kc = q * 2.0 ** -60, kc * 2.0 ** 60
    elif values == "tiny scale":
        q, kc, scale = q * 2.0 ** 35, kc * 2.0 ** 35, scale * 2.0 ** -70
    elif values == "scale past range":
        q, kc, scale = q * 2.0 ** 50, kc * 2.0 ** 50, scale * 2.0 ** -100
    elif values == "nan":
        q[k // 2] = math.nan
    ws = torch.empty(max(1, ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)), dtype=torch.uint8, device=DEV)
    o, lse = torch.full((k, h, d), math.inf, device=DEV), torch.full((k, h), math.inf, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, o, scale, q_is_compact=True, lse_sel=lse, workspace=ws)
    torch.cuda.synchronize()
    if values == "nan":
        assert bool(o[k // 2].isnan().all()) and bool(lse[k // 2].isnan().all())
        q[k // 2] = 0.0
    for i in range(h):
        qd, kd, vd = q[:, i].double(), kc[:, i].double(), vc[:, i].double()
        logits, s = qd @ kd.T.contiguous() * scale, qd.abs() @ kd.abs().T.contiguous() * scale
        lse_ref = torch.logsumexp(logits, 1)
        p = torch.softmax(logits, 1)
        off = p * (1.0 + s + (lse_ref[:, None] - logits))                      # [k, n]
        ref = p @ vd
        bound = 8 * 2.0 ** -23 * (off @ vd.abs() + off.sum(1, keepdim=True) * ref.abs()) + 2.0 ** -140
        err, lse_err, lse_bound = (o[:, i].double() - ref).abs(), (lse[:, i].double() - lse_ref).abs(), 8 * 2.0 ** -23 * (off.sum(1) + lse_ref.abs())
        if values == "nan":
            err[k // 2], lse_err[k // 2] = 0.0, 0.0
        assert bool((err <= bound).all()), (err / bound).max().item()
        assert bool((lse_err <= lse_bound).all()), (lse_err / lse_bound).max().item()


@pytest.mark.parametrize("n,h,d,k", [(1, 1, 64, 1), (65, 2, 64, 10), (700, 8, 64, 60), (33, 1, 128, 128), (97, 2, 128, 300)] + F32_EIGHT_WAVES)
def test_attn_f32_infinity_in_the_last_key(n, h, d, k):
    """Rows past the last key fill its tile with weight 0: nothing of it may reach them."""
    g = torch.Generator(device=DEV).manual_seed(n + d)
    q, kc, vc = (torch.randn(m, h, d, device=DEV, generator=g) for m in (k, n, n))
    vc[n - 1, 0, 3] = math.inf
    ws = torch.empty(max(1, ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k, h, d)), dtype=torch.uint8, device=DEV)
    o = torch.full((k, h, d), math.nan, device=DEV)
    ab.astraea_sparse_attn_fwd(q, kc, vc, None, k, o, 1.0 / math.sqrt(d), q_is_compact=True, workspace=ws)
    torch.cuda.synchronize()
    assert bool((o[:, 0, 3] == math.inf).all())
    o[:, 0, 3] = 0.0
    assert bool(o.isfinite().all())


# ... and of 128 features x 128 tokens where larger ones would leave most CUs without one: edges of the tile on both sides, ragged
# features, one tile, and contractions that end anywhere in the ring of four stages.
@pytest.mark.parametrize("n,k,c_in,c_out,gather,scatter,bias,act", [
    (5, 1, 512, 16392, True, True, True, ab.ACT_NONE), (300, 127, 576, 17000, True, False, False, ab.ACT_GELU_TANH),
    (300, 128, 640, 17024, False, True, True, ab.ACT_NONE), (300, 129, 704, 8200, True, True, True, ab.ACT_NONE),
    (700, 608, 512, 3400, True, True, True, ab.ACT_GELU_TANH), (700, 608, 1088, 4104, True, True, True, ab.ACT_NONE),
    (1100, 1000, 3072, 3072, False, False, True, ab.ACT_NONE), (1100, 1001, 576, 2056, False, True, True, ab.ACT_NONE),
    (1300, 1153, 640, 3064, True, False, True, ab.ACT_GELU_TANH), (1100, 897, 704, 2568, True, True, False, ab.ACT_NONE),
])
def test_linear_bf16_small_tile(n, k, c_in, c_out, gather, scatter, bias, act):
    test_linear_bf16_tiles(n, k, c_in, c_out, gather, scatter, bias, act, 128, features=128)


# ... and of 64 features x 64 or 128 tokens where there are not more of them than CUs: one and many steps past the ring of six stages, odd counts of
# them, ragged rows and features, one row, a full round.
@pytest.mark.parametrize("n,k,c_in,c_out,gather,scatter,bias,act,tokens", [
    (300, 127, 576, 136, True, False, False, ab.ACT_GELU_TANH, 64), (300, 128, 640, 128, False, True, True, ab.ACT_NONE, 64),
    (300, 129, 704, 264, True, True, True, ab.ACT_NONE, 64), (700, 608, 512, 3064, True, True, True, ab.ACT_GELU_TANH, 128),
    (5, 1, 512, 8, True, True, True, ab.ACT_NONE, 64), (300, 65, 576, 72, True, False, True, ab.ACT_GELU_TANH, 64),
    (300, 64, 640, 64, False, True, False, ab.ACT_NONE, 64), (800, 705, 1088, 1096, True, True, True, ab.ACT_NONE, 64),
    (800, 707, 4096, 1024, False, True, True, ab.ACT_NONE, 64), (300, 191, 704, 4600, True, True, True, ab.ACT_GELU_TANH, 64),
    (700, 608, 12288, 3072, True, True, True, ab.ACT_NONE, 128), (1100, 1001, 576, 1544, True, True, True, ab.ACT_GELU_TANH, 128),
    (1100, 1024, 640, 2048, False, True, False, ab.ACT_NONE, 128), (2100, 2047, 1152, 1000, True, False, True, ab.ACT_NONE, 128),
])
def test_linear_bf16_few_rows(n, k, c_in, c_out, gather, scatter, bias, act, tokens):
    assert ab.astraea_linear_few_rows(k, c_in, c_out) == {"tile_features": 64, "tile_tokens": tokens, "tiles": -(-k // tokens) * -(-c_out // 64)}
    plan = ab.astraea_linear_plan(ab.BF16, k, c_in, c_out)
    test_linear_bf16_tiles(n, k, c_in, c_out, gather, scatter, bias, act, plan["tile_tokens"], features=plan["tile_features"], few=tokens)


# Layers of one input in one launch, against a call each: one to three parts, widths that end inside a tile of features, every tile kind
# (few rows, in bf16 tiles of 64 and of 128 of them, many rows, deep and shallow contractions), a part without a bias, compact and placed results.  bf16 sums a contraction in one
# order whatever the tile, so its bits are the same; fp32 results are held to the bound of their products (test_linear_f32_split_range).
# "chained": a layer whose weight is the result before it gets its turn after it.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n,k,c_in,c_out,parts,chained", [
    (700, 300, 128, 264, 3, False), (2100, 2049, 512, 512, 3, False), (1300, 1000, 1024, 1096, 2, False), (90, 33, 64, 8, 3, False),
    (4000, 3900, 320, 776, 3, False), (500, 499, 192, 192, 1, False), (500, 192, 192, 192, 3, True),
    (300, 131, 576, 264, 3, False), (90, 1, 512, 72, 2, False), (700, 601, 640, 1032, 3, False), (1300, 1001, 1088, 520, 2, False),
])
def test_linear_group(dtype, n, k, c_in, c_out, parts, chained):
    g = torch.Generator(device=DEV).manual_seed(n + k)
    x = torch.randn(n, c_in, device=DEV, generator=g).to(dtype)
    ws = [torch.randn(c_out, c_in, device=DEV, generator=g).div(math.sqrt(c_in)).to(dtype) for _ in range(parts)]
    bs = [None if i == 1 else torch.randn(c_out, device=DEV, generator=g).to(dtype) for i in range(parts)]
    idx = torch.randperm(n, device=DEV, generator=g)[:k].sort().values.to(torch.int32)

    def layers():
        ys = [torch.zeros(k if i == 0 else n, c_out + 8, dtype=dtype, device=DEV)[:, :c_out] for i in range(parts)]
        w = list(ws)
        if chained:
            w[1] = ys[0] = torch.zeros(k, c_out, dtype=dtype, device=DEV)
        return [(w[i], bs[i], ys[i], i == 0) for i in range(parts)]
    la, lb = layers(), layers()
    for w, b, y, compact in la:
        ab.astraea_sparse_linear(x, w, b, idx, k, y, act=ab.ACT_GELU_TANH, y_is_compact=compact)
    ab.astraea_sparse_linear_group(x, lb, idx, k, act=ab.ACT_GELU_TANH)
    torch.cuda.synchronize()
    for (w, _, ya, _), (_, _, yb, _) in zip(la, lb):
        if dtype == torch.bfloat16 or chained:               # a launch each, of the same tiles, where chained
            assert torch.equal(ya, yb)
        else:
            # either is off by (2^-22 + c_in / 2 2^-24) of the sum of |x w|, and GELU (slope at most 1.13) by 2^-21 of its result
            size = x.double().abs()[idx.long()] @ w.double().abs().T
            a, b = (t.double() if t.shape[0] == k else t[idx.long()].double() for t in (ya, yb))
            bound = 2 * 1.13 * (2.0 ** -22 + c_in / 2 * 2.0 ** -24) * size + 2.0 ** -20 * (1 + a.abs())
            assert bool(((a - b).abs() <= bound).all())
            rest = torch.ones(n, dtype=torch.bool, device=DEV)
            rest[idx.long()] = False
            assert ya.shape[0] == k or not yb[rest].any()
