"""GPU parity: every C-ABI entry point against the CPU oracle on the same seeded inputs.

Bars: selected indices, masks, counters and moved rows bit-exact; scores bit-exact (the score
decides integers, both sides take it in fp32 with the same channel order); attention max-abs
<= 1e-4 in fp32 mode and relative L2 <= 1e-2 in bf16 mode, over the whole comparison and over every (row, head) by itself.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from conftest import assert_rel_l2, bf16_bits_to_f64, to_np
from paper_2506_05096_amd import binding as ab
from paper_2506_05096_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _sync():
    torch.cuda.synchronize()


def as_f64(a: np.ndarray) -> np.ndarray:
    return bf16_bits_to_f64(a) if a.dtype == np.uint16 else a.astype(np.float64)


# ------------------------------------------------------------------ score --

def _features(n, c, dtype, recipe, seed, stride=None):
    g = torch.Generator().manual_seed(seed)
    prev = torch.randn(n, c, generator=g)
    cur = prev + 0.1 * torch.randn(n, c, generator=g) if recipe == "drift" else torch.randn(n, c, generator=g)
    prev, cur = prev.to(dtype), cur.to(dtype)
    if stride is not None and stride != c:
        pp = torch.zeros(n, stride, dtype=dtype)
        cc = torch.zeros(n, stride, dtype=dtype)
        pp[:, :c], cc[:, :c] = prev, cur
        return cc, pp
    return cur, prev


@pytest.mark.parametrize("n,c,dtype,recipe,stride", [
    (4096, 512, torch.float32, "independent", None),      # config-0 shape
    (3001, 3072, torch.bfloat16, "drift", None),          # config-2/3 recipe, ragged token count
    (257, 520, torch.bfloat16, "drift", None),            # ragged last channel slab, vector path
    (130, 100, torch.bfloat16, "independent", None),      # rows not 16-byte aligned: element path
    (130, 100, torch.float32, "independent", 104),        # strided rows
    (1, 64, torch.float32, "independent", None),
    (64, 7, torch.float32, "independent", None),
])
@pytest.mark.parametrize("mode", [ab.DELTA_L2, ab.DELTA_MEAN_ABS, ab.DELTA_MEAN_SQ])
def test_score_bit_exact(n, c, dtype, recipe, stride, mode):
    cur, prev = _features(n, c, dtype, recipe, seed=n + c, stride=stride)
    exp = oracle.score(to_np(cur)[:, :c], to_np(prev)[:, :c], mode)
    dc, dp = cur.to(DEV), prev.to(DEV)
    out = torch.full((n,), -1.0, device=DEV)
    ab.astraea_score(dc[:, :c], dp[:, :c], out, mode)
    _sync()
    got = out.cpu().numpy()
    assert np.array_equal(got.view(np.uint32), exp.view(np.uint32)), \
        f"max |diff| {np.max(np.abs(got - exp))}, mismatches {(got != exp).sum()}"


def test_score_weight_and_penalty_bit_exact():
    n, c = 1000, 512
    cur, prev = _features(n, c, torch.bfloat16, "drift", seed=5)
    g = torch.Generator().manual_seed(6)
    w = torch.rand(n, generator=g) * 40 + 1
    cnt = torch.randint(-1, 30, (n,), generator=g, dtype=torch.int32)
    table = torch.from_numpy(oracle.penalty_table(20))
    exp = oracle.score(to_np(cur), to_np(prev), ab.DELTA_L2, lse_weight=w.numpy(), skip_count=cnt.numpy(),
                       penalty_table=table.numpy(), w_alpha=0.7, w_beta=1e-3)
    out = torch.empty(n, device=DEV)
    ab.astraea_score(cur.to(DEV), prev.to(DEV), out, ab.DELTA_L2, lse_weight=w.to(DEV), skip_count=cnt.to(DEV),
                     penalty_table=table.to(DEV), w_alpha=0.7, w_beta=1e-3)
    _sync()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), exp.view(np.uint32))


def test_score_closed_forms_on_gpu():
    # all-ones difference: sqrt(C) exactly; cur == prev: zero
    for c, expect in ((1024, 32.0), (4096, 64.0)):
        prev = torch.full((70, c), 2.0, device=DEV, dtype=torch.bfloat16)
        cur = torch.full((70, c), 3.0, device=DEV, dtype=torch.bfloat16)
        out = torch.empty(70, device=DEV)
        ab.astraea_score(cur, prev, out)
        assert torch.all(out == expect)
        ab.astraea_score(cur, cur.clone(), out)
        assert torch.all(out == 0)


# ------------------------------------------------------------------ top-k --

def _run_topk(score_t, k, with_skip=True):
    n = score_t.numel()
    ws = torch.empty(ab.workspace_bytes(ab.OP_SELECT_TOPK, n), dtype=torch.uint8, device=DEV)
    ws.random_(0, 255)                                     # the workspace needs no initialisation
    idx = torch.full((max(k, 1),), -7, dtype=torch.int32, device=DEV)
    rem = torch.full((max(n - k, 1),), -7, dtype=torch.int32, device=DEV)
    mask = torch.full((n,), 9, dtype=torch.uint8, device=DEV)
    skip0 = torch.arange(n, dtype=torch.int32) % 5
    skip = skip0.to(DEV) if with_skip else None
    ab.astraea_select_topk(score_t.to(DEV), k, idx, ws, idx_remain=rem, sel_mask=mask, skip_count=skip)
    _sync()
    return idx[:k].cpu().numpy(), rem[:n - k].cpu().numpy(), mask.cpu().numpy(), skip0.numpy(), \
        (skip.cpu().numpy() if with_skip else None)


@pytest.mark.parametrize("kind", ["normal", "lognormal", "tied", "narrow", "signed_tied"])
@pytest.mark.parametrize("n", [1, 7, 2048, 2049, 5000, 118800])
def test_topk_bit_exact(kind, n):
    s = synth.random_scores(n, 3 + n, kind)
    for k in sorted({0, 1, n // 3, (3 * n) // 10, n - 1, n} & set(range(0, n + 1))):
        e_idx, e_rem, e_mask = oracle.topk(s.numpy(), k)
        idx, rem, mask, skip0, skip = _run_topk(s, k)
        assert np.array_equal(idx, e_idx), (kind, n, k)
        assert np.array_equal(rem, e_rem), (kind, n, k)
        assert np.array_equal(mask, e_mask), (kind, n, k)
        assert np.array_equal(skip, oracle.update_skip_count(skip0, e_mask)), (kind, n, k)


@pytest.mark.parametrize("kind", ["tied", "narrow", "lognormal"])
@pytest.mark.parametrize("n", [32767, 32768, 32769, 32768 + 2048])
def test_topk_on_both_sides_of_the_single_workgroup_limit(kind, n):
    """Up to 32768 scores are selected by one workgroup with the keys in LDS, more by the multi-launch path:
    the two must agree with the oracle right at the switch, with heavily tied and narrow-band scores (whose
    threshold value is shared by many elements, so that the lowest-index rule decides) and at the budgets'
    ends."""
    s = synth.random_scores(n, 11 + n, kind)
    for k in (0, 1, n // 10, (3 * n) // 10, n // 2, n - 1, n):
        e_idx, e_rem, e_mask = oracle.topk(s.numpy(), k)
        idx, rem, mask, skip0, skip = _run_topk(s, k)
        assert np.array_equal(idx, e_idx), (kind, n, k)
        assert np.array_equal(rem, e_rem), (kind, n, k)
        assert np.array_equal(mask, e_mask), (kind, n, k)
        assert np.array_equal(skip, oracle.update_skip_count(skip0, e_mask)), (kind, n, k)


@pytest.mark.parametrize("n", [40001, 118800])
def test_topk_scores_that_are_not_16_byte_aligned(n):
    """The score array only has to be 4-byte aligned: one that starts 4 bytes into an allocation (and has an odd
    length) must give the same selection."""
    s = synth.random_scores(n + 1, 29 + n, "narrow")
    k = (3 * n) // 10
    e_idx, e_rem, e_mask = oracle.topk(s.numpy()[1:], k)
    ds = s.to(DEV)[1:]
    assert ds.data_ptr() % 16 == 4
    ws = torch.empty(ab.workspace_bytes(ab.OP_SELECT_TOPK, n), dtype=torch.uint8, device=DEV)
    idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
    rem = torch.full((n - k,), -7, dtype=torch.int32, device=DEV)
    mask = torch.full((n,), 9, dtype=torch.uint8, device=DEV)
    _check_rc = ab.lib().astraea_select_topk(ds.data_ptr(), n, k, idx.data_ptr(), rem.data_ptr(), mask.data_ptr(), None,
                                             ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert _check_rc == ab.OK
    _sync()
    assert np.array_equal(idx.cpu().numpy(), e_idx) and np.array_equal(rem.cpu().numpy(), e_rem)
    assert np.array_equal(mask.cpu().numpy(), e_mask)


def test_topk_special_values():
    s = torch.tensor([float("nan"), -0.0, 0.0, float("inf"), -float("inf"), 1.0, float("nan"), 0.0, -1e-45, 1e-45,
                      3.4e38, -3.4e38])
    for k in range(0, s.numel() + 1):
        e_idx, e_rem, e_mask = oracle.topk(s.numpy(), k)
        idx, rem, mask, _, _ = _run_topk(s, k, with_skip=False)
        assert np.array_equal(idx, e_idx) and np.array_equal(rem, e_rem) and np.array_equal(mask, e_mask), k


def test_topk_from_gpu_scores_end_to_end():
    # config-2/3 recipe: scores crowd in a narrow band with exact ties; selection must still agree
    n, c = 20000, 3072
    cur, prev = _features(n, c, torch.bfloat16, "drift", seed=77)
    sc = torch.empty(n, device=DEV)
    ab.astraea_score(cur.to(DEV), prev.to(DEV), sc)
    k = (n * 3) // 10
    e_idx, _, _ = oracle.topk(oracle.score(to_np(cur), to_np(prev)), k)
    idx, _, _, _, _ = _run_topk(sc.cpu(), k, with_skip=False)
    assert np.array_equal(idx, e_idx)


def test_topk_is_deterministic_across_runs():
    s = synth.random_scores(118800, 1, "narrow")
    a = _run_topk(s, 35640, with_skip=False)[0]
    for _ in range(3):
        assert np.array_equal(a, _run_topk(s, 35640, with_skip=False)[0])


# ------------------------------------------------------- gather / scatter --

@pytest.mark.parametrize("dtype,e", [(torch.bfloat16, 3072), (torch.float32, 512), (torch.bfloat16, 5),
                                     (torch.float32, 3), (torch.bfloat16, 8200), (torch.bfloat16, 264)])
def test_scatter_and_gather_bit_exact(dtype, e):
    g = torch.Generator().manual_seed(e)
    n, k = 777, 300
    cache = torch.randn(n, e, generator=g).to(dtype)
    src = torch.randn(k, e, generator=g).to(dtype)
    full = torch.randn(n, e, generator=g).to(dtype)
    idx = torch.randperm(n, generator=g)[:k].sort().values.to(torch.int32)
    for src_t, is_full in ((src, False), (full, True)):
        exp = to_np(cache).copy()
        oracle.scatter(exp, to_np(src_t), idx.numpy(), src_is_full=is_full)
        dc = cache.to(DEV).clone()
        ab.astraea_scatter_update(dc, src_t.to(DEV), idx.to(DEV), k, src_is_full=is_full)
        _sync()
        assert np.array_equal(to_np(dc), exp)
    # budget 0: nothing moves
    dc = cache.to(DEV).clone()
    ab.astraea_scatter_update(dc, src.to(DEV), idx.to(DEV), 0)
    _sync()
    assert np.array_equal(to_np(dc), to_np(cache))
    # gather
    dst = torch.zeros(k, e, dtype=dtype, device=DEV)
    ab.astraea_gather_rows(full.to(DEV), dst, idx.to(DEV), k)
    _sync()
    assert np.array_equal(to_np(dst), oracle.gather(to_np(full), idx.numpy()))


@pytest.mark.parametrize("dtype,e,pad", [(torch.bfloat16, 3072, 0), (torch.float32, 512, 0), (torch.bfloat16, 5, 3),
                                         (torch.bfloat16, 264, 8), (torch.float32, 3, 0)])
def test_kv_refresh_bit_exact(dtype, e, pad):
    """The K and V rows of the selected tokens in one launch: both caches equal what the oracle's cache merge
    gives buffer by buffer, rows of other tokens and the padding of wider rows keep their bits, budget 0 moves
    nothing."""
    g = torch.Generator().manual_seed(e + pad)
    n, k = 901, 333
    kc, vc, kn, vn = (torch.randn(n, e + pad, generator=g).to(dtype) for _ in range(4))
    idx = torch.randperm(n, generator=g)[:k].sort().values.to(torch.int32)
    ek, ev = to_np(kc).copy(), to_np(vc).copy()
    oracle.scatter(ek[:, :e], to_np(kn)[:, :e], idx.numpy(), src_is_full=True)
    oracle.scatter(ev[:, :e], to_np(vn)[:, :e], idx.numpy(), src_is_full=True)
    dk, dv = kc.to(DEV), vc.to(DEV)
    ab.astraea_kv_refresh(dk[:, :e], dv[:, :e], kn.to(DEV)[:, :e], vn.to(DEV)[:, :e], idx.to(DEV), k)
    _sync()
    assert np.array_equal(to_np(dk), ek) and np.array_equal(to_np(dv), ev)
    ab.astraea_kv_refresh(dk[:, :e], dv[:, :e], vn.to(DEV)[:, :e], kn.to(DEV)[:, :e], idx.to(DEV), 0)
    _sync()
    assert np.array_equal(to_np(dk), ek) and np.array_equal(to_np(dv), ev)


# -------------------------------------------------------------- attention --

def _attn_case(n, h, d, k_sel, dtype, seed, bias_std=0.0):
    g = torch.Generator().manual_seed(seed)
    q = torch.randn(n, h, d, generator=g)
    k = torch.randn(n, h, d, generator=g)
    v = torch.randn(n, h, d, generator=g)
    if bias_std:
        k = k + bias_std * torch.randn(1, h, d, generator=g)
    idx = torch.randperm(n, generator=g)[:k_sel].sort().values.to(torch.int32)
    return q.to(dtype), k.to(dtype), v.to(dtype), idx


def _run_attn(q, k, v, idx, scale, compact=False, want_lse=True):
    n, h, d = k.shape
    k_sel = idx.numel()
    o = torch.full((k_sel, h, d), float("nan"), dtype=k.dtype, device=DEV)
    lse = torch.full((k_sel, h), float("nan"), device=DEV) if want_lse else None
    wsb = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k_sel, h, d)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device=DEV) if wsb else None
    dq = q[idx.long()].contiguous().to(DEV) if compact else q.to(DEV)
    ab.astraea_sparse_attn_fwd(dq, k.to(DEV), v.to(DEV), None if compact else idx.to(DEV), k_sel, o, scale,
                               q_is_compact=compact, lse_sel=lse, workspace=ws)
    _sync()
    return as_f64(to_np(o)), (lse.cpu().numpy().astype(np.float64) if want_lse else None)


@pytest.mark.parametrize("n,h,d,k_sel", [(300, 2, 64, 77), (1000, 3, 128, 333), (33, 1, 64, 33), (129, 2, 128, 1)])
def test_attn_f32_matches_oracle(n, h, d, k_sel):
    q, k, v, idx = _attn_case(n, h, d, k_sel, torch.float32, seed=n)
    scale = 1.0 / math.sqrt(d)
    eo, else_ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    for compact in (False, True):
        o, lse = _run_attn(q, k, v, idx, scale, compact=compact)
        assert np.max(np.abs(o - eo)) <= 1e-4, np.max(np.abs(o - eo))
        assert np.max(np.abs(lse - else_)) <= 1e-4


@pytest.mark.parametrize("n,h,k_sel,bias", [(1000, 3, 333, 0.0), (64, 1, 64, 0.0), (129, 2, 1, 0.0),
                                            (2500, 2, 130, 0.5), (4096, 2, 128, 0.0),
                                            (1, 1, 1, 0.0), (1, 24, 1, 0.0), (63, 2, 63, 0.0), (191, 1, 7, 0.0)])
def test_attn_bf16_matches_oracle(n, h, k_sel, bias):
    d = 128
    q, k, v, idx = _attn_case(n, h, d, k_sel, torch.bfloat16, seed=n + 1, bias_std=bias)
    scale = 1.0 / math.sqrt(d)
    eo, else_ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    for compact in (False, True):
        o, lse = _run_attn(q, k, v, idx, scale, compact=compact)
        assert_rel_l2(o, eo, tag=f"bf16 attention n={n} h={h} k_sel={k_sel} compact={compact}")
        assert np.max(np.abs(lse - else_)) <= 2e-2


def test_attn_bf16_peaked_and_uniform_rows():
    # peaked: one key dominates a row by a wide margin -> that V row; uniform: zero queries -> mean of V.
    n, h, d = 700, 2, 128
    g = torch.Generator().manual_seed(4)
    v = torch.randn(n, h, d, generator=g).bfloat16()
    k = torch.zeros(n, h, d)
    k[123, :, 0] = 64.0
    q = torch.zeros(n, h, d)
    q[:, :, 0] = 16.0                        # logit 1024 * scale for key 123, 0 elsewhere
    idx = torch.arange(0, n, 5, dtype=torch.int32)
    o, _ = _run_attn(q.bfloat16(), k.bfloat16(), v, idx, 1.0 / math.sqrt(d))
    assert np.array_equal(o, np.broadcast_to(as_f64(to_np(v))[123][None], o.shape))
    o, lse = _run_attn(torch.zeros(n, h, d).bfloat16(), k.bfloat16(), v, idx, 1.0 / math.sqrt(d))
    vm = as_f64(to_np(v)).mean(axis=0)
    assert np.max(np.abs(o - vm[None])) < 2e-3
    assert np.max(np.abs(lse - math.log(n))) < 1e-4


@pytest.mark.parametrize("shape", ["ramp", "jump", "late_peak_after_floor"])
def test_attn_bf16_logits_that_outgrow_the_first_tile(shape):
    """The online softmax keeps a running row max that it only raises lazily; these rows make it rise far and
    often.  Logits along one head-dim direction, so that their size is controlled exactly:
    ramp  - logits rise by ~6 to ~23 nats per 128 keys (the max is raised many times);
    jump  - flat, then single keys 35 to 283 nats above everything before them;
    late_peak_after_floor - the first keys lie up to ~180 nats below the rest."""
    n, h, d = 1500, 2, 128
    g = torch.Generator().manual_seed(11)
    v = torch.randn(n, h, d, generator=g)
    k = 0.05 * torch.randn(n, h, d, generator=g)
    q = 0.05 * torch.randn(n, h, d, generator=g)
    a = torch.tensor([8.0, 16.0, 32.0]).repeat(n // 3)        # per-query gain
    q[:, :, 0] = a[:, None]
    j = torch.arange(n, dtype=torch.float32)
    if shape == "ramp":
        b = j / 16.0
    elif shape == "jump":
        b = torch.zeros(n)
        b[700], b[1200], b[1499] = 50.0, 100.0, 99.0
    else:
        b = torch.full((n,), 64.0)
        b[:128] = 0.0
        b[900] = 70.0
    k[:, :, 0] = b[:, None]
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    idx = torch.arange(0, n, 2, dtype=torch.int32)
    scale = 1.0 / math.sqrt(d)
    eo, else_ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    o, lse = _run_attn(q, k, v, idx, scale)
    assert np.all(np.isfinite(lse))
    assert_rel_l2(o, eo, tag=shape)
    # lse is 50 to 280 here and the logits behind it reach 400 in the log2 units the kernel works in, where
    # one fp32 ulp is 3e-5: a handful of roundings at that size
    assert np.max(np.abs(lse - else_) / np.maximum(1.0, np.abs(else_))) <= 3e-5


@pytest.mark.parametrize("rise_nats", [20.0, 45.0])
def test_attn_bf16_rows_that_outgrow_their_first_tile_by_a_tolerated_margin(rise_nats):
    """The main launch fixes a row's exponent offset at the max over its first key tile; later logits may exceed
    it by up to 2^80 before the row is handed to the exact form.  Here every logit past the first tile lies 20 or
    45 nats (29 or 65 powers of two) above the first tile's, with a few single keys another 6 nats up: inside
    the margin, so these rows are served with a stale offset, and must still meet the bar row by row."""
    n, h, d = 1300, 2, 128
    g = torch.Generator().manual_seed(23)
    v = torch.randn(n, h, d, generator=g)
    k = 0.05 * torch.randn(n, h, d, generator=g)
    q = 0.05 * torch.randn(n, h, d, generator=g)
    scale = 1.0 / math.sqrt(d)
    q[:, :, 0] = 8.0
    b = torch.full((n,), rise_nats / (8.0 * scale))
    b[:64] = 0.0
    b[[300, 777, 1299]] += 6.0 / (8.0 * scale)
    k[:, :, 0] = b[:, None]
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    idx = torch.arange(0, n, 3, dtype=torch.int32)
    eo, else_ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    o, lse = _run_attn(q, k, v, idx, scale)
    assert_rel_l2(o, eo, tag=f"rise {rise_nats}")
    assert np.max(np.abs(lse - else_) / np.maximum(1.0, np.abs(else_))) <= 3e-5


@pytest.mark.parametrize("h,k_sel,groups", [(12, 1400, 1), (24, 1100, 2)])
def test_attn_bf16_only_the_workgroups_that_need_it_are_redone(h, k_sel, groups):
    """A handful of selected rows meet one key whose logit lies hundreds of nats above everything in their first
    tile (their exponentials overflow under the first tile's offset), all other rows are ordinary.  The
    workgroups holding those rows repeat their sweep in the exact form, the others do not; every row, redone or not,
    of items cut into key ranges or of key groups, must match the oracle, and twice the same call the same bits."""
    n, d = 4100, 128
    assert ab.astraea_attn_key_groups(n, h, k_sel) == groups and ab.astraea_attn_plan(n, h, k_sel)["splits"] > 1
    q, k, v, idx = _attn_case(n, h, d, k_sel, torch.bfloat16, seed=404)
    hot = idx[[3, 300, 1000, k_sel - 1]].long()       # rows of the first, the last and two other query tiles
    q[hot, :, 0] = 64.0
    k[3000, :, 0] = 64.0                              # logit 4096 / sqrt(128) = 362 nats for the hot rows
    k[17, 5, 0] = 48.0                                # and a second, smaller peak inside the first tile of head 5
    scale = 1.0 / math.sqrt(d)
    eo, else_ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    o, lse = _run_attn(q, k, v, idx, scale)
    assert_rel_l2(o, eo, tag="hot rows among ordinary ones")
    assert np.max(np.abs(lse - else_) / np.maximum(1.0, np.abs(else_))) <= 2e-2
    o2, lse2 = _run_attn(q, k, v, idx, scale)
    assert np.array_equal(o, o2) and np.array_equal(lse, lse2)
    # and written straight into a cached buffer: the same bits in the rows idx names, nothing else touched
    g = torch.Generator().manual_seed(8)
    cache0 = torch.randn(n, h * d, generator=g).bfloat16()
    cache = cache0.to(DEV)
    wsb = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k_sel, h, d)
    ws = torch.empty(wsb, dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_update_fwd(q.to(DEV), k.to(DEV), v.to(DEV), idx.to(DEV), k_sel, cache, scale, workspace=ws)
    _sync()
    got = to_np(cache)
    assert np.array_equal(as_f64(got[idx.numpy()]).reshape(k_sel, h, d), o)
    rest = np.setdiff1d(np.arange(n), idx.numpy())
    assert np.array_equal(got[rest], to_np(cache0)[rest])


@pytest.mark.parametrize("n,h,k_sel", [
    (4100, 24, 1100),     # 9 query tiles of 128 x 24 heads = 27 items per XCD, each in 2 key groups of 33 and 32 tiles
    (4100, 12, 1400),     # 6 query tiles x 12 heads = 9 items per XCD -> 3 key ranges of the 65 tiles (uneven split)
    (3000, 24, 2800),     # 33 items per XCD: a whole round, and one cut
    (1500, 8, 256),       # 1 item per XCD, cut into as many key ranges as there are tiles allow
    (700, 24, 2000 // 3), # 6 query tiles of 128 x 24 heads = 18 items per XCD, each in 2 key groups of 6 and 5 tiles
    (200, 3, 190),        # fewer items than XCDs
    (65, 5, 3),           # two tiles, one of them a single key
    (129, 5, 3),          # three tiles, the last a single key
])
def test_attn_bf16_split_items_match_oracle(n, h, k_sel):
    """Shapes chosen to exercise the budget-aware launch: items of the last round are cut along the keys
    and merged; the result must not depend on how the work was cut."""
    d = 128
    q, k, v, idx = _attn_case(n, h, d, k_sel, torch.bfloat16, seed=7 * n + h)
    scale = 1.0 / math.sqrt(d)
    eo, else_ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    o, lse = _run_attn(q, k, v, idx, scale)
    assert_rel_l2(o, eo, tag=f"split items n={n} h={h} k_sel={k_sel}")
    assert np.max(np.abs(lse - else_)) <= 2e-2
    # determinism: the same call twice gives the same bits
    o2, _ = _run_attn(q, k, v, idx, scale)
    assert np.array_equal(o, o2)


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float32, 64)])
def test_attention_accepts_head_major_and_packed_layouts(dtype, d):
    """The same numbers laid out three ways must give the same bits: token-major [N, H, d]; head-major
    [H, N, d] (the layout of the paper's FLOPs appendix) viewed through strides; and one packed [N, 3, H, d]
    buffer holding Q, K and V side by side (what a fused projection writes)."""
    n, h, k_sel = 900, 3, 250
    q, k, v, idx = _attn_case(n, h, d, k_sel, dtype, seed=77)
    scale = 1.0 / math.sqrt(d)
    wsb = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k_sel, h, d)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device=DEV) if wsb else None

    def run(qq, kk, vv):
        o = torch.full((k_sel, h, d), float("nan"), dtype=dtype, device=DEV)
        ab.astraea_sparse_attn_fwd(qq, kk, vv, idx.to(DEV), k_sel, o, scale, workspace=ws)
        _sync()
        return to_np(o)

    base = run(q.to(DEV), k.to(DEV), v.to(DEV))
    hm = [t.permute(1, 0, 2).contiguous().to(DEV).permute(1, 0, 2) for t in (q, k, v)]       # [H, N, d] storage
    assert hm[0].stride(0) == d and hm[0].stride(1) == n * d
    assert np.array_equal(run(*hm), base)
    packed = torch.stack([q, k, v], dim=1).contiguous().to(DEV)                               # [N, 3, H, d]
    assert np.array_equal(run(packed[:, 0], packed[:, 1], packed[:, 2]), base)
    eo, _ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    got = as_f64(base)
    if dtype == torch.float32:
        assert np.max(np.abs(got - eo)) <= 1e-4
    else:
        assert_rel_l2(got, eo, tag="layouts")


@pytest.mark.parametrize("dtype,d,n_ctx,k_sel", [(torch.bfloat16, 128, 77, 1000), (torch.bfloat16, 128, 256, 5000),
                                                  (torch.float32, 64, 120, 700)])
def test_cross_attention_of_selected_rows(dtype, d, n_ctx, k_sel):
    """Cross-attention is a per-token layer too (each video token attends to the same short context), so it is
    computed for the selected rows only: compact queries of the selected tokens, keys/values of another, shorter
    sequence.  More queries than keys, a key count far below one key tile's multiple."""
    h = 3
    g = torch.Generator().manual_seed(n_ctx)
    q = torch.randn(k_sel, h, d, generator=g).to(dtype)
    k = torch.randn(n_ctx, h, d, generator=g).to(dtype)
    v = torch.randn(n_ctx, h, d, generator=g).to(dtype)
    scale = 1.0 / math.sqrt(d)
    eo, else_ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), None, scale, q_is_compact=True)
    o = torch.full((k_sel, h, d), float("nan"), dtype=dtype, device=DEV)
    lse = torch.full((k_sel, h), float("nan"), device=DEV)
    wsb = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n_ctx, k_sel, h, d)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device=DEV) if wsb else None
    ab.astraea_sparse_attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), None, k_sel, o, scale, q_is_compact=True, lse_sel=lse,
                               workspace=ws)
    _sync()
    got = as_f64(to_np(o))
    if dtype == torch.float32:
        assert np.max(np.abs(got - eo)) <= 1e-4
    else:
        assert_rel_l2(got, eo, tag="cross-attention")
    # the bf16 kernel sums the bf16-rounded probabilities (the values its second product uses): few keys, little averaging
    assert np.max(np.abs(lse.cpu().numpy() - else_)) <= (1e-4 if dtype == torch.float32 else 1e-3)


# ------------------------------------------- attention fused with the cache update --

@pytest.mark.parametrize("dtype,n,h,d,k_sel,pad", [
    (torch.bfloat16, 1000, 3, 128, 333, 0), (torch.bfloat16, 4100, 24, 128, 1100, 0),   # second shape has split items
    (torch.bfloat16, 700, 2, 128, 700, 64), (torch.float32, 300, 2, 64, 77, 0), (torch.float32, 515, 3, 128, 130, 8)])
def test_attn_update_equals_attention_then_scatter(dtype, n, h, d, k_sel, pad):
    """astraea_sparse_attn_update_fwd == astraea_sparse_attn_fwd + astraea_scatter_update, bit for bit, and rows
    outside idx_sel (and the padding columns of a wider cache row) keep their bits."""
    q, k, v, idx = _attn_case(n, h, d, k_sel, dtype, seed=3 * n + h)
    scale = 1.0 / math.sqrt(d)
    g = torch.Generator().manual_seed(n)
    e = h * d
    cache0 = torch.randn(n, e + pad, generator=g).to(dtype)
    wsb = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k_sel, h, d)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device=DEV) if wsb else None
    dq, dk, dv, didx = q.to(DEV), k.to(DEV), v.to(DEV), idx.to(DEV)
    # two steps
    o = torch.empty(k_sel, h, d, dtype=dtype, device=DEV)
    lse_a = torch.empty(k_sel, h, device=DEV)
    ab.astraea_sparse_attn_fwd(dq, dk, dv, didx, k_sel, o, scale, lse_sel=lse_a, workspace=ws)
    cache_a = cache0.to(DEV)
    ab.astraea_scatter_update(cache_a[:, :e], o.view(k_sel, e), didx, k_sel, src_is_full=False)
    # one step
    cache_b = cache0.to(DEV)
    lse_b = torch.empty(k_sel, h, device=DEV)
    ab.astraea_sparse_attn_update_fwd(dq, dk, dv, didx, k_sel, cache_b[:, :e], scale, lse_sel=lse_b, workspace=ws)
    _sync()
    a, b = to_np(cache_a), to_np(cache_b)
    assert np.array_equal(a, b)
    assert np.array_equal(lse_a.cpu().numpy(), lse_b.cpu().numpy())
    rest = np.setdiff1d(np.arange(n), idx.numpy())
    assert np.array_equal(b[rest], to_np(cache0)[rest])
    assert np.array_equal(b[:, e:], to_np(cache0)[:, e:])
    # and against the oracle on the selected rows
    eo, _ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    got = as_f64(b[idx.numpy()][:, :e]).reshape(k_sel, h, d)
    if dtype == torch.float32:
        assert np.max(np.abs(got - eo)) <= 1e-4
    else:
        assert_rel_l2(got, eo, tag="attention fused with the cache update")


# ------------------------------------------------------------ kernel timer --

@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float32, 64)])
def test_kernel_timer_counts_attention_launches_and_leaves_results_alone(dtype, d):
    """With the timer on, each attention call adds one timed launch whose duration is positive and no longer than
    the whole call measured around it; outputs are the bits the untimed call gives; off again, nothing is counted."""
    n, h, k_sel = 2000, 2, 600
    q, k, v, idx = _attn_case(n, h, d, k_sel, dtype, seed=17)
    scale = 1.0 / math.sqrt(d)
    wsb = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k_sel, h, d)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device=DEV) if wsb else None
    dq, dk, dv, didx = q.to(DEV), k.to(DEV), v.to(DEV), idx.to(DEV)
    o0 = torch.empty(k_sel, h, d, dtype=dtype, device=DEV)
    ab.astraea_sparse_attn_fwd(dq, dk, dv, didx, k_sel, o0, scale, workspace=ws)
    _sync()
    ab.kernel_timer(True)
    try:
        assert ab.kernel_times_ms() == []
        o1 = torch.empty_like(o0)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(3):
            ab.astraea_sparse_attn_fwd(dq, dk, dv, didx, k_sel, o1, scale, workspace=ws)
        b.record()
        _sync()
        ms = ab.kernel_times_ms()
        assert len(ms) == 3 and all(t > 0.0 for t in ms)
        assert sum(ms) <= a.elapsed_time(b) * 1.05
    finally:
        ab.kernel_timer(False)
    ab.astraea_sparse_attn_fwd(dq, dk, dv, didx, k_sel, o1, scale, workspace=ws)
    _sync()
    assert ab.kernel_times_ms() == []
    assert np.array_equal(to_np(o0), to_np(o1))


# ------------------------------------------------------------- determinism --

@pytest.mark.parametrize("n,h,k_sel,groups,splits", [(4100, 12, 1400, 1, 3), (4100, 24, 1100, 2, 2), (2025, 24, 608, 4, 3)])
def test_every_kernel_gives_the_same_bits_on_every_run(n, h, k_sel, groups, splits):
    """No result depends on the order in which workgroups happen to run: three runs of each call on the same
    inputs are bit-identical (the split attention items are merged in a fixed order, and so are key groups, the top-k compaction
    is by index, nothing accumulates through atomics)."""
    d, c = 128, 520
    g = torch.Generator().manual_seed(77)
    xc, xp = torch.randn(n, c, generator=g).bfloat16().to(DEV), torch.randn(n, c, generator=g).bfloat16().to(DEV)
    q, k, v = (torch.randn(n, h, d, generator=g).bfloat16().to(DEV) for _ in range(3))
    w = (torch.randn(264, h * d, generator=g) / 55.0).bfloat16().to(DEV)
    assert ab.astraea_attn_plan(n, h, k_sel)["splits"] == splits and ab.astraea_attn_key_groups(n, h, k_sel) == groups
    ws_t = torch.empty(ab.workspace_bytes(ab.OP_SELECT_TOPK, n), dtype=torch.uint8, device=DEV)
    ws_a = torch.empty(ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k_sel, h, d), dtype=torch.uint8, device=DEV)
    runs = []
    for _ in range(3):
        score = torch.empty(n, device=DEV)
        idx = torch.empty(n, dtype=torch.int32, device=DEV)
        o = torch.empty(k_sel, h, d, dtype=torch.bfloat16, device=DEV)
        lse = torch.empty(k_sel, h, device=DEV)
        y = torch.empty(k_sel, 264, dtype=torch.bfloat16, device=DEV)
        ab.astraea_score(xc, xp, score)
        ab.astraea_select_topk(score, k_sel, idx, ws_t)
        ab.astraea_sparse_attn_fwd(q, k, v, idx, k_sel, o, 1.0 / math.sqrt(d), lse_sel=lse, workspace=ws_a)
        ab.astraea_sparse_linear(o.view(k_sel, h * d), w, None, None, k_sel, y, act=ab.ACT_GELU_TANH, x_is_compact=True)
        _sync()
        runs.append([to_np(score), idx[:k_sel].cpu().numpy(), to_np(o), to_np(lse), to_np(y)])
        ws_a.random_(0, 255)                                # nothing may depend on what the workspace held
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
    # the fp32 attention too
    qf, kf, vf = (t[:, :2, :64].float().contiguous() for t in (q, k, v))
    outs = []
    for _ in range(3):
        o = torch.empty(k_sel, 2, 64, device=DEV)
        ab.astraea_sparse_attn_fwd(qf, kf, vf, torch.from_numpy(runs[0][1]).to(DEV), k_sel, o, 0.125)
        _sync()
        outs.append(to_np(o))
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


# --------------------------------------------- fp32 attention: key-range shares --

@pytest.mark.parametrize("n,h,d,k_sel", [(4096, 8, 64, 2048), (1000, 3, 128, 333), (2100, 1, 64, 5), (257, 2, 64, 257)])
def test_attn_f32_key_range_shares_match_oracle_and_the_unsplit_run(n, h, d, k_sel):
    """A small fp32 selection is cut into key ranges when a workspace is given (the fp32 configuration: 4
    shares); without one every work item sweeps all keys.  Both must meet the fp32 bar against the oracle, also
    when the rows go straight into a cached buffer."""
    q, k, v, idx = _attn_case(n, h, d, k_sel, torch.float32, seed=5 * n + d)
    scale = 1.0 / math.sqrt(d)
    wsb = ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, k_sel, h, d)
    if (n, k_sel) != (257, 257):
        assert wsb > 0                                      # these shapes are cut
    eo, el = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy(), scale)
    dq, dk, dv, di = q.to(DEV), k.to(DEV), v.to(DEV), idx.to(DEV)
    outs = []
    for ws in (torch.empty(max(wsb, 1), dtype=torch.uint8, device=DEV), None):
        o = torch.full((k_sel, h, d), float("nan"), device=DEV)
        lse = torch.full((k_sel, h), float("nan"), device=DEV)
        ab.astraea_sparse_attn_fwd(dq, dk, dv, di, k_sel, o, scale, lse_sel=lse, workspace=ws)
        _sync()
        got = o.cpu().numpy().astype(np.float64)
        assert np.max(np.abs(got - eo)) <= 1e-4
        assert np.max(np.abs(lse.cpu().numpy() - el)) <= 1e-4
        outs.append(got)
    assert np.max(np.abs(outs[0] - outs[1])) <= 2e-6        # same rows, another summation order
    cache0 = torch.randn(n, h * d + 8, generator=torch.Generator().manual_seed(n))
    cache = cache0.to(DEV)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device=DEV)
    ab.astraea_sparse_attn_update_fwd(dq, dk, dv, di, k_sel, cache[:, :h * d], scale, workspace=ws)
    _sync()
    got = cache.cpu().numpy()
    assert np.max(np.abs(got[idx.numpy()][:, :h * d].reshape(k_sel, h, d) - eo)) <= 1e-4
    rest = np.setdiff1d(np.arange(n), idx.numpy())
    assert np.array_equal(got[rest], cache0.numpy()[rest]) and np.array_equal(got[:, h * d:], cache0.numpy()[:, h * d:])


def test_attn_f32_layer_workspace_sized_once_serves_the_small_budgets():
    """A layer sizes its attention workspace once, for the largest selection.  The fp32 path cuts small
    selections into more key ranges than large ones, so that size must cover them: at N = 8192, H = 8 the
    full selection is not cut at all, yet at a 25 % budget the cut must be in use (its partial results land
    in the workspace) and the rows must meet the fp32 bar."""
    from paper_2506_05096_amd.layer import LayerStep
    n, h, d = 8192, 8, 64
    layer = LayerStep(n, h, d, torch.float32, device=DEV)
    assert layer.attn_ws is not None and layer.attn_ws.numel() >= ab.workspace_bytes(ab.OP_SPARSE_ATTN, n, n // 4, h, d) > 0
    q, k, v, idx = _attn_case(n, h, d, n // 4, torch.float32, seed=91)
    t = {"q": q.to(DEV), "k_cache": k.to(DEV), "v_cache": v.to(DEV)}
    layer.idx_sel[:n // 4].copy_(idx.to(DEV))
    layer.attn_ws.fill_(0xAB)
    layer.step_attn(t, n // 4)
    _sync()
    assert int((layer.attn_ws != 0xAB).sum().item()) > 0, "the key-range split did not run: no partial results were written"
    rows = np.unique(np.concatenate([[0, 1, n // 4 - 1], np.random.default_rng(3).integers(0, n // 4, 61)]))
    eo, _ = oracle.sparse_attn(to_np(q), to_np(k), to_np(v), idx.numpy()[rows], 1.0 / math.sqrt(d))
    got = layer.o_sel[:n // 4].cpu().numpy().astype(np.float64)[rows]
    assert np.max(np.abs(got - eo)) <= 1e-4
