// astraea_select_topk: I_sel, I_remain = TopK(S_token, theta) (paper, Algorithm 1 step 3).
//
// Exact, deterministic selection of the k largest fp32 scores with lowest-index tie-break:
//   1. scores map to order-preserving 32-bit keys (-0 -> +0, NaN -> lowest key);
//   2. radix passes, most significant digit first, find the key T of the k-th largest element and `need`, the number
//      of elements equal to T that are still selected;
//   3. the selected indices are compacted in ascending index order: an element is selected iff key > T, or
//      key == T and fewer than `need` equal elements precede it.  Ranks come from wavefront ballots and counts.
// The score array (4N bytes) stays in the caches; the step is latency-bound.  By the number of scores:
//   * up to 32768: one launch, every workgroup with all keys in registers, sharing the outputs.  (A single workgroup that streams more scores than
//     it holds from L2 in every pass was measured too: one CU's loads are latency-bound, 129 us at 118800 scores.)
//   * up to 786432, if the workspace holds a slot per workgroup: a launch per digit and one for the outputs.  us, indices
//     alone / every output, by this and by the next form: 33000 scores 23 / 23 and 34 / 36, 118800 24 / 24 and 43 / 45, 262144
//     27 / 28 and 57 / 59, 786432 36 / 37 and 111 / 115 (scores of one magnitude; others 1 - 2 us less).  The limit bounds
//     the slots: every workgroup reads all of them in every launch.
//   * more, or a smaller workspace: three histogram launches (11 + 11 + 10 bits) whose counts are merged by integer
//     global atomics (order-independent) and whose last workgroup (atomic ticket) resolves the digit, a count and an emit
//     launch, and one before them that clears the state.
#include <mutex>

#include "common.h"

namespace astraea {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 8;                       // consecutive elements per thread
constexpr int kChunk = kThreads * kItems;       // elements per workgroup
constexpr int kBins = 2048;
constexpr int kNumPass = 3;
__constant__ const int kShift[kNumPass] = {21, 10, 0};
__constant__ const int kBits[kNumPass] = {11, 11, 10};

struct SelectState {
    uint32_t prefix;      // key bits decided so far
    uint32_t mask;        // which bits those are
    uint32_t k_rem;       // how many elements are still to be taken among those matching the prefix
    uint32_t ticket;      // workgroups finished in the current launch
    uint32_t pad[60];
};
static_assert(sizeof(SelectState) == 256, "state block is one 256-byte line");

// workspace layout: [SelectState][hist kBins u32][cnt_gt nb u32][cnt_eq nb u32]
__host__ __device__ inline size_t ws_hist_off() { return sizeof(SelectState); }
__host__ __device__ inline size_t ws_cnt_off() { return sizeof(SelectState) + kBins * sizeof(uint32_t); }

__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t b = __float_as_uint(s);
    if ((b & 0x7fffffffu) > 0x7f800000u) return 0u;        // NaN: below every number
    if (b == 0x80000000u) b = 0u;                           // -0 == +0
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Set bits of a ballot below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// k > 0: empty prefix, the passes refine it.  k == 0: the passes are skipped and the threshold is
// the key no score maps to (all ones), so nothing compares above or equal to it with need = 0.
__global__ void topk_init_kernel(SelectState *st, uint32_t *hist, uint32_t k)
{
    for (int i = threadIdx.x; i < kBins; i += blockDim.x) hist[i] = 0;
    if (threadIdx.x == 0) {
        st->prefix = k ? 0u : 0xffffffffu;
        st->mask = 0;
        st->k_rem = k;
        st->ticket = 0;
    }
}

// One radix pass.  PASS is the digit position (0 = most significant).
template <int PASS>
__global__ __launch_bounds__(kThreads) void topk_hist_kernel(const float *__restrict__ score, int64_t N,
                                                             SelectState *st, uint32_t *hist)
{
    __shared__ uint32_t lh[kBins];
    __shared__ uint32_t wave_tot[kThreads / kWave];
    __shared__ uint32_t is_last;
    const int shift = kShift[PASS];
    const uint32_t nb = 1u << kBits[PASS];
    for (int i = threadIdx.x; i < kBins; i += kThreads) lh[i] = 0;
    __syncthreads();
    const uint32_t prefix = st->prefix, mask = st->mask;
    const int64_t base = (int64_t)blockIdx.x * kChunk;
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        int64_t i = base + it * kThreads + threadIdx.x;       // order is irrelevant for counting
        if (i < N) {
            uint32_t key = score_key(score[i]);
            if ((key & mask) == prefix) atomicAdd(&lh[(key >> shift) & (nb - 1)], 1u);
        }
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nb; b += kThreads) {
        uint32_t c = lh[b];
        if (c) atomicAdd(&hist[b], c);
    }
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) is_last = (atomicAdd(&st->ticket, 1u) == gridDim.x - 1) ? 1u : 0u;
    __syncthreads();
    if (!is_last) return;
    __threadfence();

    // Last workgroup: walk the bins from the largest digit down until k_rem elements are covered.
    // Thread t owns bins [hi - t*per, hi - (t+1)*per) in descending order.
    const uint32_t per = nb / kThreads;                    // 8 or 4
    const uint32_t k_rem = st->k_rem;
    uint32_t cnt[8];
    uint32_t mine = 0;
    for (uint32_t j = 0; j < per; ++j) {
        uint32_t b = nb - 1 - (threadIdx.x * per + j);
        cnt[j] = __hip_atomic_load(&hist[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mine += cnt[j];
    }
    // exclusive prefix over threads (descending bins): wave scan, then across waves
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    uint32_t incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        uint32_t o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == kWave - 1) wave_tot[wv] = incl;
    __syncthreads();
    uint32_t before = incl - mine;
    for (int w = 0; w < wv; ++w) before += wave_tot[w];
    // the digit is the first bin (descending) whose running count reaches k_rem
    uint32_t run = before;
    for (uint32_t j = 0; j < per; ++j) {
        uint32_t b = nb - 1 - (threadIdx.x * per + j);
        if (run < k_rem && run + cnt[j] >= k_rem) {
            st->prefix = prefix | (b << shift);
            st->mask = mask | ((nb - 1) << shift);
            st->k_rem = k_rem - run;
        }
        run += cnt[j];
    }
    // reset for the next launch
    for (int i = threadIdx.x; i < kBins; i += kThreads) hist[i] = 0;
    if (threadIdx.x == 0) st->ticket = 0;
}

// Per-workgroup counts of keys above / equal to the threshold; the last workgroup turns them into
// exclusive offsets over workgroups (ascending index order).
__global__ __launch_bounds__(kThreads) void topk_count_kernel(const float *__restrict__ score, int64_t N,
                                                              SelectState *st, uint32_t *cnt_gt, uint32_t *cnt_eq)
{
    __shared__ uint32_t red_gt[kThreads / kWave], red_eq[kThreads / kWave];
    __shared__ uint32_t is_last;
    const uint32_t T = st->prefix;
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    uint32_t g = 0, e = 0;
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        int64_t i = base + it * kThreads + threadIdx.x;
        if (i < N) {
            uint32_t key = score_key(score[i]);
            g += key > T;
            e += key == T;
        }
    }
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        g += __shfl_xor(g, d);
        e += __shfl_xor(e, d);
    }
    if (lane == 0) {
        red_gt[wv] = g;
        red_eq[wv] = e;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sg = 0, se = 0;
        for (int w = 0; w < kThreads / kWave; ++w) {
            sg += red_gt[w];
            se += red_eq[w];
        }
        cnt_gt[blockIdx.x] = sg;
        cnt_eq[blockIdx.x] = se;
        __threadfence();
        is_last = (atomicAdd(&st->ticket, 1u) == gridDim.x - 1) ? 1u : 0u;
    }
    __syncthreads();
    if (!is_last) return;
    __threadfence();

    // exclusive scan of both count arrays over workgroups, by this one workgroup
    __shared__ uint32_t carry_g, carry_e;
    __shared__ uint32_t wt_g[kThreads / kWave], wt_e[kThreads / kWave];
    if (threadIdx.x == 0) {
        carry_g = 0;
        carry_e = 0;
    }
    __syncthreads();
    const uint32_t nblk = gridDim.x;
    for (uint32_t b0 = 0; b0 < nblk; b0 += kThreads) {
        uint32_t b = b0 + threadIdx.x;
        uint32_t vg = 0, ve = 0;
        if (b < nblk) {
            vg = __hip_atomic_load(&cnt_gt[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ve = __hip_atomic_load(&cnt_eq[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        uint32_t ig = vg, ie = ve;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            uint32_t og = __shfl_up(ig, d), oe = __shfl_up(ie, d);
            if (lane >= d) {
                ig += og;
                ie += oe;
            }
        }
        if (lane == kWave - 1) {
            wt_g[wv] = ig;
            wt_e[wv] = ie;
        }
        __syncthreads();
        uint32_t pg = carry_g + ig - vg, pe = carry_e + ie - ve;
        for (int w = 0; w < wv; ++w) {
            pg += wt_g[w];
            pe += wt_e[w];
        }
        if (b < nblk) {
            cnt_gt[b] = pg;
            cnt_eq[b] = pe;
        }
        __syncthreads();
        if (threadIdx.x == kThreads - 1) {
            carry_g = pg + vg;
            carry_e = pe + ve;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) st->ticket = 0;
}

// Writes idx_sel / idx_remain / mask / skip counters.  Thread t owns elements
// [base + t*kItems, base + (t+1)*kItems), so ranks follow index order.
__global__ __launch_bounds__(kThreads) void topk_emit_kernel(const float *__restrict__ score, int64_t N,
                                                             const SelectState *st, const uint32_t *off_gt,
                                                             const uint32_t *off_eq, int32_t *__restrict__ idx_sel,
                                                             int32_t *__restrict__ idx_remain,
                                                             uint8_t *__restrict__ sel_mask,
                                                             int32_t *__restrict__ skip_count)
{
    __shared__ uint32_t wt_g[kThreads / kWave], wt_e[kThreads / kWave];
    const uint32_t T = st->prefix, need = st->k_rem;
    const int64_t base = (int64_t)blockIdx.x * kChunk + (int64_t)threadIdx.x * kItems;
    uint32_t gt_bits = 0, eq_bits = 0;
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        int64_t i = base + it;
        if (i < N) {
            uint32_t key = score_key(score[i]);
            gt_bits |= (uint32_t)(key > T) << it;
            eq_bits |= (uint32_t)(key == T) << it;
        }
    }
    const uint32_t mg = __popc(gt_bits), me = __popc(eq_bits);
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    uint32_t ig = mg, ie = me;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        uint32_t og = __shfl_up(ig, d), oe = __shfl_up(ie, d);
        if (lane >= d) {
            ig += og;
            ie += oe;
        }
    }
    if (lane == kWave - 1) {
        wt_g[wv] = ig;
        wt_e[wv] = ie;
    }
    __syncthreads();
    uint32_t g_before = off_gt[blockIdx.x] + ig - mg;     // keys > T before this thread's first element
    uint32_t e_before = off_eq[blockIdx.x] + ie - me;     // keys == T before it
    for (int w = 0; w < wv; ++w) {
        g_before += wt_g[w];
        e_before += wt_e[w];
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        int64_t i = base + it;
        if (i >= N) break;
        const bool g = (gt_bits >> it) & 1u, e = (eq_bits >> it) & 1u;
        const uint32_t sel_before = g_before + (e_before < need ? e_before : need);
        const bool sel = g || (e && e_before < need);
        if (sel)
            idx_sel[sel_before] = (int32_t)i;
        else if (idx_remain)
            idx_remain[i - sel_before] = (int32_t)i;
        if (sel_mask) sel_mask[i] = sel ? 1 : 0;
        if (skip_count) skip_count[i] = sel ? 0 : skip_count[i] + 1;
        g_before += g;
        e_before += e;
    }
}

// ---- small inputs: the whole selection in one launch of workgroups that each do all of it, the keys in registers, and share the outputs.  Wave w owns the elements
// [w*items*64, (w+1)*items*64), element (w*items + j)*64 + lane in register j, so that loads and stores are coalesced and
// ranks in index order come from ballots.  The keys' range is found first and the passes look at its bits only: digit 1 is
// (key - lowest) >> shift, up to 2048 bins, digit 2 the next 11 bits of the keys that share it, and so on until the shift
// is 0 (at most three passes; scores of one magnitude need two).  That spreads scores of similar size, which the top
// bits of the key would put into one or two bins; equal scores find four counters per bin, and the lowest are not counted at all.
// Bound by instructions issued on one CU and by the chain of barriers.  Measured, indices alone / with every output (before:
// keys in LDS, digits at fixed bits, a contiguous run of elements per thread): 4096 scores 10.0 / 11.4 -> 6.9 / 7.1 us, 17550
// 20.0 / 40.2 -> 12.8 / 15.5, 32768 30.1 / 77.7 -> 21.4 / 26.3; 17550 scores, 70 % of them 0, 22.7 / 42.3 -> 15.0 / 17.4 (with the
// lowest counted 20.8 / 23.2), 25000, nearly all 0, 28.3 / 58.2 -> 19.7 / 23.4 (32.5 / 36.1), 17550 half 1 and half -1 24.4 / 44.6 ->
// 19.5 / 22.0.  A run-time count of elements per thread took 18.1 / 20.5 at 17550, eight copies of the histogram side by side
// 20.5 / 23.5; a digit that many lanes share counted by ballot cost all other distributions 0.5 us; a first digit of 8 bits with 32 copies cost
// most distributions 0.3 - 0.9 us (17550 half 1 and half -1 21.8 -> 19.0).
// The outputs are a store of 4 bytes and more per element from one CU, and their order takes ballots.  So ITEMS / 2 workgroups do the same
// selection, each on a CU, and a thread of each writes the outputs of two elements.  One workgroup / now, us, indices alone and every output:
// 4096 scores 6.9 / 7.1 -> 6.5 / 6.7, 17550 13.2 / 15.7 -> 11.6 / 11.7, 32768 21.7 / 26.7 -> 18.4 / 18.6; two workgroups 12.2 / 13.0 at 17550.
constexpr int kSmallMax = 32768;
constexpr int kOutItems = 2;                // elements of a thread whose outputs a workgroup writes
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kCopyPitch = kBins + 16;       // of the histogram's copies: their counters lie in different banks
constexpr uint32_t kPad = 0xffffffffu;      // stands for no element; above every key (the largest is +inf's, 0xff800000)

// Writes the outputs of a workgroup whose wave w owns ITEMS * 64 consecutive elements, element first + 64 j in register j: ranks in
// index order come from ballots.  g_before and e_before count the keys above / equal to T in front of the workgroup's elements.
// PARTS workgroups may share the elements: all count, and each writes the outputs of its part of a wave's registers, whose counters
// `skip` holds.
template <int ITEMS, int PARTS>
__device__ __forceinline__ void emit_in_order(const uint32_t (&key)[ITEMS], const int32_t (&skip)[ITEMS / PARTS], int first, int wave, int lane,
                                              uint32_t T, uint32_t need, uint32_t g_before, uint32_t e_before, uint32_t *wt_a,
                                              uint32_t *wt_b, int32_t *__restrict__ idx_sel, int32_t *__restrict__ idx_remain,
                                              uint8_t *__restrict__ sel_mask, int32_t *__restrict__ skip_count, int part)
{
    static_assert(ITEMS % PARTS == 0, "whole registers");
    auto above = [&](uint32_t kk) { return kk - (T + 1) < kPad - (T + 1); };       // kk > T and an element
    uint32_t mg = 0, me = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        mg += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(above(key[j])));
        me += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(key[j] == T));
    }
    if (lane == 0) {
        wt_a[wave] = mg;
        wt_b[wave] = me;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
        g_before += w < wave ? wt_a[w] : 0u;
        e_before += w < wave ? wt_b[w] : 0u;
    }
    g_before = __builtin_amdgcn_readfirstlane(g_before);      // in front of the wave's present 64 elements from here on
    e_before = __builtin_amdgcn_readfirstlane(e_before);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = first + j * kWave;
        bool sel = above(key[j]);
        const uint64_t gm = __builtin_amdgcn_ballot_w64(sel), em = __builtin_amdgcn_ballot_w64(key[j] == T);
        uint32_t sel_before = g_before + lanes_below(gm);
        if (em == 0) {
            sel_before += e_before < need ? e_before : need;
        } else {
            const uint32_t eb = e_before + lanes_below(em);
            sel_before += eb < need ? eb : need;
            sel = sel || (key[j] == T && eb < need);
        }
        if (PARTS == 1 || j / (ITEMS / PARTS) == part) {
            if (sel)
                idx_sel[sel_before] = i;
            else if (idx_remain && key[j] != kPad)
                idx_remain[(uint32_t)i - sel_before] = i;
            if (key[j] != kPad) {
                if (sel_mask) sel_mask[i] = sel ? 1 : 0;
                if (skip_count) skip_count[i] = sel ? 0 : skip[j % (ITEMS / PARTS)] + 1;
            }
        }
        g_before += (uint32_t)__popcll(gm);
        e_before += (uint32_t)__popcll(em);
    }
}

template <int ITEMS>
__global__ __launch_bounds__(kSmallThreads) void topk_small_kernel(const float *__restrict__ score, int32_t N, uint32_t k,
                                                                   int32_t *__restrict__ idx_sel,
                                                                   int32_t *__restrict__ idx_remain,
                                                                   uint8_t *__restrict__ sel_mask,
                                                                   int32_t *__restrict__ skip_count)
{
    // copies of the histogram, by lane: equal digits of a wave meet 16 (32) to a counter instead of 64; few scores pay more for
    // clearing and reading four than they gain (50 scores 6.85 us with four, 6.45 with two)
    constexpr int kCopies = ITEMS == 2 ? 2 : 4;
    __shared__ __attribute__((aligned(16))) uint32_t hist[kCopyPitch * kCopies];
    __shared__ uint32_t wt_a[kSmallWaves], wt_b[kSmallWaves];
    __shared__ uint32_t s_base, s_krem;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int first = wave * ITEMS * kWave + lane;                      // element j of this thread: first + 64 j
    uint32_t key[ITEMS];
    constexpr int PARTS = ITEMS / kOutItems;
    const int part = PARTS == 1 ? 0 : blockIdx.x;                       // the elements whose outputs, and counters, are this workgroup's
    int32_t skip[kOutItems];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = first + j * kWave < N ? first + j * kWave : N - 1;     // unconditional loads stay in flight together
        key[j] = __float_as_uint(score[i]);
    }
    if (skip_count) {
#pragma unroll
        for (int j = 0; j < kOutItems; ++j) {
            const int i = first + (part * kOutItems + j) * kWave;
            skip[j] = skip_count[i < N ? i : N - 1];
        }
    }
    for (int i = tid; i < kCopyPitch * kCopies / 4; i += kSmallThreads) reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0, 0, 0, 0);
    uint32_t *mine = hist + (lane & (kCopies - 1)) * kCopyPitch;
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t kk = score_key(__uint_as_float(key[j]));
        lo = kk < lo ? kk : lo;                                     // the last element's key again where there is none
        hi = kk > hi ? kk : hi;
        key[j] = first + j * kWave < N ? kk : kPad;
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        const uint32_t l = __shfl_xor(lo, d), h = __shfl_xor(hi, d);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    if (lane == 0) {
        wt_a[wave] = lo;
        wt_b[wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
        lo = wt_a[w] < lo ? wt_a[w] : lo;
        hi = wt_b[w] > hi ? wt_b[w] : hi;
    }
    // k == 0: a threshold no key reaches, nothing is selected
    uint32_t T = kPad - 1, need = 0;
    if (k > 0) {
        // the candidates are the keys in [base, base + last]; k_rem of them are still to be taken
        uint32_t base = __builtin_amdgcn_readfirstlane(lo), last = __builtin_amdgcn_readfirstlane(hi) - base, k_rem = k;
        for (;;) {
            const int width = last ? 32 - __builtin_clz(last) : 0;
            const int shift = width > 11 ? width - 11 : 0;
            // Keys equal to the lowest of the range are not counted (the walk below ends at them anyway): often many tokens share
            // the lowest score, and all their atomics would meet on the counters of one bin.
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t off = key[j] - base;
                if (off - 1 < last) atomicAdd(&mine[off >> shift], 1u);
            }
            __syncthreads();
            // the digit: walking the bins from the largest down, the first whose running count reaches k_rem.
            // Thread t owns bins 2047 - 2t and 2046 - 2t.
            const uint32_t top = kBins - 1 - 2 * tid;
            uint2 *cells = reinterpret_cast<uint2 *>(hist + top - 1);
            uint32_t c0 = 0, c1 = 0;
#pragma unroll
            for (int c = 0; c < kCopies; ++c) {
                const uint2 u = cells[c * (kCopyPitch / 2)];
                c1 += u.x;
                c0 += u.y;
            }
            if (tid == kSmallThreads - 1) c1 += k_rem;          // bin 0, with the uncounted keys: the last resort
            uint32_t incl = c0 + c1;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t o = __shfl_up(incl, d);
                if (lane >= d) incl += o;
            }
            if (lane == kWave - 1) wt_a[wave] = incl;
#pragma unroll
            for (int c = 0; c < kCopies; ++c) cells[c * (kCopyPitch / 2)] = make_uint2(0, 0);           // for the next pass
            __syncthreads();
            uint32_t run = incl - (c0 + c1);
#pragma unroll
            for (int w = 0; w < kSmallWaves; ++w) run += w < wave ? wt_a[w] : 0u;
            if (run < k_rem && run + c0 + c1 >= k_rem) {          // true for exactly one thread
                const bool second = run + c0 < k_rem;
                s_base = base + ((second ? top - 1 : top) << shift);
                s_krem = k_rem - run - (second ? c0 : 0u);
            }
            __syncthreads();
            base = __builtin_amdgcn_readfirstlane(s_base);
            k_rem = __builtin_amdgcn_readfirstlane(s_krem);
            if (shift == 0) break;
            last = (1u << shift) - 1;
        }
        T = base;
        need = k_rem;
    }
    // last read of wt_a before the barriers above (k == 0: for the key range, unused then)
    emit_in_order<ITEMS, PARTS>(key, skip, first, wave, lane, T, need, 0u, 0u, wt_a, wt_b, idx_sel, idx_remain, sel_mask, skip_count, part);
}

// ---- more scores than one workgroup takes: a launch for each of three digits and one for the outputs.  A workgroup owns 12288
// elements, laid out as in the kernel above.  Its part of a pass is a slot of its own in the workspace, for every bin the number of
// its candidates in that bin or a higher one, 16 bits each.  The next launch adds up the slots: the digit is the highest bin whose sum
// reaches what is left to be taken, and the sum over the slots in front of a workgroup's own says how many larger keys precede its
// elements.  Every workgroup does that for itself, so nothing is cleared, counted by tickets or merged by atomics, and no launch ends with
// one workgroup at work alone.  Passes 0 and 2 use the same slots: pass 2 writes them after pass 1 has read them.
// Bound by the start of four launches and, in each, the chain of load, histogram, scan and store (6 us apiece at 118800 scores).
constexpr int kSlotItems = 12;
constexpr int kSlotChunk = kSlotItems * kSmallThreads;
// Workgroups that share the writing of a chunk's outputs.  Each repeats the sums over the slots, which only pays while every one of them has a
// CU of its own: four, 256 at the most scores that come here.  us, every output, with 1 / 2 / 4 / 6 / 12: 33000 scores 25.2 / 24.4 / 23.8 /
// 23.6 / 23.3, 118800 25.8 / 24.9 / 24.3 / 24.2 / 23.9, 262144 30.7 / 29.9 / 29.4 / 29.4 / 36.1, 786432 40.8 / 40.4 / 40.0 / 49.9 / 60.9
constexpr int kEmitParts = 4;
// Slots that a thread has in flight.  3 to 64 of them are added up: more in flight save round trips, but the branches around those that are
// not there are passed.  us, indices alone, with 10 / 16 / 22 / 32: 33000 scores 22.5 / 23.0 / 23.7 / 25.8, 118800 23.8 / 24.0 / 24.6 / 26.7, 262144
// 27.9 / 27.4 / 26.3 / 27.9, 786432 38.6 / 36.3 / 36.0 / 36.7; 16 is best over the range
constexpr int kSlotBatch = 16;
constexpr int64_t kSlotMax = 64 * (int64_t)kSlotChunk;
constexpr int kSlotBits[3] = {11, 10, 11};
constexpr int kSlotShift[3] = {21, 11, 0};
constexpr int kSlotWordsA = 1 << (kSlotBits[0] - 1), kSlotWordsB = 1 << (kSlotBits[1] - 1);        // of 32 bits, a slot of passes 0 and 2 / pass 1

// What a workgroup knows after a pass: the threshold's digits so far, how many elements are still to be taken among those that share
// them, how many larger keys lie in front of its elements.
struct SlotRecord {
    uint32_t prefix, k_rem, above, pad;
};

// workspace layout: [slots of passes 0 and 2][slots of pass 1][records], one of each per workgroup
constexpr size_t slot_bytes(int64_t N)
{
    const size_t n_wg = (size_t)((N + kSlotChunk - 1) / kSlotChunk);
    return n_wg * ((kSlotWordsA + kSlotWordsB) * sizeof(uint32_t) + sizeof(SlotRecord));
}

struct SlotShared {
    uint32_t tot[kSlotWordsA + 1], pre[kSlotWordsA + 1];
    uint32_t digit, k_rem, above, equal;
};

// The digit of a pass from its slots.  equal counts the keys with that digit in front of workgroup `me`.
template <int WORDS>
__device__ __forceinline__ void resolve_digit(const uint32_t *__restrict__ slots, int n_wg, int me, uint32_t k_rem, SlotShared &sh)
{
    const int t = threadIdx.x;
    uint32_t lo = 0, hi = 0, pre_lo = 0, pre_hi = 0;       // bins 2t and 2t + 1: over all workgroups, over those in front
    if (t < WORDS) {
        for (int w0 = 0; w0 < n_wg; w0 += kSlotBatch) {
            uint32_t v[kSlotBatch];
#pragma unroll
            for (int j = 0; j < kSlotBatch; ++j)
                if (w0 + j < n_wg) v[j] = slots[(w0 + j) * WORDS + t];
#pragma unroll
            for (int j = 0; j < kSlotBatch; ++j)
                if (w0 + j < n_wg) {
                    const uint32_t u = v[j];
                    pre_lo += w0 + j < me ? u & 0xffffu : 0u;
                    pre_hi += w0 + j < me ? u >> 16 : 0u;
                    lo += u & 0xffffu;
                    hi += u >> 16;
                }
        }
        sh.tot[t] = lo;
        sh.pre[t] = pre_lo;
    }
    if (t == 0) sh.tot[WORDS] = sh.pre[WORDS] = 0;
    __syncthreads();
    if (t < WORDS) {
        const uint32_t next = sh.tot[t + 1], pre_next = sh.pre[t + 1];
        // sums fall from bin to bin, bin 0 has all the candidates: true for exactly one bin
        if (lo >= k_rem && next < k_rem) {
            const bool upper = hi >= k_rem;
            sh.digit = 2 * t + (upper ? 1 : 0);
            sh.k_rem = k_rem - (upper ? next : hi);
            sh.above = upper ? pre_next : pre_hi;
            sh.equal = upper ? pre_hi - pre_next : pre_lo - pre_hi;
        }
    }
    __syncthreads();
}

template <int PASS>
__global__ __launch_bounds__(kSmallThreads) void topk_slot_kernel(const float *__restrict__ score, int32_t N, uint32_t k,
                                                                  const uint32_t *__restrict__ slots_in, uint32_t *__restrict__ slots_out,
                                                                  SlotRecord *__restrict__ records)
{
    constexpr int kCopies = 4;
    constexpr int BINS = 1 << kSlotBits[PASS], SHIFT = kSlotShift[PASS];
    __shared__ __attribute__((aligned(16))) uint32_t hist[kCopyPitch * kCopies];
    __shared__ SlotShared sh;
    __shared__ uint32_t wt[kSmallWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int first = (int)blockIdx.x * kSlotChunk + wave * kSlotItems * kWave + lane;
    uint32_t key[kSlotItems];
#pragma unroll
    for (int j = 0; j < kSlotItems; ++j)
        key[j] = __float_as_uint(score[first + j * kWave < N ? first + j * kWave : N - 1]);
    for (int i = tid; i < kCopyPitch * kCopies / 4; i += kSmallThreads) reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0, 0, 0, 0);
    SlotRecord rec = {0u, k, 0u, 0u};
    if (PASS > 0) {
        constexpr int P = PASS > 0 ? PASS - 1 : 0;
        if (PASS > 1) rec = records[blockIdx.x];
        resolve_digit<(1 << kSlotBits[P]) / 2>(slots_in, gridDim.x, blockIdx.x, rec.k_rem, sh);
        rec = SlotRecord{rec.prefix | (sh.digit << kSlotShift[P]), sh.k_rem, rec.above + sh.above, 0u};
        if (tid == 0) records[blockIdx.x] = rec;
    } else {
        __syncthreads();
    }
    uint32_t *mine = hist + (lane & (kCopies - 1)) * kCopyPitch;
#pragma unroll
    for (int j = 0; j < kSlotItems; ++j) {
        const uint32_t kk = score_key(__uint_as_float(key[j]));
        constexpr int TOP = PASS > 0 ? kSlotShift[PASS > 0 ? PASS - 1 : 0] : 0;
        const bool candidate = PASS == 0 || (kk ^ rec.prefix) >> TOP == 0;
        if (candidate && first + j * kWave < N) atomicAdd(&mine[(kk >> SHIFT) & (BINS - 1)], 1u);
    }
    __syncthreads();
    // thread t owns bins BINS - 1 - 2t and BINS - 2 - 2t
    uint32_t c0 = 0, c1 = 0;
    if (tid < BINS / 2) {
        const uint2 *cells = reinterpret_cast<const uint2 *>(hist + BINS - 2 - 2 * tid);
#pragma unroll
        for (int c = 0; c < kCopies; ++c) {
            const uint2 u = cells[c * (kCopyPitch / 2)];
            c1 += u.x;
            c0 += u.y;
        }
    }
    uint32_t incl = c0 + c1;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == kWave - 1) wt[wave] = incl;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) incl += w < wave ? wt[w] : 0u;
    if (tid < BINS / 2) slots_out[(int)blockIdx.x * (BINS / 2) + BINS / 2 - 1 - tid] = incl | (incl - c1) << 16;
}

// k == 0: a threshold no key reaches.
__global__ __launch_bounds__(kSmallThreads) void topk_slot_emit_kernel(const float *__restrict__ score, int32_t N, uint32_t k,
                                                                       const uint32_t *__restrict__ slots,
                                                                       const SlotRecord *__restrict__ records,
                                                                       int32_t *__restrict__ idx_sel, int32_t *__restrict__ idx_remain,
                                                                       uint8_t *__restrict__ sel_mask, int32_t *__restrict__ skip_count)
{
    __shared__ SlotShared sh;
    __shared__ uint32_t wt_a[kSmallWaves], wt_b[kSmallWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int first = (int)blockIdx.x * kSlotChunk + wave * kSlotItems * kWave + lane;
    uint32_t key[kSlotItems];
#pragma unroll
    for (int j = 0; j < kSlotItems; ++j)
        key[j] = __float_as_uint(score[first + j * kWave < N ? first + j * kWave : N - 1]);
    // the counters that this workgroup writes, and no others: the chunk's other workgroups write theirs at the same time
    constexpr int kMine = kSlotItems / kEmitParts;
    int32_t skip[kMine];
#pragma unroll
    for (int j = 0; j < kMine; ++j) {
        const int i = first + ((int)blockIdx.y * kMine + j) * kWave;
        if (skip_count && i < N) skip[j] = skip_count[i];
    }
    uint32_t T = kPad - 1, need = 0, above = 0, equal = 0;
    if (k > 0) {
        const SlotRecord rec = records[blockIdx.x];
        resolve_digit<kSlotWordsA>(slots, gridDim.x, blockIdx.x, rec.k_rem, sh);
        T = __builtin_amdgcn_readfirstlane(rec.prefix | sh.digit);
        need = __builtin_amdgcn_readfirstlane(sh.k_rem);
        above = rec.above + sh.above;
        equal = sh.equal;
    }
#pragma unroll
    for (int j = 0; j < kSlotItems; ++j)
        key[j] = first + j * kWave < N ? score_key(__uint_as_float(key[j])) : kPad;
    emit_in_order<kSlotItems, kEmitParts>(key, skip, first, wave, lane, T, need, above, equal, wt_a, wt_b, idx_sel, idx_remain, sel_mask,
                                          skip_count, (int)blockIdx.y);
}

// ---- astraea_select_topk_static: the same selection for callers that cannot allocate.  The selection state,
// the histogram and the per-workgroup counts live in this file-scope device array instead of a caller's
// workspace: 256 B of state + 8 KiB of histogram + 8 B per 2048 scores, or the slots, 6160 B per 12288 scores: 385 KiB
// for the largest input that uses them.  Every GPU the library runs on holds its own copy, at its own address, until the
// process ends.  In host code the array's name only stands for the symbol: the address kernels are given is
// the one hipGetSymbolAddress returns for the device that is current, looked up once per device.
constexpr int64_t kStaticMaxN = (int64_t)1 << 22;
constexpr size_t kStaticSlotBytes = slot_bytes(kSlotMax);
constexpr size_t kStaticCountBytes = sizeof(SelectState) + kBins * sizeof(uint32_t) + 2 * (size_t)(kStaticMaxN / kChunk) * sizeof(uint32_t);
constexpr size_t kStaticBytes = kStaticSlotBytes > kStaticCountBytes ? kStaticSlotBytes : kStaticCountBytes;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void *g_scratch_ptr[kMaxDevices] = {};

}  // namespace

int64_t topk_static_max_n() { return kStaticMaxN; }

// Device address of `scratch` on the current device (first use on a device looks it up and keeps it).
int topk_static_scratch(void **ptr_out)
{
    static_assert(kStaticBytes % 256 == 0, "scratch size keeps the 256-byte granularity of the workspace");
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(ASTRAEA_ERR_HIP, "astraea_select_topk_static: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(ASTRAEA_ERR_UNSUPPORTED, "astraea_select_topk_static: device ordinal %d not below %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(ASTRAEA_ERR_HIP, "astraea_select_topk_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *ptr_out = g_scratch_ptr[dev];
    return ASTRAEA_OK;
}

size_t topk_static_bytes() { return kStaticBytes; }

size_t topk_min_workspace_bytes(int64_t N)
{
    const int64_t nblk = (N + kChunk - 1) / kChunk;
    size_t b = ws_cnt_off() + 2 * (size_t)(nblk > 0 ? nblk : 1) * sizeof(uint32_t);
    return (b + 255) & ~(size_t)255;
}

size_t topk_workspace_bytes(int64_t N)
{
    const size_t least = topk_min_workspace_bytes(N), slots = (slot_bytes(N) + 255) & ~(size_t)255;
    return N > kSmallMax && N <= kSlotMax && slots > least ? slots : least;
}

int launch_select_topk(const float *score, int64_t N, int64_t k, int32_t *idx_sel, int32_t *idx_remain,
                       uint8_t *sel_mask, int32_t *skip_count, void *workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (N == 0) return ASTRAEA_OK;
    if (N <= kSmallMax) {
        auto go = [&](auto kernel, int items) {
            hipLaunchKernelGGL(kernel, dim3(items / kOutItems), dim3(kSmallThreads), 0, stream, score, (int32_t)N, (uint32_t)k, idx_sel,
                               idx_remain, sel_mask, skip_count);
        };
        // elements per thread, rounded up to an even number: a constant, so that nothing is tested per element and
        // all loads go out together
        switch ((N + 2 * kSmallThreads - 1) / (2 * kSmallThreads)) {
        case 1: go(topk_small_kernel<2>, 2); break;
        case 2: go(topk_small_kernel<4>, 4); break;
        case 3: go(topk_small_kernel<6>, 6); break;
        case 4: go(topk_small_kernel<8>, 8); break;
        case 5: go(topk_small_kernel<10>, 10); break;
        case 6: go(topk_small_kernel<12>, 12); break;
        case 7: go(topk_small_kernel<14>, 14); break;
        case 8: go(topk_small_kernel<16>, 16); break;
        case 9: go(topk_small_kernel<18>, 18); break;
        case 10: go(topk_small_kernel<20>, 20); break;
        case 11: go(topk_small_kernel<22>, 22); break;
        case 12: go(topk_small_kernel<24>, 24); break;
        case 13: go(topk_small_kernel<26>, 26); break;
        case 14: go(topk_small_kernel<28>, 28); break;
        case 15: go(topk_small_kernel<30>, 30); break;
        default: go(topk_small_kernel<32>, 32); break;
        }
        return check_launch("astraea_select_topk");
    }
    if (N <= kSlotMax && workspace_bytes >= slot_bytes(N)) {
        const unsigned n_wg = (unsigned)((N + kSlotChunk - 1) / kSlotChunk);
        uint32_t *slots_a = reinterpret_cast<uint32_t *>(workspace), *slots_b = slots_a + (size_t)n_wg * kSlotWordsA;
        SlotRecord *records = reinterpret_cast<SlotRecord *>(slots_b + (size_t)n_wg * kSlotWordsB);
        auto pass = [&](auto kernel, const uint32_t *in, uint32_t *out) {
            hipLaunchKernelGGL(kernel, dim3(n_wg), dim3(kSmallThreads), 0, stream, score, (int32_t)N, (uint32_t)k, in, out, records);
        };
        if (k > 0) {
            pass(topk_slot_kernel<0>, slots_b, slots_a);
            pass(topk_slot_kernel<1>, slots_a, slots_b);
            pass(topk_slot_kernel<2>, slots_b, slots_a);
        }
        hipLaunchKernelGGL(topk_slot_emit_kernel, dim3(n_wg, kEmitParts), dim3(kSmallThreads), 0, stream, score, (int32_t)N, (uint32_t)k, slots_a,
                           records, idx_sel, idx_remain, sel_mask, skip_count);
        return check_launch("astraea_select_topk");
    }
    const unsigned nblk = (unsigned)((N + kChunk - 1) / kChunk);
    SelectState *st = reinterpret_cast<SelectState *>(workspace);
    uint32_t *hist = reinterpret_cast<uint32_t *>((char *)workspace + ws_hist_off());
    uint32_t *cnt_gt = reinterpret_cast<uint32_t *>((char *)workspace + ws_cnt_off());
    uint32_t *cnt_eq = cnt_gt + nblk;
    hipLaunchKernelGGL(topk_init_kernel, dim3(1), dim3(kThreads), 0, stream, st, hist, (uint32_t)k);
    if (k > 0) {
        hipLaunchKernelGGL(topk_hist_kernel<0>, dim3(nblk), dim3(kThreads), 0, stream, score, N, st, hist);
        hipLaunchKernelGGL(topk_hist_kernel<1>, dim3(nblk), dim3(kThreads), 0, stream, score, N, st, hist);
        hipLaunchKernelGGL(topk_hist_kernel<2>, dim3(nblk), dim3(kThreads), 0, stream, score, N, st, hist);
    }
    hipLaunchKernelGGL(topk_count_kernel, dim3(nblk), dim3(kThreads), 0, stream, score, N, st, cnt_gt, cnt_eq);
    hipLaunchKernelGGL(topk_emit_kernel, dim3(nblk), dim3(kThreads), 0, stream, score, N, st, cnt_gt, cnt_eq, idx_sel,
                       idx_remain, sel_mask, skip_count);
    return check_launch("astraea_select_topk");
}

}  // namespace astraea
