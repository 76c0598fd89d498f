// astraea_sparse_attn_fwd, fp32 mode (paper, Algorithm 1 step 6: Softmax(Q_sel K^T / sqrt(d)) V over
// all N keys for the selected queries only).
//
// Everything stays in fp32: QK^T and PV run on the fp32 matrix instruction
// v_mfma_f32_32x32x2_f32, the softmax is the online (running max / running sum) form.
// Both products are computed transposed, S^T = K Q^T and O^T = V^T P^T, so that a lane owns one
// query column in every accumulator: row max, row sum and the rescale factor are per-lane values
// (one exchange between lane l and lane l+32), and the S^T accumulator registers feed the second
// product directly as its B operand.
//
// Shape on gfx950:
//  * workgroup = 4 waves x 32 queries, two workgroups per CU; keys are swept in tiles of 32.  K and V tiles go from global
//    memory straight into two LDS stages (global_load_lds_dwordx4), one tile ahead, one barrier per tile; 16-byte
//    chunks are XOR-swizzled inside a row, so that reads meet no bank conflicts.
//  * the first product's contraction is permuted: a lane reads 8 consecutive floats of its key row (two 16-byte reads) and
//    MFMA j of the step takes index pair {j, 8 + j}; the second product reads V by the float, 32 consecutive ones of a row.
//  * bound by the matrix pipe (4096 flops per MFMA in 64 clocks, 157 TFLOP/s) plus the vector instructions, which do not
//    overlap fp32 MFMAs.  So a row's exponent offset is not its exact running max: it is raised, to kSlack above the max so
//    far, only when a logit passes it, which after the first tiles is rare, and the other tiles rescale nothing and exchange
//    nothing between lanes: per logit half a max, an fma, an exponential and an add.  Probabilities stay at most 1 and the
//    arguments that matter close to 0, as under a running max, so accumulators overflow no earlier than theirs and the error is
//    no larger.  (An offset left at the first tile's max takes no max at all and is 2 - 5 % faster, but overflows on rows
//    that rise by r powers of two over values of 2^(128 - r), and its error grows with the rise, 6.5e-7 -> 11e-7 at 45 nats.)
// Measured (call with merge; before: tiles staged through registers between two barriers, running max, 4-byte K reads):
// 2048 queries x 4096 keys x 8 heads x 64 190 -> 153 us (112 TFLOP/s), 6000 x 6000 x 24 x 64 2292 -> 1816, 3000 x 6000 x 24 x
// 128 3431 -> 2129, 250 x 2500 x 8 x 128 79 -> 53.  Error against 64 bits, both: 6.7e-7 at the first, 6.5e-7 for rows that rise
// by 10, 30 or 45 nats; kSlack 1 / 2 / 3 / 4 at the first: 6.72 / 6.73 / 6.73 / 6.75e-7, 153.5 / 152.9 / 151.4 / 151.2 us.  Not
// bound by the number of workgroups per CU (forced to two: no change).
#include <type_traits>

#include "gfx950.h"

namespace astraea {
namespace {


constexpr int kWaves = 4;
constexpr int kBq = 32 * kWaves;   // queries per workgroup
constexpr int kBk = 32;            // keys per tile
constexpr float kSlack = 1.0f;     // log2 units by which a raised exponent offset lies above the row's max so far

__device__ __forceinline__ float xhalf_max(float x)
{
    // max of lane l and lane l^32
    float o = __shfl_xor(x, 32);
    return fmaxf(x, o);
}
__device__ __forceinline__ float xhalf_sum(float x) { return x + __shfl_xor(x, 32); }

__device__ __forceinline__ float lds_read_f32(uint32_t addr)
{
    return *reinterpret_cast<const float __attribute__((address_space(3))) *>((uintptr_t)addr);
}

// FAR: 32 rows span 4 GiB or more, copies take 64-bit lane addresses.
template <int D, bool FAR>
__global__ __launch_bounds__(kWaves *kWave, 2) void attn_f32_kernel(
    const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v, int64_t N, int32_t H,
    int64_t q_stride_n, int64_t q_stride_h, int64_t kv_stride_n, int64_t kv_stride_h,
    const int32_t *__restrict__ idx_sel, int64_t k_sel, int q_is_compact, float scale_log2e,
    float *__restrict__ o_sel, int64_t o_stride_n, int o_scatter, float *__restrict__ lse_sel, int32_t splits,
    int64_t tiles_per_split, float *__restrict__ partial)
{
    constexpr int kPartialPitch = D + 4;   // a share's row: D accumulators, running max, row sum (16-byte aligned)
    constexpr int DB = D / 32, DS = D / 16;
    constexpr int kRowBytes = D * 4, kTileBytes = kBk * kRowBytes, kStageBytes = 2 * kTileBytes;   // K tile, then V tile
    constexpr int kRowsPerCopy = 1024 / kRowBytes;                   // a copy instruction fills 1 KiB of a tile
    constexpr int kCopies = kTileBytes / 1024 / kWaves;              // per wave and tile, K and V each
    __shared__ __attribute__((aligned(1024))) char lds[2 * kStageBytes];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int qc = lane & 31, hf = lane >> 5;
    const int head = blockIdx.y;
    const int64_t r0 = (int64_t)blockIdx.x * kBq + wave * 32;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    // blockIdx.z takes one of `splits` consecutive key ranges (the budget-aware launch: a small selection
    // does not fill the chip with whole sweeps)
    const int64_t ntiles = (N + kBk - 1) / kBk;
    const int64_t t_begin = (int64_t)blockIdx.z * tiles_per_split;
    const int64_t t_end = t_begin + tiles_per_split < ntiles ? t_begin + tiles_per_split : ntiles;

    // ---- tile copies.  Instruction i of this wave fills rows kRowsPerCopy * (wave + 4 i) .. of the K and of the V tile.
    // Physical chunk p of row r holds logical chunk p ^ (r & 15) of K (a read takes one chunk of each of 32 rows) and
    // p ^ 8 * ((r / 4) & 1) of V (a read takes 128 bytes of rows r and r + 4).
    // Past the last tile of the range the last one is copied again, into a stage that nothing reads.
    const int64_t row_pitch = kv_stride_n * 4, tile_pitch = row_pitch * kBk;
    const char *kb = reinterpret_cast<const char *>(k + (int64_t)head * kv_stride_h);
    const char *vb = reinterpret_cast<const char *>(v + (int64_t)head * kv_stride_h);
    const int c_row = lane / (kRowBytes / 16), c_chunk = lane % (kRowBytes / 16);
    using Off = std::conditional_t<FAR, int64_t, uint32_t>;
    Off koff[kCopies], voff[kCopies];            // this lane's byte offsets inside a tile
    auto offsets = [&](int64_t rows) __attribute__((always_inline)) {      // of a tile with this many valid rows: those past them re-read the last
#pragma unroll
        for (int i = 0; i < kCopies; ++i) {
            const int r = kRowsPerCopy * (wave + kWaves * i) + c_row;
            const int64_t from = (r < rows ? r : rows - 1) * row_pitch;
            koff[i] = (Off)(from + ((c_chunk ^ (r & 15)) << 4));
            voff[i] = (Off)(from + ((c_chunk ^ (((r >> 2) & 1) << 3)) << 4));
        }
    };
    auto copy = [&](const char *kt, const char *vt, uint32_t stage, int n) __attribute__((always_inline)) {       // copy n of 2 * kCopies of a tile
        const int i = n >> 1;
        const char *src = n & 1 ? vt : kt;
        const Off off = n & 1 ? voff[i] : koff[i];
        const uint32_t dst = lds0 + stage + (n & 1 ? kTileBytes : 0) + (wave + kWaves * i) * 1024;
        if (FAR) dma16_far(src + off, dst);
        else dma16(src, (uint32_t)off, dst);
    };
    auto rows_of = [&](int64_t t) { return N - t * kBk < kBk ? N - t * kBk : (int64_t)kBk; };
    offsets(rows_of(t_begin));
#pragma unroll
    for (int n = 0; n < 2 * kCopies; ++n) copy(kb + t_begin * tile_pitch, vb + t_begin * tile_pitch, 0, n);

    // Q operand: lane holds query column qc, head-dim elements 16 s + 8 hf + j in qreg[8 s + j]
    int64_t r = r0 + qc;
    if (r > k_sel - 1) r = k_sel - 1;                    // ragged last tile: duplicate a valid row, never stored
    // an index outside [0, N) reads a valid row instead
    const int64_t qrow = q_is_compact ? r : (int64_t)clamp_row(idx_sel[r], (int32_t)N);
    const float *qp = q + qrow * q_stride_n + (int64_t)head * q_stride_h + 8 * hf;
    float qreg[D / 2];
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        const floatx4 lo = *reinterpret_cast<const floatx4 *>(qp + 16 * s), hi = *reinterpret_cast<const floatx4 *>(qp + 16 * s + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            qreg[8 * s + j] = lo[j];
            qreg[8 * s + 4 + j] = hi[j];
        }
    }
    // a load still counted as pending at the loop header would make the compiler wait on the copies inside the loop
#pragma unroll
    for (int s = 0; s < D / 2; ++s) asm volatile("" : "+v"(qreg[s]));

    // ---- LDS read offsets inside a stage; the stage is a constant of the unrolled loop.
    // K fragment (s, half): row qc, logical chunk 4 s + 2 hf + half; s >= 4 adds 256 bytes
    uint32_t ka[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) ka[u] = lds0 + qc * kRowBytes + (((4 * (u >> 1) + 2 * hf + (u & 1)) ^ (qc & 15)) << 4);
    // V fragment (i, b): row (i/4)*8 + 4 hf + i%4, float 32 b + qc; b >= 2 adds 256 bytes
    uint32_t va[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
        va[b] = lds0 + kTileBytes + 4 * hf * kRowBytes + (((8 * b + (qc >> 2)) ^ (hf << 3)) << 4) + 4 * (qc & 3);

    floatx16 oacc[DB];
    float m_run = -INFINITY;   // exponent offset of the row, in log2 units: at least the max of its scaled logits so far
    float l_run = 0.0f;        // this lane's share of the running sum
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[b][i] = 0.0f;

    // One tile out of stage PAR; the copies of the next tile go out behind the first MFMAs.
    auto tile = [&](int64_t t, auto par_tag) __attribute__((always_inline)) {
        constexpr uint32_t at = decltype(par_tag)::value * kStageBytes, next = kStageBytes - at;
        // tile t has landed, for every wave, and every wave is past its last read of tile t - 1
        wait_dma();
        __builtin_amdgcn_s_barrier();
        const int64_t tn = t + 1 < t_end ? t + 1 : t;
        if ((tn + 1) * kBk > N) offsets(N - tn * kBk);         // only the last tile can be ragged
        const char *kt = kb + tn * tile_pitch, *vt = vb + tn * tile_pitch;

        // S^T[key, q] = sum_d K[key, d] Q[q, d]
        floatx4 kf[2][2];
        float vf[2][4 * DB];
        auto read_k = [&](int s, int half) { kf[s & 1][half] = lds_read_f32x4(ka[2 * (s & 3) + half] + (at + (s >> 2) * 256)); };
        auto read_v = [&](int g, int u) {          // u = 4 keys of group g by DB blocks
            const int i = 4 * g + u / DB, b = u % DB;
            vf[g & 1][u] = lds_read_f32(va[b & 1] + (at + (8 * (i >> 2) + (i & 3)) * kRowBytes + (b >> 1) * 256));
        };
        read_k(0, 0);
        read_k(0, 1);
        floatx16 sacc;
#pragma unroll
        for (int i = 0; i < 16; ++i) sacc[i] = 0.0f;
#pragma unroll
        for (int s = 0; s < DS; ++s)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s & 1][j >> 2][j & 3], qreg[8 * s + j], sacc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (s + 1 < DS) {
                    if (j < 2) read_k(s + 1, j);
                    } else {
#pragma unroll
                    for (int u = 0; u < 4 * DB; ++u)
                        if (u * 8 / (4 * DB) == j) read_v(0, u);
                }
                if (s < 2 && j >= 3 && j < 3 + kCopies) copy(kt, vt, next, s * kCopies + j - 3);
                __builtin_amdgcn_sched_barrier(0);
            }
        // register i of sacc: key = 32 t + (i/4)*8 + hf*4 + i%4, query = qc
        if ((t + 1) * kBk > N) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (t * kBk + (i >> 2) * 8 + hf * 4 + (i & 3) >= N) sacc[i] = -INFINITY;
        }
        // A logit above its row's offset raises it, to kSlack above the row's max.  Lanes look at their own half of the keys;
        // only when one of them finds something do the halves meet and the accumulators get rescaled.
        float tmax = sacc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, sacc[i]);
        if (__builtin_amdgcn_ballot_w64(tmax * scale_log2e > m_run) != 0) {
            tmax = xhalf_max(tmax) * scale_log2e;
            const float m_new = tmax > m_run ? tmax + kSlack : m_run;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);          // 0 on the first tile
            l_run *= alpha;
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[b][i] *= alpha;
            m_run = m_new;
        }
        float ps[2] = {0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            sacc[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], scale_log2e, -m_run));
            ps[i & 1] += sacc[i];
        }
        l_run += ps[0] + ps[1];
        // O^T[d, q] += sum_key V[key, d] P^T[key, q]; MFMA i contracts keys (i/4)*8 + i%4 (+4 in the upper half)
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int b = 0; b < DB; ++b) {
                oacc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[(i >> 2) & 1][(i & 3) * DB + b], sacc[i], oacc[b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (i < 12) read_v((i >> 2) + 1, (i & 3) * DB + b);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    int64_t t = t_begin;
    for (; t + 1 < t_end; t += 2) {
        tile(t, P0{});
        tile(t + 1, P1{});
    }
    if (t < t_end) tile(t, P0{});
    const float l_tot = xhalf_sum(l_run);
    wait_dma();                // the copies past the last tile
    const int64_t rr = r0 + qc;
    if (rr >= k_sel) return;
    if (splits > 1) {
        // a key-range share: unnormalised accumulators, running max and row sum go to the workspace
        float *pp = partial + (((int64_t)blockIdx.z * k_sel + rr) * H + head) * kPartialPitch;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4 *>(pp + b * 32 + g * 8 + hf * 4) =
                    make_float4(oacc[b][4 * g], oacc[b][4 * g + 1], oacc[b][4 * g + 2], oacc[b][4 * g + 3]);
        if (hf == 0) {
            pp[D] = m_run;
            pp[D + 1] = l_tot;
        }
        return;
    }
    const float inv = 1.0f / l_tot;
    // compact output row rr, or straight into the cached buffer's row of that token
    const int64_t orow = o_scatter ? (int64_t)idx_sel[rr] : rr;
    float *op = o_sel + orow * o_stride_n + (int64_t)head * D;
    if (!o_scatter || (uint64_t)orow < (uint64_t)N)      // a row index outside the cached buffer writes nothing
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            // registers 4g..4g+3: head-dim b*32 + g*8 + hf*4 + 0..3
            float4 o4 = make_float4(oacc[b][4 * g] * inv, oacc[b][4 * g + 1] * inv, oacc[b][4 * g + 2] * inv,
                                    oacc[b][4 * g + 3] * inv);
            *reinterpret_cast<float4 *>(op + b * 32 + g * 8 + hf * 4) = o4;
        }
    if (lse_sel && hf == 0) lse_sel[rr * H + head] = (m_run + log2f(l_tot)) * 0.69314718055994530942f;
}

// Combines the key-range shares: with m* = max_s m_s and w_s = 2^(m_s - m*), O = sum_s w_s O_s / sum_s w_s l_s.
// One thread per (selected row, head, 4 head-dim elements), shares visited in order.
template <int D>
__global__ __launch_bounds__(256) void merge_f32_kernel(const float *__restrict__ partial, int32_t splits, int32_t H,
                                                        int64_t k_sel, int64_t n_rows, const int32_t *__restrict__ idx_sel,
                                                        float *__restrict__ o_sel, int64_t o_stride_n, int o_scatter,
                                                        float *__restrict__ lse_sel)
{
    constexpr int Q4 = D / 4, kPartialPitch = D + 4;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t rh = id / Q4;
    const int d4 = (int)(id % Q4) * 4;
    if (rh >= k_sel * H) return;
    const int64_t rr = rh / H;
    const int head = (int)(rh % H);
    const int64_t share = k_sel * H * (int64_t)kPartialPitch;
    const float *base = partial + rh * kPartialPitch;
    float m_star = -INFINITY;
    for (int s = 0; s < splits; ++s) m_star = fmaxf(m_star, base[s * share + D]);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float l = 0.0f;
    for (int s = 0; s < splits; ++s) {
        const float *ps = base + s * share;
        const float w = exp2f(ps[D] - m_star);
        const float4 o = *reinterpret_cast<const float4 *>(ps + d4);
        acc.x += w * o.x;
        acc.y += w * o.y;
        acc.z += w * o.z;
        acc.w += w * o.w;
        l += w * ps[D + 1];
    }
    const float inv = 1.0f / l;
    const int64_t orow = o_scatter ? (int64_t)idx_sel[rr] : rr;
    if (!o_scatter || (uint64_t)orow < (uint64_t)n_rows)
        *reinterpret_cast<float4 *>(o_sel + orow * o_stride_n + (int64_t)head * D + d4) =
            make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
    if (lse_sel && d4 == 0) lse_sel[rh] = (m_star + log2f(l)) * 0.69314718055994530942f;
}

// Key-range shares per work item: enough workgroups for two waves per SIMD of the chip, shares of at least 8 key
// tiles, at most 8 shares.  Large selections get 1 (no workspace, no merge).
static int32_t f32_splits(int64_t N, int32_t H, int64_t k_sel)
{
    const int64_t waves = ((k_sel + kBq - 1) / kBq) * H * kWaves;
    const int64_t ntiles = (N + kBk - 1) / kBk;
    int64_t s = 2048 / (waves > 0 ? waves : 1);
    if (s > ntiles / 8) s = ntiles / 8;
    if (s > 8) s = 8;
    return s < 2 ? 1 : (int32_t)s;
}

}  // namespace

// Partial-result bytes the key-range split needs at exactly k_sel selected queries (0 when it is not cut).
static size_t f32_partial_bytes(int64_t N, int32_t H, int32_t D, int64_t k_sel)
{
    if (N <= 0 || H <= 0 || k_sel <= 0) return 0;
    const int32_t s = f32_splits(N, H, k_sel);
    return s > 1 ? (size_t)s * (size_t)k_sel * (size_t)H * (size_t)(D + 4) * sizeof(float) : 0;
}

// What astraea_workspace_bytes names: enough for every selection of up to k_sel queries.  The need is not
// monotone in k_sel (fewer queries are cut into more shares), so a buffer sized once for the largest budget
// must cover the smaller ones too: the maximum over k' <= k_sel.  Within one count of query tiles the share
// count is fixed and the need grows with k', so only tile multiples (and k_sel itself) are candidates, and
// past 2048 waves nothing is cut any more.
size_t attn_f32_workspace_bytes(int64_t N, int32_t H, int32_t D, int64_t k_sel)
{
    if (N <= 0 || H <= 0 || k_sel <= 0) return 0;
    size_t need = f32_partial_bytes(N, H, D, k_sel);
    const int64_t t_max = 2048 / ((int64_t)H * kWaves) + 1;
    for (int64_t t = 1; t <= t_max && t * kBq <= k_sel; ++t) {
        const size_t b = f32_partial_bytes(N, H, D, t * kBq);
        if (b > need) need = b;
    }
    return need;
}

int launch_attn_f32(const void *q, const void *k, const void *v, int64_t N, int32_t H, int32_t D, int64_t q_stride_n,
                    int64_t q_stride_h, int64_t kv_stride_n, int64_t kv_stride_h, const int32_t *idx_sel,
                    int64_t k_sel, int q_is_compact, float scale, void *o_sel, int64_t o_stride_n, int o_scatter,
                    float *lse_sel, void *workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (k_sel == 0) return ASTRAEA_OK;
    // the split is an option: without a workspace of the size astraea_workspace_bytes names, every work item
    // sweeps all keys itself
    int32_t splits = f32_splits(N, H, k_sel);
    if (splits > 1 && (!workspace || workspace_bytes < f32_partial_bytes(N, H, D, k_sel))) splits = 1;
    const int64_t ntiles = (N + kBk - 1) / kBk;
    const int64_t tps = (ntiles + splits - 1) / splits;
    if ((int64_t)(splits - 1) * tps >= ntiles) splits = (int32_t)((ntiles + tps - 1) / tps);   // no empty share
    float *partial = (float *)workspace;
    dim3 grid((unsigned)((k_sel + kBq - 1) / kBq), (unsigned)H, (unsigned)splits), block(kWaves * kWave);
    const float c = scale * 1.44269504088896340736f;
    kernel_timer_begin(stream);
    const bool far = kv_stride_n * 4 * kBk >= (int64_t)1 << 32;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, (const float *)q, (const float *)k, (const float *)v, N, H,
                           q_stride_n, q_stride_h, kv_stride_n, kv_stride_h, idx_sel, k_sel, q_is_compact, c,
                           (float *)o_sel, o_stride_n, o_scatter, lse_sel, splits, tps, partial);
    };
    if (D == 64) go(far ? attn_f32_kernel<64, true> : attn_f32_kernel<64, false>);
    else go(far ? attn_f32_kernel<128, true> : attn_f32_kernel<128, false>);
    kernel_timer_end(stream);
    if (splits > 1) {
        const int64_t threads = k_sel * H * (D / 4);
        const dim3 mgrid((unsigned)((threads + 255) / 256));
        if (D == 64)
            hipLaunchKernelGGL(merge_f32_kernel<64>, mgrid, dim3(256), 0, stream, partial, splits, H, k_sel, N, idx_sel,
                               (float *)o_sel, o_stride_n, o_scatter, lse_sel);
        else
            hipLaunchKernelGGL(merge_f32_kernel<128>, mgrid, dim3(256), 0, stream, partial, splits, H, k_sel, N, idx_sel,
                               (float *)o_sel, o_stride_n, o_scatter, lse_sel);
    }
    return check_launch("astraea_sparse_attn_fwd(f32)");
}

}  // namespace astraea
