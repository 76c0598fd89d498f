// astraea_score: selection metric S_token (paper Sec. 3.2 "Selection Metric"; Algorithm 1 steps 1-2).
//
// The score decides which tokens are selected, so its fp32 value is defined to the bit: per token
// one accumulator walks the channels in ascending order.  One lane owns a token's accumulator and the
// rest of the design is about feeding it: both feature arrays are read in 16-byte vectors along the
// rows, turned into fp32 differences, and handed over through an LDS tile whose row t the lane of
// token t walks.  A chain step takes 5.4 clocks (2.2 ns), so 3072 channels are 6.9 us however many tokens there are.
//
// Two kernels, by the number of tokens:
//  * score_kernel: a workgroup of two waves owns 16 tokens.  The first wave loads slabs of [16 tokens x 128
//    channels] of both arrays, 32 KiB in flight, and writes the differences into one of two LDS tiles; the second runs the chains, half a
//    slab behind and reading 64 channels ahead of them, with one barrier per slab.  16 tokens per workgroup instead of 64 per wave is what a
//    short sequence needs: at 17550 tokens 64 per wave make 275 waves, one per CU, and each slab's
//    load latency, its conversion and its chain came one after the other.  Cold arrays, 64 per wave -> this
//    kernel, its chain waiting for each slab's reads: 2025 x 3072 bf16 63 -> 14.5 us; 17550 x 3072 80 -> 41 us (5.3 TB/s); 16384 x 512 13.1 -> 8.8;
//    4096 x 512 fp32 14.3 -> 8.5; 36000 x 3072 89.8 -> 74.5.  Tried: one wave for both jobs 22 and 49 us at
//    2025 and 17550 tokens; slabs of 8 x 512 B the same, 32 x 128 B 20 us at 2025.
//  * score_wide_kernel: a wave owns 64 tokens and does both jobs (a [64 x 128 byte] slab, the next one in flight).
//    With three such waves per CU or more the latencies are covered and all 64 lanes run chains: 111 us
//    (6.7 TB/s) at 60000 x 3072 and 217 us at 118800 x 3072, against 116 and 220 for the other kernel.  Arrays that
//    the memory-side cache may still hold need fewer: there the latencies are shorter, see launch_score.
//
// HBM-bound: 2*C*sizeof(T) bytes read and 4 written per token.
#include <type_traits>

#include "common.h"

#pragma clang fp contract(off)

namespace astraea {
namespace {

typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

constexpr int kWideWavesPerBlock = 4;
constexpr int kWideTok = 64;            // tokens per wave (lane == token in the reduce phase)
constexpr int kWideSegBytes = 128;      // bytes of each row handled per slab
constexpr int kWideVecPerLane = 8;      // 64 rows * 8 vec16 per row / 64 lanes
// The wide kernel is for at least this many tokens, three waves per CU; where both arrays fit in the memory-side cache, for
// fewer (launch_score has the figures).
constexpr int64_t kWideMinTokens = 3 * 256 * kWideTok;
constexpr int64_t kWideMinCachedBf16 = 28672, kWideMinCachedF32 = 20480;
constexpr int64_t kCacheBytes = (int64_t)256 << 20;

constexpr int kTok = 16;            // tokens per workgroup; lane t < kTok of the second wave reduces token t
// fp32 slabs have 64 channels above this many tokens, two workgroups per CU: there the arrays' rate is the time, and a workgroup is over sooner that is
// half a slab behind; below it the chain is, which meets half as many barriers in slabs of 128.  64 / 128 channels, us hot: 2025 x 3072 12.8 / 11.2, 4000 x
// 1536 8.8 / 8.9, 5000 x 2048 16.0 / 15.6, 9000 x 1024 12.8 / 13.3, 14000 x 512 10.2 / 10.9, 16300 x 1024 22.1 / 23.1.
constexpr int64_t kShortSlabTokens = 8192;
constexpr int kInFlight = 32 << 10;  // bytes of both arrays

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// 16-byte load; with NT the load carries the streaming hint (the line is not kept in L2)
template <bool NT, typename T> __device__ __forceinline__ uint4v load16(const T *p)
{
    if (NT) return __builtin_nontemporal_load(reinterpret_cast<const uint4v *>(p));
    return *reinterpret_cast<const uint4v *>(p);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int kPerVec = 4;        // elements of a 16-byte vector
    __device__ static float load(const float *p) { return *p; }
    __device__ static void diff(const uint4v &a, const uint4v &b, float *d)
    {
        d[0] = __uint_as_float(a.x) - __uint_as_float(b.x);
        d[1] = __uint_as_float(a.y) - __uint_as_float(b.y);
        d[2] = __uint_as_float(a.z) - __uint_as_float(b.z);
        d[3] = __uint_as_float(a.w) - __uint_as_float(b.w);
    }
};
template <> struct Elem<uint16_t> {
    static constexpr int kPerVec = 8;
    __device__ static float load(const uint16_t *p) { return __uint_as_float(((uint32_t)*p) << 16); }
    __device__ static void diff(const uint4v &a, const uint4v &b, float *d)
    {
        d[0] = bf16_lo(a.x) - bf16_lo(b.x);
        d[1] = bf16_hi(a.x) - bf16_hi(b.x);
        d[2] = bf16_lo(a.y) - bf16_lo(b.y);
        d[3] = bf16_hi(a.y) - bf16_hi(b.y);
        d[4] = bf16_lo(a.z) - bf16_lo(b.z);
        d[5] = bf16_hi(a.z) - bf16_hi(b.z);
        d[6] = bf16_lo(a.w) - bf16_lo(b.w);
        d[7] = bf16_hi(a.w) - bf16_hi(b.w);
    }
};

// Delta from the channel sum, then the weights and the penalty of the metric.
template <int MODE>
__device__ __forceinline__ float finish_score(float acc, int64_t C, int64_t tok, const float *__restrict__ lse_weight,
                                              const int32_t *__restrict__ skip_count,
                                              const float *__restrict__ penalty_table, int32_t table_len, float w_alpha,
                                              float w_beta)
{
    float delta = (MODE == ASTRAEA_DELTA_L2) ? sqrtf(acc) : acc / (float)C;
    float sig = lse_weight ? delta * lse_weight[tok] : delta;
    float sc = w_alpha * sig;
    if (skip_count) {
        int32_t n = skip_count[tok];
        n = n < 0 ? 0 : n;
        n = n > table_len - 1 ? table_len - 1 : n;
        sc = __builtin_fmaf(w_beta, penalty_table[n], sc);
    }
    return sc;
}

// Publishes the loading wave's LDS writes to the reducing wave and its reads to the loading one.  Outstanding global
// loads stay outstanding across it.
__device__ __forceinline__ void publish()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// SEG: channels handled per slab.
template <typename T, int MODE, bool VEC, bool NT, int SEG>
__global__ __launch_bounds__(2 * kWave) void score_kernel(
    const T *__restrict__ x_cur, const T *__restrict__ x_prev, int64_t N, int64_t C, int64_t row_stride,
    const float *__restrict__ lse_weight, const int32_t *__restrict__ skip_count,
    const float *__restrict__ penalty_table, int32_t table_len, float w_alpha, float w_beta,
    float *__restrict__ score_out)
{
    constexpr int EPV = Elem<T>::kPerVec;              // elements per 16-byte vector
    constexpr int kDepth = kInFlight / (2 * kTok * SEG * (int)sizeof(T));        // slabs in flight
    constexpr int kVecPerRow = SEG / EPV, kRowsPerLoad = kWave / kVecPerRow, kVecPerLane = kTok / kRowsPerLoad;
    constexpr int PLANES = EPV / 4;                    // a vector's floats are kept as 16-byte pieces, piece p in plane p
    constexpr int PLANE = 4 * kVecPerRow;              // floats
    constexpr int PITCH = SEG + 4;                     // floats; the 16 row reads of a piece hit distinct banks
    __shared__ __attribute__((aligned(16))) float tile[2][kTok * PITCH];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t tok0 = (int64_t)blockIdx.x * kTok;
    const int32_t nslab = (int32_t)((C + SEG - 1) / SEG);

    if (wave == 0) {
        // load slot j of this lane: row j*kRowsPerLoad + lane/kVecPerRow of the slab, 16-byte vector lane%kVecPerRow
        const int vrow = lane / kVecPerRow, vcol = lane % kVecPerRow;
        const char *bc = reinterpret_cast<const char *>(x_cur + tok0 * row_stride);
        const char *bp = reinterpret_cast<const char *>(x_prev + tok0 * row_stride);
        uint32_t row_off[kVecPerLane];
#pragma unroll
        for (int j = 0; j < kVecPerLane; ++j) {
            int64_t row = j * kRowsPerLoad + vrow;
            if (tok0 + row > N - 1) row = N - 1 - tok0;   // ragged last workgroup: re-read a valid row, result unused
            row_off[j] = (uint32_t)(row * row_stride * (int64_t)sizeof(T));
        }
        // Loads are unconditional, so that the wait for one slab never has to cover the next one's: past the last
        // whole vector of the row a lane reads that vector again, and its difference counts as +0.
        const int32_t c_lane = vcol * EPV, c_last = (int32_t)(C - C % EPV - EPV);
        uint4v ra[kDepth][kVecPerLane], rb[kDepth][kVecPerLane];
        auto issue = [&](int32_t s, auto buf_tag) __attribute__((always_inline)) {
            constexpr int B = decltype(buf_tag)::value;
            if (!VEC) return;
            const uint32_t c = (s * SEG + c_lane < c_last ? s * SEG + c_lane : c_last) * (uint32_t)sizeof(T);
#pragma unroll
            for (int j = 0; j < kVecPerLane; ++j) {
                ra[B][j] = load16<NT>(bc + (row_off[j] + c));
                rb[B][j] = load16<NT>(bp + (row_off[j] + c));
            }
            __builtin_amdgcn_sched_barrier(0);         // the waits count on this order
        };
        int wt = 0;                                    // the tile written next
        // differences of slab s -> LDS tile
        auto slab = [&](int32_t s, auto buf_tag) __attribute__((always_inline)) {
            constexpr int B = decltype(buf_tag)::value;
            const int32_t c0 = s * SEG;
            auto differences = [&](auto whole_tag) __attribute__((always_inline)) {
                const bool keep = decltype(whole_tag)::value || c0 + c_lane <= c_last;
#pragma unroll
                for (int j = 0; j < kVecPerLane; ++j) {
                    float d[EPV];
                    if (VEC) {
                        Elem<T>::diff(ra[B][j], rb[B][j], d);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) d[e] = keep ? d[e] : 0.0f;
                    } else {
#pragma unroll
                        for (int e = 0; e < EPV; ++e) {
                            const int32_t c = c0 + c_lane + e;
                            // channels past C contribute +0, which leaves the accumulator unchanged
                            d[e] = (c < C) ? Elem<T>::load(reinterpret_cast<const T *>(bc + row_off[j]) + c) -
                                             Elem<T>::load(reinterpret_cast<const T *>(bp + row_off[j]) + c)
                                       : 0.0f;
                        }
                    }
                    float *dst = tile[wt] + (j * kRowsPerLoad + vrow) * PITCH + vcol * 4;
#pragma unroll
                    for (int p = 0; p < PLANES; ++p)
                        *reinterpret_cast<float4 *>(dst + p * PLANE) = make_float4(d[4 * p], d[4 * p + 1], d[4 * p + 2], d[4 * p + 3]);
                }
            };
            if (c0 + SEG <= C)
                differences(std::true_type{});
            else
                differences(std::false_type{});
        };
        using B0 = std::integral_constant<int, 0>;
        using B1 = std::integral_constant<int, 1>;
        using B2 = std::integral_constant<int, 2>;
        using B3 = std::integral_constant<int, 3>;
        issue(0, B0{});
        issue(1, B1{});
        if constexpr (kDepth == 4) {
            issue(2, B2{});
            issue(3, B3{});
        }
        auto step = [&](int32_t s, auto buf_tag) __attribute__((always_inline)) {
            slab(s, buf_tag);
            issue(s + kDepth, buf_tag);
            publish();
            wt ^= 1;
        };
        int32_t s = 0;
        for (; s + kDepth <= nslab; s += kDepth) {
            step(s, B0{});
            step(s + 1, B1{});
            if constexpr (kDepth == 4) {
                step(s + 2, B2{});
                step(s + 3, B3{});
            }
        }
        auto last = [&](int32_t at, auto buf_tag) __attribute__((always_inline)) {
            if (at >= nslab) return;
            slab(at, buf_tag);
            publish();
            wt ^= 1;
        };
        last(s, B0{});
        if constexpr (kDepth == 4) {
            last(s + 1, B1{});
            last(s + 2, B2{});
        }
        publish();                       // the chains' last one
        return;
    }

    // The chains.  A dependent instruction per channel is their time, so little else may stand among them: pieces are read 64 channels ahead, in
    // the first half of the instructions of the 64 channels before their own, and waited for once.  Nine reads at the head of a slab waited
    // for there, and a wait for each later one, took 3.9 ns a channel; this takes 2.2: 2025 x 3072 bf16 hot / cold 14.7 / 17.9 -> 11.7 / 15.0 us,
    // 17550 x 3072 39.6 / 43.7 -> 37.0 / 41.5, 40000 x 3072 77.4 -> 75.5; fp32, slabs of 64 channels then, 900 x 3072 14.1 -> 10.8 hot, 3000 x 3072
    // 14.4 -> 12.2.  The barrier lies between the halves of a slab: all of it has been read there, so two tiles do, and the first half of a slab waits for
    // no other.  At the head of the slab, with a third tile: 16384 x 512 fp32 12.6 us for 11.5 and, of rows that are not aligned, whose workgroups
    // registers and LDS then held to six on a CU, 28000 x 511 bf16 56 for 35.  Two loading waves: 13.1 and 39.3 us at the first two sizes; four, with
    // six slabs in flight, 12.4 and 55.9.
    float acc = 0.0f;
    // Pieces that are read at a time: half of a slab's, or a quarter where the loads take few registers (68 in all; 132 with half slabs, three waves on a SIMD)
    constexpr int UNITS = VEC ? 2 : 4, UNIT = SEG / 4 / UNITS;
    float4 v[2][UNIT];
    const int t = lane % kTok;           // the other lanes do what the first kTok do
    auto read = [&](int tl, int unit, int buf, int e) __attribute__((always_inline)) {
        const int p = unit * UNIT + e;
        v[buf][e] = *reinterpret_cast<const float4 *>(tile[tl] + t * PITCH + (p % PLANES) * PLANE + (p / PLANES) * 4);
    };
    auto channel = [&](float x) __attribute__((always_inline)) {
        if (MODE == ASTRAEA_DELTA_MEAN_ABS)
            acc = acc + fabsf(x);
        else
            acc = __builtin_fmaf(x, x, acc);
    };
    auto unrolled_units = [&](auto f) __attribute__((always_inline)) {
        f(std::integral_constant<int, 0>{});
        f(std::integral_constant<int, 1>{});
        if constexpr (UNITS == 4) {
            f(std::integral_constant<int, 2>{});
            f(std::integral_constant<int, 3>{});
        }
    };
    // the chain through the unit in buffer B, and the reads of the next, unit `next` of tile tl, into the other buffer
    auto chain = [&](auto buf_tag, int tl, int next) __attribute__((always_inline)) {
        constexpr int B = decltype(buf_tag)::value;
#pragma unroll
        for (int e = 0; e < UNIT; ++e) {
            const float4 u = v[B][e];
            if (e < UNIT / 2) {
                read(tl, next, B ^ 1, 2 * e);
                read(tl, next, B ^ 1, 2 * e + 1);
            }
            channel(u.x);
            channel(u.y);
            channel(u.z);
            channel(u.w);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);            // lgkmcnt(0)
    };
    publish();                           // slab 0 is in its tile
#pragma unroll
    for (int e = 0; e < UNIT; ++e) read(0, 0, 0, e);
    __builtin_amdgcn_s_waitcnt(0xc07f);                // here and not, for the first slab's sake, in the loop
    int tl = 0;
    for (int32_t s = 0; s < nslab; ++s) {
        unrolled_units([&](auto unit_tag) __attribute__((always_inline)) {
            constexpr int u = decltype(unit_tag)::value;
            if (u == UNITS - 1) {
                // All of this slab has been read, so its tile is free, and slab s + 1 is in the other, if there is one: past the last what lies there is
                // read and not used.
                publish();
                tl ^= 1;
            }
            chain(std::integral_constant<int, u % 2>{}, tl, (u + 1) % UNITS);
        });
    }
    if (lane >= kTok) return;
    if (VEC) {
        // a width that is no multiple of a vector: its last channels, from memory
        const int64_t row = (tok0 + lane < N ? tok0 + lane : N - 1) * row_stride;
        for (int64_t c = C - C % EPV; c < C; ++c) {
            const float d = Elem<T>::load(x_cur + row + c) - Elem<T>::load(x_prev + row + c);
            acc = MODE == ASTRAEA_DELTA_MEAN_ABS ? acc + fabsf(d) : __builtin_fmaf(d, d, acc);
        }
    }
    const int64_t tok = tok0 + lane;
    if (tok >= N) return;
    score_out[tok] = finish_score<MODE>(acc, C, tok, lse_weight, skip_count, penalty_table, table_len, w_alpha, w_beta);
}

// Orders this wave's LDS traffic without a workgroup barrier.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T, int MODE, bool VEC, bool NT>
__global__ __launch_bounds__(kWideWavesPerBlock *kWave) void score_wide_kernel(
    const T *__restrict__ x_cur, const T *__restrict__ x_prev, int64_t N, int64_t C, int64_t row_stride,
    const float *__restrict__ lse_weight, const int32_t *__restrict__ skip_count,
    const float *__restrict__ penalty_table, int32_t table_len, float w_alpha, float w_beta,
    float *__restrict__ score_out)
{
    constexpr int EPV = Elem<T>::kPerVec;              // elements per 16-byte vector
    constexpr int SEG = kWideSegBytes / (int)sizeof(T);    // channels per slab
    constexpr int PITCH = SEG + 4;                     // floats; keeps b128 row reads conflict-free
    __shared__ float tile_all[kWideWavesPerBlock][kWideTok * PITCH];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    float *tile = tile_all[wave];
    const int64_t tok0 = ((int64_t)blockIdx.x * kWideWavesPerBlock + wave) * kWideTok;
    if (tok0 >= N) return;

    // load slot j of this lane: row j*8 + lane/8 of the slab, 16-byte vector lane%8 of the segment
    const int vrow = lane >> 3, vcol = lane & 7;
    const T *pc[kWideVecPerLane];
    const T *pp[kWideVecPerLane];
#pragma unroll
    for (int j = 0; j < kWideVecPerLane; ++j) {
        int64_t tok = tok0 + j * 8 + vrow;
        if (tok > N - 1) tok = N - 1;                  // ragged last wave: re-read a valid row, result unused
        pc[j] = x_cur + tok * row_stride + vcol * EPV;
        pp[j] = x_prev + tok * row_stride + vcol * EPV;
    }

    uint4v ra[kWideVecPerLane], rb[kWideVecPerLane];
    auto issue = [&](int64_t c0) {
#pragma unroll
        for (int j = 0; j < kWideVecPerLane; ++j) {
            if (VEC && c0 + SEG <= C) {
                ra[j] = load16<NT>(pc[j] + c0);
                rb[j] = load16<NT>(pp[j] + c0);
            }
        }
    };

    float acc = 0.0f;
    const int64_t nslab = (C + SEG - 1) / SEG;
    issue(0);
    for (int64_t s = 0; s < nslab; ++s) {
        const int64_t c0 = s * SEG;
        const bool fast = VEC && (c0 + SEG <= C);
        // 1. differences of this slab -> LDS tile
#pragma unroll
        for (int j = 0; j < kWideVecPerLane; ++j) {
            float d[EPV];
            if (fast) {
                Elem<T>::diff(ra[j], rb[j], d);
            } else {
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    int64_t c = c0 + vcol * EPV + e;
                    // channels past C contribute +0, which leaves the accumulator unchanged
                    d[e] = (c < C) ? Elem<T>::load(pc[j] + c0 + e) - Elem<T>::load(pp[j] + c0 + e) : 0.0f;
                }
            }
            float *dst = tile + (j * 8 + vrow) * PITCH + vcol * EPV;
#pragma unroll
            for (int e = 0; e < EPV; e += 4)
                *reinterpret_cast<float4 *>(dst + e) = make_float4(d[e], d[e + 1], d[e + 2], d[e + 3]);
        }
        // 2. next slab's loads go out before the reduce phase
        if (s + 1 < nslab) issue(c0 + SEG);
        wave_lds_sync();
        // 3. lane t reduces row t, channels ascending
        const float *row = tile + lane * PITCH;
#pragma unroll
        for (int e = 0; e < SEG; e += 4) {
            float4 v = *reinterpret_cast<const float4 *>(row + e);
            if (MODE == ASTRAEA_DELTA_MEAN_ABS) {
                acc = acc + fabsf(v.x);
                acc = acc + fabsf(v.y);
                acc = acc + fabsf(v.z);
                acc = acc + fabsf(v.w);
            } else {
                acc = __builtin_fmaf(v.x, v.x, acc);
                acc = __builtin_fmaf(v.y, v.y, acc);
                acc = __builtin_fmaf(v.z, v.z, acc);
                acc = __builtin_fmaf(v.w, v.w, acc);
            }
        }
        wave_lds_sync();
    }

    const int64_t tok = tok0 + lane;
    if (tok >= N) return;
    score_out[tok] = finish_score<MODE>(acc, C, tok, lse_weight, skip_count, penalty_table, table_len, w_alpha, w_beta);
}

template <typename T, bool VEC, bool NT>
void launch_mode(astraea_delta_mode mode, bool wide, hipStream_t st, const T *xc, const T *xp, int64_t N, int64_t C,
                 int64_t rs, const float *lw, const int32_t *sc, const float *pt, int32_t tl, float wa, float wb, float *out)
{
    const int64_t per_block = wide ? kWideWavesPerBlock * kWideTok : kTok;
    const dim3 grid((unsigned)((N + per_block - 1) / per_block)), block(wide ? kWideWavesPerBlock * kWave : 2 * kWave);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, xc, xp, N, C, rs, lw, sc, pt, tl, wa, wb, out); };
    auto pick = [&](auto mode_tag) {
        constexpr int MODE = decltype(mode_tag)::value;
        if (wide)
            go(score_wide_kernel<T, MODE, VEC, NT>);
        else if (std::is_same<T, float>::value && VEC && N > kShortSlabTokens)
            go(score_kernel<T, MODE, VEC, NT, 64>);
        else
            go(score_kernel<T, MODE, VEC, NT, 128>);
    };
    switch (mode) {
    case ASTRAEA_DELTA_L2: pick(std::integral_constant<int, ASTRAEA_DELTA_L2>{}); break;
    case ASTRAEA_DELTA_MEAN_ABS: pick(std::integral_constant<int, ASTRAEA_DELTA_MEAN_ABS>{}); break;
    default: pick(std::integral_constant<int, ASTRAEA_DELTA_MEAN_SQ>{}); break;
    }
}

}  // namespace

int launch_score(const void *x_cur, const void *x_prev, astraea_dtype dt, int64_t N, int64_t C, int64_t row_stride,
                 astraea_delta_mode mode, const float *lse_weight, const int32_t *skip_count,
                 const float *penalty_table, int32_t table_len, float w_alpha, float w_beta, float *score_out,
                 hipStream_t stream)
{
    if (N == 0) return ASTRAEA_OK;
    const int64_t es = dt == ASTRAEA_F32 ? 4 : 2;
    // Which kernel.  Past the 256 MB of the memory-side cache the line is three wide waves per CU (bf16 x 3072, us wide / 16 tokens: 36000 83.7 /
    // 71.1, 49000 94.2 / 91.1, 52000 97.5 / 100.2).  Arrays below that are either hot, still in the cache from their producer, or cold.  Cold, 16 tokens
    // win up to about the same line; hot, they lose it earlier, since the wide kernel then has less latency to cover: bf16 28000 x 512 13.0 / 12.0,
    // 36000 x 512 13.5 / 14.2, 28600 x 2048 43.3 / 44.3, 32000 x 2048 43.5 / 49.4, 32000 x 1536 33.7 / 31.4; fp32 20000 x 512
    // 14.6 / 13.4, 28000 x 512 17.6 / 18.2, 20400 x 1024 26.6 / 27.3, 24000 x 1024 28.8 / 30.2.  The lines
    // lie where neither loses hot at the width that loses first.  (A 16-token workgroup also addresses its rows with 32-bit byte offsets.)
    const int64_t bytes = 2 * N * row_stride * es;
    const int64_t line = bytes > kCacheBytes ? kWideMinTokens : dt == ASTRAEA_F32 ? kWideMinCachedF32 : kWideMinCachedBf16;
    const bool wide = N >= line || kTok * row_stride * es > 2147483647LL;
    const bool vec = C * es >= 16 && ((uintptr_t)x_cur % 16 == 0) && ((uintptr_t)x_prev % 16 == 0) && ((row_stride * es) % 16 == 0);
    // The streaming hint (the line is not kept in L2) is for arrays that are not still cached from their producer:
    // above the 256 MB of the memory-side cache, 5.96 -> 6.77 TB/s at 118800 x 3072 (wide).  Up to 24576 tokens the
    // 16-token kernel takes it from 200 MB on, where it costs little even hot: 17550 x 3072 (206 MB) cold 45.5 -> 41.6 us (as the chains were before they
    // read ahead) and hot 37.1 -> 37.8; not so below, hot 25.2 -> 29.7 at 17550 x 1024 fp32 (137 MB), nor past
    // that many tokens, hot 43.4 -> 46.5 at 28000 x 2048 bf16 (219 MB).
    const bool stream_loads = vec && bytes > (!wide && N <= 24576 ? (int64_t)200 << 20 : kCacheBytes);
#define ASTRAEA_SCORE_LAUNCH(T, VEC, NT)                                                                                  \
    launch_mode<T, VEC, NT>(mode, wide, stream, (const T *)x_cur, (const T *)x_prev, N, C, row_stride, lse_weight,        \
                            skip_count, penalty_table, table_len, w_alpha, w_beta, score_out)
    if (dt == ASTRAEA_F32) {
        if (stream_loads)
            ASTRAEA_SCORE_LAUNCH(float, true, true);
        else if (vec)
            ASTRAEA_SCORE_LAUNCH(float, true, false);
        else
            ASTRAEA_SCORE_LAUNCH(float, false, false);
    } else {
        if (stream_loads)
            ASTRAEA_SCORE_LAUNCH(uint16_t, true, true);
        else if (vec)
            ASTRAEA_SCORE_LAUNCH(uint16_t, true, false);
        else
            ASTRAEA_SCORE_LAUNCH(uint16_t, false, false);
    }
#undef ASTRAEA_SCORE_LAUNCH
    return check_launch("astraea_score");
}

}  // namespace astraea
