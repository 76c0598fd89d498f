// astraea_sparse_attn_fwd, bf16 mode, head_dim 128 (paper, Algorithm 1 step 6:
// X_out[I_sel] = Softmax(Q_sel K^T / sqrt(d)) V with every key and value kept, Sec. 3.2
// "Sparse Attention").  Flash-style: K/V are streamed once per query tile, the N x N map is never
// materialised, softmax is the online form in fp32.
//
// Shape of the computation on gfx950:
//  * both products are computed transposed, S^T = K Q^T and O^T = V^T P^T, with
//    v_mfma_f32_32x32x16_bf16.  In every accumulator a lane then owns one query column, so the row
//    max / row sum / rescale factor are per-lane scalars (one exchange between lanes l and l+32),
//    and the S^T accumulator registers, converted to bf16, are the B operand of the second
//    product as they stand: register group 8*(t%2)..+7 of key block t/2 feeds MFMA t, with the key
//    order inside the contraction permuted the same way on the V side.
//  * K/V tiles go from global memory straight into LDS (global_load_lds_dwordx4), double
//    buffered, with no register staging.  Such a load writes 64 x 16 B contiguously, so rows
//    cannot be padded; bank conflicts are avoided by an XOR swizzle of the 16-byte chunks inside
//    each 256-byte row, applied through the per-lane global address.
//  * the LDS pipe issues one wave instruction every ~4.5 clocks whatever its width, so fragments
//    must come in 16-byte reads.  K rows are head-dim contiguous, which is what S^T = K Q^T wants.
//    V is contracted over keys.  For large selections a pre-pass rewrites V once per call into 16 KiB tiles of V^T
//    ([128 head-dim rows][64 keys], keys permuted inside each group of 16 to match the register
//    order of P^T, 16-byte chunks already XOR-swizzled); the main kernel then copies a tile
//    linearly into LDS and reads every V^T fragment with one ds_read_b128.  The pre-pass moves
//    2*N*H*D*2 bytes and needs N_pad*H*D*2 bytes of workspace.  For smaller ones, where that pass is 2 to 20 % of the
//    call, V rows are copied as they lie and a fragment is two transposing reads (ds_read_b64_tr_b16).
//  * queries are gathered by index on their way through LDS into the Q fragment, which then lives in registers
//    for the whole sweep (the "gather" step of the path is fused here).
//  * the exponent offset of a row need not be its exact max: a stale one costs range, not accuracy
//    (P, the row sums and the O accumulators are floating point with 8-bit exponents).  The main
//    kernel therefore fixes each row's offset at the max over the first key tile and takes no max in
//    the sweep at all, which removes a fifth of the softmax arithmetic.  A row whose later logits
//    outgrow that offset by more than 2^80 (or overflow) shows in its final row sum, one whose rise
//    is smaller but meets values large enough to overflow the output shows in its accumulators; the workgroup
//    then sweeps its keys once more in the exact form (a max per tile, lazy rescale when it grew by
//    more than 2^kTau).  So a workgroup with such a row, or with a NaN or an infinity among its operands, takes up
//    to twice the time.  Both forms are in the one kernel: as a launch of its own over the same grid the
//    exact form cost 4 - 7 us a call with nothing to redo, and needed a flag per workgroup.
//  * workgroup ids are mapped so that the workgroups resident on one XCD work on the same head and
//    sweep the keys together; K/V tiles are then served from that XCD's L2.
//  * the two waves that share a SIMD alternate: while one runs the MFMAs of a tile the other runs
//    the exponentials of its own tile, so the matrix pipe and the VALU work at the same time.
//  * few or short work items run in workgroups of four waves instead of eight: halves of an item each on a CU of its own, or two
//    on one CU, one of which stores or loads while the other sweeps.  Fewer still run in workgroups of eight waves that share 128 or 64
//    queries and split the keys between them.
#include <type_traits>

#include "gfx950.h"

namespace astraea {
namespace {


constexpr int D = 128;
constexpr int kGroupWaves = 4;          // one wave per SIMD
constexpr int kBq = 256;                // queries per work item
constexpr int kBk = 64;                 // keys per LDS tile
constexpr int kRowBytes = D * 2;        // 256 B per key row, unpadded
constexpr int kTileBytes = kBk * kRowBytes;          // 16 KiB
constexpr int kRowsBytes = 32 * kRowBytes;           // a wave's 32 query or output rows
constexpr float kTau = 8.0f;            // exact form: lazy-rescale threshold, log2 units
constexpr float kRose = 0x1p8f;         // 2^kTau
// Exact form: the offset before the first tile.  From minus infinity, a tile of such logits alone would make NaN of their weights (as it does in the
// fast form, which the row sums then show); from here they weigh nothing and the first finite logit raises the offset.
constexpr float kLowest = -3.40282347e38f;
constexpr float kBig = 0x1p80f;         // fast form: after a final row sum above this the workgroup repeats its sweep in the exact form
constexpr int kNumXcd = 8;
constexpr int kCuPerXcd = 32;
// The pre-pass costs a read and a write of V whatever the selection, direct V tiles half as many LDS reads again per key and
// query.  Retiled against direct, same results, us: 608 queries x 2025 keys 38.5 / 32.2; 7020 x 512 64.5 / 60.0; 1755 x 17550
// 376 / 344; 7020 x 17550 1323 / 1301; 17550 x 17550 3159 / 3151; 11880 x 118800 14315 / 14225; 35640 x 118800 41688 / 41906.
// Both costs grow with the number of keys, so the line is a number of queries.
constexpr int64_t kRetileRows = 16384;

__device__ __forceinline__ float xhalf_max(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}



// ---- pre-pass: V [N, H, 128] -> tiles of V^T.  Tile (head, T) is 16 KiB at
// vt + (head * ntiles + T) * 16 KiB and holds keys 64*T .. 64*T+63: row d (128 bytes) = 8 chunks;
// logical chunk c = 2*t + hf holds keys 64*T + 16*t + 8*(j/4) + 4*hf + j%4 for j = 0..7, and is
// stored at physical chunk c ^ ((d >> 1) & 7).  Keys past N are zero.
__global__ __launch_bounds__(256) void transpose_v_kernel(const __bf16 *__restrict__ v, int64_t N, int64_t kv_stride_n,
                                                          int64_t kv_stride_h, int64_t ntiles,
                                                          char *__restrict__ vt)
{
    __shared__ uint16_t tile[kBk][D + 2];      // [key][d], odd dword pitch: column reads conflict-free
    const int64_t T = blockIdx.x;
    const int head = blockIdx.y;
    const uint16_t *vb = reinterpret_cast<const uint16_t *>(v) + (int64_t)head * kv_stride_h;
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (tid >> 4) + 16 * i, c16 = tid & 15;
        const int64_t key = T * kBk + row;
        uint4v val = {0u, 0u, 0u, 0u};
        // V is read once here: streaming hint, the lines are not kept in L2
        if (key < N) val = __builtin_nontemporal_load(reinterpret_cast<const uint4v *>(vb + key * kv_stride_n + c16 * 8));
        uint32_t *dst = reinterpret_cast<uint32_t *>(&tile[row][c16 * 8]);
        dst[0] = val[0];
        dst[1] = val[1];
        dst[2] = val[2];
        dst[3] = val[3];
    }
    __syncthreads();
    char *out = vt + ((int64_t)head * ntiles + T) * kTileBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int o = tid + 256 * i;           // output chunk id: row d = o / 8, logical chunk c = o % 8
        const int d = o >> 3, c = o & 7, t = c >> 1, hf = c & 1;
        uint32_t w[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int j0 = 2 * jj, j1 = 2 * jj + 1;
            const int k0 = 16 * t + 8 * (j0 >> 2) + 4 * hf + (j0 & 3);
            const int k1 = 16 * t + 8 * (j1 >> 2) + 4 * hf + (j1 & 3);
            w[jj] = (uint32_t)tile[k0][d] | ((uint32_t)tile[k1][d] << 16);
        }
        uint4v val = {w[0], w[1], w[2], w[3]};
        *reinterpret_cast<uint4v *>(out + d * 128 + ((c ^ ((d >> 1) & 7)) << 4)) = val;
    }
}

// 32 output rows of 256 bytes in LDS, 16-byte chunks XOR-swizzled, on their way from accumulators to whole rows:
// registers 4g..4g+3 of block b of a lane are head-dim 32*b + 8*g + 4*(lane/32) + 0..3 of row lane%32.
__device__ __forceinline__ void rows_put(uint32_t rows_lds, int b, int g, int lane, uint2v v)
{
    const int row = lane & 31;
    *reinterpret_cast<uint2v __attribute__((address_space(3))) *>(
        (uintptr_t)(rows_lds + row * kRowBytes + (((4 * b + g) ^ (row & 15)) << 4) + 8 * (lane >> 5))) = v;
}
__device__ __forceinline__ uint4v rows_get(uint32_t rows_lds, int row, int chunk)
{
    return __builtin_bit_cast(uint4v, lds_read_b128(rows_lds + row * kRowBytes + ((chunk ^ (row & 15)) << 4)));
}

// 16 bytes of result row r, which belongs to `token`: to wherever the caller asked for.
__device__ __forceinline__ void store_row(const AttnOut &out, int32_t H, int head, int64_t r, int64_t token, int chunk, uint4v val, bool valid)
{
    const int64_t at = (int64_t)head * D + 8 * chunk;
    if (out.rows && valid) *reinterpret_cast<uint4v *>(reinterpret_cast<__bf16 *>(out.rows) + r * H * D + at) = val;
    if (out.cache && valid && (uint64_t)token < (uint64_t)out.cache_rows)
        *reinterpret_cast<uint4v *>(reinterpret_cast<__bf16 *>(out.cache) + token * out.cache_stride + at) = val;
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
// The transposing LDS read: of each 16 lanes, lane 4 r + c supplies elements 4 c .. 4 c + 3 of row r, and lane i gets element i of
// the four rows.
__device__ __forceinline__ bf16x4 lds_read_tr(uint32_t addr)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                          reinterpret_cast<s16x4 __attribute__((address_space(3))) *>((uintptr_t)addr)));
}

// Budget-aware work split.  Work item = (head, tile of 256 selected queries), head-major; XCD x owns the
// contiguous item range [x * items_per_xcd, (x+1) * items_per_xcd) and workgroups reach XCDs round-robin
// by id.  With 32 CUs per XCD the items of an XCD run in rounds of 32.  The first `full_items` of each
// XCD sweep all keys; the remaining items_per_xcd - full_items (< 32, what would be a mostly idle last
// round) are each cut into `splits` key ranges of `tiles_per_split` tiles, run by as many workgroups,
// whose unnormalised partial results are combined by merge_partials_kernel.  Execution time then
// follows the number of selected tokens instead of the number of rounds.
// All of it fits 32 bits (plan_attn refuses grids past 2^31), which spares a workgroup its 64-bit divisions.
struct AttnSchedule {
    uint32_t items_per_xcd;
    uint32_t full_items;
    uint32_t tiles_per_split;
    uint32_t q_tiles;
    uint32_t splits;
};
constexpr int kPartialFloats = kBq * D + 2 * kBq;    // O^T accumulators, then running max, then row sum
constexpr int kMaxSharesPerXcd = 64;

constexpr int MFMA = 0x008, DSR = 0x100;
#define SGB(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)
// Nothing may be moved across a phase boundary: left alone, the scheduler pulls the exponentials next to
// the MFMAs that consume them, i.e. into the other phase.
#define PHASE_BARRIER()                    \
    do {                                   \
        __builtin_amdgcn_sched_barrier(0); \
        __builtin_amdgcn_s_barrier();      \
        __builtin_amdgcn_sched_barrier(0); \
    } while (0)

// RETILED: V comes from the pre-pass's V^T tiles.  Otherwise its rows are copied as they lie, in the K tile's shape, and the
// fragments are read through the transposing LDS read.
// GROUPS: groups of four waves in a workgroup (half_workgroups).  2: an item's 256 queries, the groups taking turns at the matrix pipe.  1: half
// an item's queries; two such workgroups share a CU.
// KEYS: key groups of an eight-wave workgroup (key_groups).  1: its waves have 32 queries each and sweep the same keys.  2 or 4: there are 128
// or 64 queries, and each group of waves that has them all takes a share of the keys in tiles of its own; the groups' results are merged through LDS.
template <bool RETILED, int GROUPS, int KEYS>
__global__ __launch_bounds__(GROUPS *kGroupWaves *kWave, 2 / GROUPS) void attn_bf16_kernel(
    const __bf16 *__restrict__ q, const __bf16 *__restrict__ k, const void *__restrict__ v, int64_t N, int32_t H,
    int64_t q_stride_n, int64_t q_stride_h, int64_t kv_stride_n, int64_t kv_stride_h,
    const int32_t *__restrict__ idx_sel, int64_t k_sel, int q_is_compact, float scale_log2e,
    AttnOut out, float *__restrict__ lse_sel, AttnSchedule sch, float *__restrict__ partial)
{
    static_assert(KEYS == 1 || (GROUPS == 2 && !RETILED), "key groups are for eight waves and V as it lies");
    constexpr int kWaves = GROUPS * kGroupWaves;
    constexpr int kKeyWaves = kWaves / KEYS;         // waves of a key group
    constexpr int KB = KEYS == 4 ? 1 : 2;            // blocks of 32 keys in a tile: four groups' tiles fit LDS twice at 32 keys
    constexpr int kTk = 32 * KB, kTile = kTk * kRowBytes, kBuf = 2 * kTile;
    constexpr int kMfmas = 8 * KB;                   // of either product, per tile
    // [parity][K tile | V^T tile], 64 KiB, and 8 KiB per wave for its query rows and later its output rows: behind the tiles for one
    // 8-wave workgroup per CU; from the second V tile's place on for two 4-wave ones, whose 160 KiB are the CU's whole LDS.  There the rows of
    // waves 0 and 1 lie over the whole second V buffer: query rows are read before the barrier in front of the first tile, output
    // rows are written past a barrier behind the last one (the vote's, or its own after a repeated sweep)
    constexpr uint32_t kRowsAt = GROUPS == 2 ? KEYS * 2 * kBuf : kBuf + kTile;
    constexpr uint32_t kRowsEnd = kRowsAt + kKeyWaves * kRowsBytes;      // key groups have the same query rows
    __shared__ __attribute__((aligned(1024))) char lds[kRowsEnd + (GROUPS == 2 && KEYS == 1 ? 64 : 0)];
    // one word per wave; the first K tile's place, or that of key groups' query rows, is free when they are used
    uint32_t *const wave_outgrew = reinterpret_cast<uint32_t *>(lds + (KEYS > 1 ? kRowsAt : GROUPS == 2 ? sizeof(lds) - 64 : 0));

    const int64_t ntiles = (N + kTk - 1) / kTk;
    const uint32_t total_items = (uint32_t)H * sch.q_tiles;
    const uint32_t xcd = blockIdx.x % kNumXcd, slot = blockIdx.x / (kNumXcd * (2 / GROUPS));
    uint32_t item = xcd * sch.items_per_xcd + slot;
    int tile_begin = 0, tile_end = (int)ntiles;      // at most 2^25 tiles
    int64_t pslot = -1;
    if (slot >= sch.full_items) {
        const uint32_t p = slot - sch.full_items, li = p / sch.splits, sp = p - li * sch.splits;
        item = xcd * sch.items_per_xcd + sch.full_items + li;
        tile_begin = (int)(sp * sch.tiles_per_split);
        tile_end = tile_begin + (int64_t)sch.tiles_per_split < ntiles ? tile_begin + (int)sch.tiles_per_split : (int)ntiles;
        pslot = (int64_t)(xcd * (sch.items_per_xcd - sch.full_items) + li) * sch.splits + sp;
    }
    if (item >= (xcd + 1) * sch.items_per_xcd || item >= total_items) return;
    const int head = (int)(item / sch.q_tiles);
    const int64_t qt = item - (uint32_t)head * sch.q_tiles;

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int qc = lane & 31, hf = lane >> 5;
    // the wave's place among the item's eight: a 4-wave workgroup takes one half of them
    const int iwave = KEYS > 1 ? wave % kKeyWaves : GROUPS == 2 ? wave : wave + (blockIdx.x / kNumXcd & 1) * kGroupWaves;
    const int64_t r0 = qt * (kBq / KEYS) + iwave * 32;
    if (GROUPS == 1 && r0 - wave * 32 >= k_sel) return;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    // The key group, its share of the tiles and where it keeps them.  Shares differ by a tile at most; there are at least KEYS tiles.
    const int kg = KEYS > 1 ? wave / kKeyWaves : 0;
    if (KEYS > 1) {
        tile_begin = (int)(kg * ntiles / KEYS);
        tile_end = (int)((kg + 1) * ntiles / KEYS);
    }
    const uint32_t tiles0 = lds0 + kg * 2 * kBuf;
    // part of the fragments' addresses where it differs among the waves
    const uint32_t at0 = KEYS > 1 ? tiles0 : 0, from0 = KEYS > 1 ? 0 : lds0;

    floatx16 oacc[4];
    float m_c;                 // running max of scale*log2(e)*logit actually used as exponent offset
    float l_run;               // this lane's share of the running sum

    // ---- tile DMA.  A wave instruction fills 1 KiB of a tile: lane l writes 16 bytes at 16*l.
    // K: block = 4 key rows; physical chunk p of row r holds logical chunk p ^ (r & 15).
    // V^T: the pre-pass already wrote the tile as its LDS image, so the copy is linear.
    const char *kbase = reinterpret_cast<const char *>(k + (int64_t)head * kv_stride_h);
    const char *vbase = RETILED ? reinterpret_cast<const char *>(v) + (int64_t)head * ntiles * kTile
                                : reinterpret_cast<const char *>(reinterpret_cast<const __bf16 *>(v) + (int64_t)head * kv_stride_h);
    const int64_t row_pitch = kv_stride_n * 2;       // bytes between consecutive keys
    const int d_row = lane >> 4, d_p = lane & 15;
    const uint32_t lin_off = lane * 16;
    // Rows [key0, key0 + kTk) of K or V; physical chunk p of row r holds logical chunk p ^ sw(r).
    auto dma_rows = [&](const char *base, int64_t tile, uint32_t buf, int w, auto nw_tag, int swz, bool zero_fill) __attribute__((always_inline)) {
        // a wave's rows advance by 4 NW: with 4 or 8 waves the swizzle is the same for all of them, with 2 it alternates for K
        constexpr int NW = decltype(nw_tag)::value;
        const int64_t key0 = tile * kTk;
        const char *src = base + key0 * row_pitch;
        const uint32_t dst = buf + w * 1024;
        const int row0 = 4 * w + d_row;
        const uint32_t sw = (uint32_t)((d_p ^ swz) << 4);
        const uint32_t sw_odd = NW == 2 && !zero_fill ? sw ^ 128 : sw;
        if (key0 + kTk <= N) {
            const uint32_t off = (uint32_t)row0 * (uint32_t)row_pitch;
#pragma unroll
            for (int i = 0; i < kTk / 4 / NW; ++i) dma16(src + i * 4 * NW * row_pitch, off + (i & 1 ? sw_odd : sw), dst + i * NW * 1024);
        } else {
            const int64_t last = N - 1 - key0;       // K rows past the last key re-read it (masked later); V rows are zero
#pragma unroll
            for (int i = 0; i < kTk / 4 / NW; ++i) {
                const int rr = row0 + 4 * NW * i;
                const int64_t rc = rr < last ? rr : last;
                if (!zero_fill || rr <= last)
                    dma16(src, (uint32_t)(rc * row_pitch) + (i & 1 ? sw_odd : sw), dst + i * NW * 1024);
                else
                    *reinterpret_cast<uint4v __attribute__((address_space(3))) *>((uintptr_t)(dst + i * NW * 1024 + lane * 16)) = uint4v{0u, 0u, 0u, 0u};
            }
            if (zero_fill) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    };
    // Copies one tile with NW waves taking part (this wave is number w of them): block b of the
    // tile is copied by wave b % NW.
    auto dma_v_tile = [&](int64_t tile, int par, int w, auto nw_tag) __attribute__((always_inline)) {
        constexpr int NW = decltype(nw_tag)::value;
        const uint32_t buf = tiles0 + par * kBuf + kTile;
        if (RETILED) {
            const char *src = vbase + tile * kTile + w * 1024;
#pragma unroll
            for (int i = 0; i < 16 / NW; ++i) dma16(src + i * NW * 1024, lin_off, buf + w * 1024 + i * NW * 1024);
        } else {
            dma_rows(vbase, tile, buf, w, nw_tag, d_row << 2, true);
        }
    };
    auto dma_k_tile = [&](int64_t tile, int par, int w, auto nw_tag) __attribute__((always_inline)) {
        dma_rows(kbase, tile, tiles0 + par * kBuf, w, nw_tag, (4 * w + d_row) & 15, false);
    };

    // the waves that copy a tile in the sweep, those of one phase group or of a key group, and this wave's number among them; the first
    // tiles are copied by all waves that read them
    const int grp = wave >> 2, wig = KEYS > 1 ? iwave : wave & 3, wkg = KEYS > 1 ? iwave : wave;
    using WGrp = std::integral_constant<int, (KEYS > 1 ? kKeyWaves : kGroupWaves)>;
    using WAll = std::integral_constant<int, kKeyWaves>;
    auto first_tiles = [&]() __attribute__((always_inline)) {
        dma_k_tile(tile_begin, 0, wkg, WAll{});
        dma_v_tile(tile_begin, 0, wkg, WAll{});
        if (tile_begin + 1 < tile_end) dma_k_tile(tile_begin + 1, 1, wkg, WAll{});
    };
    first_tiles();

    // ---- Q fragment: lane holds query column qc, head-dim 16*s + 8*hf + 0..7 (B operand of K Q^T).  The rows come
    // through LDS in the K tile's layout, four whole rows per copy: fragments loaded straight from global memory take
    // 16 bytes of each of 32 rows per instruction, and a short sweep waits for them.
    const int64_t row_n = k_sel - r0 < 32 ? k_sel - r0 : 32;     // rows of this wave; at most 0: none
    auto lane_row = [&](int n) { return (int64_t)n < row_n ? r0 + n : k_sel - 1; };    // ragged tile: a valid row, never stored
    // an index outside [0, N) reads a valid row instead
    const int32_t q_row = q_is_compact ? 0 : clamp_row(idx_sel[lane_row(qc)], (int32_t)N);
    const uint32_t rows_lds = lds0 + kRowsAt + wkg * kRowsBytes;
#pragma unroll
    for (int ii = 0; ii < 8 / KEYS; ++ii) {          // key groups share the copying
        const int i = ii * KEYS + kg, n = 4 * i + d_row;
        const int64_t row = q_is_compact ? lane_row(n) : (int64_t)__shfl(q_row, n);
        dma16_far(q + row * q_stride_n + (int64_t)head * q_stride_h + 8 * (d_p ^ (n & 15)), rows_lds + i * 1024);
    }
    wait_dma();
    if (KEYS > 1) __syncthreads();
    bf16x8 qf[D / 16];
#pragma unroll
    for (int s = 0; s < D / 16; ++s) qf[s] = lds_read_b128(rows_lds + qc * kRowBytes + (((2 * s + hf) ^ (qc & 15)) << 4));
    if (GROUPS == 1) __builtin_amdgcn_s_waitcnt(0xc07f);         // lgkmcnt(0): past the next barrier a V tile may lie there

    // ---- LDS read offsets relative to a buffer pair; the buffer parity and the array's base are added where
    // the offsets are used (the tile loop is unrolled by two, so the parity is a compile-time constant there
    // and lands in the read's immediate offset)
    // K fragment (kb, s): row 32*kb + qc, logical chunk 2*s + hf; kb is an immediate offset
    uint32_t ka[D / 16];
#pragma unroll
    for (int s = 0; s < D / 16; ++s) ka[s] = at0 + qc * kRowBytes + (((2 * s + hf) ^ (qc & 15)) << 4);
    // V^T fragment (tt, b): row d = 32*b + qc (128-byte rows), logical chunk 2*tt + hf; b is an immediate
    // Not retiled: lane 16 g + i of a transposing read supplies 4 head-dims of key 4 (g / 2) + i / 4 and gets head-dim
    // 16 (g % 2) + i of four keys; V fragment (tt, b) is two of them, keys 16 tt + 4 hf + 0..3 and 8 further.  va[b] is
    // their place: chunk 4 b + 2 (g % 2) + (i % 4) / 2 of that row, swizzled by 4 (row % 4).
    uint32_t va[4];
    const int tr_row = qc & 15;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        va[u] = RETILED ? kTile + qc * 128 + (((2 * u + hf) ^ ((qc >> 1) & 7)) << 4)
                        : at0 + kTile + (4 * hf + (tr_row >> 2)) * kRowBytes +
                              ((((u ^ (tr_row >> 2)) << 2) + 2 * (qc >> 4) + ((tr_row >> 1) & 1)) << 4) + 8 * (tr_row & 1);
    auto read_v = [&](int u, uint32_t at) __attribute__((always_inline)) -> bf16x8 {     // fragment tt = u / 4, b = u % 4 of the buffer pair at `at`
        if (RETILED) return lds_read_b128(from0 + va[u >> 2] + (at + (u & 3) * 32 * 128));
        const uint32_t p = from0 + va[u & 3] + (at + (u >> 2) * 16 * kRowBytes);
        const bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 8 * kRowBytes);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    floatx16 sacc[KB];         // S^T of the current tile (blocks of 32 keys)
    uint32_t pw[8 * KB];       // P^T as bf16 pairs: pw[8*kb + i] = registers 2i, 2i+1 of block kb

    // VALU phase for tile j: exponentials -> pw, row sums; in the exact form first the row max: the running
    // max is only raised (and what was accumulated under the old one rescaled) when some row's max moved up by
    // more than 2^kTau, otherwise the stale max stays in use.
    // register i of sacc[kb]: key = kTk*j + 32*kb + (i/4)*8 + hf*4 + i%4, query = qc
    auto tile_row_max = [&]() __attribute__((always_inline)) -> float {
        float tm = sacc[0][0];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i) tm = fmaxf(tm, sacc[kb][i]);
        return xhalf_max(tm) * scale_log2e;
    };
    auto softmax_tile = [&](int64_t j, auto exact_tag) __attribute__((always_inline)) {
        constexpr bool EXACT = decltype(exact_tag)::value;
        if ((j + 1) * kTk > N) {                    // only the last tile can be ragged
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = (int)(j * kTk - N) + 32 * kb + (i >> 2) * 8 + hf * 4 + (i & 3);
                    if (key >= 0) sacc[kb][i] = -INFINITY;
                }
        }
        if (EXACT) {
            const float tmax = tile_row_max();
            if (__builtin_amdgcn_ballot_w64(tmax > m_c + kTau) != 0) {
                const float m_new = fmaxf(m_c, tmax);
                const float alpha = __builtin_amdgcn_exp2f(m_c - m_new);   // 0 on the first tile
                m_c = m_new;
                l_run *= alpha;
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[b][i] *= alpha;
            }
        }
        float ps0 = 0.0f, ps1 = 0.0f;
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
        for (int u = 0; u < 8 * KB; ++u) {
            const int kb = u >> 3, i = 2 * (u & 7);
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][i], scale_log2e, -m_c));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][i + 1], scale_log2e, -m_c));
            pw[u] = pack_bf16(p0, p1);
            // the row sum adds the rounded values, the same ones the second product uses
            if (u & 1)
                ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw[u]), ones, ps1, false);
            else
                ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw[u]), ones, ps0, false);
        }
        l_run += ps0 + ps1;
        // keep the row-sum arithmetic in this phase (it is not needed until the end of the sweep, and
        // would otherwise drift behind the MFMAs of the next phase)
        asm volatile("" : "+v"(l_run));
    };

    constexpr int kAhead = 4;      // an MFMA's fragment is fetched kAhead MFMAs before it issues
    // MFMA phase.  O^T += V^T(j) P^T(j): kMfmas MFMAs, 8 to a block of 32 keys; group tt contracts the 16 keys 16*tt + {0..3, 8..11}
    // (lanes 0-31) and 16*tt + {4..7, 12..15} (lanes 32-63); V^T(j) is in the parity va[] points at.
    // Then, if WITH_QK, S^T = K Q^T for the next tile: as many, where there are two blocks of 32 keys these taking turns (two
    // consecutive MFMAs share the Q fragment and feed different accumulators).  One LDS read pipeline runs
    // through all of them.
    // The buffer parity PAR of the phase is a compile-time constant: V^T(j) is read from buffer pair PAR, K(j+1)
    // from pair PAR ^ 1.
    auto mfma_phase = [&](auto qk_tag, auto par_tag) __attribute__((always_inline)) {
        constexpr bool WITH_QK = decltype(qk_tag)::value;
        constexpr uint32_t VP = decltype(par_tag)::value * kBuf;
        constexpr uint32_t KP = (decltype(par_tag)::value ^ 1) * kBuf;
        bf16x8 vf[kMfmas], kf[kMfmas];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) vf[u] = read_v(u, VP);
#pragma unroll
        for (int u = 0; u < kMfmas; ++u) {
            const int tt = u >> 2, b = u & 3;
            uint4v p4 = {pw[4 * tt], pw[4 * tt + 1], pw[4 * tt + 2], pw[4 * tt + 3]};
            oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u], __builtin_bit_cast(bf16x8, p4), oacc[b], 0, 0, 0);
            const int n = u + kAhead;
            if (n < kMfmas)
                vf[n] = read_v(n, VP);
            else if (WITH_QK)
                kf[n - kMfmas] = lds_read_b128(from0 + ka[(n - kMfmas) / KB] + (KP + (n - kMfmas) % KB * 32 * kRowBytes));
        }
        if (WITH_QK) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) sacc[kb][i] = 0.0f;
#pragma unroll
            for (int u = 0; u < kMfmas; ++u) {
                sacc[u % KB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u], qf[u / KB], sacc[u % KB], 0, 0, 0);
                const int n = u + kAhead;
                if (n < kMfmas) kf[n] = lds_read_b128(from0 + ka[n / KB] + (KP + n % KB * 32 * kRowBytes));
            }
        }
        constexpr int kVReads = RETILED ? 1 : 2;         // LDS instructions per V fragment
        SGB(DSR, kAhead * kVReads);
#pragma unroll
        for (int u = 0; u < kMfmas - kAhead; ++u) {
            SGB(MFMA, 1);
            SGB(DSR, kVReads);
        }
        if (WITH_QK) {
#pragma unroll
            for (int u = 0; u < kMfmas; ++u) {
                SGB(MFMA, 1);
                SGB(DSR, 1);
            }
        }
        SGB(MFMA, kAhead);
    };
    // S^T of tile 0 (prologue only)
    auto qk_mfmas = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) sacc[kb][i] = 0.0f;
#pragma unroll
        for (int u = 0; u < kMfmas; ++u)
            sacc[u >> 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                lds_read_b128(from0 + ka[u & 7] + (u >> 3) * 32 * kRowBytes), qf[u & 7], sacc[u >> 3], 0, 0, 0);
    };
    // ---- ping-pong schedule.  K tile j lives in K buffer j & 1, V^T tile j in V buffer j & 1.
    // The 8 waves form two groups of 4 (one wave of each group per SIMD).  Each wave alternates a VALU
    // phase (exponentials of tile j) and an MFMA phase (second product of tile j, first product of
    // tile j+1), with a workgroup barrier after every phase.  Group 1 runs one phase behind group 0,
    // so on every SIMD one wave is in its MFMA phase while the other is in its VALU phase.  Group 1
    // also streams the tiles: during its VALU phase for tile j the buffers of V^T(j+1) and K(j+2) are
    // free (both groups are past the MFMA phase that read them), and the copies are waited for at the
    // end of its following MFMA phase, one phase before group 0 needs them.  Every wave executes the
    // same number of barriers: group 1 one more at the start, group 0 one more at the end.
    // Key groups (all waves of one are in one of these two groups) have tiles of their own, j counting from their share's first, and copy them
    // themselves, all waves of a group in the same phase: in the VALU phase for tile j they are past the barrier behind their MFMA phase for tile
    // j - 1, which read these buffers last, and each waits for its copies in front of the barrier behind the MFMA phase for tile j, the next
    // phase but one being the first that reads them.  A share that has a tile less than the longest passes two more barriers, one for either phase.
    // So the last barrier of all, group 1's behind its last tile and group 0's one more, lies behind every wave's last read of a tile: past it
    // the vote, the repeated sweep's first copies and the merge may use the tiles' place.
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    // The whole sweep.  EXACT = false: offset fixed by the first tile, no max in the sweep.  EXACT = true: a max per tile.
    auto sweep = [&](auto exact_tag) __attribute__((always_inline)) {
        constexpr bool EXACT = decltype(exact_tag)::value;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[b][i] = 0.0f;
        m_c = kLowest;
        l_run = 0.0f;
        PHASE_BARRIER();
        if (grp == 1) PHASE_BARRIER();
        qk_mfmas();                    // S^T of the first tile (K buffer 0)
        // fast form: the first tile's row max is the offset of the whole sweep (nothing is accumulated yet, so
        // nothing needs rescaling; rows past the last key were filled with copies of it and cannot raise the max)
        if (!EXACT) m_c = tile_row_max();
        PHASE_BARRIER();

        auto between_phases = [&]() __attribute__((always_inline)) {
            if (GROUPS == 2) PHASE_BARRIER();
            else __builtin_amdgcn_sched_barrier(0);
        };
        // One tile that has a successor: VALU phase of tile j, then the MFMA phase (second product of tile j from
        // V buffer PAR, first product of tile j+1 from K buffer PAR ^ 1).
        auto tile_step = [&](int j, auto par_tag) __attribute__((always_inline)) {
            constexpr int PAR = decltype(par_tag)::value;
            if (GROUPS == 1 || KEYS > 1 || grp == 1) {
                dma_v_tile(j + 1, PAR ^ 1, wig, WGrp{});
                if (j + 2 < tile_end) dma_k_tile(j + 2, PAR, wig, WGrp{});
            }
            softmax_tile(j, exact_tag);
            between_phases();
            // The wave in its MFMA phase gets issue priority over its SIMD neighbour, which is in its VALU phase.
            __builtin_amdgcn_s_setprio(3);
            mfma_phase(std::true_type{}, par_tag);
            __builtin_amdgcn_s_setprio(0);
            if (GROUPS == 1 || KEYS > 1 || grp == 1) wait_dma();
            PHASE_BARRIER();
        };
        // last tile: no next tile to prefetch or to start
        auto last_step = [&](int j, auto par_tag) __attribute__((always_inline)) {
            softmax_tile(j, exact_tag);
            between_phases();
            mfma_phase(std::false_type{}, par_tag);
            if (GROUPS == 2) PHASE_BARRIER();
        };
        // The loop is unrolled by two so that the buffer parity is a constant in each copy.  Tiles are counted in 32 bits: with 64-bit ones, whose
        // comparisons take vector instructions, and the work split in 32, the two groups' ways through the loop are laid out worse: us 64-bit
        // / 32-bit, code aligned as the build says: 35640 queries x 118800 keys x 24 heads 38648 / 38278, 11880 x 118800 13036 / 13006,
        // 7020 x 17550 1177.5 / 1173.3, 7020 x 512 52.1 / 51.1, 36000 x 77 119 / 114
        int j = tile_begin;
        for (; j < tile_end - 2; j += 2) {
            tile_step(j, P0{});
            tile_step(j + 1, P1{});
        }
        if (j + 1 < tile_end) {
            tile_step(j, P0{});
            last_step(j + 1, P1{});
        } else {
            last_step(j, P0{});
        }
        if (KEYS > 1 && tile_end - tile_begin < (int)((ntiles + KEYS - 1) / KEYS)) {      // a key group with a tile less than another
            PHASE_BARRIER();
            PHASE_BARRIER();
        }
        if (GROUPS == 2 && grp == 0) PHASE_BARRIER();
    };
    sweep(std::false_type{});
    float l_tot = xhalf_sum(l_run);
    // Did a row outgrow its offset?  Its row sum then passed 2^80, or is infinite or NaN (the comparisons are
    // written so that those fail them too), or one of its accumulators overflowed, which shows in their sum.  With a row sum of
    // at most 2^kTau no logit passed the offset by more than kTau, and the exact form would do the very same: short flat
    // sweeps skip the 64 additions (0.7 us of a 57 us call of 7020 queries x 512 keys).  The workgroup decides as one,
    // since its waves share the tiles.
    bool lost = !(l_tot <= kBig);
    const bool rose = l_tot > kRose;
    if (__builtin_amdgcn_ballot_w64(rose) != 0) {
        float o_sum = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) o_sum += (oacc[0][i] + oacc[1][i]) + (oacc[2][i] + oacc[3][i]);
        lost = lost || (rose && !(__builtin_fabsf(o_sum) < INFINITY));
    }
    const bool outgrew = __builtin_amdgcn_ballot_w64(lost) != 0;
    if (lane == 0) wave_outgrew[wave] = outgrew ? 1u : 0u;
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) any |= wave_outgrew[w];
    if (__builtin_amdgcn_readfirstlane(any) != 0) {
        if (GROUPS == 1) __syncthreads();            // every wave has read the words that the first tile is about to replace
        first_tiles();
        wait_dma();
        sweep(std::true_type{});
        if (GROUPS == 1) __syncthreads();            // every wave is past its last V tile, over which output rows are about to lie
        l_tot = xhalf_sum(l_run);
    }
    if (KEYS > 1) {
        // Merge of the key groups: with m* = max_s m_s and w_s = 2^(m_s - m*), O = sum_s w_s O_s / sum_s w_s l_s.  The tiles' place is
        // free.  Each wave has 16 KiB of it for its accumulators as they lie, [b][g][lane][4], merges 4 / KEYS of the four blocks of
        // head-dim for its queries, and keeps its offsets and sums where the blocks that it merges itself would lie.
        constexpr int kOwn = 4 / KEYS;
        int el = lane;                               // the lane number under another name, as below
        asm volatile("" : "+v"(el));
        const int e_qc = el & 31, e_row = el >> 4, e_p = el & 15;
        const int32_t o_row = out.cache ? idx_sel[lane_row(e_qc)] : 0;
        auto place = [&](int s, int b) { return lds0 + ((s * kKeyWaves + iwave) * 4 + b) * 4096; };
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (b / kOwn == kg) continue;
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<floatx4 __attribute__((address_space(3))) *>((uintptr_t)(place(kg, b) + g * 1024 + el * 16)) =
                    floatx4{oacc[b][4 * g], oacc[b][4 * g + 1], oacc[b][4 * g + 2], oacc[b][4 * g + 3]};
        }
        if (el < 32)
            *reinterpret_cast<floatx2 __attribute__((address_space(3))) *>((uintptr_t)(place(kg, kg * kOwn) + e_qc * 8)) = floatx2{m_c, l_tot};
        __syncthreads();
        float ms[KEYS], m_star = -INFINITY, l = 0.0f;
        float w[KEYS];
#pragma unroll
        for (int s = 0; s < KEYS; ++s) {
            const floatx2 ml = *reinterpret_cast<const floatx2 __attribute__((address_space(3))) *>((uintptr_t)(place(s, s * kOwn) + e_qc * 8));
            ms[s] = ml[0];
            w[s] = ml[1];
            m_star = fmaxf(m_star, ms[s]);
        }
#pragma unroll
        for (int s = 0; s < KEYS; ++s) {
            ms[s] = exp2f(ms[s] - m_star);
            l += ms[s] * w[s];
        }
        const float inv = 1.0f / l;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (b / kOwn != kg) continue;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KEYS; ++s) {
                    const floatx4 o = s == kg ? floatx4{oacc[b][4 * g], oacc[b][4 * g + 1], oacc[b][4 * g + 2], oacc[b][4 * g + 3]}
                                              : lds_read_f32x4(place(s, b) + g * 1024 + el * 16);
                    acc += ms[s] * o;
                }
                uint2v o4;
                o4[0] = pack_bf16(acc[0] * inv, acc[1] * inv);
                o4[1] = pack_bf16(acc[2] * inv, acc[3] * inv);
                rows_put(rows_lds, b, g, el, o4);
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8 / KEYS; ++i) {
            const int n = 4 * (i * KEYS + kg) + e_row;
            const int64_t token = __shfl(o_row, n);
            store_row(out, H, head, r0 + n, token, e_p, rows_get(rows_lds, n, e_p), (int64_t)n < row_n);
        }
        if (lse_sel && kg == 0 && el < 32 && (int64_t)el < row_n)
            lse_sel[(r0 + el) * H + head] = (m_star + log2f(l)) * 0.69314718055994530942f;
        return;
    }
    if (pslot >= 0) {
        // a key-range share of an item: unnormalised accumulators, running max and row sum go to the workspace;
        // merge_partials_kernel combines the shares.  The accumulators are stored as they lie, [wave][b][g][lane][4]:
        // whole lines, where rows of head-dim would put 16 bytes on each of 64 lines.
        float *pp = partial + pslot * kPartialFloats;
        const int row = iwave * 32 + qc;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4 *>(pp + (((iwave * 4 + b) * 4 + g) * kWave + lane) * 4) =
                    make_float4(oacc[b][4 * g], oacc[b][4 * g + 1], oacc[b][4 * g + 2], oacc[b][4 * g + 3]);
        if (hf == 0) {
            pp[kBq * D + row] = m_c;
            pp[kBq * D + kBq + row] = l_tot;
        }
        return;
    }
    // the lane number under another name: addresses the prologue had are computed again instead of held in registers
    // through the sweep, which has none to spare
    int el = lane;
    asm volatile("" : "+v"(el));
    const float inv = 1.0f / l_tot;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            // registers 4g..4g+3: head-dim 32*b + 8*g + 4*hf + 0..3
            uint2v o4;
            o4[0] = pack_bf16(oacc[b][4 * g] * inv, oacc[b][4 * g + 1] * inv);
            o4[1] = pack_bf16(oacc[b][4 * g + 2] * inv, oacc[b][4 * g + 3] * inv);
            rows_put(rows_lds, b, g, el, o4);
        }
    __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt(0): this wave's rows are in LDS; no other wave reads them
    const int32_t o_row = out.cache ? idx_sel[lane_row(el & 31)] : 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int n = 4 * i + (el >> 4);
        const int64_t token = __shfl(o_row, n);
        store_row(out, H, head, r0 + n, token, el & 15, rows_get(rows_lds, n, (el & 15)), (int64_t)n < row_n);
    }
    if (lse_sel && el < 32 && (int64_t)el < row_n)
        lse_sel[(r0 + el) * H + head] = (m_c + log2f(l_tot)) * 0.69314718055994530942f;
}


// Combines the key-range shares of the split items: with m* = max_s m_s and w_s = 2^(m_s - m*),
// O = sum_s w_s O_s / sum_s w_s l_s.  Workgroup (x, y) handles rows 32*y .. 32*y+31 of split item x, i.e. what wave y of
// each share stored; its wave b takes head-dim 32*b .. 32*b+31.  Bound by reading the shares (4 KiB per wave and share), which is why
// their number S is a constant: all loads of a wave go out at once, one round trip instead of one per share for the offsets and one
// per two for the sums.
template <int S>
__global__ __launch_bounds__(256) void merge_partials_kernel(const float *__restrict__ partial, AttnSchedule sch,
                                                             int32_t H, int64_t k_sel, const int32_t *__restrict__ idx_sel,
                                                             AttnOut out, float *__restrict__ lse_sel)
{
    __shared__ __attribute__((aligned(1024))) char rows[kRowsBytes];
    const uint32_t left = sch.items_per_xcd - sch.full_items;
    const uint32_t xcd = blockIdx.x / left;
    const uint32_t item = xcd * sch.items_per_xcd + sch.full_items + (blockIdx.x - xcd * left);
    if (item >= (xcd + 1) * sch.items_per_xcd || item >= (uint32_t)H * sch.q_tiles) return;
    const int head = (int)(item / sch.q_tiles);
    const int64_t r0 = (int64_t)(item - (uint32_t)head * sch.q_tiles) * kBq + 32 * blockIdx.y;
    if (r0 >= k_sel) return;
    const float *base = partial + blockIdx.x * S * (int64_t)kPartialFloats;
    const int lane = threadIdx.x & (kWave - 1), b = threadIdx.x / kWave;
    const int row = 32 * blockIdx.y + (lane & 31);
    float ms[S], ls[S];
    floatx4 os[S][4];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const float *ps = base + s * (int64_t)kPartialFloats;
        ms[s] = ps[kBq * D + row];
        ls[s] = ps[kBq * D + kBq + row];
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            os[s][g] = *reinterpret_cast<const floatx4 *>(base + s * (int64_t)kPartialFloats + (((blockIdx.y * 4 + b) * 4 + g) * kWave + lane) * 4);
    int32_t token[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t rr = r0 + 16 * i + (threadIdx.x >> 4);
        token[i] = out.cache ? idx_sel[rr < k_sel ? rr : k_sel - 1] : 0;
    }
    __builtin_amdgcn_sched_barrier(0);
    float m_star = -INFINITY;
#pragma unroll
    for (int s = 0; s < S; ++s) m_star = fmaxf(m_star, ms[s]);
    floatx4 acc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
    float l = 0.0f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const float w = exp2f(ms[s] - m_star);
        l += w * ls[s];
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[g] += w * os[s][g];
    }
    const float inv = 1.0f / l;
    const uint32_t rows_lds = (uint32_t)(uintptr_t)rows;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        uint2v o4;
        o4[0] = pack_bf16(acc[g][0] * inv, acc[g][1] * inv);
        o4[1] = pack_bf16(acc[g][2] * inv, acc[g][3] * inv);
        rows_put(rows_lds, b, g, lane, o4);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = 16 * i + (threadIdx.x >> 4), c = threadIdx.x & 15;
        const int64_t rr = r0 + n;
        if (rr >= k_sel) break;
        store_row(out, H, head, rr, token[i], c, rows_get(rows_lds, n, c), true);
    }
    if (lse_sel && threadIdx.x < 32 && r0 + lane < k_sel)
        lse_sel[(r0 + lane) * H + head] = (m_star + log2f(l)) * 0.69314718055994530942f;
}

}  // namespace

// Estimated microseconds of the last items of an XCD, `left` of them cut into s shares each.  Measured on shapes of 2 to
// 625 key tiles with 90 to 12000 queries:
//  * a key tile takes 0.72 + 0.027 n us with n of the XCD's 32 CUs at work: the chip is at its power limit and lowers its
//    clock as CUs fill up (0.96 us at 9, 1.16 at 18, 1.56 at 30), so filling the idle ones gains less than the count of
//    rounds says (1755 queries x 17550 keys x 24 heads, 21 items per XCD: 351 us whole, 320 us in 63 shares);
//  * a workgroup costs 11 us besides its tiles, one that stores a share (128 KiB) 11 + 0.13 n;
//  * merging costs 4 us and 0.2 us per share of an XCD.
// So short sweeps stay whole: 7020 queries x 512 keys 66 us whole, 84 us in shares by the count of rounds alone; 608 x
// 2025 takes 3 shares per item (37.7 us) instead of 7 (48.2).
static double tail_us(int64_t left, int64_t s, int64_t ntiles)
{
    double us = s > 1 ? 4.0 + 0.2 * (double)(left * s) : 0.0;
    for (int64_t n = left * s; n > 0; n -= kCuPerXcd) {
        const double cus = (double)(n < kCuPerXcd ? n : kCuPerXcd);
        us += 11.0 + (s > 1 ? 0.13 * cus : 0.0) + (double)((ntiles + s - 1) / s) * (0.72 + 0.027 * cus);
    }
    return us;
}

// The budget-aware split for k_sel selected queries of H heads over N keys; `slots` = workgroups per XCD.
// False when the grid would not fit.
static bool plan_attn(int64_t N, int32_t H, int64_t k_sel, AttnSchedule &sch, int64_t &slots)
{
    const int64_t ntiles = (N + kBk - 1) / kBk;
    const int64_t q_tiles = (k_sel + kBq - 1) / kBq, items = (q_tiles * H + kNumXcd - 1) / kNumXcd;
    // Items that would run in a last, partly filled round are cut along the keys into `splits` shares each (up to 8
    // per item, 64 per XCD) where that is cheaper by the estimate below.
    int64_t left = items % kCuPerXcd;
    int64_t splits = 1;
    if (left > 0) {
        double best = tail_us(left, 1, ntiles);
        for (int64_t s2 = 2; s2 <= 8 && left * s2 <= kMaxSharesPerXcd && s2 <= ntiles; ++s2) {
            if ((s2 - 1) * ((ntiles + s2 - 1) / s2) >= ntiles) continue;      // would leave an empty share
            const double cost = tail_us(left, s2, ntiles);
            if (cost < best) {
                best = cost;
                splits = s2;
            }
        }
    }
    if (splits <= 1) {
        left = 0;
        splits = 1;
    }
    slots = items - left + left * splits;
    sch.q_tiles = (uint32_t)q_tiles;
    sch.items_per_xcd = (uint32_t)items;
    sch.full_items = (uint32_t)(items - left);
    sch.splits = (uint32_t)splits;
    sch.tiles_per_split = (uint32_t)((ntiles + splits - 1) / splits);
    return slots * kNumXcd <= 2147483647LL && ntiles <= 2147483647LL;
}

// Whether the plan's workgroups run as two of four waves each.  A 4-wave workgroup copies its own key tiles, so a CU with two of them
// copies twice what one of eight waves does, and two waves on a SIMD meet as they come instead of taking turns: 3 - 5 % slower where the
// sweep is most of the time and every CU has work.  It is the faster one
//  * where every half gets a CU of its own (at most 32 per XCD): four waves with a CU to themselves sweep 8 tiles in 8.8 us, eight in 11;
//  * in short sweeps of more than one round, where rows and results of one half move under the other's sweep, provided that the halves
//    fill fewer rounds, that they are at most one to a CU in the last round, or that there are enough rounds for it not to matter.
// Eight waves / four, us: 450 queries x 900 keys x 24 heads 23.5 / 20.2, 433 x 439 x 16 14.5 / 12.5, 1564 x 966 x 12 24.9 / 22.1, 1094 x 301 x 24
// 13.0 / 11.4; two rounds and more: 36000 x 77 x 24 137 / 121, 8712 x 476 x 8 34.8 / 31.9, 2595 x 205 x 24 23.2 / 21.2, 12941 x 1227 x 16 144.5 /
// 138.8; past the lines: 3060 x 390 x 12 15.8 / 16.4 (36 halves per XCD), 6382 x 2188 x 24 164 / 169 (35 tiles), 4234 x 445 x 24 33.5 / 34.5 and
// 7020 x 512 x 24 56.6 / 57.0 (last rounds of 38 halves).
static bool half_workgroups(int32_t H, int64_t k_sel, int64_t slots, const AttnSchedule &sch)
{
    constexpr int64_t kShort = 24;                 // key tiles
    constexpr int64_t kRound = 2 * kCuPerXcd;      // halves of an XCD's round
    const int64_t items = (k_sel + kBq / 2 - 1) / (kBq / 2) * H, all = items * (sch.full_items ? 1 : sch.splits);
    if (slots <= kCuPerXcd) return all <= kNumXcd * kCuPerXcd;
    const int64_t halves = (items + kNumXcd - 1) / kNumXcd, rounds = (halves + kRound - 1) / kRound;
    return sch.splits == 1 && sch.tiles_per_split <= kShort && slots < (1 << 26) /* a grid of 2^30 at most */ &&
           (rounds > 3 || rounds < (slots + kCuPerXcd - 1) / kCuPerXcd || (halves - 1) % kRound < kCuPerXcd);
}

// How many key groups the eight waves of a workgroup form.  With few items, the halves' four waves have a SIMD each to themselves, where nothing
// runs while one of them is not in its MFMAs, and shares cost a merging launch.  Two key groups on the same 128 queries take turns at the
// matrix pipe instead, and four on 64 queries give CUs work that would have none; the price is key tiles copied for half or a quarter
// of the queries.  They are taken where every item gets a CU of its own, by estimates of the microseconds a call takes, fitted to 120 shapes of
// 2 to 170 key tiles (rms 3 %, and 0.3 % lost on choosing by them): n workgroups on an XCD, a step the key groups' tiles.  A step of four groups takes
// 0.74 us and not 0.82 in calls that repeat with their keys cached; by that, layer-steps of 6088 x 608 x 16 took 72.6 us for 62.3, 4837 x 967 x 12 65.6 for 58.8.
// Before / with them, us: 2025 keys x 608 queries x 24 heads (three shares) 31.0 / 23.2, 1497 x 615 x 24 28.7 / 17.7, 900 x 450 x 24 20.6 / 13.8,
// 1220 x 1746 x 8 26.1 / 15.6, 512 x 1000 x 8 12.6 / 9.2, 2705 x 1894 x 8 33.3 / 27.6; two groups: 1460 x 1460 x 16 29.5 / 24.7, 2072 x 1450 x 16 41.0 /
// 31.5, 3836 x 1918 x 16 68.6 / 58.1; not taken: 1992 x 317 x 4 13.4 (eight shares) / 18.5, 274 x 1479 x 16 11.1 / 11.1.
// What bounds four groups is LDS: their tiles are written for two waves each and V fragments are two reads (10454 x 1045 x 12 86 us, 63 without copies).
static int key_groups(int64_t N, int32_t H, int64_t k_sel, int64_t slots, const AttnSchedule &sch, bool narrow)
{
    const int64_t ntiles = (N + kBk - 1) / kBk, blocks = (N + 31) / 32;
    auto per_xcd = [&](int64_t queries) { return ((k_sel + queries - 1) / queries * H + kNumXcd - 1) / kNumXcd; };
    if (slots > 2 * kCuPerXcd || blocks < 4) return 1;
    const double n1 = (double)(per_xcd(128) * (sch.full_items ? 1 : sch.splits)), n2 = (double)per_xcd(128), n4 = (double)per_xcd(64);
    double best;
    if (narrow && slots <= kCuPerXcd) {
        best = 6.1 + (double)sch.tiles_per_split * (0.87 + 0.008 * n1) + (sch.splits > 1 ? 1.6 + 0.13 * n1 : 0.0);
    } else {
        const int64_t left = sch.items_per_xcd - sch.full_items, rounds = sch.full_items / kCuPerXcd, rest = left ? left : sch.full_items % kCuPerXcd;
        best = 1.042 * ((double)rounds * tail_us(kCuPerXcd, 1, ntiles) + (rest ? tail_us(rest, sch.splits, ntiles) : 0.0)) - 9.2;
    }
    int keys = 1;
    const double two = 7.6 + (double)((ntiles + 1) / 2) * (0.99 + 0.017 * n2), four = 6.2 + (double)((blocks + 3) / 4) * (0.82 + 0.0051 * n4) + 0.03 * n4;
    if (n2 <= kCuPerXcd && ntiles >= 2 && two < best) {
        best = two;
        keys = 2;
    }
    return n4 <= kCuPerXcd && four < best ? 4 : keys;
}

int attn_bf16_key_groups(int64_t N, int32_t H, int64_t k_sel)
{
    AttnSchedule sch;
    int64_t slots = 0;
    if (k_sel > kRetileRows || !plan_attn(N, H, k_sel, sch, slots)) return 1;
    return key_groups(N, H, k_sel, slots, sch, half_workgroups(H, k_sel, slots, sch));
}

int attn_bf16_plan(int64_t N, int32_t H, int64_t k_sel, int64_t plan[8])
{
    AttnSchedule sch;
    int64_t slots = 0;
    if (!plan_attn(N, H, k_sel, sch, slots)) return fail(ASTRAEA_ERR_INVALID, "astraea_attn_plan: grid too large");
    plan[0] = sch.q_tiles;
    plan[1] = sch.items_per_xcd;
    plan[2] = sch.full_items;
    plan[3] = sch.splits;
    plan[4] = sch.tiles_per_split;
    plan[5] = slots * kNumXcd * (half_workgroups(H, k_sel, slots, sch) ? 2 : 1);
    plan[6] = (N + kBk - 1) / kBk;
    plan[7] = (int64_t)kNumXcd * kMaxSharesPerXcd;
    return ASTRAEA_OK;
}

// Workspace of the bf16 path: the V^T tiles written by the pre-pass, then the partial results of the
// split items (at most kMaxSharesPerXcd shares per XCD).
static size_t vt_bytes(int64_t N, int32_t H)
{
    const int64_t ntiles = (N + kBk - 1) / kBk;
    return (size_t)ntiles * (size_t)H * kTileBytes;
}
static size_t partial_bytes() { return (size_t)kNumXcd * kMaxSharesPerXcd * kPartialFloats * sizeof(float); }
size_t attn_bf16_workspace_bytes(int64_t N, int32_t H)
{
    if (N <= 0 || H <= 0) return 0;
    const size_t b = vt_bytes(N, H) + partial_bytes();
    return (b + 255) & ~(size_t)255;
}

int launch_attn_bf16_d128(const void *q, const void *k, const void *v, int64_t N, int32_t H, int64_t q_stride_n,
                          int64_t q_stride_h, int64_t kv_stride_n, int64_t kv_stride_h, const int32_t *idx_sel,
                          int64_t k_sel, int q_is_compact, float scale, const AttnOut &out, float *lse_sel, void *workspace,
                          hipStream_t stream)
{
    if (k_sel == 0) return ASTRAEA_OK;
    // a tile's lane offsets are 32-bit: 64 rows must span less than 4 GiB
    if (kv_stride_n * 2 * kBk >= (int64_t)1 << 32)
        return fail(ASTRAEA_ERR_UNSUPPORTED, "astraea_sparse_attn_fwd: K/V token stride too large");
    const int64_t ntiles = (N + kBk - 1) / kBk;
    AttnSchedule sch;
    int64_t slots = 0;
    if (!plan_attn(N, H, k_sel, sch, slots))
        return fail(ASTRAEA_ERR_INVALID, "astraea_sparse_attn_fwd: grid too large");
    char *vt = (char *)workspace;
    float *partial = (float *)(vt + vt_bytes(N, H));
    const bool retile = k_sel > kRetileRows;
    const bool narrow = half_workgroups(H, k_sel, slots, sch);
    const int keys = retile ? 1 : key_groups(N, H, k_sel, slots, sch, narrow);
    if (keys > 1) {          // every item whole, 256 / keys queries each
        sch.q_tiles = (uint32_t)((k_sel + kBq / keys - 1) / (kBq / keys));
        slots = sch.items_per_xcd = sch.full_items = (uint32_t)(((int64_t)sch.q_tiles * H + kNumXcd - 1) / kNumXcd);
        sch.splits = 1;
    }
    const int64_t left = sch.items_per_xcd - sch.full_items;
    const int groups = narrow && keys == 1 ? 1 : 2;
    dim3 grid((unsigned)(slots * kNumXcd * (2 / groups))), block(groups * kGroupWaves * kWave);
    const float c = scale * 1.44269504088896340736f;
    if (retile)
        hipLaunchKernelGGL(transpose_v_kernel, dim3((unsigned)ntiles, (unsigned)H), dim3(256), 0, stream, (const __bf16 *)v, N,
                           kv_stride_n, kv_stride_h, ntiles, vt);
    auto go = [&](auto kernel, const void *vsrc) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, (const __bf16 *)q, (const __bf16 *)k, vsrc, N, H, q_stride_n,
                           q_stride_h, kv_stride_n, kv_stride_h, idx_sel, k_sel, q_is_compact, c, out, lse_sel, sch,
                           partial);
    };
    kernel_timer_begin(stream);
    if (keys == 4) go(attn_bf16_kernel<false, 2, 4>, v);
    else if (keys == 2) go(attn_bf16_kernel<false, 2, 2>, v);
    else if (retile && narrow) go(attn_bf16_kernel<true, 1, 1>, vt);
    else if (narrow) go(attn_bf16_kernel<false, 1, 1>, v);
    else if (retile) go(attn_bf16_kernel<true, 2, 1>, vt);
    else go(attn_bf16_kernel<false, 2, 1>, v);
    kernel_timer_end(stream);
    if (left > 0)
        with_shares((int)sch.splits, [&](auto shares) {
            hipLaunchKernelGGL(merge_partials_kernel<decltype(shares)::value>, dim3((unsigned)(left * kNumXcd), kBq / 32), dim3(256), 0, stream,
                               partial, sch, H, k_sel, idx_sel, out, lse_sel);
        });
    return check_launch("astraea_sparse_attn_fwd(bf16)");
}

}  // namespace astraea
