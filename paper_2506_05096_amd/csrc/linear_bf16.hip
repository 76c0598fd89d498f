// astraea_sparse_linear, bf16: a per-token linear layer evaluated for the selected tokens only
// (paper, Algorithm 1: Q = X_in[I_sel] W_Q; Sec. 3.2: every layer that acts on a token by itself is
// computed for the selected tokens and reused from the cache for the others; FLOPs appendix: the
// projection and MLP terms):
//     y[row_out(r), o] = act( sum_c x[row_in(r), c] * w[o, c] + bias[o] )
// Rows are gathered by index while the input tile is copied into LDS and scattered by index in the
// epilogue, so neither a compact copy of the input nor one of the output exists.
//
// Shape of the computation on gfx950:
//  * x rows and w rows are both contiguous along the contraction, which is what both operands of
//    v_mfma_f32_32x32x16_bf16 want (a lane holds 8 consecutive k of one row / column).  w feeds the A
//    operand and x the B operand, so that an accumulator lane owns one token and 4 consecutive output
//    features per register group: the epilogue packs them to 8-byte stores along the output row.
//  * workgroup = 8 waves, two per SIMD, output tile 256 features x 256 tokens, each wave 128 features
//    x 64 tokens (4 x 2 MFMA blocks, 128 accumulator registers, 3 LDS fragment reads per 4 MFMAs); or, where
//    that leaves fewer idle CUs in the last round of tiles, 192 or 128 tokens (waves of 64 x 96 or 64 x 64), or 128 features x 128
//    tokens (waves of 64 x 32; bound by the operands' way from L2, 32 KiB per step and CU).
//    One wave per SIMD with 128 x 128 (kWaves = 4, every wave copying, the step's barrier moved in
//    front of the last quarter so that no fragment read follows it) runs fewer clocks per step at a
//    lower clock rate, or the other way round: the chip holds its power limit and the two designs
//    end up within 1 % of each other.
//  * the contraction advances in steps of 64; the w tile (32 KiB) and the x tile (16 to 32) of a step go from global memory
//    straight into LDS (global_load_lds_dwordx4, per-lane addresses, so the row gather costs nothing),
//    into a ring of stages, 16-byte chunks XOR-swizzled inside each 128-byte row against bank conflicts.
//    A copy must cover whole 128-byte lines: with 64-byte pieces (a ring of four 32-deep units) the
//    L1 fetches every line from L2 twice and the kernel is 30 % slower.
//    The second wave of each SIMD issues the copy instructions of a coming step, one behind each of
//    its first 12 to 16 MFMAs, and has the higher priority: the memory pipe holds it at every copy, and its
//    neighbour's MFMAs fill exactly that time.  A 4-byte load per row, shared out among the
//    workgroups that use the row, touches the lines of two steps ahead so that the copies hit in L2.  The 128-token tile has
//    three stages, copied two ahead (128 x 128: four, three ahead), and no touches: its steps are shorter than a copy takes (all linear layers of a
//    block, 608 rows: 387 us with two stages' touches, 316 shared, 308 without).
//  * layers with fewer tiles than CUs take tiles of 64 features x 64 or 128 tokens (linear_bf16_few_kernel).
//  * workgroup ids are mapped so that the 32 workgroups resident on one XCD form an 8 x 4 block of
//    tiles: they stream 8 row tiles and 4 weight tiles through that XCD's L2 instead of 32 + 32.  The tiles
//    left after whole rounds go to all XCDs evenly.
// Measured with all of this (us; before: 256-token tiles only, blocks of 8 x 4 dealt whole to the XCDs, so that some had a
// round more than others, every workgroup touching all its rows): 35640 rows 12288 -> 3072 2146 -> 2074 (1.30 PFLOP/s); 5000
// rows 3072 -> 3072 132 -> 80, 12288 -> 3072 489 -> 292; 7020 rows 3072 -> 9216 380 -> 322, 3072 -> 3072 150 -> 119, 12288 -> 3072
// 550 -> 439; 1755 rows 3072 -> 9216 143 -> 83; 608 rows 3072 -> 3072 54 -> 33, 12288 -> 3072 190 -> 115.
#include "gfx950.h"

namespace astraea {
namespace {


constexpr int kBk = 64;                  // contraction step
constexpr int kRowBytes = kBk * 2;       // 128 B of a row per step
constexpr int kWaves = 8;                // two per SIMD
constexpr int kCopyWaves = kWaves / 2;   // the waves that issue the tile copies (the second wave of each SIMD)
constexpr int kNumXcd = 8, kCuPerXcd = 32, kCus = kNumXcd * kCuPerXcd;
constexpr int kSbM = 8, kSbN = 4;        // tiles of one XCD round: 8 token tiles x 4 feature tiles

// A 4-byte load per lane whose only purpose is to pull its 128-byte line into L2.  It is the copy form
// of the load (global -> LDS), aimed at a 256-byte scrap area every wave may scribble on: the data lands
// whenever it arrives, and with no register as its destination nothing the compiler does with registers
// in the meantime can be hit by it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"    // m0 is a reserved register; naming it as clobbered is the point
__device__ __forceinline__ void touch_line(const void *gbase, uint32_t goff, uint32_t lds_scrap)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :
                 : "s"(lds_scrap), "v"(goff), "s"(gbase)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// Nothing moves across it: the order of MFMAs, fragment reads and copies inside a step is the written one.
#define SB() __builtin_amdgcn_sched_barrier(0)

struct LinearArgs {
    const __bf16 *x;
    const int32_t *idx_sel;    // or null when neither side is indexed
    int64_t ldx;               // row stride in elements
    int32_t k_sel, c_in, c_out;
    int32_t n_rows;            // rows of the indexed buffer(s): indices outside [0, n_rows) read a valid row, write none
    int32_t x_indexed, act;
    int32_t m_tiles, n_tiles;  // token tiles, and feature tiles of all parts
    LinearParts parts;         // last: what a launch of one layer loads lies together
};

// Which tile a workgroup has: workgroup ids reach the XCDs round-robin.  The tiles are listed super-block by super-block (8 token
// tiles x 4 feature tiles, fewer at the edges); while whole rounds of 256 are left, each XCD takes 32 of the list at
// a time, and what is left after them is dealt evenly.
__device__ __forceinline__ bool find_tile(const LinearArgs &a, int &mt, int &nt)
{
    const int xcd = blockIdx.x % kNumXcd, seq = blockIdx.x / kNumXcd;
    const int tiles = a.m_tiles * a.n_tiles, whole = tiles / kCus * kCuPerXcd;
    int tile = (seq / kCuPerXcd * kNumXcd + xcd) * kCuPerXcd + seq % kCuPerXcd;
    if (seq >= whole) {
        const int left = tiles - whole * kNumXcd, per_xcd = (left + kNumXcd - 1) / kNumXcd, at = xcd * per_xcd + seq - whole;
        if (at >= left) return false;
        tile = whole * kNumXcd + at;
    }
    const int sb_row = tile / (kSbM * a.n_tiles), in_row = tile % (kSbM * a.n_tiles);
    const int sb_h = a.m_tiles - sb_row * kSbM < kSbM ? a.m_tiles - sb_row * kSbM : kSbM;
    const int sb_col = in_row / (kSbN * sb_h), inner = in_row % (kSbN * sb_h);
    mt = sb_row * kSbM + inner % sb_h, nt = sb_col * kSbN + inner / sb_h;
    return true;
}

// A wave has NB x TB MFMA blocks of 32 features x 32 tokens, a tile kBn features: <4, 2, 256> makes tiles of 256 tokens, <2, 3, 256> of
// 192, <2, 2, 256> and <2, 1, 128> of 128.
template <int NB, int TB, int kBn, bool GROUP>
__global__ __launch_bounds__(kWaves *kWave, 1) void linear_bf16_kernel(LinearArgs a)
{
    constexpr int kTileBytes = kBn * kRowBytes;                   // the w tile of a stage
    constexpr int kWn = kBn / (32 * NB), kWm = kWaves / kWn;      // waves along the features and along the tokens
    constexpr int kBm = 32 * TB * kWm;                            // tokens per tile
    constexpr int kCopiesW = kBn / 8 / kCopyWaves, kCopiesX = kBm / 8 / kCopyWaves;   // 1 KiB copies per copying wave and step
    constexpr int kCopies = kCopiesW + kCopiesX;
    // Stages of [w tile | x tile] in a ring: two, or three where they fit, with the copies one step more ahead.  A step of a
    // small tile is shorter than a copy takes, and small tiles serve layers with few of them, which nothing else hides.
    constexpr int kStageBytes = kTileBytes + kBm * kRowBytes;
    constexpr int kStages = 4 * kStageBytes <= 144 * 1024 ? 4 : 3 * kStageBytes <= 144 * 1024 ? 3 : 2;
    constexpr int kAhead = kStages - 1;
    constexpr int kTouches = kStages == 2 ? 2 : 0;     // L2 warm-up loads per copying wave and step
    constexpr int kPitch = 64 * NB + 16; // epilogue staging: the wave's features of a token, padded
    constexpr int kEpiTokens = 32 * TB;  // the wave's tokens
    constexpr int kEpiBytes = kWaves * kEpiTokens * kPitch;
    __shared__ __attribute__((aligned(1024))) char lds[kStages * kStageBytes > kEpiBytes ? kStages * kStageBytes : kEpiBytes];
    __shared__ __attribute__((aligned(256))) uint32_t scrap[kWave];      // where the L2 warm-up loads land
    // destination rows and bias of this tile, fetched while the first step's tiles are on their way: the
    // epilogue then reads them from LDS instead of waiting for global loads three times over
    __shared__ int32_t tile_rows[kBm];
    __shared__ __attribute__((aligned(16))) uint16_t tile_bias[kBn];

    int mt, nt;
    if (!find_tile(a, mt, nt)) return;
    int part_nt = nt;
    const LinearPart part = a.parts.of<GROUP>(part_nt);
    const int m0 = mt * kBm, n0 = part_nt * kBn;
    // Every argument that is used from here on is loaded here, in one round trip.  The compiler would otherwise load each next to its first
    // use, x inside the copying waves' branch: LDS reads and scalar loads share a counter and scalar loads come out of order, so with one
    // pending at the loop header each step waits for all of its fragments in front of its first MFMA instead of for three at a time.
    // 35640 rows 3072 -> 9216 / 3072 -> 3072 / 3072 -> 12288 / 12288 -> 3072, us: 1586 / 537 / 2198 / 2057 so, 1572 / 534 / 2189 / 2039 now
    asm volatile("" ::"s"(part.w), "s"(part.bias), "s"(part.y), "s"(part.ldy), "s"(part.y_indexed), "s"(a.x), "s"(a.idx_sel), "s"(a.ldx),
                 "s"(a.k_sel), "s"(a.c_in), "s"(a.c_out), "s"(a.n_rows), "s"(a.x_indexed), "s"(a.act));

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int qc = lane & 31, hf = lane >> 5;
    const int wn = wave % kWn, wm = wave / kWn;       // this wave's 32*NB features and 32*TB tokens of the tile
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    // thread t: destination row of the tile's token t (-1: not stored) and bias of its feature t
    int32_t my_row = -1;
    uint16_t my_bias = 0;
    if (tid < kBn) {
        const int m = m0 + tid;
        if (tid < kBm && m < a.k_sel) {
            my_row = m;
            if (part.y_indexed) {
                const int32_t ix = a.idx_sel[m];
                my_row = (uint32_t)ix < (uint32_t)a.n_rows ? ix : -1;
            }
        }
        const int n = n0 + tid;
        if (part.bias && n < a.c_out) my_bias = reinterpret_cast<const uint16_t *>(part.bias)[n];
    }

    // ---- tile copies.  The memory pipe accepts a 1 KiB copy instruction only every ~16 clocks per CU
    // (~57 per wave with four waves at it), so the 48 to 64 of a step hold whoever issues them for half a step.
    // The second wave of each SIMD does all of it, one copy behind each of its first MFMAs, and runs at
    // the higher priority: while it is held at a copy the first wave's MFMAs have the matrix pipe, and
    // when it is not, its own go first.  Both waves end their step at about the same time.
    // One instruction fills 8 rows of a tile; copying wave c = wave - 4 issues instructions c, c+4, ...
    // of each tile.  Lane l serves row 8*i + l/8 and the physical chunk l%8, which holds logical
    // chunk (l%8) ^ ((row/2)%8); for the rows of one wave that is the same in all its instructions, so a
    // lane's byte offset inside its rows is fixed.
    const bool copier = wave >= kCopyWaves;
    const int cw = wave & (kCopyWaves - 1);
    if (copier) __builtin_amdgcn_s_setprio(1);
    const int d_row = lane >> 3;
    const int lchunk = (lane & 7) ^ ((4 * (cw & 1) + (lane >> 4)) & 7);
    uint32_t woff[kCopiesW], xoff[kCopiesX];   // byte offsets of this lane's rows from w and x
    auto w_row = [&](int r) __attribute__((always_inline)) {
        const int n = n0 + r;            // rows past the end re-read the last one; they are never stored
        return (uint32_t)(n < a.c_out ? n : a.c_out - 1) * (uint32_t)a.c_in * 2u;
    };
    auto x_row = [&](int r) __attribute__((always_inline)) {
        const int m = m0 + r < a.k_sel ? m0 + r : a.k_sel - 1;
        const int64_t row = a.x_indexed ? (int64_t)clamp_row(a.idx_sel[m], a.n_rows) : (int64_t)m;
        return (uint32_t)(row * a.ldx * 2);
    };
#pragma unroll
    for (int t = 0; t < kCopiesW; ++t) woff[t] = w_row(8 * (cw + kCopyWaves * t) + d_row) + (uint32_t)lchunk * 16u;
#pragma unroll
    for (int t = 0; t < kCopiesX; ++t) xoff[t] = x_row(8 * (cw + kCopyWaves * t) + d_row) + (uint32_t)lchunk * 16u;
    // all index loads must have landed before the loop: a load still pending at the loop header would
    // make the compiler wait on the vector-memory counter inside it
#pragma unroll
    for (int t = 0; t < kCopiesW; ++t) asm volatile("" ::"v"(woff[t]));
#pragma unroll
    for (int t = 0; t < kCopiesX; ++t) asm volatile("" ::"v"(xoff[t]));

    const char *wg = reinterpret_cast<const char *>(part.w);
    const char *xg = reinterpret_cast<const char *>(a.x);
    // L2 warm-up: a step's 128 bytes of one row are one cache line, and this wave copies up to 64 rows of
    // each tile, so one lane per row touches all of them (lane l: the l/8-th copy's row l%8).
    // Rows come from HBM (gathered x rows) or the memory-side cache (w), whose latency exceeds one step;
    // touching them kPrefetch steps ahead lets the tile copies hit in L2.
    const uint32_t pf_w = w_row(8 * (cw + kCopyWaves * ((lane >> 3) % kCopiesW)) + (lane & 7));
    const uint32_t pf_x = x_row(8 * (cw + kCopyWaves * ((lane >> 3) % kCopiesX)) + (lane & 7));
    if (kTouches) asm volatile("" ::"v"(pf_x), "v"(pf_w));
    // The 8 token tiles of a block share its weight rows and the 4 feature tiles its token rows, so each workgroup touches an
    // eighth of the one and a quarter of the other: a load of one word of each of 64 rows holds the memory pipe like
    // four tile copies.  All linear layers of a block, 17550 tokens at 40 % / 118800 at 30 %: every workgroup touching all
    // its rows 1484 / 6689 us, no touches 1540 / 6757, shared 1340 / 6346.  (Of a layer by itself, repeated with its weights still
    // cached, no touches would be as fast.)  Whether the neighbours run at the same time matters for speed only.
    const bool touch_w = (lane & (kSbM - 1)) == mt % kSbM, touch_x = (lane & (kSbN - 1)) == nt % kSbN;
    const uint32_t scrap0 = (uint32_t)(uintptr_t)scrap;
    constexpr int kPrefetch = kAhead + 1;      // one step before the copy; 3 with copies one ahead: 2-3 % slower
    auto dma_w = [&](int t, int kstep, uint32_t stage) __attribute__((always_inline)) {
        dma16(wg + (int64_t)kstep * kRowBytes, woff[t], lds0 + stage + (cw + kCopyWaves * t) * 1024);
    };
    auto dma_x = [&](int t, int kstep, uint32_t stage) __attribute__((always_inline)) {
        dma16(xg + (int64_t)kstep * kRowBytes, xoff[t], lds0 + stage + kTileBytes + (cw + kCopyWaves * t) * 1024);
    };

    // ---- fragment offsets inside the array: row 32*block + qc of this wave's half, logical chunk 2*s + hf of k-step s
    uint32_t wa[4], xa[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const uint32_t sw = (uint32_t)(((2 * s + hf) ^ ((qc >> 1) & 7)) << 4);
        wa[s] = (wn * 32 * NB + qc) * kRowBytes + sw;
        xa[s] = kTileBytes + (wm * 32 * TB + qc) * kRowBytes + sw;
    }

    floatx16 acc[NB][TB];                // [feature block][token block]
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    const int nk = a.c_in / kBk;
    // prologue: the first stages
    if (copier) {
#pragma unroll
        for (int p = 0; p < kAhead; ++p)
#pragma unroll
            for (int t = 0; t < kCopiesW; ++t) {
                dma_w(t, p < nk ? p : nk - 1, p * kStageBytes);
                if (t < kCopiesX) dma_x(t, p < nk ? p : nk - 1, p * kStageBytes);
            }
        const int kp = kAhead < nk ? kAhead : nk - 1;
        if (kTouches && touch_w) touch_line(wg + (int64_t)kp * kRowBytes, pf_w, scrap0);
        if (kTouches && touch_x) touch_line(xg + (int64_t)kp * kRowBytes, pf_x, scrap0);
    }
    wait_dma_but<(kAhead - 1) * kCopies + kTouches>();
    if (tid < kBn) {
        if (tid < kBm) tile_rows[tid] = my_row;
        tile_bias[tid] = my_bias;
    }
    __builtin_amdgcn_s_barrier();

    bf16x8 wf[2][NB], xf[2][TB];
    // the fragments of a step's first quarter
    auto read_first = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TB; ++j) xf[0][j] = lds_read_b128(lds0 + xa[0] + j * 32 * kRowBytes);
#pragma unroll
        for (int i = 0; i < NB; ++i) wf[0][i] = lds_read_b128(lds0 + wa[0] + i * 32 * kRowBytes);
    };
    uint32_t next_stage = kAhead * kStageBytes;   // where the copies of step kk + kAhead go
    int kn = 0, kp = 0, stage = 0;       // stage: the ring position of the present step
    // Quarter s of a step, in the order written: behind each of its first MFMAs one fragment read of quarter
    // s + 1; a copying wave also puts one tile copy behind each of the step's first MFMAs, and the two warm-up
    // loads behind the next.  The memory pipe takes a copy every ~16 clocks per CU, ~57 per wave with four
    // waves at it, so a copying wave spends half a step held up at its copies; its SIMD neighbour's MFMAs
    // run in exactly that time.
    auto quarter = [&](auto s_tag) __attribute__((always_inline)) {
        constexpr int s = decltype(s_tag)::value;
        constexpr int cur = s & 1, nxt = cur ^ 1;
#pragma unroll
        for (int n = 0; n < NB * TB; ++n) {
            const int i = n / TB, j = n % TB;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[cur][i], xf[cur][j], acc[i][j], 0, 0, 0);
            constexpr int kReads = TB + NB, kPer = (kReads + NB * TB - 1) / (NB * TB);     // fragment reads of a quarter, behind an MFMA
            if (s < 3) {
#pragma unroll
                for (int u = kPer * n; u < kPer * (n + 1) && u < kReads; ++u) {
                    if (u < TB) xf[nxt][u] = lds_read_b128(lds0 + xa[(s + 1) & 3] + u * 32 * kRowBytes);
                    else wf[nxt][u - TB] = lds_read_b128(lds0 + wa[(s + 1) & 3] + (u - TB) * 32 * kRowBytes);
                }
            }
            const int c = s * NB * TB + n;              // MFMA of the step
            if (c < kCopies) {
                if (copier) {
                    if (c >= 2 * kCopiesX) dma_w(c - kCopiesX, kn, next_stage);
                    else if (c & 1) dma_x(c >> 1, kn, next_stage);
                    else dma_w(c >> 1, kn, next_stage);
                }
            } else if (c < kCopies + kTouches) {
                if (copier) {
                    if (c == kCopies) {
                        if (touch_w) touch_line(wg + (int64_t)kp * kRowBytes, pf_w, scrap0);
                    } else if (touch_x) {
                        touch_line(xg + (int64_t)kp * kRowBytes, pf_x, scrap0);
                    }
                }
            }
            SB();
        }
    };
    using Q0 = std::integral_constant<int, 0>;
    using Q1 = std::integral_constant<int, 1>;
    using Q2 = std::integral_constant<int, 2>;
    using Q3 = std::integral_constant<int, 3>;
    for (int kk = 0; kk < nk; ++kk) {
        // the last steps have nothing to prefetch: they copy the last tiles again into the idle stage
        // rather than branch around every copy
        kn = kk + kAhead < nk ? kk + kAhead : nk - 1;
        kp = kk + kPrefetch < nk ? kk + kPrefetch : nk - 1;
        read_first();
        SB();
        quarter(Q0{});
        quarter(Q1{});
        quarter(Q2{});
        quarter(Q3{});
        // the next step's tiles are complete (what may still be pending is what this step issued: its copies where they go
        // more than one step ahead, and its two warm-up loads) and this step's are no longer read: on to the next stage
        wait_dma_but<(kAhead - 1) * (kCopies + kTouches) + kTouches>();
        __builtin_amdgcn_s_barrier();
        SB();
        const uint32_t step = stage == kStages - 1 ? 0u - (kStages - 1) * kStageBytes : kStageBytes;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            wa[s] += step;
            xa[s] += step;
        }
        next_stage = stage * kStageBytes;
        stage = stage == kStages - 1 ? 0 : stage + 1;
    }

    wait_dma();
    // copies that ran on past the last step must not land in what another wave stages there
    if (kAhead > 1) __builtin_amdgcn_s_barrier();
    // ---- epilogue: bias, activation, bf16; then through LDS so that global stores cover whole rows.
    // Register group g of block (i, j): features 32*NB*wn + 32*i + 8*g + 4*hf + 0..3, token
    // 32*TB*wm + 32*j + qc of the tile.  An accumulator lane owns one token, so stores straight from the
    // registers would put 16 bytes on each of 32 rows per instruction; partial-line writes of that kind
    // cost several times the main loop's share of HBM time.  Instead each wave transposes its block
    // through its own part of LDS (rows of its features, padded by 16 bytes) and
    // writes whole 128-byte lines (4 rows x 256 bytes per instruction, or 8 x 128).  The stages are free: every
    // wave has passed the barrier behind the last step and its copies.  The region is private to the wave, so no
    // workgroup barrier is needed, only the wave's own LDS counter.
    // this lane's bias values (4 NB groups of 4 features), from the copy in LDS
    uint2v bias2[NB][4];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            bias2[i][g] = *reinterpret_cast<const uint2v *>(&tile_bias[wn * 32 * NB + 32 * i + 8 * g + 4 * hf]);
    const uint32_t ebase = lds0 + wave * (kEpiTokens * kPitch);
    constexpr int kRowLanes = 4 * NB, kRowsPerStore = kWave / kRowLanes;      // read-back: 16 bytes per lane
    const int o_row = lane / kRowLanes, o_chunk = lane % kRowLanes;
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int nl = 32 * i + 8 * g + 4 * hf;      // feature inside the wave's part
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * g + e];
                const uint2v b2 = bias2[i][g];
                v[0] += __uint_as_float(b2[0] << 16);
                v[1] += __uint_as_float(b2[0] & 0xffff0000u);
                v[2] += __uint_as_float(b2[1] << 16);
                v[3] += __uint_as_float(b2[1] & 0xffff0000u);
                if (a.act == ASTRAEA_ACT_GELU_TANH) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
                }
                uint2v o2;
                o2[0] = pack_bf16(v[0], v[1]);
                o2[1] = pack_bf16(v[2], v[3]);
                *reinterpret_cast<uint2v __attribute__((address_space(3))) *>(
                    (uintptr_t)(ebase + (32 * j + qc) * kPitch + nl * 2)) = o2;
            }
    __builtin_amdgcn_s_waitcnt(0xc07f);                      // lgkmcnt(0): this wave's LDS writes are done
#pragma unroll
    for (int it = 0; it < kEpiTokens / kRowsPerStore; ++it) {
        const int tl = kRowsPerStore * it + o_row;           // token inside the wave's part
        const int64_t orow = tile_rows[wm * 32 * TB + tl];   // -1: past the end or a bad index
        const int n = n0 + wn * 32 * NB + 8 * o_chunk;       // c_out is a multiple of 8: a chunk is all in or all out
        const uint4v val = *reinterpret_cast<const uint4v __attribute__((address_space(3))) *>(
            (uintptr_t)(ebase + tl * kPitch + o_chunk * 16));
        // written once: streaming stores leave the tiles other workgroups still read in L2 (+1-3 %)
        if (n < a.c_out && orow >= 0)
            __builtin_nontemporal_store(val, reinterpret_cast<uint4v *>(reinterpret_cast<__bf16 *>(part.y) + orow * part.ldy + n));
    }
}


// ---- Few rows: tiles of 32 WN features x 32 WM tokens, a wave a block of 32 x 32.  A wave reads all of its fragments of a step while the
// MFMAs of the step before run, from a ring whose copies, shared by all waves, are published a step early: with four MFMAs of a wave in a
// step, fragments that are read between them leave the matrix pipe waiting for LDS.  Sums are formed in the order of the kernel above.
template <int WN, int WM, bool GROUP>
__global__ __launch_bounds__(WN *WM *kWave, 1) void linear_bf16_few_kernel(LinearArgs a)
{
    constexpr int NW = WN * WM, kWRows = 32 * WN, kXRows = 32 * WM, kWBytes = kWRows * kRowBytes, kStageBytes = kWBytes + kXRows * kRowBytes;
    constexpr int kStages = 6, kAhead = kStages - 1, kCopiesW = kWRows / 8 / NW, kCopies = kCopiesW + kXRows / 8 / NW;
    constexpr int kPitch = kWRows * 2 + 16;                  // of a token's features on their way out
    static_assert(kStages * kStageBytes <= 144 * 1024 && kXRows * kPitch <= kStages * kStageBytes && kXRows <= NW * kWave, "fits");
    static_assert(kCopies <= 4, "a copy behind each of a step's MFMAs");
    __shared__ __attribute__((aligned(1024))) char lds[kStages * kStageBytes];
    __shared__ int32_t tile_rows[kXRows];
    __shared__ __attribute__((aligned(16))) uint16_t tile_bias[kWRows];

    int mt, nt;
    if (!find_tile(a, mt, nt)) return;
    int part_nt = nt;
    const LinearPart part = a.parts.of<GROUP>(part_nt);
    const int m0 = mt * kXRows, n0 = part_nt * kWRows;
    // the arguments in one round trip, as above
    asm volatile("" ::"s"(part.w), "s"(part.bias), "s"(part.y), "s"(part.ldy), "s"(part.y_indexed), "s"(a.x), "s"(a.idx_sel), "s"(a.ldx),
                 "s"(a.k_sel), "s"(a.c_in), "s"(a.c_out), "s"(a.n_rows), "s"(a.x_indexed), "s"(a.act));
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int qc = lane & 31, hf = lane >> 5, wn = wave % WN, wm = wave / WN;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    // ---- copies: instruction t of wave w fills rows 8 (w + NW t) .. of an operand's tile, physical chunk p of row r with logical p ^ (r / 2 % 8)
    const int d_row = lane >> 3, lchunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);
    uint32_t off[kCopies];               // byte offsets of this lane's rows from w and x
#pragma unroll
    for (int t = 0; t < kCopies; ++t) {
        const int r = 8 * (wave + NW * (t < kCopiesW ? t : t - kCopiesW)) + d_row;
        if (t < kCopiesW) {
            const int n = n0 + r;        // rows past the end re-read the last one; they are never stored
            off[t] = (uint32_t)(n < a.c_out ? n : a.c_out - 1) * (uint32_t)a.c_in * 2u;
        } else {
            const int m = m0 + r < a.k_sel ? m0 + r : a.k_sel - 1;
            const int64_t row = a.x_indexed ? (int64_t)clamp_row(a.idx_sel[m], a.n_rows) : (int64_t)m;
            off[t] = (uint32_t)(row * a.ldx * 2);
        }
        off[t] += (uint32_t)lchunk * 16u;
    }
    // thread t: destination row of the tile's token t (-1: not stored) and bias of its feature t
    int32_t my_row = -1;
    uint16_t my_bias = 0;
    if (tid < kXRows && m0 + tid < a.k_sel) {
        my_row = m0 + tid;
        if (part.y_indexed) {
            const int32_t ix = a.idx_sel[my_row];
            my_row = (uint32_t)ix < (uint32_t)a.n_rows ? ix : -1;
        }
    }
    if (tid < kWRows && part.bias && n0 + tid < a.c_out) my_bias = reinterpret_cast<const uint16_t *>(part.bias)[n0 + tid];
    // no load may be pending at the loop, where the counter counts copies
    asm volatile("" ::"v"(my_row), "v"((uint32_t)my_bias));
#pragma unroll
    for (int t = 0; t < kCopies; ++t) asm volatile("" ::"v"(off[t]));
    const char *wg = reinterpret_cast<const char *>(part.w), *xg = reinterpret_cast<const char *>(a.x);
    auto copy = [&](int t, int kstep, uint32_t stage) __attribute__((always_inline)) {
        const uint32_t to = lds0 + stage + (t < kCopiesW ? 0 : kWBytes) + (wave + NW * (t < kCopiesW ? t : t - kCopiesW)) * 1024;
        dma16((t < kCopiesW ? wg : xg) + (int64_t)kstep * kRowBytes, off[t], to);
    };

    // ---- fragments: row qc of this wave's part, logical chunk 2 q + hf for quarter q of a step
    uint32_t wa[4], xa[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t sw = (uint32_t)(((2 * q + hf) ^ ((qc >> 1) & 7)) << 4);
        wa[q] = lds0 + (wn * 32 + qc) * kRowBytes + sw;
        xa[q] = lds0 + kWBytes + (wm * 32 + qc) * kRowBytes + sw;
    }
    bf16x8 wf[2][4], xf[2][4];           // [step's parity][quarter]
    auto read = [&](auto par_tag, uint32_t stage) __attribute__((always_inline)) {
        constexpr int P = decltype(par_tag)::value;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            wf[P][q] = lds_read_b128(wa[q] + stage);
            xf[P][q] = lds_read_b128(xa[q] + stage);
        }
    };
    floatx16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;

    const int nk = a.c_in / kBk;
#pragma unroll
    for (int p = 0; p < kAhead; ++p)
#pragma unroll
        for (int t = 0; t < kCopies; ++t) copy(t, p < nk ? p : nk - 1, p * kStageBytes);
    wait_dma_but<(kAhead - 1) * kCopies>();
    if (tid < kXRows) tile_rows[tid] = my_row;
    if (tid < kWRows) tile_bias[tid] = my_bias;
    __builtin_amdgcn_s_barrier();
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    read(P0{}, 0);
    uint32_t next = kStageBytes, to = kAhead * kStageBytes;      // where step kk + 1 lies and where the copies of step kk + kAhead go
    auto step = [&](int kk, auto par_tag) __attribute__((always_inline)) {
        constexpr int P = decltype(par_tag)::value;
        // Step kk + 1 is there, for every wave, and every wave has its fragments of step kk - 1, whose place the copies take.  The last steps have
        // nothing to copy or to read ahead: they copy the last tiles again and read what lies there.
        wait_dma_but<(kAhead - 2) * kCopies>();
        SB();
        __builtin_amdgcn_s_barrier();
        SB();
        read(std::integral_constant<int, P ^ 1>{}, next);
        SB();
        const int kn = kk + kAhead < nk ? kk + kAhead : nk - 1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[P][q], xf[P][q], acc, 0, 0, 0);
            if (q < kCopies) copy(q, kn, to);
            SB();
        }
        next = next == (kStages - 1) * kStageBytes ? 0 : next + kStageBytes;
        to = to == (kStages - 1) * kStageBytes ? 0 : to + kStageBytes;
    };
    int kk = 0;
    for (; kk + 2 <= nk; kk += 2) {
        step(kk, P0{});
        step(kk + 1, P1{});
    }
    if (kk < nk) step(kk, P0{});
    wait_dma();
    __syncthreads();                     // nobody reads or copies into the ring any more

    // ---- register group g: features 32 wn + 8 g + 4 hf + 0..3, token 32 wm + qc; through LDS to whole rows of the tile
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int nl = wn * 32 + 8 * g + 4 * hf;
        const uint2v b2 = *reinterpret_cast<const uint2v *>(&tile_bias[nl]);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[4 * g + e];
        v[0] += __uint_as_float(b2[0] << 16);
        v[1] += __uint_as_float(b2[0] & 0xffff0000u);
        v[2] += __uint_as_float(b2[1] << 16);
        v[3] += __uint_as_float(b2[1] & 0xffff0000u);
        if (a.act == ASTRAEA_ACT_GELU_TANH) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
        }
        const uint2v o2 = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *reinterpret_cast<uint2v __attribute__((address_space(3))) *>((uintptr_t)(lds0 + (wm * 32 + qc) * kPitch + nl * 2)) = o2;
    }
    __syncthreads();
    // whole rows of the tile: 16 bytes per lane
    constexpr int kRowLanes = kWRows / 8, kRowsPerStore = NW * kWave / kRowLanes;
    const int o_chunk = tid % kRowLanes;
#pragma unroll
    for (int it = 0; it < kXRows / kRowsPerStore; ++it) {
        const int tl = kRowsPerStore * it + tid / kRowLanes, n = n0 + 8 * o_chunk;       // c_out is a multiple of 8: a chunk is all in or all out
        const int64_t orow = tile_rows[tl];
        const uint4v val = *reinterpret_cast<const uint4v __attribute__((address_space(3))) *>((uintptr_t)(lds0 + tl * kPitch + o_chunk * 16));
        if (n < a.c_out && orow >= 0)
            *reinterpret_cast<uint4v *>(reinterpret_cast<__bf16 *>(part.y) + orow * part.ldy + n) = val;
    }
}

// Estimated microseconds of a layer of `tiles` tiles and nk contraction steps: rounds of 256 workgroups, each `fixed` us besides
// its steps, a step taking `base` us while few of the CUs are at work and, past a share `from` of them, `slope` more per unit
// (the chip at its power limit).  Measured per step, 256 / 192 / 128 tokens per tile: 1.03 / 0.93 / 0.56 with a fifth of the CUs
// at work, 1.25 / 1.0 / 0.61 with two thirds, 1.52 / 1.2 / 0.83 with all.
static double layer_us(int64_t tiles, int nk, double fixed, double base, double from, double slope)
{
    auto round = [&](double share) { return fixed + nk * (base + (share > from ? (share - from) * slope : 0.0)); };
    const int64_t last = tiles % kCus;
    return (double)(tiles / kCus) * round(1.0) + (last ? round((double)last / kCus) : 0.0);
}

int64_t tiles_of(int64_t k_sel, int64_t c_out, int parts, int64_t bm, int64_t bn = 256) { return (k_sel + bm - 1) / bm * ((c_out + bn - 1) / bn) * parts; }

}  // namespace

// Tile by the estimate above.  128 x 128 is for layers whose larger tiles leave most CUs without one: a step of it takes 0.36 us (0.54
// with all CUs at work), for half the work of a 256 x 128 step.  Six layers in turn, so that weights come from memory, us a
// layer, before / with it: 608 rows 12288 -> 3072 163 / 107, 3072 -> 3072 33 / 23, 300 rows 3072 -> 9216 43 / 28, 1755 rows
// 6144 -> 1536 62 / 45, 90 rows 3072 -> 12288 47 / 32; where the larger tiles fill a round they stay, 608 rows 3072 -> 9216 48 / 59.
// Contractions below kDeep are all start and end in either tile (608 rows 128 -> 3072 9.7 / 9.8).
constexpr int32_t kDeep = 512;
static LinearTile whole_tile(int64_t k_sel, int32_t c_in, int64_t c_out, int parts, double &us)
{
    const int nk = c_in / kBk;
    const double us256 = layer_us(tiles_of(k_sel, c_out, parts, 256), nk, 9.0, 1.05, 0.4, 0.78),
                 us192 = layer_us(tiles_of(k_sel, c_out, parts, 192), nk, 7.5, 0.93, 0.6, 0.65),
                 us128 = layer_us(tiles_of(k_sel, c_out, parts, 128), nk, 6.0, 0.56, 0.6, 0.7),
                 small = layer_us(tiles_of(k_sel, c_out, parts, 128, 128), nk, 5.0, 0.36, 0.4, 0.3);
    const LinearTile wide = us256 <= us192 && us256 <= us128 ? LinearTile{256, 256} : LinearTile{256, us192 < us128 ? 192 : 128};
    us = wide.tokens == 256 ? us256 : wide.tokens == 192 ? us192 : us128;
    if (c_in < kDeep || small >= us128 || small >= us192 || small >= us256) return wide;
    us = small;
    return {128, 128};
}

LinearTile linear_bf16_tile(int64_t k_sel, int32_t c_in, int64_t c_out, int parts)
{
    double us;
    return whole_tile(k_sel, c_in, c_out, parts, us);
}

// Tiles of 64 features x 64 or 128 tokens, where there are not more of them than CUs; features 0: none.
// What bounds a layer of few tiles is what a CU takes in, 64 to 75 bytes a nanosecond of copies through LDS: smaller tiles give more CUs some of it, and a
// step of them is only as long as its copies if no wave waits for fragments.  By estimates fitted to 96 layers of blocks 1024 to 3072 wide,
// 80 to 3000 rows, weights from memory (0.1 % lost on choosing by them).  Before / with them, us: 600 rows 12288 -> 3072 106 / 77, 300 x 12288 -> 3072
// 90 / 55, 1045 x 6144 -> 1536 55 / 43, 707 x 4096 -> 1024 26.7 / 14.2, 707 x 1024 -> 1024 9.9 / 6.7, 152 x 1536 -> 4608 13.2 / 7.7, 218 x 8192 -> 2048
// 62 / 30; left to the other tiles, which win from a round and a bit on: 600 x 3072 -> 9216 49 / 63, 1885 x 1536 -> 1536 15.0 / 20.9.  128 features x 64
// tokens measured as 64 x 128 do.  Shallow contractions keep the tiles that are all start and end.
LinearTile linear_bf16_few(int64_t k_sel, int32_t c_in, int64_t c_out, int parts)
{
    double best;
    whole_tile(k_sel, c_in, c_out, parts, best);
    LinearTile tile{0, 0};
    if (c_in < kDeep) return tile;
    const double nk = (double)(c_in / kBk);
    const int64_t square = tiles_of(k_sel, c_out, parts, 64, 64), tall = tiles_of(k_sel, c_out, parts, 128, 64);
    const double us64 = 1.9 + nk * (0.191 + 0.093 * (double)square / kCus), us128 = 2.4 + nk * (0.28 + 0.121 * (double)tall / kCus);
    if (tall <= kCus && us128 < best) {
        tile = {64, 128};
        best = us128;
    }
    if (square <= kCus && us64 < best) tile = {64, 64};
    return tile;
}

int launch_linear_bf16(const void *x, const LinearPart *parts, int n_parts, const int32_t *idx_sel, int64_t k_sel, int64_t n_rows,
                       int32_t c_in, int32_t c_out, int64_t ldx, int x_indexed, int act, hipStream_t stream)
{
    if (k_sel == 0) return ASTRAEA_OK;
    LinearArgs a;
    a.x = (const __bf16 *)x;
    for (int i = 0; i < kMaxLinearParts; ++i) a.parts.part[i] = parts[i < n_parts ? i : 0];
    a.idx_sel = idx_sel;
    a.ldx = ldx;
    a.k_sel = (int32_t)k_sel;
    a.n_rows = (int32_t)n_rows;
    a.c_in = c_in;
    a.c_out = c_out;
    a.x_indexed = x_indexed;
    a.act = act;
    if (tiles_of(k_sel, c_out, n_parts, 128, 128) > 2147483647LL / 16) return fail(ASTRAEA_ERR_INVALID, "astraea_sparse_linear: grid too large");
    const LinearTile few = linear_bf16_few(k_sel, c_in, c_out, n_parts);
    const LinearTile tile = few.tokens ? few : linear_bf16_tile(k_sel, c_in, c_out, n_parts);
    auto go = [&](auto kernel, int waves = kWaves) {
        a.m_tiles = (int32_t)((k_sel + tile.tokens - 1) / tile.tokens);
        a.parts.n_tiles_each = (c_out + tile.features - 1) / tile.features;
        a.n_tiles = a.parts.n_tiles_each * n_parts;
        const int64_t t = (int64_t)a.m_tiles * a.n_tiles;
        const int64_t grid = t / kCus * kCus + (t % kCus + kNumXcd - 1) / kNumXcd * kNumXcd;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(waves * kWave), 0, stream, a);
    };
    auto choose = [&](auto group) {
        constexpr bool G = decltype(group)::value;
        if (few.tokens == 128) go(linear_bf16_few_kernel<2, 4, G>, 8);
        else if (few.tokens == 64) go(linear_bf16_few_kernel<2, 2, G>, 4);
        else if (tile.tokens == 256) go(linear_bf16_kernel<4, 2, 256, G>);
        else if (tile.tokens == 192) go(linear_bf16_kernel<2, 3, 256, G>);
        else if (tile.features == 256) go(linear_bf16_kernel<2, 2, 256, G>);
        else go(linear_bf16_kernel<2, 1, 128, G>);
    };
    if (n_parts > 1) choose(std::true_type{});
    else choose(std::false_type{});
    return check_launch("astraea_sparse_linear(bf16)");
}

}  // namespace astraea
