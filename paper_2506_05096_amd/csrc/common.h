// Internal declarations shared by the HIP translation units of libastraea (gfx950 only).
#pragma once
#include <type_traits>

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "astraea.h"

namespace astraea {

constexpr int kWave = 64;

// Records a message for astraea_last_error() and returns `status`.
int fail(int status, const char *fmt, ...);
// Checks hipGetLastError() after a launch.
int check_launch(const char *what);

// Measurement aid: while the kernel timer is on, the attention launchers bracket their main kernel with a
// pair of HIP events on the caller's stream (astraea_probe_kernel_timer / astraea_probe_kernel_ms).
void kernel_timer_begin(hipStream_t stream);
void kernel_timer_end(hipStream_t stream);

// ---- launchers (each enqueues on `stream`, arguments already validated) ----
int launch_score(const void *x_cur, const void *x_prev, astraea_dtype dt, int64_t N, int64_t C, int64_t row_stride,
                 astraea_delta_mode mode, const float *lse_weight, const int32_t *skip_count,
                 const float *penalty_table, int32_t table_len, float w_alpha, float w_beta, float *score_out,
                 hipStream_t stream);

size_t topk_workspace_bytes(int64_t N);       // for the fewest launches; with topk_min_workspace_bytes the selection takes two more
size_t topk_min_workspace_bytes(int64_t N);
int64_t topk_static_max_n();
size_t topk_static_bytes();
int topk_static_scratch(void **ptr_out);      // the library's own per-device scratch array, for astraea_select_topk_static
int launch_select_topk(const float *score, int64_t N, int64_t k, int32_t *idx_sel, int32_t *idx_remain, uint8_t *sel_mask,
                       int32_t *skip_count, void *workspace, size_t workspace_bytes, hipStream_t stream);

// dst_b / src_b: an optional second buffer pair of the same shape and strides, moved by the same launch
int launch_move_rows(void *dst, const void *src, int64_t row_bytes, int64_t dst_stride_bytes,
                     int64_t src_stride_bytes, const int32_t *idx, int64_t k_sel, int64_t n_rows, bool index_dst,
                     bool index_src, hipStream_t stream, void *dst_b = nullptr, const void *src_b = nullptr);

int launch_check_indices(const int32_t *idx_sel, int64_t k_sel, int64_t N, int32_t *counts, hipStream_t stream);

int launch_lse_weight_update(const float *lse_sel, int32_t H, int64_t N, const int32_t *idx_sel, int64_t k_sel,
                             float *lse_weight, hipStream_t stream);

// What a linear layer multiplies by and where its rows go.  Up to kMaxLinearParts layers of the same input and sizes run as one launch,
// their feature tiles one after another.
struct LinearPart {
    const void *w, *bias;      // bias or null
    void *y;
    int64_t ldy;               // row stride in elements
    int32_t y_indexed;
};
constexpr int kMaxLinearParts = 3;
struct LinearParts {
    LinearPart part[kMaxLinearParts];
    int32_t n_tiles_each;      // feature tiles of a layer
    // The layer that feature tile nt belongs to; nt becomes its own tile number.  (Chosen by selections: an index would put the parts into memory.)
    // GROUP: there may be more than one.  A launch of one does not choose: it loads the part with the kernel's other arguments, in one round trip.
    template <bool GROUP> __device__ __forceinline__ LinearPart of(int &nt) const
    {
        LinearPart p = part[0];
        if (!GROUP) return p;
        if (nt >= n_tiles_each) p = nt >= 2 * n_tiles_each ? part[2] : part[1];
        nt -= nt >= 2 * n_tiles_each ? 2 * n_tiles_each : nt >= n_tiles_each ? n_tiles_each : 0;
        return p;
    }
};

int launch_linear_bf16(const void *x, const LinearPart *parts, int n_parts, const int32_t *idx_sel, int64_t k_sel, int64_t n_rows,
                       int32_t c_in, int32_t c_out, int64_t ldx, int x_indexed, int act, hipStream_t stream);

int launch_linear_f32(const void *x, const LinearPart *parts, int n_parts, const int32_t *idx_sel, int64_t k_sel, int64_t n_rows,
                      int32_t c_in, int32_t c_out, int64_t ldx, int x_indexed, int act, hipStream_t stream);

// The tile a linear launch takes.
struct LinearTile {
    int features, tokens;
};
LinearTile linear_bf16_tile(int64_t k_sel, int32_t c_in, int64_t c_out, int parts);
LinearTile linear_bf16_few(int64_t k_sel, int32_t c_in, int64_t c_out, int parts);     // features 0: that tile is the one
LinearTile linear_f32_tile(int64_t k_sel, int64_t c_in, int64_t c_out, int parts);
int linear_f32_waves(int64_t k_sel, int64_t c_in, int64_t c_out, int parts);

// Where the attention puts row r: rows[r] of a compact [k_sel, H * D] result, and row idx_sel[r] of a cached buffer of cache_rows rows.
// Either may be null; an index outside the cached buffer writes nothing.
struct AttnOut {
    void *rows;
    void *cache;
    int64_t cache_stride, cache_rows;
};
size_t attn_bf16_workspace_bytes(int64_t N, int32_t H);
int attn_bf16_plan(int64_t N, int32_t H, int64_t k_sel, int64_t plan[8]);
int attn_bf16_key_groups(int64_t N, int32_t H, int64_t k_sel);
int launch_attn_bf16_d128(const void *q, const void *k, const void *v, int64_t N, int32_t H, int64_t q_stride_n,
                          int64_t q_stride_h, int64_t kv_stride_n, int64_t kv_stride_h, const int32_t *idx_sel,
                          int64_t k_sel, int q_is_compact, float scale, const AttnOut &out, float *lse_sel, void *workspace,
                          hipStream_t stream);
int launch_attn_f32(const void *q, const void *k, const void *v, int64_t N, int32_t H, int32_t D, int64_t q_stride_n,
                    int64_t q_stride_h, int64_t kv_stride_n, int64_t kv_stride_h, const int32_t *idx_sel,
                    int64_t k_sel, int q_is_compact, float scale, const AttnOut &out, float *lse_sel, void *workspace,
                    size_t workspace_bytes, hipStream_t stream);
size_t attn_f32_workspace_bytes(int64_t N, int32_t H, int32_t D, int64_t k_sel);
int attn_f32_plan(int64_t N, int32_t H, int32_t D, int64_t k_sel, size_t workspace_bytes, int64_t plan[8]);

// Calls f with the number of key-range shares of an item, 2 to 8, as a constant.
template <class F> void with_shares(int shares, F &&f)
{
    switch (shares) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
    }
}

}  // namespace astraea
