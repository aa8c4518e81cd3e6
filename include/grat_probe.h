/*
 * libgrat — measurement aids, not operations of the method: a register-resident MFMA-only loop, and what an
 * attention call would launch.
 *
 * The attention kernels are priced against the chip's published dense matrix rate.  What the same
 * matrix instruction sustains on a given machine with nothing else going on (no memory traffic,
 * no vector arithmetic, no waits) depends on the clock the chip holds under that load; this entry
 * point lets a benchmark measure it next to the kernels it reports on.
 */
#ifndef GRAT_PROBE_H
#define GRAT_PROBE_H

#include "grat.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Enqueues one launch of `blocks` workgroups of 256 threads (4 waves).  Every wave issues
 * iters * 8 matrix instructions of the kind the attention kernels use for `dtype`
 * (GRAT_BF16: v_mfma_f32_32x32x16_bf16, GRAT_F16: v_mfma_f32_32x32x16_f16; 32 768 flop each) on
 * four independent accumulators.  Work per launch: blocks * 4 * iters * 8 * 32 768 flop; the
 * caller times the launch (events on hip_stream).
 *
 * What the instruction sustains depends on how its operands toggle, so `data` chooses them.  In
 * every iteration accumulator v (0..3) takes A_v B_v and then A_v B'_v:
 *   data 0  all operands 1.0, B' = B;
 *   data 1  small integers, B' = B: lane l (0..63) holds, as element e (0..7),
 *             A_v = ((37 + 2v) l + 11 e + 5 + 3v) mod 9 - 4,  B_v = ((53 + 2v) l + 17 e + 2 + 3v) mod 9 - 4,
 *           in the instruction's operand layout A[i][k] and B[k][j] with i = j = l mod 32 and
 *           k = 8 (l div 32) + e;
 *   data 2  the stand-in for real activations: for v < 3 pseudo-random n / 64 with n an integer of at
 *           most 8 significant bits spread roughly like 64 N(0,1), and B' = -B, which returns these
 *           accumulators to exactly 0 (every partial sum is a multiple of 1/4096 below 2^24);
 *           v = 3 as under data 1.
 * Afterwards every lane adds up its 64 accumulator values (integers, exact) into
 * d_sink[block * 256 + thread]; the 64 sums of a wave add up to iters * 2 * sum_ij (A_v B_v)_ij
 * summed over the accumulators that count (data 0, 1: all four; data 2: v = 3) — a check that the
 * loop ran its count.
 *
 *   data    0 .. 2
 *   d_sink  DEVICE pointer, blocks * 256 int64, overwritten
 *   blocks  1 .. 65 536;  iters  1 .. 4096 (keeps every accumulator below 2^24)
 *
 * Errors: GRAT_ERR_NULL (d_sink), GRAT_ERR_BAD_DIMS (data, blocks, iters out of range),
 * GRAT_ERR_UNSUPPORTED (dtype GRAT_F32: no matrix path), GRAT_ERR_HIP; nothing is launched on an
 * error other than GRAT_ERR_HIP.  Allocates nothing, does not synchronise.
 */
grat_status grat_probe_mfma(grat_dtype dtype, int32_t data, int64_t* d_sink, int32_t blocks,
                            int32_t iters, void* hip_stream);

/* What an attention call launches (grat_probe_launch). */
typedef struct {
    int32_t mode;           /* tiles: 0 of groups, 1 of one sequence, 2 of groups and prompt rows, 3 of groups, some clipped */
    int32_t rows;           /* query rows of a workgroup */
    int32_t teams;          /* 16-bit types: teams of waves that share a workgroup's keys (1: undivided) */
    int32_t tile_keys;      /* 16-bit types: keys of an LDS tile; fp32: 0 */
    int32_t whole_tiles;    /* mixed launches: leading tiles that are not split, 0: not one */
    int32_t key_waves;      /* fp32, 16-row workgroups: waves that share the keys; else 0 */
    int32_t longest_first;  /* 1: grouped tiles go out by list length */
    int32_t tiles;          /* query tiles (mixed launches: before the split) */
    int32_t xcd_tiles;      /* tiles of the XCD that gets most */
} grat_launch_info;

/*
 * Fills *info for the call with these sizes on contiguous [B, H, N, d] tensors; host only, launches nothing.
 *   ndim 1 .. 3  grat_attention_fwd, or grat_attention_global_fwd with n_global > 0; max_kv = columns of kv_index
 *   ndim 0       grat_dense_attention_fwd over n_global tokens (grid, group, max_kv not read)
 * Errors: GRAT_ERR_NULL (info), and those of the call.
 */
grat_status grat_probe_launch(grat_dtype dtype, int32_t batch, int32_t heads, int32_t head_dim, int32_t n_global,
                              int32_t ndim, const int32_t* grid, const int32_t* group, int32_t max_kv,
                              grat_launch_info* info);

#ifdef __cplusplus
}
#endif
#endif /* GRAT_PROBE_H */
