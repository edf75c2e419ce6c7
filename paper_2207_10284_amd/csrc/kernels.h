// Launchers of the MRA-2 kernels (internal; the public interface is mra.h).
// Every launcher only enqueues on `stream` and returns hipGetLastError().
// Arguments are assumed validated by the caller (api.cpp).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "mra.h"

namespace mra {

// The forward's host-side half, shared by mra_attention_forward and the entry
// point without a workspace argument (api.cpp). forward_check runs every
// argument check of mra_attention_forward except those of the workspace,
// makes no HIP call, and on MRA_OK sets *need to the workspace bytes and
// *empty when there is nothing to compute. forward_enqueue enqueues the three
// launches of the forward with the given workspace (at least *need bytes,
// 16-byte aligned) for arguments that passed forward_check.
mra_status_t forward_check(const void* q, const void* k, const void* v, const void* out,
                           const int32_t* idx_out, const float* lse_out, int B, int H, int n,
                           int d, int block, int budget, mra_dtype_t dtype, size_t* need,
                           bool* empty);
mra_status_t forward_enqueue(const void* q, const void* k, const void* v, void* out,
                             int32_t* idx_out, float* lse_out, void* workspace, int B, int H,
                             int n, int d, int budget, mra_dtype_t dtype, void* stream);
// MRA_OK for hipSuccess; otherwise records e as the calling thread's last HIP
// error (mra_last_hip_error) and returns MRA_ERR_HIP.
mra_status_t hip_error_status(hipError_t e);

// q, k, v, g ([bh, n, d] float32) as three bfloat16 planes each, for the gradient
// passes: per 32-row block the hi, mid and lo tiles (32 x d, row-major) one after the
// other, 6 bytes per element.
hipError_t launch_split(const float* q, const float* k, const float* v, const float* g, void* qpl,
                        void* kpl, void* vpl, void* gpl, long long bh, int n, int d, hipStream_t stream);

// Block-means of q/k/v ([bh, n, d], dtype) into qp/kp/vp ([bh, n/32, d] f32);
// a NULL output skips that tensor.
hipError_t launch_pool(const void* q, const void* k, const void* v, float* qp, float* kp,
                       float* vp, long long bh, int n, int d, int dtype, hipStream_t stream);

constexpr int kMaxLevels = 8;      // resolutions above 1 of one call

// S = qp kp^T / sqrt(d) per head and level, float64 accumulation, [bh, nb, nb]
// f32 (first: filled in by the launcher).
struct CoarseLevels {
  const float *qp[kMaxLevels], *kp[kMaxLevels];
  float* S[kMaxLevels];
  int nb[kMaxLevels];
  unsigned first[kMaxLevels];
  int levels;
};
hipError_t launch_coarse_levels(CoarseLevels C, long long bh, int d, hipStream_t stream);

// The same for one level.
hipError_t launch_coarse(const float* qp, const float* kp, float* S, long long bh, int nb, int d,
                         hipStream_t stream);

// Debug aid: every 32-bit word of p[0 .. bytes/4) set to `pattern`.
hipError_t launch_fill(void* p, size_t bytes, uint32_t pattern, hipStream_t stream);

// Top-m column blocks per row of S, ascending, into idx [bh, nb, m].
hipError_t launch_select(const float* S, int32_t* idx, long long bh, int nb, int m,
                         hipStream_t stream);

// The same among the children of the parent level's kept blocks parent_idx
// [bh, nbp, mp] (nbp = nb / r <= 1024) of each row's parent row.
hipError_t launch_select_among(const float* S, int32_t* idx, const int32_t* parent_idx, long long bh, int nb, int m,
                               int nbp, int mp, hipStream_t stream);

// Low-resolution term (cmax, csum, cvec) of the blocks not listed in idx.
hipError_t launch_coarse_term(const float* S, const int32_t* idx, const float* vp, float* cmax,
                              float* csum, float* cvec, long long bh, int nb, int d, int m,
                              hipStream_t stream);

// Head-wide selection (one budget per head over all nb x nb blocks, optional
// diagonal priors) into idx [bh, nb, nb]: ascending rows padded with -1.
hipError_t launch_select_global(const float* S, int32_t* idx, long long bh, int nb, int budget,
                                int prior_diagonal, hipStream_t stream);

// Coarse logits and selection in one pass (the logits kept in LDS), for the
// sparse-only variant; same arithmetic and order as the two calls above.
hipError_t launch_select_fused(const float* qp, const float* kp, int32_t* idx, long long bh,
                               int nb, int d, int m, hipStream_t stream);

// Coarse logits, selection and low-resolution term in one pass, the logits
// kept in LDS (same arithmetic and order as the three calls above).
hipError_t launch_select_term_fused(const float* qp, const float* kp, int32_t* idx,
                                    const float* vp, float* cmax, float* csum, float* cvec,
                                    long long bh, int nb, int d, int m, hipStream_t stream);

// Selected 32x32 tiles, merge with the low-resolution term (or none if cmax is
// NULL) and normalise into out [bh, n, d] of dtype; if lse is not NULL, each
// query's natural log normaliser into lse [bh, n] f32.
hipError_t launch_tile(const void* q, const void* k, const void* v, const int32_t* idx,
                       const float* cmax, const float* csum, const float* cvec, void* out, float* lse,
                       long long bh, int n, int d, int m, int dtype, hipStream_t stream);

// Gradient pass (bwd.hip) of one MRA-2 forward with the selection held fixed.
// Inputs q, k, v, out (Z), dout (G) [bh, n, d] of dtype; lse [bh, n] f32 (the
// forward's natural log normalisers); idx [bh, n/32, m] (entries outside
// [0, n/32) ignored, the others distinct); coarse = false for the
// sparse-only variant. Outputs dq, dk, dv [bh, n, d] of dtype. The remaining
// pointers are workspace: pooled rows (coarse only) [bh, nb, d] f32; the
// planes of q, k, v and dout (launch_split; float32 only: the bfloat16 passes
// read raw tiles); ld [bh*nb, 64] f32 (per block-row: 32 log normalisers in
// log2 units, then 32 deltas); bias [bh*n] x 16 bytes (bfloat16 only, else
// NULL: per query the bfloat16 triples hi + mid + lo of -L_i/c and of
// -delta_i, the A operand that adds both to the column pass's products);
// bits [bh*nb, ceil(nb/32)] u32; gh, dqp, dkp, dvp [bh, nb, d] f32 and W, dS
// [bh, nb, nb] f32 (coarse only).
struct BwdArgs {
  const void *q, *k, *v, *out, *dout;
  const float* lse;
  const int32_t* idx;
  void *dq, *dk, *dv;
  long long bh;
  int n, d, m, dtype;
  bool coarse;
  bool pooled_in;                 // qp, kp, vp hold the block means already
  float *qp, *kp, *vp;
  void *q_pl, *k_pl, *v_pl, *g_pl;
  float* ld;
  uint32_t* bias;
  uint32_t* bits;
  float *gh, *W, *dS, *dqp, *dkp, *dvp;
};
hipError_t launch_bwd(const BwdArgs& args, hipStream_t stream);

// More resolutions R = {s_0 > ... > s_{L-1} = 32, 1} (multilevel.hip).
// Means of several levels from the scale-32 means [bh, nb, d] (f32): level l's
// rows[l] = bh nb / r[l] rows of each tensor into dst[l][0 .. 2].
struct PoolUp {
  float* dst[kMaxLevels][3];
  long long rows[kMaxLevels];
  int r[kMaxLevels];
};
hipError_t launch_pool_up(const float* qp, const float* kp, const float* vp, const PoolUp& P, int levels, int d,
                          hipStream_t stream);
// The levels of R = {s_0 > ... > s_{L-1} = 32, 1}: per level l the coarse
// logits S [bh, nb_l, nb_l], the kept blocks idx [bh, nb_l, m_l] (entries
// outside [0, nb_l) ignored), the pooled values vp [bh, nb_l, d] and
// r_l = s_l / 32.
struct LevelTerm {
  const float* S[kMaxLevels];
  const int32_t* idx[kMaxLevels];
  const float* vp[kMaxLevels];
  int nb[kMaxLevels], m[kMaxLevels], r[kMaxLevels];
  int levels;
};
// Low-resolution term (cmax, csum, cvec) of every 32-block-row: at every
// level, the candidate blocks its ancestor did not keep.
hipError_t launch_coarse_term_levels(const LevelTerm& T, float* cmax, float* csum, float* cvec,
                                     long long bh, int d, hipStream_t stream);

}  // namespace mra
