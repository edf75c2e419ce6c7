// Gradients of the MRA-2 output with the selection held fixed (Sec. 4.2 eq.
// actual_approx_mat_form, Sec. 4.3 Alg. 2; R = {b, 1}, b = 32).
//
// Query i of block-row x takes a softmax over the fine logits P_ij = c Q_i.K_j
// of the columns j of its refined blocks T_x and, with the low-resolution
// term, over the coarse logits S~[x,y] + ln b of the other blocks y, applied
// to the rows V_j and V~_y. With L_i its log normaliser (saved by the
// forward), G = dZ and delta_i = G_i . Z_i, each logit's gradient is its
// probability times (G_i . value - delta_i):
//   fine:   dP_ij = e^{P_ij - L_i} (G_i . V_j - delta_i)
//           dQ_i += c sum_j dP_ij K_j,   dK_j += c sum_i dP_ij Q_i,
//           dV_j += sum_i e^{P_ij - L_i} G_i
//   coarse: the 32 queries of block-row x share S~[x,y]. For a reference m_x,
//           W[x,y] = b e^{S~[x,y] - m_x} (0 for y in T_x),
//           G^_x = sum_{i in x} e^{m_x - L_i} G_i,  d^_x = sum e^{m_x - L_i} delta_i:
//           dS~[x,y] = W[x,y] (V~_y . G^_x - d^_x),   dV~_y = sum_x W[x,y] G^_x,
//           dQ~_x = c sum_y dS~[x,y] K~_y,           dK~_y = c sum_x dS~[x,y] Q~_x.
//           A pooled row is a block mean, so its gradient reaches each of the
//           block's 32 rows divided by 32.
// m_x = min_{i in x} L_i keeps both exponentials at most 1: every L_i is at
// least each coarse logit S~[x,y] + ln b of its own row.
//
// Kernels, in launch order (for float32 after split_kernel of pool.hip, which
// writes the planes):
//  * bwd_rows_kernel: per block-row (a wave; 16 per workgroup): a 256-byte
//    record of the 32 log normalisers (log2 units) and the 32 deltas, the
//    selection as a bitmap; with the coarse
//    term also G^, d^ and the row's W, dS~ and dQ~ (K~ and V~ staged through
//    LDS 64 blocks at a time).
//  * bwd_cols_kernel: per column block (a wave; 16 per workgroup): dK~, dV~.
//  * bwd_dq_*_kernel: per block-row (a wave, float32 a pair), over its refined tiles: the
//    products K_y Q_x^T and V_y G_x^T on the matrix cores, then
//    dQ^T += K_y^T dP^T.
//  * bwd_dkdv_*_kernel: per column block (a wave, float32 a pair), over the block-rows that
//    refined it (ascending): dV^T += G_x^T A, dK^T += c Q_x^T dP. For raw
//    tiles the row pass also writes, per query, the bfloat16 triples of
//    -L_i/c and -delta_i, which enter the products as one more contraction
//    step, so a lane holding 16 queries needs no per-query registers.
//  * bwd_tiles_*_kernel: both tile passes in one launch where the rows are few,
//    without the column pass up to 32 blocks per head.
//  * bwd_lengths_kernel, bwd_order_kernel: before the column pass of many column
//    blocks, their order by falling list length.
// Tile operands: for bfloat16 raw 32-row tiles of the inputs (copied into LDS
// under a swizzle that serves row and transposed reads); for float32 the same
// tiles of three bfloat16 planes.
#include "common.h"
#include "kernels.h"
#include "tile_ops.h"

namespace mra {

constexpr int kBwdRows = 16;              // waves (block-rows) per workgroup of the row pass
constexpr int kBwdTileWaves = 4;          // waves per workgroup of the tile passes
constexpr int kBwdCols = 16;              // column blocks per workgroup of the column pass

template <int DT>
__device__ __forceinline__ float elem_lo(uint32_t w) {
  return DT == BF16 ? bf16_to_f32(w & 0xFFFFu) : __uint_as_float(w);
}

__device__ __forceinline__ f32x4 mfma16x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// x as hi + mid + lo, each rounded to bfloat16 in turn (the two differences
// are exact in float32, so the sum is x to about 2^-24 |x|).
__device__ __forceinline__ uint32_t split3_bf16(float x, uint32_t& mid_lo) {
  const __bf16 hi = (__bf16)x;
  const float r1 = x - (float)hi;
  const __bf16 mid = (__bf16)r1;
  const __bf16 lo = (__bf16)(r1 - (float)mid);
  mid_lo = (uint32_t)__builtin_bit_cast(uint16_t, mid) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
  return __builtin_bit_cast(uint16_t, hi);
}

// One query's bias operand for the column pass: the bfloat16 elements
// [hi(x), mid(x), lo(x), hi(y), mid(y), lo(y), 0, 0].
__device__ __forceinline__ u32x4 bias_operand(float x, float y) {
  uint32_t xm, ym;
  const uint32_t xh = split3_bf16(x, xm), yh = split3_bf16(y, ym);
  return u32x4{xh | (xm << 16), (xm >> 16) | (yh << 16), ym, 0u};
}

// Sum over the N consecutive lanes of each group of N (N a power of two up to
// 32), in every lane of the group.
template <int N>
__device__ __forceinline__ float sum_within(float v) {
  auto dpp = [](float x, auto ctl) {
    return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), decltype(ctl)::value, 0xF, 0xF, true));
  };
  if constexpr (N >= 2) v += dpp(v, std::integral_constant<int, 0xB1>{});     // lane ^ 1
  if constexpr (N >= 4) v += dpp(v, std::integral_constant<int, 0x4E>{});     // lane ^ 2
  if constexpr (N >= 8) v += dpp(v, std::integral_constant<int, 0x141>{});    // mirror in 8
  if constexpr (N >= 16) v += dpp(v, std::integral_constant<int, 0x140>{});   // mirror in 16
  if constexpr (N >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return v;
}

// Sum over the lanes l, l + N, l + 2N, ... (N = 4, 8, 16 or 32), in every lane.
template <int N>
__device__ __forceinline__ float sum_across(float v) {
  auto ror = [](float x, auto ctl) {
    return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), decltype(ctl)::value, 0xF, 0xF, true));
  };
  if constexpr (N <= 4) v += ror(v, std::integral_constant<int, 0x124>{});    // rotated by 4 in 16
  if constexpr (N <= 8) v += ror(v, std::integral_constant<int, 0x128>{});    // by 8
  if constexpr (N <= 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return halves_sum(v);
}

// ---------------------------------------------------------------------------
// Row pass: one wave per block-row x for the per-row terms (the record, the
// bitmap, G^_x, d^_x), then with the coarse term the 16 rows of the
// workgroup together, 128 column blocks per step, on the float32 matrix cores
// (v_mfma_f32_16x16x4_f32; A: 16 rows x 4, B: 4 x 16 columns, lane l holds
// A[l%16][l/16] and B[l/16][l%16], and D[4(l/16)+r][l%16] in register r):
// The per-row terms are one pass over G and Z in whole-row loads (each load 64
// consecutive chunks of 16 bytes): the chunk products are summed over the lanes
// of a row for delta_i and, weighted, over the rows for G^. (Half a row per
// lane touched 64 cache lines per load, and G^ read G a second time, two or four
// bytes per lane.) Training step, before -> after: 32 heads x 1504 x 128 float32
// 377 -> 334 us, 48 heads x 1024 x 128 bfloat16 120 -> 114, 16 heads x 32768 x 128
// 2421 -> 2392, 96 heads x 4096 x 64 429 -> 426.
//  1. S~ = Q~_x K~_y^T and G^_x V~_y^T: one 16 x 16 tile per wave, the
//     contraction over dims taken four at a time from 16-byte loads;
//  2. W and dS~ for the 16 x 128 entries (two per thread), written out;
//  3. dQ~_x += dS~ K~_y: wave (dim tile, part of the step's columns), the
//     partial sums added in part order at the end.
template <int DT, int D, bool COARSE>
__global__ __launch_bounds__(kBwdRows * kWave) __attribute__((amdgpu_waves_per_eu(8, 8))) void bwd_rows_kernel(
    const void* __restrict__ gin, const void* __restrict__ zin, const float* __restrict__ lse,
    const int32_t* __restrict__ idx, const float* __restrict__ qp, const float* __restrict__ kp,
    const float* __restrict__ vp, float* __restrict__ ld, uint32_t* __restrict__ bias,
    uint32_t* __restrict__ bits, float* __restrict__ gh, float* __restrict__ Wout,
    float* __restrict__ dSout, float* __restrict__ dqp, int nb, int m, float scale) {
  using Cfg = TileCfg<DT, D>;
  using elem = typename Cfg::elem;
  constexpr int PER = DT == BF16 ? 8 : 4, CPR = D / PER;   // elements per 16-byte chunk, chunks per row
  constexpr int R = kWave / CPR, NI = 32 / R;              // rows per load, loads of a block-row
  constexpr int BT = NI <= 4 ? NI : 2;                     // loads of G and of Z in flight (more spill at d = 128)
  constexpr int PQ = D + 4;                                 // LDS pitch of the Q~, G^ rows
  constexpr int YC = 128;                                   // column blocks per step
  constexpr int PP = YC + 1, PD = YC + 4;
  constexpr int NTD = D / 16, KQ = kBwdRows / NTD, YK = YC / KQ;
  static_assert(KQ * kBwdRows * D <= 2 * kBwdRows * PP, "dQ~ partials fit the step buffer");
  __shared__ __attribute__((aligned(16))) float Qx[COARSE ? kBwdRows * PQ : 1];
  __shared__ __attribute__((aligned(16))) float Gx[COARSE ? kBwdRows * PQ : 1];
  __shared__ float Pst[COARSE ? 2 * kBwdRows * PP : 1];    // a step's S~, G^V~^T; then dQ~ partials
  __shared__ float Ds[COARSE ? kBwdRows * PD : 1];
  __shared__ float wq[kBwdRows][32], dls[kBwdRows][32];
  __shared__ float rowm[kBwdRows], rowd[kBwdRows];
  __shared__ uint32_t bm_all[kBwdRows][64];                 // nb <= 2048 bits

  const int tid = threadIdx.x;
  const int w = wave_uniform(tid / kWave);
  const int lane = lane_id(), j = lane & 31, h = lane >> 5;
  const int groups = (nb + kBwdRows - 1) / kBwdRows;
  const long long lwg = xcd_remap(blockIdx.x, gridDim.x);
  const long long bh = lwg / groups;
  const int x0 = (int)(lwg - bh * groups) * kBwdRows;
  const bool active = x0 + w < nb;                          // wave-uniform
  const long long g = bh * nb + x0 + w;                     // this wave's block-row
  const int nbw = (nb + 31) / 32;
  uint32_t* bm = bm_all[w];

  if (active) {
    // the first 64 selection entries, the log normaliser and Q~_x are requested
    // first, so their latency overlaps that of the rows of G and Z
    const int ysel0 = lane < m ? idx[g * m + lane] : -1;
    const float L = lse[g * 32 + j];
    float qv[(D + kWave - 1) / kWave];
    if constexpr (COARSE) {
#pragma unroll
      for (int p = 0; p * kWave < D; ++p) qv[p] = p * kWave + lane < D ? qp[g * D + p * kWave + lane] : 0.0f;
    }
    // G and Z, whole rows per load: lane l of load i holds 16 bytes (chunk c) of
    // row i R + l / CPR
    const u32x4* gp = reinterpret_cast<const u32x4*>(reinterpret_cast<const elem*>(gin) + g * 32 * D) + lane;
    const u32x4* zp = reinterpret_cast<const u32x4*>(reinterpret_cast<const elem*>(zin) + g * 32 * D) + lane;
    u32x4 gw[BT], zw[BT];
    auto load = [&](int i0) {
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        gw[b] = gp[(i0 + b) * kWave];
        zw[b] = zp[(i0 + b) * kWave];
      }
    };
    load(0);
    // the selection as a bitmap (entries outside [0, nb) ignored)
    for (int i = lane; i < nbw; i += kWave) bm[i] = 0u;
    wave_lds_sync();
    if (ysel0 >= 0 && ysel0 < nb) atomicOr(&bm[ysel0 >> 5], 1u << (ysel0 & 31));
    for (int i0 = kWave; i0 < m; i0 += kWave) {
      const int y = i0 + lane < m ? idx[g * m + i0 + lane] : -1;
      if (y >= 0 && y < nb) atomicOr(&bm[y >> 5], 1u << (y & 31));
    }
    float mref = 0.0f, wi = 0.0f;
    if constexpr (COARSE) {
      mref = -wave_max(-L);                                 // min over the 32 queries
      wi = exp2f((mref - L) * kLog2e);
      if (h == 0) wq[w][j] = wi;
    }
    wave_lds_sync();
    for (int i = lane; i < nbw; i += kWave) bits[g * nbw + i] = bm[i];
    // delta_i = G_i . Z_i and G^_x = sum_i w_i G_i from the same registers
    float ga[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) ga[e] = 0.0f;
    const int r0 = lane / CPR;
#pragma unroll 1
    for (int i0 = 0; i0 < NI; i0 += BT) {
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        const int r = (i0 + b) * R + r0;
        const float wr = COARSE ? wq[w][r] : 0.0f;
        float part = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g0 = elem_lo<DT>(gw[b][e]);
          part = fmaf(g0, elem_lo<DT>(zw[b][e]), part);
          if constexpr (COARSE) ga[DT == BF16 ? 2 * e : e] = fmaf(wr, g0, ga[DT == BF16 ? 2 * e : e]);
          if constexpr (DT == BF16) {
            const float g1 = __uint_as_float(gw[b][e] & 0xFFFF0000u);
            part = fmaf(g1, __uint_as_float(zw[b][e] & 0xFFFF0000u), part);
            if constexpr (COARSE) ga[2 * e + 1] = fmaf(wr, g1, ga[2 * e + 1]);
          }
        }
        part = sum_within<CPR>(part);
        if (lane % CPR == 0) dls[w][r] = part;
      }
      if (i0 + BT < NI) load(i0 + BT);
    }
    wave_lds_sync();
    const float dl = dls[w][j];
    if (h == 0) {                                           // the block-row's record
      ld[g * 64 + j] = L * kLog2e;
      ld[g * 64 + 32 + j] = dl;
      if (bias != nullptr)
        *reinterpret_cast<u32x4*>(bias + (g * 32 + j) * 4) = bias_operand(-L / scale, -dl);
    }
    if constexpr (COARSE) {
      const float dhat = wave_sum(h == 0 ? wi * dl : 0.0f);
      if (lane == 0) {
        rowm[w] = mref;
        rowd[w] = dhat;
      }
#pragma unroll
      for (int e = 0; e < PER; ++e) ga[e] = sum_across<CPR>(ga[e]);
      if (lane < CPR) {
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) {
          const f32x4 v = {ga[4 * q], ga[4 * q + 1], ga[4 * q + 2], ga[4 * q + 3]};
          *reinterpret_cast<f32x4*>(Gx + w * PQ + lane * PER + 4 * q) = v;
          *reinterpret_cast<f32x4*>(gh + g * D + lane * PER + 4 * q) = v;
        }
      }
#pragma unroll
      for (int p = 0; p * kWave < D; ++p)
        if (p * kWave + lane < D) Qx[w * PQ + p * kWave + lane] = qv[p];
    }
  } else if constexpr (COARSE) {
    for (int dd = lane; dd < D; dd += kWave) Gx[w * PQ + dd] = Qx[w * PQ + dd] = 0.0f;
  }
  if constexpr (!COARSE) return;
  __syncthreads();                                          // Q~, G^, rowm, rowd, bitmaps

  // K~, V~ of the head as buffers: loads past row nb read as zero
  const unsigned hbytes = (unsigned)nb * D * (unsigned)sizeof(float);
  const i32x4 krs = buffer_rsrc(kp + bh * (long long)nb * D, hbytes);
  const i32x4 vrs = buffer_rsrc(vp + bh * (long long)nb * D, hbytes);
  const int lr = lane & 15, lg = lane >> 4;
  const int kind = w >> 3, t = w & 7;                       // step 1: S~ (0) or G^V~^T (1), columns 16t..
  const float* arow = (kind ? Gx : Qx) + lr * PQ + 4 * lg;
  const i32x4 brs = kind ? vrs : krs;
  const int nt = w % NTD, kq = w / NTD;                     // step 3: dims 16nt.., columns kq*YK..
  const int b1lane = ((16 * t + lr) * D + 4 * lg) * (int)sizeof(float);
  const int b3lane = ((kq * YK + lg) * D + 16 * nt + lr) * (int)sizeof(float);
  f32x4 accq = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int y0 = 0; y0 < nb; y0 += YC) {
    const int ystep = y0 * D * (int)sizeof(float);
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int UG = D / 16 < 4 ? D / 16 : 4;             // 16-byte loads in flight per group
#pragma unroll
    for (int u0 = 0; u0 < D / 16; u0 += UG) {
      f32x4 bq[UG];
#pragma unroll
      for (int u = 0; u < UG; ++u)
        bq[u] = mra_raw_buffer_load_f32x4(brs, b1lane + ystep + 16 * (u0 + u) * (int)sizeof(float), 0, 0);
#pragma unroll
      for (int u = 0; u < UG; ++u) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(arow + 16 * (u0 + u));
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mfma16x4(a[e], bq[u][e], acc);   // dims 16(u0+u) + 4(l/16) + e
      }
    }
    __syncthreads();                                        // the previous step's Pst, Ds consumed
#pragma unroll
    for (int r = 0; r < 4; ++r) Pst[(kind * kBwdRows + 4 * lg + r) * PP + 16 * t + lr] = acc[r];
    __syncthreads();
    for (int e = tid; e < kBwdRows * YC; e += kBwdRows * kWave) {
      const int i = e / YC, yl = e % YC, y = y0 + yl;
      float dsv = 0.0f;
      if (x0 + i < nb && y < nb) {
        float wv = 0.0f;
        if (!((bm_all[i][y >> 5] >> (y & 31)) & 1u)) {
          wv = (float)kBlock * exp2f(fmaf(Pst[i * PP + yl], scale, -rowm[i]) * kLog2e);
          dsv = wv * (Pst[(kBwdRows + i) * PP + yl] - rowd[i]);
        }
        const long long gi = bh * nb + x0 + i;
        Wout[gi * nb + y] = wv;
        dSout[gi * nb + y] = dsv;
      }
      Ds[i * PD + yl] = dsv;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < YK / 4; ++s) {
      const int yl = kq * YK + 4 * s + lg;
      const float b = mra_raw_buffer_load_f32(krs, b3lane + ystep + 4 * s * D * (int)sizeof(float), 0, 0);
      accq = mfma16x4(Ds[lr * PD + yl], b, accq);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) Pst[(kq * kBwdRows + 4 * lg + r) * D + 16 * nt + lr] = accq[r];
  __syncthreads();
  if (active) {
    for (int dd = lane; dd < D; dd += kWave) {
      float sum = Pst[w * D + dd];
#pragma unroll
      for (int q = 1; q < KQ; ++q) sum += Pst[(q * kBwdRows + w) * D + dd];
      dqp[g * D + dd] = sum * scale;
    }
  }
}

// The block-rows x whose selection holds column block y (bit y of row x's
// bitmap), ascending, into list (LDS); returns their count (wave-uniform).
// The bitmap words of kColBatch groups of 64 rows are all requested before
// the first is used (rows past nb read row nb - 1's word and are dropped).
constexpr int kColBatch = 8;
template <class T>
__device__ __forceinline__ int column_list(const uint32_t* __restrict__ bits, long long hb, int nbw, int y,
                                           int nb, T* list) {
  const int lane = lane_id();
  int cnt = 0;
  for (int x0 = 0; x0 < nb; x0 += kColBatch * kWave) {
    uint32_t wv[kColBatch];
#pragma unroll
    for (int u = 0; u < kColBatch; ++u) {
      const int x = min(x0 + kWave * u + lane, nb - 1);
      wv[u] = bits[(hb + x) * nbw + (y >> 5)];
    }
#pragma unroll
    for (int u = 0; u < kColBatch; ++u) {
      const int x = x0 + kWave * u + lane;
      const bool ok = x < nb && ((wv[u] >> (y & 31)) & 1u);
      const uint64_t mk = __ballot(ok);
      if (ok) list[cnt + bits_below(mk)] = (T)x;
      cnt += __popcll(mk);
    }
  }
  wave_lds_sync();
  return wave_uniform(cnt);
}

// ---------------------------------------------------------------------------
// Column pass: dK~_y = c sum_x dS~[x,y] Q~_x and dV~_y = sum_x W[x,y] G^_x for
// 16 column blocks per workgroup on the float32 matrix cores, the contraction
// over the block-rows x in ascending order, four per matrix-core step. A wave
// takes one quantity and TW = min(4, D/16) dim tiles at once, with the dims
// permuted inside its group of 16 TW: tile t, column n is dim 16 TW g +
// TW n + t, so each lane reads its TW consecutive dims of a row of Q~ or G^
// with one load (and stores its TW dims of an output row with one store),
// and the column of W or dS serves all TW products.
constexpr int kColsBatch = 8;                             // matrix-core steps per batch of loads

template <int D>
struct ColsCfg {
  static constexpr int kTW = D / 16 < 4 ? D / 16 : 4;      // dim tiles per wave
  static constexpr int kGroups = D / (16 * kTW);            // dim groups
  static constexpr int kWaves = 2 * kGroups;                // (quantity, group) per wave
};

template <int TW>
__device__ __forceinline__ void load_tw(i32x4 rs, int off, float (&b)[TW]) {
  if constexpr (TW == 4) {
    const f32x4 v = mra_raw_buffer_load_f32x4(rs, off, 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) b[t] = v[t];
  } else if constexpr (TW == 2) {
    const f32x2 v = mra_raw_buffer_load_f32x2(rs, off, 0, 0);
    b[0] = v[0];
    b[1] = v[1];
  } else {
    b[0] = mra_raw_buffer_load_f32(rs, off, 0, 0);
  }
}

template <int D>
__global__ __launch_bounds__(ColsCfg<D>::kWaves * kWave) void bwd_cols_kernel(
    const float* __restrict__ qp, const float* __restrict__ gh, const float* __restrict__ W,
    const float* __restrict__ dS, float* __restrict__ dkp, float* __restrict__ dvp, int nb,
    float scale) {
  constexpr int TW = ColsCfg<D>::kTW;
  const int w = wave_uniform(threadIdx.x / kWave);
  const int lane = lane_id(), lr = lane & 15, lg = lane >> 4;
  const int groups = (nb + kBwdCols - 1) / kBwdCols;
  const long long lwg = xcd_remap(blockIdx.x, gridDim.x);
  const long long bh = lwg / groups;
  const int y0 = (int)(lwg - bh * groups) * kBwdCols;
  const long long hb = bh * nb;                             // first block of the head
  const int y = y0 + lr;
  const int kind = w / ColsCfg<D>::kGroups, dg = w % ColsCfg<D>::kGroups;
  const int d0 = 16 * TW * dg + TW * lr;                    // this lane's first dim
  // A[y][x] = A[x * nb + y] (column y) and B[x][d0 ..] of the head as
  // buffers: reads past the head's last row or column come back as zero
  // (those columns' outputs are not stored)
  const i32x4 ars = buffer_rsrc((kind ? W : dS) + hb * nb, (unsigned)nb * nb * (unsigned)sizeof(float));
  const i32x4 brs = buffer_rsrc((kind ? gh : qp) + hb * D, (unsigned)nb * D * (unsigned)sizeof(float));
  int ao = (lg * nb + y) * (int)sizeof(float), bo = (lg * D + d0) * (int)sizeof(float);
  f32x4 acc[TW];
#pragma unroll
  for (int t = 0; t < TW; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // kColsBatch steps of four block-rows per batch, every load of a batch in
  // flight before its products (rows past nb read as zero)
  for (int xs = 0; xs < nb; xs += 4 * kColsBatch) {
    float a[kColsBatch], b[kColsBatch][TW];
#pragma unroll
    for (int u = 0; u < kColsBatch; ++u) {
      a[u] = mra_raw_buffer_load_f32(ars, ao + u * 4 * nb * (int)sizeof(float), 0, 0);
      load_tw<TW>(brs, bo + u * 4 * D * (int)sizeof(float), b[u]);
    }
#pragma unroll
    for (int u = 0; u < kColsBatch; ++u)
#pragma unroll
      for (int t = 0; t < TW; ++t) acc[t] = mfma16x4(a[u], b[u][t], acc[t]);
    ao += 4 * kColsBatch * nb * (int)sizeof(float);
    bo += 4 * kColsBatch * D * (int)sizeof(float);
  }
  // lane: rows y0 + 4 lg + r, dims d0 + t
  float* out = kind ? dvp : dkp;
  const float f = kind ? 1.0f : scale;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int yy = y0 + 4 * lg + r;
    if (yy >= nb) continue;
    float* o = out + (hb + yy) * D + d0;
    if constexpr (TW == 4) {
      *reinterpret_cast<f32x4*>(o) = f32x4{acc[0][r] * f, acc[1][r] * f, acc[2][r] * f, acc[3][r] * f};
    } else {
#pragma unroll
      for (int t = 0; t < TW; ++t) o[t] = acc[t][r] * f;
    }
  }
}

// Stores a 32 x D block from d-major tiles acc (lane: row j; register r of
// tile t: dim 32t + 8(r/4) + 4h + r%4) as acc * a + (add ? add[dim] / 32 : 0).
// The add terms are loaded first, all at once. bfloat16: lanes l and l^32
// hold dims 4h..4h+3 of the groups rg (even, odd); they exchange one group so
// that each stores 8 contiguous dims (16 bytes).
template <int DT, int D>
__device__ __forceinline__ void store_block(typename TileCfg<DT, D>::elem* dst,
                                            const f32x16 (&acc)[D / 32], float a,
                                            const float* add) {
  constexpr int NT = D / 32;
  const int lane = lane_id(), j = lane & 31, h = lane >> 5;
  auto* row = dst + (long long)j * D;
  constexpr float inv = 1.0f / kBlock;
  f32x4 c4[NT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg)
      c4[t][rg] = add != nullptr ? *reinterpret_cast<const f32x4*>(add + 32 * t + 8 * rg + 4 * h)
                                 : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    u32x2 pend = {0u, 0u};
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      const int d0 = 32 * t + 8 * rg + 4 * h;
      float z[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = fmaf(acc[t][4 * rg + e], a, c4[t][rg][e] * inv);
      if constexpr (DT == BF16) {
        const u32x2 pr = {pack_bf16x2(z[0], z[1]), pack_bf16x2(z[2], z[3])};
        if ((rg & 1) == 0) {
          pend = pr;
        } else {
          const u32x2 send = h ? pend : pr;                 // h = 0 sends its odd group, h = 1 its even one
          u32x2 recv;
          recv[0] = (uint32_t)__shfl_xor((int)send[0], 32);
          recv[1] = (uint32_t)__shfl_xor((int)send[1], 32);
          const u32x4 st = h ? u32x4{recv[0], recv[1], pr[0], pr[1]} : u32x4{pend[0], pend[1], recv[0], recv[1]};
          *reinterpret_cast<u32x4*>(row + 32 * t + 8 * (rg - 1) + 8 * h) = st;
        }
      } else {
        const f32x4 st = {z[0], z[1], z[2], z[3]};
        *reinterpret_cast<f32x4*>(row + d0) = st;
      }
    }
  }
}

// bfloat16 pairs of 16 float32 values in register order (the B operand of
// mfma_acc_bf16).
__device__ __forceinline__ void pack16(const float (&v)[16], uint32_t (&pk)[8]) {
#pragma unroll
  for (int rr = 0; rr < 8; ++rr) {
    bf16x2 pb;
    pb[0] = (__bf16)v[2 * rr];
    pb[1] = (__bf16)v[2 * rr + 1];
    pk[rr] = __builtin_bit_cast(uint32_t, pb);
  }
}

// C = X0 Y0^T + A B^T (bfloat16, row layout): the product of one more
// contraction step x0, y0 (16 elements of each row) followed by the KC chunks
// of a and b.
template <int KC>
__device__ __forceinline__ f32x16 mfma_abt_from(const u32x4 (&a)[KC], const u32x4 (&b)[KC], u32x4 x0, u32x4 y0) {
  f32x16 c;
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] = 0.0f;
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x0), __builtin_bit_cast(bf16x8, y0), c, 0, 0, 0);
#pragma unroll
  for (int k = 0; k < KC; ++k)
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[k]), __builtin_bit_cast(bf16x8, b[k]), c, 0, 0, 0);
  return c;
}

// ---------------------------------------------------------------------------
// bfloat16: the passes read raw 32-row tiles of the inputs themselves, no
// packed copies. A tile (32 consecutive rows, 2d bytes each) is
// copied with direct-to-LDS loads of whole rows, every lane fetching the
// 16-byte block that belongs at its LDS position under an XOR swizzle of the
// blocks within a row (raw_offset / raw_copy_offset), and read both in the row
// layout (ds_read_b128: 16 lanes = 16 rows per pass) and transposed
// (ds_read_b64_tr_b16: 32 lanes = 4 rows x 64 bytes per pass). One swizzle
// serves both: for d = 64 the even rows of 16 consecutive rows take 8
// different block positions, and so do the odd ones (row reads), and rows r
// and r + 2 of a group of four take positions in opposite halves of the row
// (transposed reads); for d = 32 rows r, r + 4, r + 8, r + 12 take 4
// different positions; for d = 128 see the d = 128 kernels below. The
// swizzle has period 16 in the row, so the transposed reads 16 rows further
// use the same lane address plus an immediate offset; reads 8 rows further
// need a second address. The copy offsets repeat with period 4 (d = 128),
// 2 (d = 64) or 1 (d = 32) in the copy index.
template <int D>
__host__ __device__ constexpr int raw_swz_b(int r) {
  return D == 128 ? 4 * (r & 3) + ((r >> 2) & 3) : (D == 64 ? 4 * ((r >> 1) & 1) + ((r >> 2) & 3) : (r >> 2) & 3);
}

// This lane's offsets for the raw tiles of the gradient passes.
template <int D>
struct RawB {
  static constexpr int KC = D / 16, NT = D / 32;
  static constexpr int TB = 64 * D;                           // bytes of a 32-row tile
  static constexpr int KP = D == 128 ? 4 : (D == 64 ? 2 : 1); // period of the copy offsets
  unsigned cp[KP];                                            // copy sources of copies i mod KP (less their KB)
  uint32_t rr[KC];                                            // row-layout chunk c
  uint32_t tr[NT][2];                                         // transposed column tile t, half e
  __device__ __forceinline__ void init() {
    const int lane = lane_id(), h = lane >> 5, j = lane & 31, i16 = lane & 15;
#pragma unroll
    for (int q = 0; q < KP; ++q) cp[q] = (unsigned)(raw_copy_offset<D, raw_swz_b<D>>(q, lane) - q * 1024);
#pragma unroll
    for (int c = 0; c < KC; ++c) rr[c] = (uint32_t)raw_offset<D, raw_swz_b<D>>(j, (D / 2) * h + 8 * c);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 2; ++e)
        tr[t][e] = (uint32_t)raw_offset<D, raw_swz_b<D>>(4 * h + i16 / 4 + 8 * e,
                                                         32 * t + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3));
  }
};

// Two raw tiles, C 1 KB copies each, as buffer loads to LDS: the heads' rows
// are the resources ra and rb, the tiles' byte offsets ta and tb go in the
// scalar offset (outside the hardware range check: callers copy validated
// blocks only), this lane's swizzled source offset of copy i (cp[i mod KP],
// the offsets repeat with period KP) in the vector offset.
template <int C, int KP>
__device__ __forceinline__ void copy_raw_pair_buf(i32x4 ra, i32x4 rb, unsigned ta, unsigned tb,
                                                  const unsigned (&cp)[KP], lptr_t as, lptr_t bs) {
  if constexpr (C > 0) {
    copy_raw_pair_buf<C - 1, KP>(ra, rb, ta, tb, cp, as, bs);
    constexpr int i = C - 1;
    buffer_load_lds16(ra, as + i * 1024, cp[i % KP], ta + i * 1024);
    buffer_load_lds16(rb, bs + i * 1024, cp[i % KP], tb + i * 1024);
  }
}

// One raw tile, C 1 KB copies, as buffer loads to LDS (as copy_raw_pair_buf).
template <int C, int KP>
__device__ __forceinline__ void copy_raw_buf(i32x4 rs, unsigned t, const unsigned (&cp)[KP], lptr_t dst) {
#pragma unroll
  for (int i = 0; i < C; ++i) buffer_load_lds16(rs, dst + i * 1024, cp[i % KP], t + i * 1024);
}

// Row-layout chunks of the raw tile at base + OFF.
template <int OFF, int KC>
__device__ __forceinline__ void raw_rows(uint32_t base, const uint32_t (&rr)[KC], u32x4 (&v)[KC]) {
#pragma unroll
  for (int c = 0; c < KC; ++c) v[c] = lds_read16<OFF>(base + rr[c]);
}

// Transposed chunks c = u*NT + t (c < VC) of the raw tile at base + OFF: two
// transposing reads each, the halves 8 rows apart, 16 u rows further on.
template <int D, int OFF, int C, int VC>
struct RawTrB {
  static constexpr int NT = D / 32;
  static __device__ __forceinline__ void run(uint32_t base, const uint32_t (&tr)[NT][2], u32x4* v) {
    if constexpr (C < VC) {
      constexpr int u = C / NT, t = C % NT, o = OFF + 16 * u * 2 * D;
      const u32x2 a = lds_read_tr16<o>(base + tr[t][0]);
      const u32x2 b = lds_read_tr16<o>(base + tr[t][1]);
      v[C] = u32x4{a[0], a[1], b[0], b[1]};
      RawTrB<D, OFF, C + 1, VC>::run(base, tr, v);
    }
  }
};

// The operands of the coarse-term gradients of a column block (see
// bwd_cols_kernel), for the passes that form them on their own: with few column
// blocks per head a launch for them costs more than their sums.
struct ColTerms {
  const float *dS, *qp, *W, *gh;
};
constexpr int kOwnBlocks = 32;

// out (LDS, D floats) = f sum_x A[x, y] B[x, :] over the head's nb <= kOwnBlocks
// block-rows, in ascending order (one wave, lanes over the dims).
template <int D>
__device__ __forceinline__ void own_term(const float* __restrict__ A, const float* __restrict__ B, long long hb, int y,
                                         int nb, float f, float* out) {
  const int lane = lane_id();
  constexpr int P = (D + kWave - 1) / kWave;
  float acc[P];
#pragma unroll
  for (int p = 0; p < P; ++p) acc[p] = 0.0f;
  constexpr int UB = 8;                                     // block-rows per batch of loads
  for (int x0 = 0; x0 < nb; x0 += UB) {
    float a[UB], b[UB][P];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const long long x = hb + min(x0 + u, nb - 1);
      a[u] = x0 + u < nb ? A[x * nb + y] : 0.0f;
#pragma unroll
      for (int p = 0; p < P; ++p) b[u][p] = B[x * D + min(p * kWave + lane, D - 1)];
    }
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int p = 0; p < P; ++p) acc[p] = fmaf(a[u], b[u][p], acc[p]);
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (p * kWave + lane < D) out[p * kWave + lane] = acc[p] * f;
}

// Adds the accumulators of waves 1 .. SPLIT - 1 to wave 0's through LDS: `slot`
// (w) is wave w's own LDS region of 32 x d floats, idle by now. Every wave calls
// it; only wave 0's acc is the sum afterwards.
template <int SPLIT, int NT, class Slot>
__device__ __forceinline__ void add_parts(f32x16 (&acc)[NT], int w, Slot slot) {
  const int lane = lane_id();
  if (w != 0) {
    f32x4* to = reinterpret_cast<f32x4*>(slot(w)) + lane;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        to[(4 * t + q) * kWave] = f32x4{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
  }
  __syncthreads();
  if (w != 0) return;
#pragma unroll
  for (int p = 1; p < SPLIT; ++p) {
    const f32x4* from = reinterpret_cast<const f32x4*>(slot(p)) + lane;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = from[(4 * t + q) * kWave];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][4 * q + e] += v[e];
      }
  }
}

// dQ (bf16, d <= 64): one wave per block-row; a slot holds the raw tiles K_y
// and V_y (K^T is read transposed from the K tile). The next tile is copied once
// the current one is in registers. SPLIT > 1: the workgroup's waves share one
// block-row, wave p taking the tiles p, p + SPLIT, ...
// wg: the logical workgroup; slots, addl, lists: the workgroup's LDS (WAVES
// slots of 2 tiles, WAVES vectors, WAVES lists of m entries).
template <int D, bool COARSE, int WAVES, int SPLIT>
__device__ __forceinline__ void dq_tr_body(
    long long wg, unsigned char* slots, float* addl, int32_t* lists,
    const void* __restrict__ qin, const void* __restrict__ gin, const void* __restrict__ kin,
    const void* __restrict__ vin, const int32_t* __restrict__ idx,
    const float* __restrict__ ld, const float* __restrict__ dqp, void* __restrict__ dq, int nb,
    int m, long long rows, float scale, float scale_log2) {
  using Cfg = TileCfg<BF16, D>;
  using elem = typename Cfg::elem;
  using R = RawB<D>;
  constexpr int KC = Cfg::kKChunks, VC = Cfg::kVChunks, NT = Cfg::kNT;
  constexpr int TB = R::TB;
  constexpr int SLOT = 2 * TB;
  static_assert(KC == R::KC && KC <= 4 && VC <= 4, "raw tiles of d <= 64");
  static_assert(SPLIT == 1 || SPLIT == WAVES, "a workgroup per row");
  const int w = wave_uniform(threadIdx.x / kWave);
  const int lane = lane_id(), jq = lane & 31;
  const long long g = SPLIT > 1 ? wg : wg * WAVES + w;
  if (g >= rows) return;                                    // a shared row: all waves; else no barriers below
  const long long bh = g / nb;
  float* add = addl + w * add_lds_floats(D);
  if constexpr (COARSE) prefetch_vec_lds<D>(dqp + g * D, (lptr_t)add);
  // the row's operands are requested before its list, whose wait covers them
  u32x4 qf[KC], gf[KC];
  load_rows<BF16, D>(reinterpret_cast<const elem*>(qin) + g * 32 * D, qf);
  load_rows<BF16, D>(reinterpret_cast<const elem*>(gin) + g * 32 * D, gf);
  const float lq = ld[g * 64 + jq], dl = ld[g * 64 + 32 + jq];
  int32_t* myidx = lists + w * m;
  int cnt = stage_selection(idx + g * m, m, nb, myidx);
  if constexpr (SPLIT > 1) {
    myidx += w;
    cnt = (cnt - w + SPLIT - 1) / SPLIT;
  }
  wait_loads<0>();
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

  R ro;
  ro.init();
  const i32x4 krs = buffer_rsrc(static_cast<const char*>(kin) + (size_t)bh * nb * TB, (unsigned)nb * TB);
  const i32x4 vrs = buffer_rsrc(static_cast<const char*>(vin) + (size_t)bh * nb * TB, (unsigned)nb * TB);
  const uint32_t base = lds_addr(slots + w * SLOT);
  auto issue = [&](int y) {
    const lptr_t dst = (lptr_t)(slots + w * SLOT);
    copy_raw_pair_buf<KC, R::KP>(krs, vrs, (unsigned)y * TB, (unsigned)y * TB, ro.cp, dst, dst + TB);
  };
  if (cnt > 0) issue(list_entry(myidx));
  for (int i = 0; i < cnt; ++i) {
    const int yn = i + 1 < cnt ? list_entry(myidx + SPLIT * (i + 1)) : 0;
    wait_loads<0>();                                        // tile i landed
    u32x4 kf[KC], vf[KC], tf[VC];
    raw_rows<0>(base, ro.rr, kf);
    raw_rows<TB>(base, ro.rr, vf);
    RawTrB<D, 0, 0, VC>::run(base, ro.tr, tf);
    lds_done(kf);
    lds_done(vf);
    lds_done(tf);
    if (i + 1 < cnt) issue(yn);
    const f32x16 s = mfma_abt<KC>(kf, qf);
    const f32x16 pv = mfma_abt<KC>(vf, gf);
    float ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      ds[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2, -lq)) * (pv[r] - dl);
    uint32_t pk[8];
    pack16(ds, pk);
    mfma_acc_bf16<NT>(acc, pk, [&](int c) { return tf[c]; });
  }
  wait_loads<0>();
  if constexpr (SPLIT > 1) {
    add_parts<SPLIT>(acc, w, [&](int p) { return slots + p * SLOT; });
    if (w != 0) return;
  }
  store_block<BF16, D>(reinterpret_cast<elem*>(dq) + g * 32 * D, acc, scale, COARSE ? add : nullptr);
}

template <int D, bool COARSE, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void bwd_dq_tr_kernel(
    const void* __restrict__ qin, const void* __restrict__ gin, const void* __restrict__ kin,
    const void* __restrict__ vin, const int32_t* __restrict__ idx,
    const float* __restrict__ ld, const float* __restrict__ dqp, void* __restrict__ dq, int nb,
    int m, long long rows, float scale, float scale_log2) {
  __shared__ __attribute__((aligned(16))) unsigned char slots[WAVES * 2 * RawB<D>::TB];
  __shared__ __attribute__((aligned(16))) float addl[COARSE ? WAVES * add_lds_floats(D) : 1];
  extern __shared__ int32_t sidx_all[];
  dq_tr_body<D, COARSE, WAVES, 1>(xcd_remap(blockIdx.x, gridDim.x), slots, addl, sidx_all, qin, gin, kin, vin, idx, ld,
                                  dqp, dq, nb, m, rows, scale, scale_log2);
}

// dK, dV (bf16, d <= 64): one wave per column block; a slot holds the raw
// tiles Q_x and G_x and block-row x's bias operands (Q^T and G^T are read
// transposed). The log normalisers and deltas enter the two products of a
// tile through one more matrix-core step each (A: the queries' bias operands,
// B: ones at the positions of the first or of the second triple), so the
// products come out as Q_i.K_j - L_i/c and G_i.V_j - delta_i, and each lane
// needs one 16-byte read for the 16 queries it holds.
// SPLIT > 1: SPLIT waves share the column block, wave p taking the entries p,
// p + SPLIT, ... of its list.
// OWN: dK~_y and dV~_y are formed here instead of read (T: their operands).
// gy: the column block; slots, addl, lists: the workgroup's LDS (SPLIT slots of
// 2 tiles and the bias operands, two vectors, SPLIT lists of nb entries).
template <int D, bool COARSE, int SPLIT, bool OWN>
__device__ __forceinline__ void dkdv_tr_body(
    long long gy, unsigned char* slots, float* addl, int32_t* lists, const ColTerms& T,
    const void* __restrict__ kin, const void* __restrict__ vin, const void* __restrict__ qin,
    const void* __restrict__ gin, const uint32_t* __restrict__ bits,
    const uint32_t* __restrict__ bias, const float* __restrict__ dkp, const float* __restrict__ dvp,
    void* __restrict__ dk, void* __restrict__ dv, int nb, float scale, float scale_log2) {
  using Cfg = TileCfg<BF16, D>;
  using elem = typename Cfg::elem;
  using R = RawB<D>;
  constexpr int KC = Cfg::kKChunks, VC = Cfg::kVChunks, NT = Cfg::kNT;
  constexpr int TB = R::TB, RB = 32 * 16;                   // bytes of a raw tile, of a block-row's bias operands
  constexpr int SLOT = 2 * TB + RB;
  static_assert(KC == R::KC && KC <= 4 && VC <= 4, "raw tiles of d <= 64");
  const int w = wave_uniform(threadIdx.x / kWave);
  const int lane = lane_id();
  const long long bh = gy / nb;
  if constexpr (COARSE) {
    if (!OWN && w == 0) {
      prefetch_vec_lds<D>(dkp + gy * D, (lptr_t)addl);
      prefetch_vec_lds<D>(dvp + gy * D, (lptr_t)(addl + add_lds_floats(D)));
    }
  }
  const int y = (int)(gy - bh * nb);
  const long long hb = bh * nb;
  const int nbw = (nb + 31) / 32;

  // the block's operands are requested before its list, whose wait covers them
  u32x4 kf[KC], vf[KC];
  load_rows<BF16, D>(reinterpret_cast<const elem*>(kin) + gy * 32 * D, kf);
  load_rows<BF16, D>(reinterpret_cast<const elem*>(vin) + gy * 32 * D, vf);
  // block-rows whose selection holds y, ascending
  int32_t* myx = lists + w * nb;
  int cnt = column_list(bits, hb, nbw, y, nb, myx);
  if constexpr (SPLIT > 1) {
    myx += w;
    cnt = (cnt - w + SPLIT - 1) / SPLIT;
  }
  if constexpr (OWN) {                                      // the first and the last wave, one quantity each
    if (w == 0) own_term<D>(T.dS, T.qp, hb, y, nb, scale, addl);
    if (w == SPLIT - 1) own_term<D>(T.W, T.gh, hb, y, nb, 1.0f, addl + add_lds_floats(D));
  }
  wait_loads<0>();
  f32x16 ak[NT], av[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) ak[t][r] = av[t][r] = 0.0f;
  // B operands of the bias steps: lane l holds B[k = 8 (l/32) + e][l % 32]
  const bool lo_half = lane < 32;
  const u32x4 ones_l = lo_half ? u32x4{0x3F803F80u, 0x00003F80u, 0u, 0u} : u32x4{0u, 0u, 0u, 0u};
  const u32x4 ones_d = lo_half ? u32x4{0u, 0x3F800000u, 0x3F803F80u, 0u} : u32x4{0u, 0u, 0u, 0u};

  R ro;
  ro.init();
  const i32x4 qrs = buffer_rsrc(static_cast<const char*>(qin) + (size_t)hb * TB, (unsigned)nb * TB);
  const i32x4 grs = buffer_rsrc(static_cast<const char*>(gin) + (size_t)hb * TB, (unsigned)nb * TB);
  const i32x4 brs = buffer_rsrc(reinterpret_cast<const char*>(bias) + (size_t)hb * RB, (unsigned)nb * RB);
  const uint32_t base = lds_addr(slots + w * SLOT);
  const uint32_t boff = (uint32_t)(2 * TB) + 16u * (lane & 31);   // this lane's query's bias operand
  auto issue = [&](int x) {
    const lptr_t dst = (lptr_t)(slots + w * SLOT);
    copy_raw_pair_buf<KC, R::KP>(qrs, grs, (unsigned)x * TB, (unsigned)x * TB, ro.cp, dst, dst + TB);
    mra_raw_buffer_load_lds(brs, dst + 2 * TB, 4, lane * 4, x * RB, 0, 0);
    mra_raw_buffer_load_lds(brs, dst + 2 * TB + 256, 4, lane * 4, x * RB + 256, 0, 0);
  };
  if (cnt > 0) issue(list_entry(myx));
  for (int i = 0; i < cnt; ++i) {
    const int xn = i + 1 < cnt ? list_entry(myx + SPLIT * (i + 1)) : 0;
    wait_loads<0>();                                        // tile i landed
    u32x4 qa[KC], ga[KC], qt[VC], gtc[VC], ba[1];
    raw_rows<0>(base, ro.rr, qa);
    raw_rows<TB>(base, ro.rr, ga);
    RawTrB<D, 0, 0, VC>::run(base, ro.tr, qt);
    RawTrB<D, TB, 0, VC>::run(base, ro.tr, gtc);
    ba[0] = lds_read16<0>(base + boff);
    lds_done(qa);
    lds_done(ga);
    lds_done(qt);
    lds_done(gtc);
    lds_done(ba);
    if (i + 1 < cnt) issue(xn);
    const f32x16 s = mfma_abt_from<KC>(qa, kf, ba[0], ones_l);   // lane: key, 16 queries
    const f32x16 pv = mfma_abt_from<KC>(ga, vf, ba[0], ones_d);
    float a[16], ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      a[r] = __builtin_amdgcn_exp2f(s[r] * scale_log2);
      ds[r] = a[r] * pv[r];
    }
    uint32_t pa8[8], pd8[8];
    pack16(a, pa8);
    pack16(ds, pd8);
    mfma_acc_bf16<NT>(av, pa8, [&](int c) { return gtc[c]; });
    mfma_acc_bf16<NT>(ak, pd8, [&](int c) { return qt[c]; });
  }
  wait_loads<0>();
  if constexpr (SPLIT > 1) {
    auto slot = [&](int p) { return slots + p * SLOT; };
    add_parts<SPLIT>(ak, w, slot);
    __syncthreads();                                        // wave 0 has read them
    add_parts<SPLIT>(av, w, slot);
    if (w != 0) return;
  }
  store_block<BF16, D>(reinterpret_cast<elem*>(dk) + gy * 32 * D, ak, scale, COARSE ? addl : nullptr);
  store_block<BF16, D>(reinterpret_cast<elem*>(dv) + gy * 32 * D, av, 1.0f, COARSE ? addl + add_lds_floats(D) : nullptr);
}

template <int D, bool COARSE>
__global__ __launch_bounds__(kWave) void bwd_dkdv_tr_kernel(
    const void* __restrict__ kin, const void* __restrict__ vin, const void* __restrict__ qin,
    const void* __restrict__ gin, const uint32_t* __restrict__ bits,
    const uint32_t* __restrict__ bias, const float* __restrict__ dkp, const float* __restrict__ dvp,
    void* __restrict__ dk, void* __restrict__ dv, int nb, float scale, float scale_log2) {
  __shared__ __attribute__((aligned(16))) unsigned char slots[2 * RawB<D>::TB + 32 * 16];
  __shared__ __attribute__((aligned(16))) float addl[COARSE ? 2 * add_lds_floats(D) : 1];
  extern __shared__ int32_t sidx_all[];
  dkdv_tr_body<D, COARSE, 1, false>(xcd_remap(blockIdx.x, gridDim.x), slots, addl, sidx_all, ColTerms{}, kin, vin, qin,
                                    gin, bits, bias, dkp, dvp, dk, dv, nb, scale, scale_log2);
}

// Both passes of a call with few rows in one launch (they are independent, and
// each alone leaves most of the chip idle): workgroups 0 .. rows - 1 the column
// blocks, whose lists can be the longer ones, then the block-rows. Training step
// (GPU time, before -> after; up to 32 blocks per head without the column pass):
// 12 heads x 512 x 64: 39.0 -> 32.7 us, 48 heads: 47.7 -> 43.0, 12 heads x 2048:
// 62.5 -> 58.4; float32 12 heads x 512 x 64: 77.6 -> 64.3, 4 heads x 2048 x 128:
// 128 -> 110.
template <int D, bool COARSE, int SPLIT, bool OWN>
__global__ __launch_bounds__(SPLIT * kWave) void bwd_tiles_tr_kernel(
    ColTerms T, const void* __restrict__ qin, const void* __restrict__ gin, const void* __restrict__ kin,
    const void* __restrict__ vin, const int32_t* __restrict__ idx, const uint32_t* __restrict__ bits,
    const float* __restrict__ ld, const uint32_t* __restrict__ bias, const float* __restrict__ dqp,
    const float* __restrict__ dkp, const float* __restrict__ dvp, void* __restrict__ dq, void* __restrict__ dk,
    void* __restrict__ dv, int nb, int m, int rows, float scale, float scale_log2) {
  __shared__ __attribute__((aligned(16))) unsigned char slots[SPLIT * (2 * RawB<D>::TB + 32 * 16)];
  __shared__ __attribute__((aligned(16))) float addl[COARSE ? SPLIT * add_lds_floats(D) : 1];
  extern __shared__ int32_t sidx_all[];
  const int b = blockIdx.x;
  if (b < rows)
    dkdv_tr_body<D, COARSE, SPLIT, OWN>(xcd_remap(b, rows), slots, addl, sidx_all, T, kin, vin, qin, gin, bits, bias,
                                        dkp, dvp, dk, dv, nb, scale, scale_log2);
  else
    dq_tr_body<D, COARSE, SPLIT, SPLIT>(xcd_remap(b - rows, rows), slots, addl, sidx_all, qin, gin, kin, vin, idx, ld,
                                        dqp, dq, nb, m, rows, scale, scale_log2);
}

// bfloat16, d = 128: raw 8 KB tiles of 32 rows x 256 bytes under the same
// kind of swizzle (block b of row r at b ^ (4 (r mod 4) + (r / 4 mod 4)):
// sixteen consecutive rows take sixteen positions for the row reads, four
// consecutive rows four groups of four for the transposed reads; copy offsets
// of period 4). A tile's operands are too many registers at this width to be
// read at once, so each is read just before its products: the row chunks of
// one tile, then of the other, then the transposed chunks.

// dQ (bf16, d = 128): one wave per block-row, one slot per wave (K_y and V_y);
// the next tile is copied once the current one has been read.
template <bool COARSE, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void bwd_dq_tr128_kernel(
    const void* __restrict__ qin, const void* __restrict__ gin, const void* __restrict__ kin,
    const void* __restrict__ vin, const int32_t* __restrict__ idx,
    const float* __restrict__ ld, const float* __restrict__ dqp, void* __restrict__ dq, int nb,
    int m, long long row0, long long rows, int in_step, float scale, float scale_log2) {
  constexpr int D = 128;
  using Cfg = TileCfg<BF16, D>;
  using elem = typename Cfg::elem;
  using R = RawB<D>;
  constexpr int KC = Cfg::kKChunks, VC = Cfg::kVChunks, NT = Cfg::kNT;
  constexpr int TB = R::TB;
  static_assert(KC == R::KC && VC == KC, "row and transposed chunks of a tile");
  __shared__ __attribute__((aligned(16))) unsigned char slots[WAVES][2 * TB];
  __shared__ __attribute__((aligned(16))) float addl[WAVES][COARSE ? D : 1];
  extern __shared__ int32_t sidx_all[];
  const int w = wave_uniform(threadIdx.x / kWave);
  const int lane = lane_id(), jq = lane & 31;
  const long long g = row0 + xcd_remap(blockIdx.x, gridDim.x) * (long long)WAVES + w;
  if (g >= rows) return;                                    // no workgroup barriers below
  const long long bh = g / nb;
  if constexpr (COARSE) prefetch_vec_lds<D>(dqp + g * D, (lptr_t)addl[w]);
  // the row's operands are requested before its list, whose wait covers them
  u32x4 qf[KC], gf[KC];
  load_rows<BF16, D>(reinterpret_cast<const elem*>(qin) + g * 32 * D, qf);
  load_rows<BF16, D>(reinterpret_cast<const elem*>(gin) + g * 32 * D, gf);
  const float lq = ld[g * 64 + jq], dl = ld[g * 64 + 32 + jq];
  int32_t* myidx = sidx_all + w * m;
  const int cnt = stage_selection(idx + g * m, m, nb, myidx);
  wait_loads<0>();
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

  R ro;
  ro.init();
  const i32x4 krs = buffer_rsrc(static_cast<const char*>(kin) + (size_t)bh * nb * TB, (unsigned)nb * TB);
  const i32x4 vrs = buffer_rsrc(static_cast<const char*>(vin) + (size_t)bh * nb * TB, (unsigned)nb * TB);
  const uint32_t base = lds_addr(slots[w]);
  const lptr_t kdst = (lptr_t)slots[w], vdst = kdst + TB;
  // the slot's halves are refilled separately: V_y's as soon as its rows are
  // read (they are read first), K_y's once its rows and K_y^T are read
  if (cnt > 0) {
    const int y = list_entry(myidx);
    copy_raw_buf<KC, R::KP>(vrs, (unsigned)y * TB, ro.cp, vdst);
    copy_raw_buf<KC, R::KP>(krs, (unsigned)y * TB, ro.cp, kdst);
  }
  for (int i = 0; i < cnt; ++i) {
    wait_loads<KC>();                                       // V_y landed (K_y may be in flight)
    const int yn = i + 1 < cnt ? list_entry(myidx + i + 1) : 0;
    u32x4 op[KC];
    raw_rows<TB>(base, ro.rr, op);                          // V_y rows
    lds_done(op);
    if (i + 1 < cnt) {
      copy_raw_buf<KC, R::KP>(vrs, (unsigned)yn * TB, ro.cp, vdst);
      wait_loads<KC>();                                     // K_y landed
    } else {
      wait_loads<0>();
    }
    const f32x16 pv = mfma_abt<KC>(op, gf);
    raw_rows<0>(base, ro.rr, op);                           // K_y rows
    lds_done(op);
    const f32x16 s = mfma_abt<KC>(op, qf);
    RawTrB<D, 0, 0, VC>::run(base, ro.tr, op);             // K_y^T
    lds_done(op);
    if (i + 1 < cnt) copy_raw_buf<KC, R::KP>(krs, (unsigned)yn * TB, ro.cp, kdst);
    if (in_step) wait_loads<0>();
    float ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      ds[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2, -lq)) * (pv[r] - dl);
    uint32_t pk[8];
    pack16(ds, pk);
    mfma_acc_bf16<NT>(acc, pk, [&](int c) { return op[c]; });
  }
  wait_loads<0>();
  store_block<BF16, D>(reinterpret_cast<elem*>(dq) + g * 32 * D, acc, scale, COARSE ? addl[w] : nullptr);
}

// dK, dV (bf16, d = 128): one wave per column block, two slots (raw Q_x, G_x
// and the block-row's bias operands), the per-query terms entering the
// products as in bwd_dkdv_tr_kernel.
template <bool COARSE>
__global__ __launch_bounds__(kWave) void bwd_dkdv_tr128_kernel(
    const void* __restrict__ kin, const void* __restrict__ vin, const void* __restrict__ qin,
    const void* __restrict__ gin, const uint32_t* __restrict__ bits, const uint32_t* __restrict__ order,
    const uint32_t* __restrict__ bias, const float* __restrict__ dkp, const float* __restrict__ dvp,
    void* __restrict__ dk, void* __restrict__ dv, int nb, long long rows, float scale,
    float scale_log2) {
  constexpr int D = 128;
  using Cfg = TileCfg<BF16, D>;
  using elem = typename Cfg::elem;
  using R = RawB<D>;
  constexpr int KC = Cfg::kKChunks, VC = Cfg::kVChunks, NT = Cfg::kNT;
  constexpr int TB = R::TB, RB = 32 * 16;
  constexpr int N = 2 * KC + 2;                             // loads per tile
  constexpr int SLOT = 2 * TB + RB;
  static_assert(KC == R::KC && VC == KC, "row and transposed chunks of a tile");
  __shared__ __attribute__((aligned(16))) unsigned char slots[2][SLOT];
  __shared__ __attribute__((aligned(16))) float addl[2][COARSE ? D : 1];
  extern __shared__ int32_t sidx_all[];
  const int lane = lane_id();
  long long gy = xcd_remap(blockIdx.x, gridDim.x);
  if (gy >= rows) return;
  if (order != nullptr) gy = wave_uniform((int)order[gy]);
  const long long bh = gy / nb;
  if constexpr (COARSE) {
    prefetch_vec_lds<D>(dkp + gy * D, (lptr_t)addl[0]);
    prefetch_vec_lds<D>(dvp + gy * D, (lptr_t)addl[1]);
  }
  const int y = (int)(gy - bh * nb);
  const long long hb = bh * nb;
  const int nbw = (nb + 31) / 32;

  // the block's operands are requested before its list, whose wait covers them
  u32x4 kf[KC], vf[KC];
  load_rows<BF16, D>(reinterpret_cast<const elem*>(kin) + gy * 32 * D, kf);
  load_rows<BF16, D>(reinterpret_cast<const elem*>(vin) + gy * 32 * D, vf);
  // block-rows whose selection holds y, ascending
  int32_t* myx = sidx_all;
  const int cnt = column_list(bits, hb, nbw, y, nb, myx);
  wait_loads<0>();
  f32x16 ak[NT], av[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) ak[t][r] = av[t][r] = 0.0f;
  const bool lo_half = lane < 32;
  const u32x4 ones_l = lo_half ? u32x4{0x3F803F80u, 0x00003F80u, 0u, 0u} : u32x4{0u, 0u, 0u, 0u};
  const u32x4 ones_d = lo_half ? u32x4{0u, 0x3F800000u, 0x3F803F80u, 0u} : u32x4{0u, 0u, 0u, 0u};

  R ro;
  ro.init();
  const i32x4 qrs = buffer_rsrc(static_cast<const char*>(qin) + (size_t)hb * TB, (unsigned)nb * TB);
  const i32x4 grs = buffer_rsrc(static_cast<const char*>(gin) + (size_t)hb * TB, (unsigned)nb * TB);
  const i32x4 brs = buffer_rsrc(reinterpret_cast<const char*>(bias) + (size_t)hb * RB, (unsigned)nb * RB);
  const uint32_t a0 = lds_addr(slots[0]);
  const uint32_t boff = (uint32_t)(2 * TB) + 16u * (lane & 31);
  auto issue = [&](int x, int sl) {
    const lptr_t dst = (lptr_t)slots[sl];
    copy_raw_pair_buf<KC, R::KP>(qrs, grs, (unsigned)x * TB, (unsigned)x * TB, ro.cp, dst, dst + TB);
    mra_raw_buffer_load_lds(brs, dst + 2 * TB, 4, lane * 4, x * RB, 0, 0);
    mra_raw_buffer_load_lds(brs, dst + 2 * TB + 256, 4, lane * 4, x * RB + 256, 0, 0);
  };
  if (cnt > 0) issue(list_entry(myx), 0);
  if (cnt > 1) issue(list_entry(myx + 1), 1);
  for (int i = 0; i < cnt; ++i) {
    if (i + 1 < cnt) wait_loads<N>();                       // tile i landed, i+1 may not have
    else wait_loads<0>();
    const uint32_t base = a0 + (uint32_t)((i & 1) * SLOT);
    u32x4 op[KC], ba[1];
    ba[0] = lds_read16<0>(base + boff);
    raw_rows<0>(base, ro.rr, op);                           // Q_x rows
    lds_done(ba);
    lds_done(op);
    const f32x16 s = mfma_abt_from<KC>(op, kf, ba[0], ones_l);   // lane: key, 16 queries
    raw_rows<TB>(base, ro.rr, op);                          // G_x rows
    lds_done(op);
    const f32x16 pv = mfma_abt_from<KC>(op, vf, ba[0], ones_d);
    float a[16], ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      a[r] = __builtin_amdgcn_exp2f(s[r] * scale_log2);
      ds[r] = a[r] * pv[r];
    }
    uint32_t pa8[8], pd8[8];
    pack16(a, pa8);
    pack16(ds, pd8);
    RawTrB<D, 0, 0, VC>::run(base, ro.tr, op);             // Q_x^T
    lds_done(op);
    mfma_acc_bf16<NT>(ak, pd8, [&](int c) { return op[c]; });
    RawTrB<D, TB, 0, VC>::run(base, ro.tr, op);            // G_x^T
    lds_done(op);
    if (i + 2 < cnt) issue(list_entry(myx + i + 2), i & 1);   // the slot has been read
    mfma_acc_bf16<NT>(av, pa8, [&](int c) { return op[c]; });
  }
  wait_loads<0>();
  store_block<BF16, D>(reinterpret_cast<elem*>(dk) + gy * 32 * D, ak, scale, COARSE ? addl[0] : nullptr);
  store_block<BF16, D>(reinterpret_cast<elem*>(dv) + gy * 32 * D, av, 1.0f, COARSE ? addl[1] : nullptr);
}

// ---------------------------------------------------------------------------
// float32 (on the bfloat16 matrix cores, tile_ops.h). split_kernel writes
// Q, K, V and dZ as planes: per 32-row block the hi, mid and lo tiles one after
// the other, each a raw bfloat16 tile of the layout above, so a wave reads its
// operands as planes and splits only the 16 values it computes per tile.
// The float32 matrix instructions bounded these passes and their operands in
// registers left one wave per SIMD at d = 128. Measured before -> after, the
// copies in operand order and the planes included: 32 heads x 4096 x 32, budget 8 (small-4096): dQ 81 -> 47, dK/dV
// 136 -> 70, copies / planes 29 -> 26 us; 32 heads x 1504 x 128, budget 8: dQ 197 -> 85,
// dK/dV 473 -> 117, copies / planes 33 -> 37 us.
//
// Both passes give a block-row or column block to a pair of waves that walk
// its tiles together, each wave holding one fixed operand. The tile's planes
// are copied into one LDS slot per workgroup (12 KB per 32 dims), half by each
// wave; two barriers per tile: A, behind which both halves and the exchanged
// values are there, and B, behind which the slot has been read and is refilled
// while the second products run.

// C = A B^T over the planes of one raw tile at `base` (A, read from LDS plane
// by plane, the smallest products first) and the fixed operand f.
template <int D, int KC>
__device__ __forceinline__ f32x16 mfma3_abt(uint32_t base, const uint32_t (&rr)[KC], const u32x4 (&f)[3][KC]) {
  constexpr int TB = RawB<D>::TB;
  f32x16 c;
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] = 0.0f;
  u32x4 a[KC];
  auto step = [&](const u32x4 (&b)[KC]) {
#pragma unroll
    for (int k = 0; k < KC; ++k)
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[k]), __builtin_bit_cast(bf16x8, b[k]), c, 0, 0, 0);
  };
  raw_rows<2 * TB>(base, rr, a);
  lds_done(a);
  step(f[0]);
  raw_rows<TB>(base, rr, a);
  lds_done(a);
  step(f[1]);
  step(f[0]);
  raw_rows<0>(base, rr, a);
  lds_done(a);
  step(f[2]);
  step(f[1]);
  step(f[0]);
  return c;
}

// The planes of block-row g's 32 rows in the row layout.
template <int D, int KC>
__device__ __forceinline__ void load_planes(const void* planes, long long g, u32x4 (&f)[3][KC]) {
  using elem = typename TileCfg<BF16, D>::elem;
#pragma unroll
  for (int q = 0; q < 3; ++q) load_rows<BF16, D>(reinterpret_cast<const elem*>(planes) + (g * 3 + q) * 32 * D, f[q]);
}

// One tile's planes (3 KC copies of 1 KB) HBM/L2 -> LDS.
template <int D>
__device__ __forceinline__ void copy_planes(i32x4 rs, int block, const RawB<D>& ro, lptr_t dst) {
  constexpr int TB = RawB<D>::TB;
#pragma unroll
  for (int q = 0; q < 3; ++q)
    copy_raw_buf<D / 16, RawB<D>::KP>(rs, (unsigned)block * (3 * TB) + q * TB, ro.cp, dst + q * TB);
}

// This wave's LDS accesses complete, then the workgroup's barrier.
__device__ __forceinline__ void pair_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// dQ (float32): a pair of waves per block-row x. Wave 0 forms S = K_y Q_x^T
// and the weights, wave 1 V_y G_x^T - delta; each then takes half of the
// keys: they exchange the other half's values (8 per lane), form
// dP and add K_y^T dP over their 16 keys to a full 32 x d accumulator. The two
// accumulators are added at the end.
// A workgroup's LDS in the float32 passes: REC block-row records, ADD vectors of
// coarse-term gradients (the dQ pass needs no record and one vector: at d = 128
// that leaves room for a third workgroup per CU).
template <int D, int REC, int ADD>
struct SplitLds {
  __attribute__((aligned(16))) unsigned char slot[2][3 * RawB<D>::TB];
  __attribute__((aligned(16))) float ex[16 * kWave];
  __attribute__((aligned(16))) float rec[REC ? REC : 1][REC ? 64 : 4];
  __attribute__((aligned(16))) float addl[ADD][add_lds_floats(D)];
};

template <int D, bool COARSE, class Lds>
__device__ __forceinline__ void dq_split_body(
    long long g, Lds& S, uint16_t* list_all,
    const void* __restrict__ qpl, const void* __restrict__ gpl, const void* __restrict__ kpl,
    const void* __restrict__ vpl, const int32_t* __restrict__ idx, const float* __restrict__ ld,
    const float* __restrict__ dqp, float* __restrict__ dq, int nb, int m, float scale, float scale_log2) {
  using R = RawB<D>;
  constexpr int KC = R::KC, NT = R::NT, TB = R::TB;
  auto& slot = S.slot;
  float* const ex[2] = {S.ex, S.ex + 8 * kWave};
  float* addl = S.addl[0];
  const int w = wave_uniform(threadIdx.x / kWave);
  const int lane = lane_id(), jq = lane & 31;
  const long long bh = g / nb;
  if constexpr (COARSE)
    if (w == 0) prefetch_vec_lds<D>(dqp + g * D, (lptr_t)addl);
  // the row's operands are requested before its list, whose wait covers them
  const float own = ld[g * 64 + 32 * w + jq];               // log normaliser (log2 units) or delta
  u32x4 fx[3][KC];                                          // Q_x or G_x
  load_planes<D>(w ? gpl : qpl, g, fx);
  uint16_t* myidx = list_all + w * m;
  const int cnt = stage_selection(idx + g * m, m, nb, myidx);
  wait_loads<0>();
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

  R ro;
  ro.init();
  const i32x4 trs = buffer_rsrc(static_cast<const char*>(w ? vpl : kpl) + (size_t)bh * nb * 3 * TB, (unsigned)nb * 3 * TB);
  const lptr_t dst = (lptr_t)slot[w];
  const uint32_t base = lds_addr(slot[w]);                  // the tile this wave copies
  const uint32_t ktr = lds_addr(slot[0]) + (uint32_t)(16 * w * 2 * D);   // this wave's 16 keys of K_y
  if (cnt > 0) copy_planes<D>(trs, list_entry(myidx), ro, dst);
  for (int i = 0; i < cnt; ++i) {
    const int yn = i + 1 < cnt ? list_entry(myidx + i + 1) : 0;
    wait_loads<0>();                                        // own half of tile i landed
    const f32x16 x = mfma3_abt<D>(base, ro.rr, fx);         // lane: query, 16 keys
    float a[16];
    if (w == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) a[r] = __builtin_amdgcn_exp2f(fmaf(x[r], scale_log2, -own));
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) a[r] = x[r] - own;
    }
    // registers 8u .. 8u + 7: the keys of half u; wave 0 sends half 1, wave 1 half 0
    float mine[8];
    {
      f32x4* o = reinterpret_cast<f32x4*>(ex[w]) + lane;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = w == 0 ? a[8 + 4 * q + e] : a[4 * q + e];
          mine[4 * q + e] = w == 0 ? a[4 * q + e] : a[8 + 4 * q + e];
        }
        o[64 * q] = v;
      }
    }
    pair_barrier();                                         // A
    {
      const f32x4* o = reinterpret_cast<const f32x4*>(ex[1 - w]) + lane;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4 v = o[64 * q];
#pragma unroll
        for (int e = 0; e < 4; ++e) mine[4 * q + e] *= v[e];
      }
    }
    u32x4 tr[3][NT];
    RawTrB<D, 2 * TB, 0, NT>::run(ktr, ro.tr, tr[2]);
    RawTrB<D, TB, 0, NT>::run(ktr, ro.tr, tr[1]);
    RawTrB<D, 0, 0, NT>::run(ktr, ro.tr, tr[0]);
    lds_done(tr[2]);
    lds_done(tr[1]);
    lds_done(tr[0]);
    pair_barrier();                                         // B
    if (i + 1 < cnt) copy_planes<D>(trs, yn, ro, dst);
    u32x4 pk[3];
    split8(mine, pk);
#pragma unroll
    for (int s = 2; s >= 0; --s)                            // p + q = s, the smallest products first
#pragma unroll
      for (int p = 0; p <= s; ++p)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, tr[p][t]),
                                                           __builtin_bit_cast(bf16x8, pk[s - p]), acc[t], 0, 0, 0);
  }
  wait_loads<0>();
  // wave 1's sums through the slot (32 d floats; every tile has been read)
  f32x4* part = reinterpret_cast<f32x4*>(slot) + lane;
  if (w != 0) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        part[(4 * t + q) * 64] = f32x4{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
  }
  pair_barrier();
  if (w != 0) return;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = part[(4 * t + q) * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][4 * q + e] += v[e];
    }
  store_block<F32, D>(dq + g * 32 * D, acc, scale, COARSE ? addl : nullptr);
}

// dK, dV (float32): a pair of waves per column block y. Wave 0 forms
// S = Q_x K_y^T, the weights A and dV^T += G_x^T A; wave 1 forms G_x V_y^T,
// takes the weights from wave 0 and adds dK^T += Q_x^T dP.
template <int D, bool COARSE, bool OWN, class Lds>
__device__ __forceinline__ void dkdv_split_body(
    long long gy, Lds& S, uint16_t* list_all, const ColTerms& T,
    const void* __restrict__ kpl, const void* __restrict__ vpl, const void* __restrict__ qpl,
    const void* __restrict__ gpl, const uint32_t* __restrict__ bits, const float* __restrict__ ld,
    const float* __restrict__ dkp, const float* __restrict__ dvp, float* __restrict__ dk,
    float* __restrict__ dv, int nb, float scale, float scale_log2) {
  using R = RawB<D>;
  constexpr int KC = R::KC, NT = R::NT, TB = R::TB, VC = 2 * NT;
  auto& slot = S.slot;
  auto& ex = S.ex;
  auto& rec = S.rec;
  auto& addl = S.addl;
  const int w = wave_uniform(threadIdx.x / kWave);
  const int lane = lane_id(), h = lane >> 5;
  const long long bh = gy / nb, hb = bh * nb;
  const int y = (int)(gy - hb);
  if constexpr (COARSE && !OWN) prefetch_vec_lds<D>((w ? dkp : dvp) + gy * D, (lptr_t)addl[w]);
  u32x4 fx[3][KC];                                          // K_y or V_y, requested before the list
  load_planes<D>(w ? vpl : kpl, gy, fx);
  // block-rows whose selection holds y, ascending (each wave keeps its own list)
  uint16_t* myx = list_all + w * nb;
  const int cnt = column_list(bits, hb, (nb + 31) / 32, y, nb, myx);
  if constexpr (OWN) own_term<D>(w ? T.dS : T.W, w ? T.qp : T.gh, hb, y, nb, w ? scale : 1.0f, addl[w]);
  wait_loads<0>();
  f32x16 acc[NT];                                           // dV^T or dK^T
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

  R ro;
  ro.init();
  const i32x4 trs = buffer_rsrc(static_cast<const char*>(w ? gpl : qpl) + (size_t)hb * 3 * TB, (unsigned)nb * 3 * TB);
  const i32x4 xrs = buffer_rsrc(ld + hb * 64, (unsigned)nb * 256u);
  const lptr_t dst = (lptr_t)slot[w], xdst = (lptr_t)rec[w];
  const uint32_t base = lds_addr(slot[w]), other = lds_addr(slot[1 - w]);
  const uint32_t ra = lds_addr(rec[w]) + 128u * w + 16u * h;   // this half's queries: L (wave 0) or delta
  auto issue = [&](int x) {
    copy_planes<D>(trs, x, ro, dst);
    mra_raw_buffer_load_lds(xrs, xdst, 4, lane * 4, x * 256, 0, 0);   // the block-row's record
  };
  if (cnt > 0) issue(list_entry(myx));
  for (int i = 0; i < cnt; ++i) {
    const int xn = i + 1 < cnt ? list_entry(myx + i + 1) : 0;
    wait_loads<0>();                                        // own half of tile i landed
    u32x4 own[4];                                           // queries 8q + 4h + e
    own[0] = lds_read16<0>(ra);
    own[1] = lds_read16<32>(ra);
    own[2] = lds_read16<64>(ra);
    own[3] = lds_read16<96>(ra);
    lds_done(own);
    const f32x16 x = mfma3_abt<D>(base, ro.rr, fx);         // lane: key, 16 queries
    float a[16];
    f32x4* o = reinterpret_cast<f32x4*>(ex) + lane;
    if (w == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) a[r] = __builtin_amdgcn_exp2f(fmaf(x[r], scale_log2, -__uint_as_float(own[r / 4][r % 4])));
#pragma unroll
      for (int q = 0; q < 4; ++q) o[64 * q] = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) a[r] = x[r] - __uint_as_float(own[r / 4][r % 4]);
    }
    pair_barrier();                                         // A
    if (w != 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = o[64 * q];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * q + e] *= v[e];
      }
    }
    u32x4 tr[3][VC];
    RawTrB<D, 2 * TB, 0, VC>::run(other, ro.tr, tr[2]);
    RawTrB<D, TB, 0, VC>::run(other, ro.tr, tr[1]);
    RawTrB<D, 0, 0, VC>::run(other, ro.tr, tr[0]);
    lds_done(tr[2]);
    lds_done(tr[1]);
    lds_done(tr[0]);
    pair_barrier();                                         // B
    if (i + 1 < cnt) issue(xn);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float half[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) half[e] = a[8 * u + e];
      u32x4 pk[3];
      split8(half, pk);
#pragma unroll
      for (int s = 2; s >= 0; --s)
#pragma unroll
        for (int p = 0; p <= s; ++p)
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, tr[p][u * NT + t]),
                                                             __builtin_bit_cast(bf16x8, pk[s - p]), acc[t], 0, 0, 0);
    }
  }
  wait_loads<0>();
  store_block<F32, D>((w ? dk : dv) + gy * 32 * D, acc, w ? scale : 1.0f, COARSE ? addl[w] : nullptr);
}

template <int D, bool COARSE>
__global__ __launch_bounds__(2 * kWave) void bwd_dq_split_kernel(
    const void* __restrict__ qpl, const void* __restrict__ gpl, const void* __restrict__ kpl,
    const void* __restrict__ vpl, const int32_t* __restrict__ idx, const float* __restrict__ ld,
    const float* __restrict__ dqp, float* __restrict__ dq, int nb, int m, float scale, float scale_log2) {
  __shared__ SplitLds<D, 0, 1> S;
  extern __shared__ uint16_t list_all[];                    // [2][m]
  dq_split_body<D, COARSE>(xcd_remap(blockIdx.x, gridDim.x), S, list_all, qpl, gpl, kpl, vpl, idx, ld, dqp, dq, nb, m,
                           scale, scale_log2);
}

template <int D, bool COARSE>
__global__ __launch_bounds__(2 * kWave) void bwd_dkdv_split_kernel(
    const void* __restrict__ kpl, const void* __restrict__ vpl, const void* __restrict__ qpl,
    const void* __restrict__ gpl, const uint32_t* __restrict__ bits, const uint32_t* __restrict__ order, const float* __restrict__ ld,
    const float* __restrict__ dkp, const float* __restrict__ dvp, float* __restrict__ dk,
    float* __restrict__ dv, int nb, float scale, float scale_log2) {
  __shared__ SplitLds<D, 2, 2> S;
  extern __shared__ uint16_t list_all[];                    // [2][nb]
  long long gy = xcd_remap(blockIdx.x, gridDim.x);
  if (order != nullptr) gy = wave_uniform((int)order[gy]);
  dkdv_split_body<D, COARSE, false>(gy, S, list_all, ColTerms{}, kpl, vpl, qpl, gpl, bits,
                                    ld, dkp, dvp, dk, dv, nb, scale, scale_log2);
}

// Both in one launch (as bwd_tiles_tr_kernel).
template <int D, bool COARSE, bool OWN>
__global__ __launch_bounds__(2 * kWave) void bwd_tiles_split_kernel(
    ColTerms T, const void* __restrict__ qpl, const void* __restrict__ gpl, const void* __restrict__ kpl,
    const void* __restrict__ vpl, const int32_t* __restrict__ idx, const uint32_t* __restrict__ bits,
    const float* __restrict__ ld, const float* __restrict__ dqp, const float* __restrict__ dkp,
    const float* __restrict__ dvp, float* __restrict__ dq, float* __restrict__ dk, float* __restrict__ dv, int nb, int m,
    int rows, float scale, float scale_log2) {
  __shared__ SplitLds<D, 2, 2> S;
  extern __shared__ uint16_t list_all[];
  const int b = blockIdx.x;
  if (b < rows)
    dkdv_split_body<D, COARSE, OWN>(xcd_remap(b, rows), S, list_all, T, kpl, vpl, qpl, gpl, bits, ld, dkp, dvp, dk, dv,
                                    nb, scale, scale_log2);
  else
    dq_split_body<D, COARSE>(xcd_remap(b - rows, rows), S, list_all, qpl, gpl, kpl, vpl, idx, ld, dqp, dq, nb, m, scale,
                             scale_log2);
}

// Column blocks in the order of falling list length, within each of the launch's
// equal ranges of them (order: rows entries): first the lengths, one workgroup per head and 32 columns, a lane per
// block-row and one ballot per column.
constexpr int kOrderWaves = 4;
__global__ __launch_bounds__(kOrderWaves * kWave) void bwd_lengths_kernel(const uint32_t* __restrict__ bits,
                                                                          uint16_t* __restrict__ len, int nb) {
  __shared__ int part[kOrderWaves][32];
  const int nbw = (nb + 31) / 32, lane = lane_id(), w = wave_uniform(threadIdx.x / kWave);
  const long long bh = blockIdx.x / nbw, hb = bh * nb;
  const int wd = (int)(blockIdx.x - bh * nbw);
  int mine = 0;                                             // lane c: column 32 wd + c
  for (int x0 = w * kWave; x0 < nb; x0 += kOrderWaves * kWave) {
    const int x = x0 + lane;
    const uint32_t v = x < nb ? bits[(hb + x) * nbw + wd] : 0u;
#pragma unroll
    for (int c = 0; c < 32; ++c) {
      const int n = __popcll(__ballot((v >> c) & 1u));
      if (lane == c) mine += n;
    }
  }
  if (lane < 32) part[w][lane] = mine;
  __syncthreads();
  const int y = 32 * wd + threadIdx.x;
  if (threadIdx.x < 32 && y < nb) {
    int n = 0;
#pragma unroll
    for (int q = 0; q < kOrderWaves; ++q) n += part[q][threadIdx.x];
    len[hb + y] = (uint16_t)n;
  }
}

// then a counting sort, one workgroup per range. Blocks of equal length come in
// any order: it decides only where and when a block is worked on.
constexpr int kOrderThreads = 1024;
constexpr int kXcds = 8;                  // ranges of xcd_remap
// bfloat16, d = 128: least tiles per row and rounds of resident column blocks to order them
constexpr int kOrderTiles = 16, kOrderRounds = 4;
__global__ __launch_bounds__(kOrderThreads) void bwd_order_kernel(const uint16_t* __restrict__ len,
                                                                  uint32_t* __restrict__ order, int nb, int rows) {
  __shared__ int off[2049];
  const int tid = threadIdx.x, parts = gridDim.x, p = blockIdx.x;
  const int q = rows / parts, r = rows % parts;
  const int i0 = p * q + (p < r ? p : r), i1 = i0 + q + (p < r);
  for (int i = tid; i <= nb; i += kOrderThreads) off[i] = 0;
  __syncthreads();
  for (int i = i0 + tid; i < i1; i += kOrderThreads) atomicAdd(&off[len[i]], 1);
  __syncthreads();
  if (tid < kWave) {                                        // where each length starts, longest first
    int run = i0;
    for (int l0 = nb; l0 >= 0; l0 -= kWave) {
      const int l = l0 - tid;
      const int mine = l >= 0 ? off[l] : 0;
      int incl = mine;
      for (int o = 1; o < kWave; o <<= 1) {
        const int other = __shfl_up(incl, o);
        if (tid >= o) incl += other;
      }
      if (l >= 0) off[l] = run + incl - mine;
      run += __shfl(incl, kWave - 1);
    }
  }
  __syncthreads();
  for (int i = i0 + tid; i < i1; i += kOrderThreads) order[atomicAdd(&off[len[i]], 1)] = (uint32_t)i;
}

// Writes the order of the column blocks within each of `parts` equal ranges of
// them to the grid of W (nothing reads it any more; six bytes per column block,
// so nb > 1) and returns it.
static const uint32_t* launch_order(const BwdArgs& A, int parts, hipStream_t stream) {
  const int nb = A.n / kBlock;
  const long long rows = A.bh * nb;
  uint32_t* order = reinterpret_cast<uint32_t*>(A.W);
  uint16_t* len = reinterpret_cast<uint16_t*>(order + rows);
  bwd_lengths_kernel<<<(unsigned)(A.bh * ((nb + 31) / 32)), kOrderWaves * kWave, 0, stream>>>(A.bits, len, nb);
  bwd_order_kernel<<<parts, kOrderThreads, 0, stream>>>(len, order, nb, (int)rows);
  return order;
}

// ---------------------------------------------------------------------------
// Few rows: dQ and dK/dV share one launch (bfloat16 d = 128 excepted: its two
// kernels fill their CUs' LDS and registers differently).
template <int DT, int D>
static bool tiles_in_one_launch(const BwdArgs& A) {
  const long long rows = A.bh * (A.n / kBlock);
  if (DT == BF16) return D <= 64 && row_split(rows, A.m) > 1;
  return rows <= 4 * kCus;
}

// own: the column blocks form dK~ and dV~ themselves (with tiles_in_one_launch).
template <int DT, int D, bool COARSE>
static void launch_tiles_t(const BwdArgs& A, bool own, hipStream_t stream) {
  const ColTerms T = {A.dS, A.qp, A.W, A.gh};
  const bool one_launch = tiles_in_one_launch<DT, D>(A);
  using Cfg = TileCfg<DT, D>;
  const int nb = A.n / kBlock;
  const long long rows = A.bh * nb;
  const float scale = (float)(1.0 / sqrt((double)D));
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));
  const unsigned wgs = (unsigned)((rows + kBwdTileWaves - 1) / kBwdTileWaves);
  const size_t smem_dq = (size_t)kBwdTileWaves * A.m * sizeof(int32_t);
  constexpr int W = kBwdTileWaves;
  if constexpr (DT == BF16 && Cfg::kKChunks <= 4 && Cfg::kVChunks <= 4) {
    // one column block per workgroup in every column pass: column lists differ in
    // length (a workgroup keeps its resources until its longest list is done),
    // rows all have m tiles
    const int split = row_split(rows, A.m);
    if (split == 1) {
      bwd_dq_tr_kernel<D, COARSE, W><<<wgs, W * kWave, smem_dq, stream>>>(
          A.q, A.dout, A.k, A.v, A.idx, A.ld, A.dqp, A.dq, nb, A.m, rows, scale, scale_log2);
      bwd_dkdv_tr_kernel<D, COARSE><<<(unsigned)rows, kWave, nb * sizeof(int32_t), stream>>>(
          A.k, A.v, A.q, A.dout, A.bits, A.bias, A.dkp, A.dvp, A.dk, A.dv, nb, scale, scale_log2);
    } else {
      const size_t lists = (size_t)split * (nb > A.m ? nb : A.m) * sizeof(int32_t);
#define MRA_TILES(S, OWN) \
  bwd_tiles_tr_kernel<D, COARSE, S, OWN><<<2 * (unsigned)rows, S * kWave, lists, stream>>>( \
      T, A.q, A.dout, A.k, A.v, A.idx, A.bits, A.ld, A.bias, A.dqp, A.dkp, A.dvp, A.dq, A.dk, A.dv, nb, A.m, \
      (int)rows, scale, scale_log2)
      if (split == 4) { if (own) MRA_TILES(4, COARSE); else MRA_TILES(4, false); }
      else { if (own) MRA_TILES(2, COARSE); else MRA_TILES(2, false); }
#undef MRA_TILES
    }
  } else if constexpr (DT == BF16 && D == 128) {
    auto kernel = bwd_dq_tr128_kernel<COARSE, W>;
    // in rounds, where a head's K and V exceed an XCD's L2, with the waves kept
    // in step (as the forward's tile pass): 16 heads of 32768 x 128, budget 32:
    // 655 -> 598 us
    long long chunk = (size_t)4 * A.n * D > kL2PerXcd ? resident_items(kernel, W * kWave, smem_dq, W) : 0;
    if (chunk <= 0) chunk = rows;
    for (long long r0 = 0; r0 < rows; r0 += chunk) {
      const long long r1 = r0 + chunk < rows ? r0 + chunk : rows;
      kernel<<<(unsigned)((r1 - r0 + W - 1) / W), W * kWave, smem_dq, stream>>>(
          A.q, A.dout, A.k, A.v, A.idx, A.ld, A.dqp, A.dq, nb, A.m, r0, r1, chunk < rows, scale, scale_log2);
    }
    // Heads whose Q and dZ tiles exceed an XCD's L2: the column blocks in the
    // order of falling list length. Neighbours then have lists of like length, so
    // the blocks an XCD works on walk the head at the same pace (the pass is bound
    // by bytes from beyond the L2), and its longest lists do not come last. 16
    // heads of 32768 x 128, budget 32 (lists of 2 to 95): training step 2550 ->
    // 2422 us, the two launches included. It takes several rounds of resident
    // blocks and lists that are long against the two launches (backward without ->
    // with, us, budget 16 / 32): 4 x 32768: 374 -> 365 / 526 -> 484, 8 x 16384:
    // 284 -> 270 / 424 -> 392, 16 x 8224: 295 -> 293 / 440 -> 441; budget 8 loses (4
    // x 32768: 285 -> 297), and so do three rounds (12 x 8224, budget 16: 215 ->
    // 231) and fewer: all resident, the launches are all that is added (1 x 8224,
    // budget 16: 94 -> 102). Below d = 128 nothing is gained (12 heads of 32768 x
    // 64: 717 and 716 us). The grid of W serves as scratch: nothing reads it any more.
    auto dkdv = bwd_dkdv_tr128_kernel<COARSE>;
    const size_t lists = nb * sizeof(int32_t);
    const uint32_t* order = nullptr;
    if (A.m >= kOrderTiles && (size_t)4 * A.n * D > kL2PerXcd) {
      const long long resident = resident_items(dkdv, kWave, lists, 1);
      if (resident > 0 && rows >= kOrderRounds * resident) order = launch_order(A, (int)A.bh, stream);
    }
    dkdv<<<(unsigned)rows, kWave, lists, stream>>>(
        A.k, A.v, A.q, A.dout, A.bits, order, A.bias, A.dkp, A.dvp, A.dk, A.dv, nb, rows, scale, scale_log2);
  } else {
    if (!one_launch) {
      bwd_dq_split_kernel<D, COARSE><<<(unsigned)rows, 2 * kWave, 2 * A.m * sizeof(uint16_t), stream>>>(
          A.q_pl, A.g_pl, A.k_pl, A.v_pl, A.idx, A.ld, A.dqp, static_cast<float*>(A.dq), nb, A.m, scale, scale_log2);
      // More column blocks than are resident at once (at d = 128 two workgroups
      // per CU): the order of falling list length over each XCD's range, or the
      // longest lists, which start at any time, end the pass alone. Training step,
      // the two launches included: 32 heads x 1504 x 128, budget 8 (lists of up to
      // 21, three rounds): 337 -> 319 us; 32 x 4096 x 32: 216 -> 207; 12 x 4096 x
      // 64, budget 16: 278 -> 266; 4 x 16384 x 128, budget 32: 1333 -> 1237. With
      // all of them resident it only costs its launches (40 x 1024 x 32: 74 -> 79),
      // and bfloat16 (d <= 64), whose passes wait more on L2, loses by working on
      // all heads of a range at once: 96 x 4096 x 64: 409 -> 429.
      auto dkdv = bwd_dkdv_split_kernel<D, COARSE>;
      const size_t lists = 2 * nb * sizeof(uint16_t);
      const long long resident = resident_items(dkdv, 2 * kWave, lists, 1);
      const uint32_t* order = nb > 1 && resident > 0 && rows > resident ? launch_order(A, kXcds, stream) : nullptr;
      dkdv<<<(unsigned)rows, 2 * kWave, lists, stream>>>(
          A.k_pl, A.v_pl, A.q_pl, A.g_pl, A.bits, order, A.ld, A.dkp, A.dvp, static_cast<float*>(A.dk),
          static_cast<float*>(A.dv), nb, scale, scale_log2);
    } else {
      const size_t lists = (size_t)2 * (nb > A.m ? nb : A.m) * sizeof(uint16_t);
#define MRA_TILES(OWN) \
  bwd_tiles_split_kernel<D, COARSE, OWN><<<2 * (unsigned)rows, 2 * kWave, lists, stream>>>( \
      T, A.q_pl, A.g_pl, A.k_pl, A.v_pl, A.idx, A.bits, A.ld, A.dqp, A.dkp, A.dvp, static_cast<float*>(A.dq), \
      static_cast<float*>(A.dk), static_cast<float*>(A.dv), nb, A.m, (int)rows, scale, scale_log2)
      if (own) MRA_TILES(COARSE); else MRA_TILES(false);
#undef MRA_TILES
    }
  }
}

template <int DT, int D>
static void launch_bwd_t(const BwdArgs& A, hipStream_t stream) {
  const int nb = A.n / kBlock;
  const float scale = (float)(1.0 / sqrt((double)D));
  const long long groups = (nb + kBwdRows - 1) / kBwdRows;
  const unsigned wg_rows = (unsigned)(A.bh * groups);
  if (A.coarse) {
    bwd_rows_kernel<DT, D, true><<<wg_rows, kBwdRows * kWave, 0, stream>>>(
        A.dout, A.out, A.lse, A.idx, A.qp, A.kp, A.vp, A.ld, A.bias, A.bits, A.gh, A.W, A.dS, A.dqp, nb,
        A.m, scale);
    const bool own = nb <= kOwnBlocks && tiles_in_one_launch<DT, D>(A);
    if (!own) {
      const unsigned wg_cols = (unsigned)(A.bh * ((nb + kBwdCols - 1) / kBwdCols));
      bwd_cols_kernel<D><<<wg_cols, ColsCfg<D>::kWaves * kWave, 0, stream>>>(
          A.qp, A.gh, A.W, A.dS, A.dkp, A.dvp, nb, scale);
    }
    launch_tiles_t<DT, D, true>(A, own, stream);
  } else {
    bwd_rows_kernel<DT, D, false><<<wg_rows, kBwdRows * kWave, 0, stream>>>(
        A.dout, A.out, A.lse, A.idx, A.qp, A.kp, A.vp, A.ld, A.bias, A.bits, A.gh, A.W, A.dS, A.dqp, nb,
        A.m, scale);
    launch_tiles_t<DT, D, false>(A, false, stream);
  }
}

hipError_t launch_bwd(const BwdArgs& A, hipStream_t stream) {
  hipError_t e = hipSuccess;
  // the pooled rows of the coarse term, unless given; the bfloat16 tile passes
  // read raw tiles of Q, K, V and G = dZ, the float32 ones their planes
  if (A.coarse && !A.pooled_in)
    e = launch_pool(A.q, A.k, A.v, A.qp, A.kp, A.vp, A.bh, A.n, A.d, A.dtype, stream);
  if (e == hipSuccess && A.dtype == F32)
    e = launch_split(static_cast<const float*>(A.q), static_cast<const float*>(A.k), static_cast<const float*>(A.v),
                     static_cast<const float*>(A.dout), A.q_pl, A.k_pl, A.v_pl, A.g_pl, A.bh, A.n, A.d, stream);
  if (e != hipSuccess) return e;
  if (A.dtype == BF16) {
    if (A.d == 32) launch_bwd_t<BF16, 32>(A, stream);
    else if (A.d == 64) launch_bwd_t<BF16, 64>(A, stream);
    else launch_bwd_t<BF16, 128>(A, stream);
  } else {
    if (A.d == 32) launch_bwd_t<F32, 32>(A, stream);
    else if (A.d == 64) launch_bwd_t<F32, 64>(A, stream);
    else launch_bwd_t<F32, 128>(A, stream);
  }
  return hipGetLastError();
}

}  // namespace mra
