// High-resolution part of MRA-2 and the output (Sec. 4.2 eq.
// actual_approx_mat_form with mu_{1,i,j} = exp(P_ij); Sec. 4.3 Alg. 2 at
// scale 1; Sec. 2.1 row normalisation D^).
//
// One wave owns one block-row x (32 queries). For every selected column block
// y, in ascending order, it computes the 32x32 tile S = c Q_x K_y^T on the
// matrix cores (block-sparse SDDMM), turns it into softmax weights and row sums
// (online softmax), and accumulates P V_y (block-sparse SpMM). At the end the
// result is merged with the block-row's low-resolution term (M_x, c_x, L_x)
// and normalised.
//
// Matrix-core layout (v_mfma_f32_32x32x16_bf16):
//  * S is formed transposed, S^T = K_y Q_x^T, so lane l holds query l%32 and
//    16 of its 32 key scores (keys 8(r/4) + 4(l/32) + r%4 in register r).
//    That is already the B-operand layout of O^T += V_y^T P^T up to a fixed
//    permutation of the key index, so P never moves between lanes; only the
//    row max crosses the two half-waves.
//  * The contraction index over d is permuted too: lane half h = l/32 takes
//    the contiguous half [h*d/2, (h+1)*d/2) of each Q and K row.
//  * float32 operands (Q, K, V and the weights) are split in registers into
//    three bfloat16 planes whose sum they are, and each product is the six
//    plane products that matter (tile_ops.h). The float32 matrix instructions
//    (64 cycles for 32x32x2) bounded the tile: 4096 cycles of them at d = 64
//    against 1536 for the plane products (48 of 32 cycles), plus about 2000 of
//    vector work, half of it the splitting. Measured before -> after: 16 heads x 4096 x 32,
//    budget 8 (small-4096): 47.5 -> 38.9 us; 24 heads x 4096 x 64, budget 16:
//    127 -> 93.6 us; 32 heads x 1504 x 128, budget 8: 84 (plus 11 for the
//    copies of K and V in operand order that it needed) -> 66 us.
//
// tile_stream_kernel copies the next selected tile's rows HBM/L2 -> a
// wave-private LDS slot with direct-to-LDS loads while the current one is
// computed from registers. float32 rows of 128 columns are shared by two waves.
//
// The softmax reference is set once per row (restart on overflow). Workgroup order
// is remapped so each XCD processes a contiguous range of heads and keeps
// their K/V tiles in its L2.
#include "common.h"
#include "kernels.h"
#include "tile_ops.h"

namespace mra {

// Reference point of the online softmax (log2 units). The weights of a tile
// are exp2(s * c * log2(e) - mrun) for the row's reference mrun, which need
// not be the running max: any reference works as long as weights and
// accumulators stay finite, because the final normalisation uses the same
// reference. mrun is set to the exact max of the row's first tile plus
// kRefMargin; later tiles only check that their weights sum to at most
// 2^kWeightCap per lane (far inside float32 and bfloat16 range, 2^128, even
// summed over 65536 keys). If a tile exceeds it, the row is computed again with
// the exact max over all its tiles as the reference, where no weight exceeds 1.
// The loop body thus has no 16-way max, no cross-lane exchange and no branch
// that rescales O. The margin makes that restart rare: a later logit must
// exceed the first tile's max by 96 (log2 units, 66.5 nats) to trigger it,
// while the row's largest weight stays at least 2^-32, far above the float32
// and bfloat16 underflow threshold 2^-126 (and bfloat16 rounding is relative,
// so the precision of the weights does not change).
constexpr float kWeightCap = 0x1p64f;
constexpr float kRefMargin = 32.0f;

__device__ __forceinline__ float tile_max(const f32x16& s) {
  float a = s[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) a = __builtin_elementwise_maximum(a, s[r]);
  return a;
}

// Accumulator state and arithmetic of one block-row (32 queries) in one wave.
// HALVES = 2 (float32, rows of 2 D columns): a pair of waves shares the row,
// each holding D of the columns (its part of Q, K, V and the output).
template <int DT, int D, bool COARSE, int HALVES>
struct TileRow {
  using Cfg = TileCfg<DT, D>;
  using elem = typename Cfg::elem;
  static constexpr int NT = Cfg::kNT, KC = Cfg::kKChunks, PITCH = D * HALVES;
  static constexpr int QP = DT == BF16 ? 1 : 3, QC = D / 16;
  f32x16 o[NT];
  float mrun, lrun, sl2;
  bool first;                                      // no reference yet
  u32x4 qf[QP][QC];                                // Q_x; float32: its bfloat16 planes

  // Q_x as the B operand: each lane reads d/2 contiguous elements of one row
  // (Q: the wave's first column).
  __device__ __forceinline__ void init(const elem* Q, int x, float scale_log2) {
    const int lane = lane_id(), jq = lane & 31, h = lane >> 5;
    const u32x4* qrow = reinterpret_cast<const u32x4*>(Q + (long long)(x * 32 + jq) * PITCH + (D / 2) * h);
    if constexpr (DT == BF16) {
#pragma unroll
      for (int s = 0; s < KC; ++s) qf[0][s] = qrow[s];
    } else {
      u32x4 raw[KC];
#pragma unroll
      for (int s = 0; s < KC; ++s) raw[s] = qrow[s];
      split_chunks(raw, qf);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
    mrun = -INFINITY;                              // no fine block: no weight
    lrun = 0.0f;
    sl2 = scale_log2;
    first = true;
  }

  // S^T = K_y Q_x^T (HALVES = 2: over this wave's columns)
  __device__ __forceinline__ f32x16 scores(const u32x4 (&kf)[KC]) const {
    if constexpr (DT == BF16) {
      return mfma_abt<KC>(kf, qf[0]);
    } else {
      u32x4 kp[3][QC];
      split_chunks(kf, kp);
      f32x16 c;
#pragma unroll
      for (int r = 0; r < 16; ++r) c[r] = 0.0f;
#pragma unroll
      for (int p = 2; p >= 0; --p)                 // the smallest products first
#pragma unroll
        for (int q = 2 - p; q >= 0; --q)
#pragma unroll
          for (int k = 0; k < QC; ++k)
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kp[p][k]),
                                                        __builtin_bit_cast(bf16x8, qf[q][k]), c, 0, 0, 0);
      return c;
    }
  }

  // Max of this tile's scores for this lane's query, in log2 units (lanes l
  // and l^32 share a query).
  __device__ __forceinline__ float tile_ref(const f32x16& s) const {
    return halves_max(tile_max(s)) * sl2;
  }

  // Start the row again with a fixed reference (no weight above 1).
  __device__ __forceinline__ void restart(float ref) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
    lrun = 0.0f;
    mrun = ref;
    first = false;
  }

  // bfloat16 weights of one tile into pk (two per register, the operand
  // order of the second product); returns their sum in float32.
  __device__ __forceinline__ float weights_bf16(const f32x16& s, uint32_t (&pk)[8]) const {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    float t = 0.0f;
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(s[2 * rr], sl2, -mrun));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(s[2 * rr + 1], sl2, -mrun));
      bf16x2 pb;
      pb[0] = (__bf16)p0;
      pb[1] = (__bf16)p1;
      t = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, t, false);   // sum of the rounded weights
      pk[rr] = __builtin_bit_cast(uint32_t, pb);
    }
    return t;
  }

  __device__ __forceinline__ float weights_f32(const f32x16& s, float (&p)[16]) const {
    float t = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], sl2, -mrun));
      t += p[r];
    }
    return t;
  }

  // Softmax weights of one tile and O^T += V_y^T P^T. `va(c)` yields the
  // 16-byte A-operand chunk c of V_y^T for this lane. Returns false if some
  // weight of the row may have exceeded the cap (the caller then restarts
  // the row); with check == false the caller guarantees it cannot.
  template <class VA>
  __device__ __forceinline__ bool accumulate(const f32x16& s, bool check, VA va) {
    float t;
    if constexpr (DT == BF16) {
      uint32_t pk[8];
      t = weights_bf16(s, pk);
      mfma_acc_bf16<NT>(o, pk, va);
    } else {
      float p[16];
      t = weights_f32(s, p);
      mfma_acc_split<NT>(o, p, va);
    }
    lrun += t;
    return !check || __ballot(!(t <= kWeightCap)) == 0;
  }

  // Merge with the low-resolution term, normalise and store the 32 x d block;
  // if lse is not NULL also each query's log normaliser, ln of the row sum of
  // A^ (natural units).
  // cmaxg, csumg, cv: the block-row's coarse-term maximum, sum and vector
  // (its D floats, in LDS or global memory); Out: the wave's first column
  __device__ __forceinline__ void finish(elem* Out, float* lse, int x, long long g, float cmaxg,
                                         float csumg, const float* cv) {
    const int lane = lane_id(), jq = lane & 31, h = lane >> 5;
    const float ltot = halves_sum(lrun);
    float af = 1.0f, bc = 0.0f, den = ltot, Mt = mrun;
    if constexpr (COARSE) {
      const float Mx = cmaxg * kLog2e;
      Mt = fmaxf(mrun, Mx);
      af = exp2f(mrun - Mt);
      bc = exp2f(Mx - Mt);
      den = ltot * af + csumg * bc;
    }
    if (lse != nullptr && h == 0) lse[g * 32 + jq] = (log2f(den) + Mt) * kLn2;
    const float inv = 1.0f / den;
    const float ao = af * inv, bv = bc * inv;       // z = o * ao + cvec * bv
    elem* orow = Out + (long long)(x * 32 + jq) * PITCH;
    u32x2 pend = {0u, 0u};                          // bf16: the even group's 4 values
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const int d0 = 32 * t + 8 * rg + 4 * h;
        float z[4];
        f32x4 c4 = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (COARSE) c4 = *reinterpret_cast<const f32x4*>(cv + d0);
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = COARSE ? fmaf(o[t][4 * rg + e], ao, c4[e] * bv) : o[t][4 * rg + e] * ao;
        if constexpr (DT == BF16) {
          bf16x2 lo, hi;
          lo[0] = (__bf16)z[0]; lo[1] = (__bf16)z[1];
          hi[0] = (__bf16)z[2]; hi[1] = (__bf16)z[3];
          const u32x2 pr = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
          // lanes l and l^32 hold dims 4h..4h+3 of groups rg (even, odd):
          // exchange so that lane h = 0 stores the even group's 8 dims and
          // lane h = 1 the odd group's, 16 contiguous bytes each
          if ((rg & 1) == 0) {
            pend = pr;
          } else {
            const u32x2 send = h ? pend : pr;          // h = 0 sends its odd group, h = 1 its even one
            u32x2 recv;
            recv[0] = (uint32_t)__shfl_xor((int)send[0], 32);
            recv[1] = (uint32_t)__shfl_xor((int)send[1], 32);
            const u32x4 st = h ? u32x4{recv[0], recv[1], pr[0], pr[1]} : u32x4{pend[0], pend[1], recv[0], recv[1]};
            *reinterpret_cast<u32x4*>(orow + 32 * t + 8 * (rg - 1) + 8 * h) = st;
          }
        } else {
          const f32x4 st = {z[0], z[1], z[2], z[3]};
          *reinterpret_cast<f32x4*>(orow + d0) = st;
        }
      }
    }
  }
};

// ---------------------------------------------------------------------------
// Raw K/V tiles in LDS (bfloat16, d <= 64). A 32-row tile of K (or V) is 4 KB
// (d = 64) of consecutive rows in HBM. It is copied with direct-to-LDS loads
// of whole rows (each 1 KB load covers 1024 / (2d) complete rows, so it
// touches as many cache lines as a contiguous copy), but each lane fetches
// the 16-byte block that belongs at its LDS position under an XOR swizzle of
// the blocks within a row: block b of row r sits at block b ^ f(r). With the
// swizzles below the matrix-core operand reads are free of bank conflicts
// (checked with a CPU model of the LDS banks):
//   K, row layout, ds_read_b128 (16 lanes = 16 rows per pass): lane (h, j)
//     reads row j, block (d/16) h + s;
//   V^T, transposed layout, ds_read_b64_tr_b16 (32 lanes per pass): within a
//     group of 16 lanes, lane 4k + g supplies 4 columns of row key0 + k and
//     lane i receives element i % 4 of lane (4k + i/4)'s 8 bytes as value k;
//     two reads (key0 = 16u + 4h and 16u + 8 + 4h) fill the 8 keys of a
//     chunk in the order the weights of the second product hold them.
template <int D>
__host__ __device__ constexpr int raw_swz_k(int r) {
  return D == 128 ? r & 15 : (D == 64 ? (r >> 1) & 7 : (r >> 2) & 3);
}
template <int D>
__host__ __device__ constexpr int raw_swz_v(int r) {
  return D == 128 ? 4 * (r & 3) : (D == 64 ? ((r >> 1) & 1) << 2 : 0);
}

// The 1 KB copies of a raw K tile and of a raw V tile (32 x d bfloat16: d/16
// copies each), buffer loads to LDS: the head's rows are one buffer resource,
// the tile's offset goes in the scalar offset and the lane's swizzled source
// offset in the vector offset, so a copy costs no vector instruction. Copy i
// moves source and destination by i KB; the swizzled lane offsets repeat with
// period 2 (K, d = 64: the swizzle of row r depends on r / 2), 4 (K, d = 128:
// r mod 16) or 1 in the copy index, so koff holds the offsets of copies
// i mod 4 and voff the V offset.
template <int I>
__device__ __forceinline__ void copy_raw_tiles_buf(i32x4 krs, i32x4 vrs, unsigned ktile, unsigned vtile,
                                                   const unsigned (&koff)[4], unsigned voff, lptr_t ks,
                                                   lptr_t vs) {
  if constexpr (I > 0) {
    copy_raw_tiles_buf<I - 1>(krs, vrs, ktile, vtile, koff, voff, ks, vs);
    constexpr int i = I - 1;
    buffer_load_lds16(krs, ks + i * 1024, koff[i & 3], ktile + i * 1024);
    buffer_load_lds16(vrs, vs + i * 1024, voff, vtile + i * 1024);
  }
}

// Transposed V chunks c = u NT + t (c < VC) of a raw tile: two transposing
// reads each, 8 rows apart, from this lane's column-tile address vt[t].
template <int D, int C, int VC>
struct RawTrChunks {
  static constexpr int NT = D / 32, RB = 2 * D;
  static __device__ __forceinline__ void run(const uint32_t* vt, u32x4* v) {
    if constexpr (C < VC) {
      constexpr int u = C / NT, t = C % NT;
      const u32x2 lo = lds_read_tr16<16 * u * RB>(vt[t]);
      const u32x2 hi = lds_read_tr16<(16 * u + 8) * RB>(vt[t]);
      v[C] = u32x4{lo[0], lo[1], hi[0], hi[1]};
      RawTrChunks<D, C + 1, VC>::run(vt, v);
    }
  }
};

// Raw float32 tiles (d <= 64). K: 4d-byte rows, the byte geometry of a
// bfloat16 tile of 2d columns, so its copies, swizzle and row-layout reads are
// those above with D2 = 2d (element (r, c) at raw_offset<D2>(r, 2c)). V is read
// transposed, four consecutive keys of one column per 16-byte operand chunk,
// with two ds_read2st64_b32 (keys 8a + 4h + e, e = 0, 1 and 2, 3, 256 bytes
// apart in LDS); rows are placed so that neither read has a bank conflict
// (CPU-modelled): d = 32 (128-byte rows): row r of each group of eight at
// slot 2 (r mod 4) + (r / 4 mod 2), so rows r and r + 4 fall in opposite bank
// halves; d = 64 (256-byte rows): the two 128-byte halves of rows with
// r / 4 odd swapped.
template <int D>
__host__ __device__ constexpr int f32v_slot(int r) {
  return D == 32 ? 8 * (r >> 3) + 2 * (r & 3) + ((r >> 2) & 1) : r;
}
template <int D>
__host__ __device__ constexpr int f32v_offset(int r, int c) {
  return f32v_slot<D>(r) * (4 * D) + 16 * ((c >> 2) ^ (D == 64 ? 8 * ((r >> 2) & 1) : 0)) + 4 * (c & 3);
}
// Source byte offset (within the V tile) of the 16 bytes lane `lane` copies to
// LDS byte i * 1024 + 16 lane.
template <int D>
__device__ __forceinline__ int f32v_copy_offset(int i, int lane) {
  const int rb = 4 * D, q = i * 1024 + 16 * lane, sl = q / rb, b = (q % rb) / 16;
  if (D == 32) return (8 * (sl >> 3) + 4 * (sl & 1) + ((sl >> 1) & 3)) * rb + 16 * b;
  return sl * rb + 16 * (b ^ (8 * ((sl >> 2) & 1)));
}

// The K copies (KPB-periodic lane offsets, as copy_raw_tiles_buf) and the V
// copies of a raw float32 tile (period 1 for d = 32, 2 for d = 64). STEP: source
// bytes between copies (1 KB; 2 KB where the tile is half of its rows).
template <int I, int STEP>
__device__ __forceinline__ void copy_raw_f32_buf(i32x4 krs, i32x4 vrs, unsigned ktile, unsigned vtile,
                                                 const unsigned (&koff)[4], const unsigned (&voff)[2], lptr_t ks,
                                                 lptr_t vs) {
  if constexpr (I > 0) {
    copy_raw_f32_buf<I - 1, STEP>(krs, vrs, ktile, vtile, koff, voff, ks, vs);
    constexpr int i = I - 1;
    buffer_load_lds16(krs, ks + i * 1024, koff[i & 3], ktile + i * STEP);
    buffer_load_lds16(vrs, vs + i * 1024, voff[i & 1], vtile + i * STEP);
  }
}

// Transposed V chunks c = 4 t + a (c < VC) of a raw float32 tile: keys
// 8a + 4h + e of column 32 t + i, from this lane's column-tile address vt[t].
template <int D, int C, int VC>
struct RawF32TrChunks {
  static constexpr int K64 = D == 32 ? 4 : 8;          // 256-byte units between key groups a
  static __device__ __forceinline__ void run(const uint32_t* vt, u32x4* v) {
    if constexpr (C < VC) {
      constexpr int t = C / 4, a = C % 4;
      const u32x2 lo = lds_read2st64<K64 * a, K64 * a + 1>(vt[t]);
      const u32x2 hi = lds_read2st64<K64 * a + 2, K64 * a + 3>(vt[t]);
      v[C] = u32x4{lo[0], lo[1], hi[0], hi[1]};
      RawF32TrChunks<D, C + 1, VC>::run(vt, v);
    }
  }
};

// ---------------------------------------------------------------------------
// One wave per block-row, K/V staged through a wave-private LDS slot:
// the next selected tile is copied HBM/L2 -> LDS with direct-to-LDS loads
// while the current one is computed from registers. Prefetching into LDS
// instead of registers leaves room for four waves per SIMD.
constexpr int kStreamWaves = 4;

// HALVES = 2 (float32 rows of 128 columns): the workgroup's two waves share one
// block-row, each working on 64 of the columns like the d = 64 kernel, with one
// exchange per tile: the scores are the sum of the two waves' products.
//
// SPLIT > 1: the workgroup's SPLIT waves share one block-row, wave p taking the
// tiles p, p + SPLIT, ... of its list; the sums are added through LDS at the end.
// All of them weigh relative to the reference of the row's first tile, which wave
// 0 has (and restart together, relative to the max over the whole list), so the
// weights, bfloat16 ones included, are those that one wave alone would form,
// whatever SPLIT: a call's sums differ from an unsplit one's in their order only.
template <int DT, int D, bool COARSE, int WAVES, int HALVES, int SPLIT>
__global__ __launch_bounds__(WAVES * kWave) void tile_stream_kernel(
    const void* __restrict__ qv, const void* __restrict__ kv, const void* __restrict__ vv,
    const int32_t* __restrict__ idx, const float* __restrict__ cmax,
    const float* __restrict__ csum, const float* __restrict__ cvec, void* __restrict__ outv,
    float* __restrict__ lse, int n, int nb, int m, long long row0, long long rows, int in_step, float scale_log2) {
  using Cfg = TileCfg<DT, D>;
  using elem = typename Cfg::elem;
  constexpr int KC = Cfg::kKChunks, VC = Cfg::kVChunks, CH = Cfg::kChunks;
  static_assert(CH <= 16, "operands of a tile are held in registers");
  static_assert(DT == BF16 || D <= 64, "raw tiles: bfloat16, or float32 with at most 64 columns per wave");
  static_assert(HALVES == 1 || (HALVES == 2 && DT == F32 && WAVES == 2), "a pair of waves per row");
  static_assert(SPLIT == 1 || (SPLIT == WAVES && HALVES == 1), "a workgroup per row");
  constexpr int DR = D * HALVES;                     // columns of a row
  constexpr bool F32RAW = DT == F32;
  constexpr int D2 = F32RAW ? 2 * D : D;             // the bfloat16 geometry of the K tile
  // the slots are their own LDS object, apart from the selection lists, so
  // reading a list does not wait for loads in flight into a slot
  __shared__ __attribute__((aligned(16))) u32x4 slot_all[WAVES][CH * 64];
  // Tiles of 8 KB per part (two waves per SIMD) fetch the coarse term's
  // vector into LDS while the tiles run (its maximum and sum are loaded then
  // too): with two waves per SIMD, reading it after the last tile exposed its
  // latency at every row's end; at four waves per SIMD the other waves hide
  // it, and the extra load at the row's start cost more than it saved.
  constexpr bool kTermAhead = COARSE && D2 >= 128;
  __shared__ __attribute__((aligned(16))) float cvl[WAVES][kTermAhead ? add_lds_floats(D) : 1];
  __shared__ __attribute__((aligned(16))) float ex[HALVES == 2 ? 2 : 1][2][HALVES == 2 ? 16 * kWave : 1];
  // waves that share a row: their references (first wave 0's; in a restart each
  // wave's max), their weights' sums and whether some weight grew too large
  __shared__ float refs[SPLIT > 1 ? SPLIT : 1][SPLIT > 1 ? kWave : 1];
  __shared__ float sums[SPLIT > 1 ? SPLIT : 1][SPLIT > 1 ? kWave : 1];
  __shared__ int grown[SPLIT > 1 ? SPLIT : 1];
  extern __shared__ int32_t sidx_all[];

  const int w = wave_uniform(threadIdx.x / kWave);
  const int lane = lane_id();
  const long long wg = xcd_remap(blockIdx.x, gridDim.x);
  // global block-row (rows row0 .. rows - 1); one per workgroup where waves share it
  const long long g = HALVES == 2 || SPLIT > 1 ? row0 + wg : row0 + wg * WAVES + w;
  if (g >= rows) return;                             // waves that share a row: all; else no barriers below
  const int part = SPLIT > 1 ? w : 0;                // this wave's tiles: part, part + SPLIT, ...
  const int col0 = HALVES == 2 ? w * D : 0;          // this wave's first column
  float cmaxg = 0.0f, csumg = 0.0f;
  if constexpr (kTermAhead) {
    prefetch_vec_lds<D>(cvec + g * DR + col0, (__attribute__((address_space(3))) char*)cvl[w]);
    cmaxg = cmax[g];
    csumg = csum[g];
  }
  const long long bh = g / nb;
  const int x = (int)(g - bh * nb);
  const long long hoff = bh * (long long)n * DR + col0;
  int32_t* myidx = sidx_all + w * m;
  // Q_x's loads are issued first, so their latency overlaps the staging of
  // the selection list
  TileRow<DT, D, COARSE, HALVES> row;
  row.init(reinterpret_cast<const elem*>(qv) + hoff, x, scale_log2);
  m = stage_selection(idx + g * m, m, nb, myidx);  // valid entries only, in order
  const bool tiles = m > 0;                        // of the row; wave 0 has the first
  if constexpr (SPLIT > 1) {
    myidx += part;
    m = (m - part + SPLIT - 1) / SPLIT;
  }
  wait_loads<0>();                                 // Q_x too (the list's loads came after it)
  // the head's K and V rows (tile y at byte y * 32 d e)
  constexpr unsigned TILE = KC * 1024u * HALVES;
  static_assert(KC == VC, "tiles of K and V");
  const char* kslab = static_cast<const char*>(kv) + (size_t)bh * nb * TILE;
  const char* vslab = static_cast<const char*>(vv) + (size_t)bh * nb * TILE;
  // this lane's source offsets for the copies (see copy_raw_tiles_buf) and its
  // LDS read offsets (K chunk c; V^T column tile t)
  constexpr int NT = TileCfg<DT, D>::kNT;
  constexpr int KPB = D2 == 128 ? 4 : (D2 == 64 ? 2 : 1);  // period of the K copy offsets
  // a byte of this wave's (half) tile -> its byte in the whole rows
  auto in_rows = [&](int b) {
    return HALVES == 1 ? b : (b / (2 * D2)) * (2 * D2 * HALVES) + b % (2 * D2) + col0 * (int)sizeof(elem);
  };
  unsigned koffq[4];                                 // K source offsets of copies i mod 4
#pragma unroll
  for (int q = 0; q < 4; ++q)
    koffq[q] = in_rows(raw_copy_offset<D2, raw_swz_k<D2>>(q % KPB, lane)) - (q % KPB) * 1024 * HALVES;
  const i32x4 krs = buffer_rsrc(kslab, (unsigned)nb * TILE);
  const i32x4 vrs = buffer_rsrc(vslab, (unsigned)nb * TILE);
  const int h = lane >> 5, j = lane & 31, i16 = lane & 15;
  int kread[KC], vread[NT];
#pragma unroll
  for (int c = 0; c < KC; ++c) kread[c] = raw_offset<D2, raw_swz_k<D2>>(j, (D2 / 2) * h + 8 * c);
  unsigned voff0 = 0, voffq[2] = {0u, 0u};
  if constexpr (F32RAW) {
#pragma unroll
    for (int q = 0; q < 2; ++q) voffq[q] = in_rows(f32v_copy_offset<D>(q, lane)) - q * 1024 * HALVES;
#pragma unroll
    for (int t = 0; t < NT; ++t) vread[t] = KC * 1024 + f32v_offset<D>(4 * h, 32 * t + j);
  } else {
    voff0 = raw_copy_offset<D, raw_swz_v<D>>(0, lane);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      vread[t] = KC * 1024 +
                 raw_offset<D, raw_swz_v<D>>(4 * h + i16 / 4, 32 * t + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3));
  }
  auto issue = [&](int y) {
    unsigned char* slot = reinterpret_cast<unsigned char*>(slot_all[w]);
    auto* ks = (__attribute__((address_space(3))) char*)slot;
    auto* vs = (__attribute__((address_space(3))) char*)(slot + KC * 1024);
    if constexpr (F32RAW)
      copy_raw_f32_buf<KC, 1024 * HALVES>(krs, vrs, (unsigned)y * TILE, (unsigned)y * TILE, koffq, voffq, ks, vs);
    else
      copy_raw_tiles_buf<KC>(krs, vrs, (unsigned)y * TILE, (unsigned)y * TILE, koffq, voff0, ks, vs);
  };
  // the tile's scores: for a pair the sum of the two waves' products, the same
  // in both (two buffers in turn, so one barrier per tile orders them)
  int exb = 0;
  auto whole_scores = [&](const u32x4 (&kf)[KC]) -> f32x16 {
    f32x16 s = row.scores(kf);
    if constexpr (HALVES == 2) {
      f32x4* mine = reinterpret_cast<f32x4*>(ex[exb][w]) + lane;
      const uint32_t theirs = lds_addr(ex[exb][1 - w]) + 16u * lane;
#pragma unroll
      for (int q = 0; q < 4; ++q) mine[64 * q] = f32x4{s[4 * q], s[4 * q + 1], s[4 * q + 2], s[4 * q + 3]};
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      u32x4 t[4];
      lds_read_chunks<4>(theirs, t);
      lds_done(t);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] += __uint_as_float(t[r / 4][r % 4]);
      exb ^= 1;
    }
    return s;
  };
  // The reference of the row's first tile (mine: wave 0's); every wave of a shared
  // row calls it once.
  auto row_reference = [&](float mine) -> float {
    if constexpr (SPLIT == 1) {
      return mine;
    } else {
      if (w == 0) refs[0][lane] = mine;
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      float ref;                                     // in one block with its wait, as list_entry
      asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(ref) : "v"(lds_addr(&refs[0][lane])) : "memory");
      return ref;
    }
  };
  // The list holds valid blocks only. The entry after the next is read before
  // the wait for a tile, so the refill is issued as soon as the slot is read.
  auto pass = [&](bool check) -> bool {
    if (m > 0) issue(list_entry(myidx));
    for (int i = 0; i < m; ++i) {
      const bool more = i + 1 < m;                   // wave-uniform
      const int yn = more ? list_entry(myidx + SPLIT * (i + 1)) : 0;
      wait_loads<0>();                               // tile i is in the slot
      u32x4 kf[KC], vf[VC];
      const uint32_t base = lds_addr(slot_all[w]);
#pragma unroll
      for (int c = 0; c < KC; ++c) kf[c] = lds_read16<0>(base + kread[c]);
      uint32_t va[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) va[t] = base + vread[t];
      if constexpr (F32RAW) RawF32TrChunks<D, 0, VC>::run(va, vf);
      else RawTrChunks<D, 0, VC>::run(va, vf);
      lds_done(kf);
      lds_done(vf);
      if (more) issue(yn);                           // refill the slot just read
      if (in_step) wait_loads<0>();                  // launched in rounds: see launch_stream_c
      const f32x16 s = whole_scores(kf);
      if (row.first) {                               // wave-uniform: the first tile of the first pass
        row.mrun = row_reference(row.tile_ref(s) + kRefMargin);
        row.first = false;
      }
      if (!row.accumulate(s, check, [&](int c) { return vf[c]; })) {
        wait_loads<0>();                             // the slot is idle again
        return false;
      }
    }
    return true;
  };
  // this wave's largest score, per query
  auto largest = [&]() -> float {
    float mx = -INFINITY;
    for (int i = 0; i < m; ++i) {
      const int yy = list_entry(myidx + SPLIT * i);
      u32x4 kf[KC];
      const u32x4* krow = reinterpret_cast<const u32x4*>(reinterpret_cast<const elem*>(kslab + (size_t)yy * TILE) +
                                                         (long long)j * DR + col0 + (D / 2) * h);
#pragma unroll
      for (int c = 0; c < KC; ++c) kf[c] = krow[c];
      mx = __builtin_elementwise_maximum(mx, row.tile_ref(whole_scores(kf)));
    }
    return mx;
  };
  // false: some weight grew too large, and the row is computed again relative to
  // its exact max
  const bool fits = pass(true);
  if constexpr (SPLIT == 1) {
    if (!fits) {
      row.restart(largest());
      pass(false);
    }
  } else {
    if (m == 0 && tiles) row_reference(0.0f);        // a wave without a tile meets the others
    // the sums, and the accumulators of waves 1 .. SPLIT - 1 in their slots (32 x d
    // floats each), behind a barrier
    auto share = [&]() {
      const float l = halves_sum(row.lrun);
      sums[w][lane] = l;
      if (w != 0) {
        f32x4* to = reinterpret_cast<f32x4*>(slot_all[w]) + lane;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            to[(4 * t + q) * kWave] = f32x4{row.o[t][4 * q], row.o[t][4 * q + 1], row.o[t][4 * q + 2], row.o[t][4 * q + 3]};
      }
      __syncthreads();
      return l;
    };
    if (lane == 0) grown[w] = !fits;
    float lt = share();
    int any = 0;
#pragma unroll
    for (int p = 0; p < SPLIT; ++p) any |= grown[p];
    if (wave_uniform(any)) {                         // all waves of the row, or none
      refs[w][lane] = largest();
      __syncthreads();
      float mx = refs[0][lane];
#pragma unroll
      for (int p = 1; p < SPLIT; ++p) mx = __builtin_elementwise_maximum(mx, refs[p][lane]);
      row.restart(mx);
      pass(false);
      lt = share();
    }
    if (w != 0) return;
#pragma unroll
    for (int p = 1; p < SPLIT; ++p) {
      lt += sums[p][lane];
      const f32x4* from = reinterpret_cast<const f32x4*>(slot_all[p]) + lane;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = from[(4 * t + q) * kWave];
#pragma unroll
          for (int e = 0; e < 4; ++e) row.o[t][4 * q + e] += v[e];
        }
    }
    row.lrun = h == 0 ? lt : 0.0f;                   // finish() adds the halves
  }
  if constexpr (kTermAhead) {
    wait_loads<0>();                                 // the coarse-term vector is in LDS
    row.finish(reinterpret_cast<elem*>(outv) + hoff, w == 0 || HALVES == 1 ? lse : nullptr, x, g, cmaxg, csumg, cvl[w]);
  } else {
    row.finish(reinterpret_cast<elem*>(outv) + hoff, w == 0 || HALVES == 1 ? lse : nullptr, x, g,
               COARSE ? cmax[g] : 0.0f, COARSE ? csum[g] : 0.0f, COARSE ? cvec + g * DR + col0 : nullptr);
  }
}

// ---------------------------------------------------------------------------
// Raw K/V tiles of up to 8 KB per wave stream through LDS.
//
// Where a head's K and V exceed an XCD's L2 (4 MB), the pass is launched one
// occupancy round of block-rows at a time: every block-row of a launch starts
// together and walks its (ascending) selection in step with its neighbours,
// so the blocks the XCD's resident rows touch at any moment stay close
// together and more of them hit L2. Within one launch, later rows start as
// earlier ones finish and the rows drift apart over the head. For the same
// reason a wave there waits for its refill as soon as it is issued (in_step):
// that costs the overlap of copy and arithmetic within a wave, which the other
// waves of the SIMD provide, and keeps the rows closer together: 16 heads of
// 32768 x 128 bfloat16, budget 32: 490 us with the wait, 548 without. Heads that
// fit L2 are launched whole (a launch per round costs more than it saves there)
// and without the wait.
//
// Where the block-rows alone leave most of the chip idle, two or four waves
// share a row (row_split). The fewer its tiles, the fewer rows it takes for the
// sharing to cost more than it gives, at bfloat16, whose tiles are short, and at
// d = 128, where the shared rows' kernels hold two waves per SIMD, first.
// Forward, GPU time, us; 1 and 2 waves per row (512 and 1024 rows in heads of
// 128 blocks, 768 in heads of 16):
//             512 rows       768 rows                        1024 rows
//   tiles     2              2          4          8          2          4          8
//   bf16  32  14.2 14.3      13.4 13.4  14.3 13.9  15.8 14.7  14.4 14.6  15.5 15.3  17.0 16.4
//   bf16  64  16.4 16.3      15.6 15.8  17.2 17.0  18.3 17.5  17.2 17.8  18.4 18.8  20.7 20.2
//   bf16 128  22.0 21.5      22.7 23.1  25.1 25.2  28.2 27.0  26.6 27.4  29.9 29.5  31.6 32.2
//   f32   32  16.0 15.7      15.9 16.0  18.0 17.7  22.1 20.8  16.6 17.0  20.0 20.0  23.6 22.6
//   f32   64  20.7 20.0      21.7 21.3  26.5 25.0  32.9 31.2  25.3 25.6  29.1 30.3  37.6 36.8
template <int DT, int D>
static int shared_rows_per_cu(int m) {
  if (m >= 8) return D == 128 ? 3 : 4;
  return DT == F32 || m >= 4 ? 3 : 2;
}
template <int DT, int D, bool COARSE, int HALVES, int SPLIT>
static void launch_stream_s(const void* q, const void* k, const void* v, const int32_t* idx,
                            const float* cmax, const float* csum, const float* cvec, void* out,
                            float* lse, long long bh, int n, int m, float scale_log2, hipStream_t stream) {
  // waves, block-rows per workgroup
  constexpr int W = SPLIT > 1 ? SPLIT : (HALVES == 2 ? 2 : kStreamWaves), R = SPLIT > 1 ? 1 : W / HALVES;
  const int nb = n / kBlock;
  const long long rows = bh * nb;
  const size_t smem = (size_t)W * m * sizeof(int32_t);     // per-wave selection lists
  auto kernel = tile_stream_kernel<DT, D, COARSE, W, HALVES, SPLIT>;
  const size_t head_kv = (size_t)2 * n * D * HALVES * (DT == BF16 ? 2 : 4);
  long long chunk = SPLIT == 1 && head_kv > kL2PerXcd ? resident_items(kernel, W * kWave, smem, R) : 0;
  if (chunk <= 0) chunk = rows;
  for (long long r0 = 0; r0 < rows; r0 += chunk) {
    const long long r1 = r0 + chunk < rows ? r0 + chunk : rows;
    const unsigned blocks = (unsigned)((r1 - r0 + R - 1) / R);
    kernel<<<blocks, W * kWave, smem, stream>>>(q, k, v, idx, cmax, csum, cvec, out, lse, n, nb, m, r0, r1,
                                                chunk < rows, scale_log2);
  }
}

template <int DT, int D, bool COARSE, int HALVES>
static void launch_stream_c(const void* q, const void* k, const void* v, const int32_t* idx,
                            const float* cmax, const float* csum, const float* cvec, void* out,
                            float* lse, long long bh, int n, int m, float scale_log2, hipStream_t stream) {
  if constexpr (HALVES == 1) {
    const int split = row_split(bh * (n / kBlock), m, shared_rows_per_cu<DT, D>(m));
    if (split == 4)
      return launch_stream_s<DT, D, COARSE, 1, 4>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
    if (split == 2)
      return launch_stream_s<DT, D, COARSE, 1, 2>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
  }
  launch_stream_s<DT, D, COARSE, HALVES, 1>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
}

template <int DT, int D, int HALVES = 1>
static void launch_stream(const void* q, const void* k, const void* v, const int32_t* idx,
                          const float* cmax, const float* csum, const float* cvec, void* out,
                          float* lse, long long bh, int n, int m, float scale_log2, hipStream_t stream) {
  if (cmax)
    launch_stream_c<DT, D, true, HALVES>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
  else
    launch_stream_c<DT, D, false, HALVES>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
}

hipError_t launch_tile(const void* q, const void* k, const void* v, const int32_t* idx,
                       const float* cmax, const float* csum, const float* cvec, void* out, float* lse,
                       long long bh, int n, int d, int m, int dtype, hipStream_t stream) {
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)d));
  if (dtype == BF16) {
    if (d == 32) launch_stream<BF16, 32>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
    else if (d == 64) launch_stream<BF16, 64>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
    else launch_stream<BF16, 128>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
  } else {
    if (d == 32) launch_stream<F32, 32>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
    else if (d == 64) launch_stream<F32, 64>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
    else launch_stream<F32, 64, 2>(q, k, v, idx, cmax, csum, cvec, out, lse, bh, n, m, scale_log2, stream);
  }
  return hipGetLastError();
}

}  // namespace mra
