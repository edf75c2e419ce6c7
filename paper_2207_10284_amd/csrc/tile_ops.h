// Matrix-core operands and products of one 32x32 tile (v_mfma_f32_32x32x16_bf16),
// shared by the forward tile pass and the two gradient passes.
//
// Operand layouts (bf16: 8 elements per 16-byte chunk, f32: 4):
//  * Row layout, 32 rows x d: lane (h, j) = (l/32, l%32) holds row j,
//    columns (d/2)h + e*s .. +e-1 in chunk s (KC chunks).
//  * Transposed layout, d rows x 32 (the A operand of C^T += X^T P^T), VC chunks
//    per lane, ordered as the B-operand registers of a tile product hold the 32
//    contraction indices: bf16 chunk u*NT + t (NT = d/32) of lane (h, j) is
//    X[16u + 8(s/4) + 4h + s%4][32t + j], s = 0..7; f32 chunk t*4 + a is
//    X[8a + 4h + kk][32t + j], kk = 0..3.
//  * A product C = A B^T of two row-layout operands leaves, in lane l,
//    column l%32 of C (B's row) and its rows 8(r/4) + 4(l/32) + r%4 in
//    register r. Those 16 values are directly the B operand of the next
//    product over the same index (mfma_acc_*), so weights never move between
//    lanes.
//
// float32 on the bfloat16 matrix cores: a float32 value is the sum of three
// bfloat16 values (hi: its upper half, mid: the remainder rounded, lo: what is
// left, at most eight bits), so a float32 product is the sum of the products of
// the planes. The six with plane indices p + q <= 2 are formed, the smallest
// first, and the other three (at most 2^-23 of the product each) dropped. Six
// 32x32x16 products of 32 cycles do the work of eight 32x32x2 float32 products of
// 64. Relative error of whole calls against float64 (2-norm), with the float32
// instruction, whose every step rounds, and with the planes: 24 heads x 4096 x 64,
// four resolutions: 1.9e-6, 0.7e-6; training, 32 heads x 1504 x 128: 2.2e-6, 2.0e-6.
// The low planes of a value below 2^-110 are no normal bfloat16 numbers: what of
// it is below 2^-126 may be lost.
#pragma once

#include "common.h"

namespace mra {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int DT, int D>
struct TileCfg {
  static constexpr int kNT = D / 32;                            // output tiles over d
  // 16-byte transposed-layout chunks per lane per tile
  static constexpr int kVChunks = DT == BF16 ? 2 * kNT : 4 * kNT;
  static constexpr int kKChunks = DT == BF16 ? D / 16 : D / 8;  // 16-byte row-layout chunks per lane
  static constexpr int kChunks = kKChunks + kVChunks;           // 1 KB chunks per K/V tile
  using elem = typename std::conditional<DT == BF16, uint16_t, float>::type;
};

// Row j = l%32 of a 32-row block at `rows` (row-major, D columns) in the row
// layout: lane half h reads columns [h*D/2, (h+1)*D/2).
template <int DT, int D>
__device__ __forceinline__ void load_rows(const typename TileCfg<DT, D>::elem* rows,
                                          u32x4 (&f)[TileCfg<DT, D>::kKChunks]) {
  const int lane = lane_id(), j = lane & 31, h = lane >> 5;
  const u32x4* p = reinterpret_cast<const u32x4*>(rows + (long long)j * D + (D / 2) * h);
#pragma unroll
  for (int s = 0; s < TileCfg<DT, D>::kKChunks; ++s) f[s] = p[s];
}

// C = A B^T over the d columns, both in the row layout (bfloat16).
template <int KC>
__device__ __forceinline__ f32x16 mfma_abt(const u32x4 (&a)[KC], const u32x4 (&b)[KC]) {
  f32x16 s;
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
  for (int k = 0; k < KC; ++k)
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[k]),
                                                __builtin_bit_cast(bf16x8, b[k]), s, 0, 0, 0);
  return s;
}

// o[t] (d rows 32t.., 32 columns) += X^T W for bfloat16 weights pk (two per
// register, in the order of a product's result registers); `xa(c)` yields
// the 16-byte transposed-layout chunk c of X.
template <int NT, class XA>
__device__ __forceinline__ void mfma_acc_bf16(f32x16 (&o)[NT], const uint32_t (&pk)[8], XA xa) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const u32x4 pw = {pk[4 * u], pk[4 * u + 1], pk[4 * u + 2], pk[4 * u + 3]};
    const bf16x8 pb = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
      o[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa(u * NT + tt)), pb, o[tt], 0, 0, 0);
  }
}

// Two float32 values as three bfloat16 pairs whose sums they are (finite
// inputs): hi the upper halves (truncated, so nothing overflows), mid the
// remainder rounded, lo the rest, which has at most eight significant bits.
// A remainder x - hi is one dot product of the pair with (-1, 0) or (0, -1);
// the two constants are kept in registers, since the compiler encodes the first
// as the inline constant -1.0, which the instruction does not read as that pair.
__device__ __forceinline__ void split2(float x, float y, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  uint32_t px = 0x0000BF80u, py = 0xBF800000u;
  asm("" : "+s"(px), "+s"(py));
  const bf16x2 pick_x = __builtin_bit_cast(bf16x2, px), pick_y = __builtin_bit_cast(bf16x2, py);
  hi = __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
  const bf16x2 h2 = __builtin_bit_cast(bf16x2, hi);
  const float rx = __builtin_amdgcn_fdot2_f32_bf16(h2, pick_x, x, false);
  const float ry = __builtin_amdgcn_fdot2_f32_bf16(h2, pick_y, y, false);
  bf16x2 m2, l2;
  m2[0] = (__bf16)rx;
  m2[1] = (__bf16)ry;
  l2[0] = (__bf16)__builtin_amdgcn_fdot2_f32_bf16(m2, pick_x, rx, false);
  l2[1] = (__bf16)__builtin_amdgcn_fdot2_f32_bf16(m2, pick_y, ry, false);
  mid = __builtin_bit_cast(uint32_t, m2);
  lo = __builtin_bit_cast(uint32_t, l2);
}

// Eight values as the three planes of a 16-byte operand chunk.
__device__ __forceinline__ void split8(const float (&v)[8], u32x4 (&pl)[3]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t h, m, l;
    split2(v[2 * q], v[2 * q + 1], h, m, l);
    pl[0][q] = h;
    pl[1][q] = m;
    pl[2][q] = l;
  }
}

// The float32 row-layout chunks f (four columns each) of a block as bfloat16
// planes in the bfloat16 row layout (eight columns per chunk): a lane's chunks
// 2k and 2k + 1 are the eight columns of plane chunk k.
template <int KC>
__device__ __forceinline__ void split_chunks(const u32x4 (&f)[KC], u32x4 (&pl)[3][KC / 2]) {
#pragma unroll
  for (int k = 0; k < KC / 2; ++k) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(f[2 * k + e / 4][e % 4]);
    u32x4 c[3];
    split8(v, c);
#pragma unroll
    for (int q = 0; q < 3; ++q) pl[q][k] = c[q];
  }
}

// The same for float32 weights p (one per register): weights and X as
// bfloat16 planes, the products of the planes with p + q <= 2, the smallest
// first. `xa(c)` yields the float32 transposed-layout chunk c = 4t + a of X;
// chunks a = 2u and 2u + 1 are the eight rows of the bfloat16 chunk (u, t).
template <int NT, class XA>
__device__ __forceinline__ void mfma_acc_split(f32x16 (&o)[NT], const float (&p)[16], XA xa) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[8 * u + e];
    u32x4 pk[3];
    split8(v, pk);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const u32x4 x0 = xa(4 * t + 2 * u), x1 = xa(4 * t + 2 * u + 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = __uint_as_float(x0[e]);
        v[4 + e] = __uint_as_float(x1[e]);
      }
      u32x4 xp[3];
      split8(v, xp);
#pragma unroll
      for (int s = 2; s >= 0; --s)
#pragma unroll
        for (int q = 0; q <= s; ++q)
          o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xp[q]),
                                                         __builtin_bit_cast(bf16x8, pk[s - q]), o[t], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ void wait_lds_reads() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Wait until at most N vector-memory loads are outstanding (they complete in
// issue order, so the older ones have landed). The builtin, unlike an asm
// s_waitcnt, tells the compiler's own wait insertion what has landed: without
// that, operands loaded before a loop cost a wait for every copy in flight in
// each of its iterations.
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "six bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);   // vmcnt; the other counters free
  asm volatile("" ::: "memory");
}

// Slot reads are issued as inline assembly: the compiler cannot tell the
// slot's parts apart and, seeing loads in flight into LDS, would wait for all
// of them before any slot read. Here the caller's wait_loads<> covers the part
// being read; lds_done() waits for the reads and ties each value to that wait
// so that no use is scheduled before it.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

template <int OFF>
__device__ __forceinline__ u32x4 lds_read16(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF) : "memory");
  return v;
}

// v[i] = chunk C0 + i of a part (chunks 1 KB apart) for this lane, i < C
template <int I, int C, int C0>
struct LdsChunks {
  static __device__ __forceinline__ void run(uint32_t addr, u32x4* v) {
    v[I] = lds_read16<(C0 + I) * 1024>(addr);
    LdsChunks<I + 1, C, C0>::run(addr, v);
  }
};
template <int C, int C0>
struct LdsChunks<C, C, C0> {
  static __device__ __forceinline__ void run(uint32_t, u32x4*) {}
};

template <int C, int C0 = 0>
__device__ __forceinline__ void lds_read_chunks(uint32_t addr, u32x4 (&v)[C]) {
  LdsChunks<0, C, C0>::run(addr, v);
}

template <int C>
__device__ __forceinline__ void lds_done(u32x4 (&v)[C]) {
  wait_lds_reads();
#pragma unroll
  for (int c = 0; c < C; ++c) asm volatile("" : "+v"(v[c]));
}

// gfx950's transposing read (ds_read_b64_tr_b16): within each group of 16
// lanes, lane i receives as value k (k = 0..3) the 16-bit element i%4 of the
// 8 bytes at the address that lane 4k + i/4 of the group supplies.
template <int OFF>
__device__ __forceinline__ u32x2 lds_read_tr16(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF) : "memory");
  return v;
}

// Two dwords per lane from addr + 256 OFF0 and addr + 256 OFF1 bytes
// (ds_read2st64_b32: offsets in units of 64 dwords).
template <int OFF0, int OFF1>
__device__ __forceinline__ u32x2 lds_read2st64(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(v) : "v"(addr), "i"(OFF0), "i"(OFF1) : "memory");
  return v;
}

// Entry of a block list in LDS, in one asm block with its wait: for an
// ordinary read the compiler may first wait for every copy in flight to LDS.
__device__ __forceinline__ int list_entry(const int32_t* p) {
  int v;
  asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(lds_addr(p)) : "memory");
  return wave_uniform(v);
}
__device__ __forceinline__ int list_entry(const uint16_t* p) {
  int v;
  asm volatile("ds_read_u16 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(lds_addr(p)) : "memory");
  return wave_uniform(v);
}

typedef __attribute__((address_space(3))) char* lptr_t;

// Raw bfloat16 tiles in LDS (d <= 64): a 32-row tile of consecutive rows
// (2d bytes each) copied with direct-to-LDS loads whose lanes each fetch the
// 16-byte block that belongs at their LDS position under an XOR swizzle F of
// the blocks within a row: block b of row r sits at block b ^ F(r).
// Byte offset of element (r, c) of such a tile in LDS:
template <int D, int (*F)(int)>
__host__ __device__ constexpr int raw_offset(int r, int c) {
  return r * (2 * D) + ((((2 * c) >> 4) ^ F(r)) << 4) + ((2 * c) & 15);
}

// Source byte offset (within the tile) of the 16 bytes lane `lane` copies to
// LDS byte i * 1024 + 16 lane under swizzle F.
template <int D, int (*F)(int)>
__device__ __forceinline__ int raw_copy_offset(int i, int lane) {
  const int q = i * 1024 + 16 * lane, r = q / (2 * D), blk = (q % (2 * D)) / 16;
  return r * (2 * D) + ((blk ^ F(r)) << 4);
}

// Buffer loads straight to LDS (16 bytes per lane): a raw buffer resource for
// `bytes` bytes from `base`, and one load of the 16 bytes at base + soff +
// voff into LDS byte dst + 16 lane. The hardware range check covers the
// vector and immediate offsets only, not the scalar offset, so a load is in
// bounds only because every caller validates the block it copies first (the
// tile passes take only block ids in [0, nb), filtered when the selection is
// staged); the resource's size is not a safety net for the scalar offset.
__device__ void mra_raw_buffer_load_lds(i32x4 rsrc, __attribute__((address_space(3))) void* lds, int size,
                                        int voffset, int soffset, int offset,
                                        int aux) __asm("llvm.amdgcn.raw.buffer.load.lds");

__device__ __forceinline__ void buffer_load_lds16(i32x4 rsrc, __attribute__((address_space(3))) char* dst,
                                                  unsigned voff, unsigned soff) {
  mra_raw_buffer_load_lds(rsrc, dst, 16, (int)voff, (int)soff, 0, 0);
}

// The D floats at src (a block's coarse-term vector, used by an epilogue)
// into LDS at dst with direct-to-LDS dword loads, 256 bytes per load (lanes
// past D read zero), so their latency passes during the tiles; a wait for the
// load counter (the tile copies' or one before the epilogue) completes them.
template <int D>
__device__ __forceinline__ void prefetch_vec_lds(const float* src, __attribute__((address_space(3))) char* dst) {
  const i32x4 rs = buffer_rsrc(src, (unsigned)D * (unsigned)sizeof(float));
  const int lane = lane_id();
#pragma unroll
  for (int p = 0; p < (D + 63) / 64; ++p) mra_raw_buffer_load_lds(rs, dst + 256 * p, 4, (lane + 64 * p) * 4, 0, 0, 0);
}
constexpr int add_lds_floats(int d) { return d < 64 ? 64 : d; }

// Copies a list of m block ids into LDS keeping only the entries in [0, nb),
// in their order, and returns how many there are (wave-uniform). Reading the
// ids from LDS keeps them off the vector-memory counter, so prefetched loads
// stay in flight; dropping entries outside [0, nb) here (the padding of a
// head-wide selection, for instance) keeps them out of the loop.
template <class T>
__device__ __forceinline__ int stage_selection(const int32_t* __restrict__ row, int m, int nb, T* dst) {
  const int lane = lane_id();
  int cnt = 0;
  for (int i0 = 0; i0 < m; i0 += kWave) {
    const int y = i0 + lane < m ? row[i0 + lane] : -1;
    const bool ok = y >= 0 && y < nb;
    const uint64_t mk = __ballot(ok);
    if (ok) dst[cnt + __popcll(mk & lanemask_lt())] = (T)y;
    cnt += __popcll(mk);
  }
  wave_lds_sync();
  return wave_uniform(cnt);
}

}  // namespace mra
