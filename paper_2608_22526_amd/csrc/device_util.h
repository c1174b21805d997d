// Device helpers shared by the readout kernels and the fused merge + commit
// launch (gfx950 only).
#pragma once

#include <algorithm>

#include "rs3_internal.h"

namespace rs3 {

// Loads through global (not generic) pointers: the compiler then counts
// them on the vector memory counter alone, and a wait for one of them does
// not have to drain every outstanding load.
#define RS3_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ T gload(const T* p) {
  return *(const RS3_GLOBAL T*)p;
}

// Stores through global pointers, for the same reason: a generic (flat)
// store counts on the LDS counter too, so a later wait for an LDS read would
// also wait for the store to land.
template <class T>
__device__ __forceinline__ void gstore(T* p, const T& v) {
  *(RS3_GLOBAL T*)p = v;
}

// Non-temporal (streaming) accesses for data that is written once and read
// once: the readout's split partials.  The merge reads every partial with
// pload; k_attn_g2, and k_attn when the readout launches it, write them
// with pstore.  Measured on the 64x64 one-object frame: the stores gave
// 1.2-1.4 % more frames/s, the loads another 1.6 %, and the attention of the
// next frame got faster too (the partials, about 3.7 MB a frame, no longer
// crowd the bank's key/value tiles out of the L2); with k_attn's stores as
// well the projected 64x64 frame gained 5 %, the other readout workloads
// 0.2-0.9 %.  The same marking was slower for the energies and projected
// queries of the energy launch, which the next launch reads back, and for
// the partials of the stack's attentions, which its own merge reads.
template <class T>
__device__ __forceinline__ void pstore(T* p, const T& v) {
  __builtin_nontemporal_store(v, (RS3_GLOBAL T*)p);
}
template <class T>
__device__ __forceinline__ T pload(const T* p) {
  return __builtin_nontemporal_load((const RS3_GLOBAL T*)p);
}

// Loads of wave-uniform values that earlier launches wrote (bank headers,
// descriptors, selected counts): through the constant address space the
// compiler uses scalar loads, which are counted apart from the vector loads,
// so waiting for them does not wait for the operand loads issued before.
#define RS3_CONST __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ T sload(const T* p) {
  return *(const RS3_CONST T*)p;
}

// Waits for loaded values and hands them on as values the compiler did not
// see being loaded: a loop that uses them then carries no pending load to
// its head, where the compiler would otherwise wait for every outstanding
// load (the key/value DMA included) in each iteration.
__device__ __forceinline__ void settle(int& a, uint32_t& b, uint32_t& c) {
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(a), "+v"(b), "+v"(c)::"memory");
}

// Keeps a loaded value alive on a path that does not use it, so the load is
// issued before the branch rather than sunk past it (an early exit would
// otherwise delay every load that only the main path uses).
template <class T>
__device__ __forceinline__ void keep(const T& v) {
  asm volatile("" ::"v"(v));
}
template <class T>
__device__ __forceinline__ void keep_s(const T& v) {
  asm volatile("" ::"s"(v));
}

// Work-group blk of c.blocks (256 threads) of a grid copy, a chunk per thread:
// read once and written to up to COPY_GROUP output grids (more of them go to
// further work-groups: a small grid shared by many objects would otherwise be
// written by a few CUs).  Grids past 2,048 work-groups each loop.  64 grids of 8
// MiB: 172 us; 2,048 work-groups in all with four chunks in flight per
// thread took 216.
constexpr int COPY_GROUP = 4;
inline int copy_blocks(const Rs3CopyArgs& c) {
  const int64_t groups = (c.copies + COPY_GROUP - 1) / COPY_GROUP, single = (c.n_x * c.count + 255) / 256;
  return (int)(std::min<int64_t>(single, 2048 * (int64_t)c.n_x) * groups);
}

__device__ __forceinline__ void copy_block(const Rs3CopyArgs& c, int blk) {
  const int64_t total = c.n_x * c.count;
  const int groups = (c.copies + COPY_GROUP - 1) / COPY_GROUP, cg = blk % groups;
  const int p0 = cg * COPY_GROUP, p1 = min(p0 + COPY_GROUP, c.copies);
  const int64_t step = (int64_t)(c.blocks / groups) * 256;
  for (int64_t i = (int64_t)(blk / groups) * 256 + threadIdx.x; i < total; i += step) {
    const int64_t xi = c.n_x == 1 ? 0 : total >> 31 ? i / c.count : (uint32_t)i / (uint32_t)c.count;
    const u32x4 v = gload((const u32x4*)c.X + xi * c.x_stride + (i - xi * c.count));
    u32x4* y = (u32x4*)c.Y + xi * c.y_stride + (i - xi * c.count);
    for (int p = p0; p < p1; ++p) gstore(y + p * c.y_stride, v);
  }
}

__device__ __forceinline__ int sel_count_of(const Rs3ReadoutArgs& a, int o, BankDev& b,
                                            bool report) {
  int cnt = gload(a.sel_count + (a.sel_stride ? o : 0));
  if (cnt > a.max_sel || cnt < 0) {
    if (report) set_err(b.hdr, RS3_E_INVALID);
    cnt = cnt < 0 ? 0 : a.max_sel;
  }
  return cnt;
}

// True iff sel[r] is in range and larger than its predecessor.
__device__ __forceinline__ bool sel_ok(const int32_t* sel, int r, int mn) {
  int i = sel[r];
  return i >= 0 && i < mn && (r == 0 || sel[r - 1] < i);
}

// D = A(32x2) * B(2x32) + C.  Lane l supplies A row l%32 and B column l%32 at
// k = l/32; the 16 results lie as in mfma32 (column l%32, rows c_row).
// A contraction of 8 consecutive channels takes four of these on a 16-byte
// chunk per operand: lane group g = l/32 holds channels 4g .. 4g+3 of the
// eight, and step e multiplies channels e and 4+e.
__device__ __forceinline__ f32x16 mfma32f(const f32x4& a, const f32x4& b, f32x16 c) {
#pragma unroll
  for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], c, 0, 0, 0);
  return c;
}

// Partials of the tiled attention (k_attn_tile), per row, head and split: the
// normalised O as f16 times a power of two of the row's own, (m, l) as two
// floats.  l is brought to [1, 2) and its exponent added to m, which leaves
// the exponent field of the second float for the scale: 2^e of O, e that of the
// row's largest value less 14, so that f16 has its 11 bits down to 2^-28 of
// it.  Not above 0 (empty, or no number): nothing to decode.  The one-wave
// attention stores O as bf16 and l as it is.
__device__ __forceinline__ float part_sum(float l) {   // l in [1, 2)
  return __uint_as_float((__float_as_uint(l) & 0x007fffffu) | 0x3f800000u);
}
__device__ __forceinline__ float part_scale(float l) { return __uint_as_float(__float_as_uint(l) & 0x7f800000u); }

// The two values of a word of partial O.
template <bool F16>
__device__ __forceinline__ float part_lo(uint32_t x) {
  if constexpr (F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)(x & 0xffffu));
  return __uint_as_float(x << 16);
}
template <bool F16>
__device__ __forceinline__ float part_hi(uint32_t x) {
  if constexpr (F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)(x >> 16));
  return __uint_as_float(x & 0xffff0000u);
}

template <int CTRL>
__device__ __forceinline__ float dppf(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over the 64 lanes, the same value in every lane: within rows of 16
// lanes by DPP (quad swaps, half-row and row mirrors), then across rows by
// v_permlane16_swap and v_permlane32_swap.  Each step adds a lane to a
// partner that adds it back, so every lane holds the same bits.
__device__ __forceinline__ float wave_sum(float v) {
  v += dppf<0xB1>(v);    // quad_perm(1, 0, 3, 2)
  v += dppf<0x4E>(v);    // quad_perm(2, 3, 0, 1)
  v += dppf<0x141>(v);   // row_half_mirror
  v += dppf<0x140>(v);   // row_mirror
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Maximum over the 64 lanes by the same exchange pattern.
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dppf<0xB1>(v));
  v = fmaxf(v, dppf<0x4E>(v));
  v = fmaxf(v, dppf<0x141>(v));
  v = fmaxf(v, dppf<0x140>(v));
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

}  // namespace rs3
