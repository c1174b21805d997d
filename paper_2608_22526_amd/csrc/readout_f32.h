// fp32 readout on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: exact fp32
// products, fp32 accumulation): device code of its merge step, shared by the
// merge kernel and the fused merge + commit launch.
#pragma once

#include "device_util.h"

namespace rs3 {

// One 32x32 output block of the projection: each of the four waves contracts a
// quarter of the channels, the partial blocks meet in LDS, and thread t ends
// with row t/8, columns 4*(t%8) .. +3.
constexpr int RF_THREADS = 256;
constexpr int RF_ROWS = 32;
constexpr int RF_PITCH = 36;   // floats: 16-byte rows

__device__ __forceinline__ f32x4 rf_reduce(const f32x16& acc, float* red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int r = 0; r < 16; ++r) red[(wave * 32 + c_row(r, lane)) * RF_PITCH + (lane & 31)] = acc[r];
  lds_barrier();
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) s += *(const f32x4*)(red + (w * 32 + (tid >> 3)) * RF_PITCH + 4 * (tid & 7));
  return s;
}

// Merge of the key splits, output projection and residual scatter of rows
// [32 ry, +32) of object o by MF_THREADS threads:
//   1. the split weights of every (head, row), from the (m, l) of the splits;
//   2. the merged rows to LDS, one 16-byte chunk per thread and step, eight
//      splits of it in flight;
//   3. y = x + O W_o on 16x16x4 fp32 MFMAs, a wave per 16 rows x 16 columns.
// Bound by the latency of step 2: 16 splits of 32 rows x 256 channels are
// 0.5 MB per block, which 1,024 threads hold in flight in two rounds (four
// waves that each merged their own operand, once per 32 columns, took 50 us).
// Plain loads and stores for the partials: the L2 and the last-level cache
// hold them (streaming ones, as the bf16 partials use, had every round go to
// memory).
// dyn: merged rows [32][D+4], weights [H*S][32], live [32] floats.
constexpr int MF_THREADS = 1024;
inline size_t merge_f32_lds(int D, int HS) { return (size_t)(32 * (D + 4) + 32 * HS + 32) * 4; }

__device__ __forceinline__ f32x4 mfma16f(const f32x4& a, const f32x4& b, f32x4 c) {
  // lane l: A row and B column l%16, channels 4*(l/16) .. +3 of sixteen; the
  // results are rows 4*(l/16) + r, column l%16
#pragma unroll
  for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
  return c;
}

__device__ __forceinline__ void merge_f32_block(const Rs3ReadoutArgs& a, int o, int ry, float* dyn) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = ry * RF_ROWS, S = a.S, H = a.H, D = a.D, C = a.C, OP = D + 4;
  float* os = dyn;
  float* wl = os + 32 * OP;        // [h][s][row]
  float* live = wl + 32 * H * S;   // [row]: 1 if a head of the row has weight on a key
  const int32_t* sel = a.sel_idx + (int64_t)o * a.sel_stride;
  int cnt = gload(a.sel_count + (a.sel_stride ? o : 0));
  // the rows this thread stores: rt + r, r < 4
  const int rt = 16 * (wave & 1) + 4 * (lane >> 4);
  int cell[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = min(r0 + rt + r, a.max_sel - 1);
    const int c = gload(sel + i), prev = i > 0 ? gload(sel + i - 1) : -1;
    cell[r] = c >= 0 && c < a.mn && prev < c ? c : -1;
  }
  if (cnt < 0 || cnt > a.max_sel) {
    if (tid == 0 && r0 == 0) set_err(a.banks[o]->hdr, RS3_E_INVALID);
    cnt = cnt < 0 ? 0 : a.max_sel;
  }
  if (r0 >= cnt) return;
  if (tid < 32) live[tid] = 0.f;
  lds_barrier();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (r0 + rt + r >= cnt)
      cell[r] = -1;
    else if (cell[r] < 0 && wave < 2)
      set_err(a.banks[o]->hdr, RS3_E_INVALID);
  }
  // split weights e^(m_s - M) / sum_s e^(m_s - M) l_s
  for (int q = tid; q < 32 * H; q += MF_THREADS) {
    const int row = q & 31, h = q >> 5, rc = min(r0 + row, a.max_sel - 1);
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const float* ml = a.ML + (((int64_t)o * S * a.max_sel + rc) * H + h) * 2;
    const int64_t st = (int64_t)a.max_sel * H * 2;
    float M = -INFINITY, den = 0.f;
#pragma unroll 8
    for (int s = 0; s < S; ++s) M = fmaxf(M, gload(ml + s * st));
#pragma unroll 8
    for (int s = 0; s < S; ++s) {
      const f32x2 v = gload((const f32x2*)(ml + s * st));
      const float w = v[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(v[0] - M);
      den = fmaf(w, v[1], den);
      wl[(h * S + s) * 32 + row] = w;
    }
    const float inv = den > 0.f ? 1.f / den : 0.f;
    for (int s = 0; s < S; ++s) wl[(h * S + s) * 32 + row] *= inv;
    if (den > 0.f) live[row] = 1.f;   // from any head: one may have no finite logit
  }
  lds_barrier();
  const int lg_dh = 31 - __clz(a.d_h), cpr = D / 4;
  const int64_t sst = (int64_t)a.max_sel * D;
  for (int q = tid; q < 32 * cpr; q += MF_THREADS) {
    const int row = q / cpr, c = 4 * (q - row * cpr);
    const float* w = wl + ((c >> lg_dh) * S) * 32 + row;
    const float* op = (const float*)a.Opart + ((int64_t)o * S * a.max_sel + min(r0 + row, a.max_sel - 1)) * D + c;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < S; s0 += 8) {
      f32x4 p[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) p[j] = gload((const f32x4*)(op + min(s0 + j, S - 1) * sst));
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // an empty split leaves its partial unwritten: its weight is 0
        const float ws = s0 + j < S ? w[32 * min(s0 + j, S - 1)] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = ws > 0.f ? fmaf(ws, p[j][e], v[e]) : v[e];
      }
    }
    *(f32x4*)(os + row * OP + c) = v;
  }
  lds_barrier();
  const float* oa = os + (16 * (wave & 1) + (lane & 15)) * OP + 4 * (lane >> 4);
  const int nu = D / 16;   // units of 16 channels (D is a multiple of 32)
  for (int cb = wave >> 1; 16 * cb < C; cb += MF_THREADS / 128) {
    const int c = 16 * cb + (lane & 15);
    const float* wo = (const float*)a.WoT + (int64_t)min(c, C - 1) * D + 4 * (lane >> 4);
    float x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      x[r] = gload((const float*)a.X + (int64_t)o * a.x_stride + (int64_t)max(cell[r], 0) * C + min(c, C - 1));
    f32x4 c0 = {}, c1 = {};   // two chains: shorter sums
    for (int u0 = 0; u0 < nu; u0 += 8) {
      f32x4 w[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = gload((const f32x4*)(wo + 16 * min(u0 + j, nu - 1)));
#pragma unroll
      for (int j = 0; j < 8; j += 2)
        if (u0 + j < nu) {
          c0 = mfma16f(*(const f32x4*)(oa + 16 * (u0 + j)), w[j], c0);
          c1 = mfma16f(*(const f32x4*)(oa + 16 * (u0 + j + 1)), w[j + 1], c1);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (cell[r] < 0 || c >= C) continue;
      // no resident key: x bit for bit
      gstore((float*)a.Y + (int64_t)o * a.y_stride + (int64_t)cell[r] * C + c,
             live[rt + r] > 0.f ? x[r] + (c0[r] + c1[r]) : x[r]);
    }
  }
}

}  // namespace rs3
