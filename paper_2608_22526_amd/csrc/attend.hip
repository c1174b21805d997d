// Bare attention core of the readout (Eq. 6 without the projections):
// O_h = softmax(Q_h K_h^T / sqrt(d_h)) V_h on already-projected tensors.
//
// bf16: the tensors are laid out as a one-frame bank in the caller's
// workspace (k_attend_prep), the readout's split-KV attention kernel runs on
// it unchanged, and k_attend_merge combines the key splits into fp32 O.
// fp32: k_attend_f32_tile, 32 queries of a head per work-group on the matrix
// cores; k_attend_f32, one work-group per query row and FMA loops, for head
// widths outside {32, 64, 128}.
#include "device_util.h"

namespace rs3 {

// grid (max(ntile*H, nqb), 2), block 256.
//  y = 0: block (tile t, head h) copies keys 64t..64t+63 of head h into the
//         K^ tile ([64][d_h]) and, transposed in LDS so that every store is 16
//         bytes of a row, the V^ tile ([d_h][64] in slot order), zero-filling
//         past n_kv (28,672 keys, two heads of 128: 10.8 us; 2-byte stores
//         of each value took 21.4); (t, 0) writes the tile's list entry, and
//         block (0, 0) the bank descriptor, header and query count.
//  y = 1: block b scales 256 chunks of 8 query values by qscale into Qs.
__global__ __launch_bounds__(256) void k_attend_prep(AttendPrepArgs p) {
  const int tid = threadIdx.x;
  const int D = p.H * p.d_h;
  if (blockIdx.y == 1) {
    const int64_t chunk = (int64_t)blockIdx.x * 256 + tid;
    if (chunk * 8 >= (int64_t)p.n_q * D) return;
    const u32x4 v = *(const u32x4*)(p.Q + chunk * 8);
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = pack_bf16x2(__uint_as_float(v[e] << 16) * p.qscale, __uint_as_float(v[e] & 0xffff0000u) * p.qscale);
    *(u32x4*)(p.Qs + chunk * 8) = w;
    return;
  }
  if (blockIdx.x == 0 && tid == 0) {
    BankDev d = {};
    d.cap = p.ntile * KT;
    d.f_max = 1;
    d.n_pin = 0;
    d.d_kv = p.d_h;
    d.H = p.H;
    d.d_h = p.d_h;
    d.dtype = RS3_BF16;
    d.n_tiles_cap = p.ntile;
    d.Khat = p.Khat;
    d.Vhat = p.Vhat;
    d.hdr = p.hdr;
    d.tiles = p.tiles;
    *p.desc = d;
    for (int w = 0; w < HDR_WORDS; ++w) p.hdr[w] = 0;
    p.hdr[HDR_NTILES] = p.ntile;
    p.hdr[HDR_NKEYS] = (int)p.n_kv;
    p.hdr[HDR_PLEN] = -1;
    *p.count = p.n_q;
  }
  const int t = blockIdx.x / p.H, h = blockIdx.x - t * p.H;
  if (t >= p.ntile) return;
  const int d_h = p.d_h, cpr = d_h / 8, n = KT * cpr, pitch = d_h / 2 + 1;
  bf16_t* kt = p.Khat + ((int64_t)t * p.H + h) * KT * d_h;
  bf16_t* vt = p.Vhat + ((int64_t)t * p.H + h) * d_h * KT;
  extern __shared__ uint32_t sv[];   // V rows [64][pitch]
  for (int q0 = tid; q0 < n; q0 += 512) {
    u32x4 kv[2], vv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {   // keys past n_kv read the last one, without a branch
      const int q = min(q0 + 256 * i, n - 1);
      const int64_t j = (int64_t)t * KT + q / cpr, at = ((j < p.n_kv ? j : p.n_kv - 1) * p.H + h) * d_h + 8 * (q % cpr);
      kv[i] = gload((const u32x4*)(p.K + at));
      vv[i] = gload((const u32x4*)(p.V + at));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = q0 + 256 * i, r = q / cpr, c = q - r * cpr;
      if (q >= n) break;
      if ((int64_t)t * KT + r >= p.n_kv) kv[i] = vv[i] = u32x4{0, 0, 0, 0};
      gstore((u32x4*)(kt + r * d_h + 8 * c), kv[i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) sv[r * pitch + 4 * c + e] = vv[i][e];
    }
  }
  __syncthreads();
  const bf16_t* sh = (const bf16_t*)sv;
  for (int q = tid; q < 8 * d_h; q += 256) {   // channel q/8, slots 8*(q%8) .. +7; vslot is its own inverse
    const int d = q >> 3, s0 = 8 * (q & 7);
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = sh[2 * pitch * vslot(s0 + 2 * e) + d] | (uint32_t)sh[2 * pitch * vslot(s0 + 2 * e + 1) + d] << 16;
    gstore((u32x4*)(vt + 8 * (int64_t)q), w);
  }
  if (h == 0 && tid == 0) {
    const int64_t left = p.n_kv - (int64_t)t * KT;
    TileEnt e;
    e.tile = t;
    e.pad = 0;
    e.mask = left >= KT ? ~0ull : ((1ull << left) - 1ull);
    p.tiles[t] = e;
  }
}

// One thread per (query row, 8-column chunk): online log-sum-exp merge of
// the SA key splits into fp32 O [n_q][D].
__global__ __launch_bounds__(256) void k_attend_merge(Rs3ReadoutArgs a, int SA, float* O) {
  const int D = a.D, cpr = D / 8;
  const int64_t it = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (it >= (int64_t)a.max_sel * cpr) return;
  const int row = (int)(it / cpr), d0 = 8 * (int)(it - (int64_t)row * cpr), h = d0 / a.d_h;
  float M = -INFINITY, W = 0.f;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int s = 0; s < SA; ++s) {
    const int64_t prow = (int64_t)s * a.max_sel + row;
    const float m = a.ML[(prow * a.H + h) * 2], l = a.ML[(prow * a.H + h) * 2 + 1];
    if (!(l > 0.f)) continue;
    const u32x4 v = *(const u32x4*)((const bf16_t*)a.Opart + prow * D + d0);
    if (m > M) {
      const float sc = __builtin_amdgcn_exp2f(M - m);
      W *= sc;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] *= sc;
      M = m;
    }
    float w = __builtin_amdgcn_exp2f(m - M) * part_sum(l);
    W += w;
    w *= part_scale(l);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += w * part_lo<true>(v[e]);
      acc[2 * e + 1] += w * part_hi<true>(v[e]);
    }
  }
  const float inv = W > 0.f ? 1.f / W : 0.f;
  float* out = O + (int64_t)row * D + d0;
  *(f32x4*)out = f32x4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
  *(f32x4*)(out + 4) = f32x4{acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv};
}

// fp32 on the matrix cores: grid (ceil(n_q/32), H), NW waves, no workspace.  The
// waves own the same 32 queries of one head and take the 32-key groups w, w +
// NW, ...; as in k_attn_f32 the logits are computed transposed and the weights
// feed the value product from their registers, accumulator register r holding
// keys 8*(r/4) + 4*(lane/32) + r%4.  Keys and values come straight from the
// caller's rows: a key row per lane in 16-byte chunks, the values of one key and
// 32 channels per load.  Keys past n_kv re-read the last one with weight 0.  The
// waves' states merge in LDS.  Bound by the latency of the loads (few waves per
// work-group, their loads of one 32-key group in flight); 173 queries, 723 keys,
// four heads of 64: 628 us with a work-group per query, 23 us here; 2,048 x 2,048,
// four heads of 128: 5,727 and 111 us (77 TFLOP/s); 4 x 7,000, one head of 64:
// 1,478 and 158 us.
template <int DH, int NW>
__global__ __launch_bounds__(64 * NW, DH <= 32 ? 4 : 2) void k_attend_f32_tile(const float* Q, const float* K, const float* V, int n_q,
                                                             int64_t n_kv, int H, float qscale, float* O) {
  constexpr int OP = DH + 4;
  extern __shared__ __attribute__((aligned(16))) float xo[];   // [NW][32][OP], then (m, l) [NW][32][2]
  const int h = blockIdx.y, row0 = blockIdx.x * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5, l31 = lane & 31;
  const int64_t D = (int64_t)H * DH;
  const float* qp = Q + min(row0 + l31, n_q - 1) * D + h * DH + 4 * g;
  f32x4 q[DH / 8];
#pragma unroll
  for (int i = 0; i < DH / 8; ++i) q[i] = gload((const f32x4*)(qp + 8 * i)) * qscale;
  f32x16 acc[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt) acc[dt] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;
  for (int64_t j0 = 32 * wave; j0 < n_kv; j0 += 32 * NW) {
    const int64_t jk = j0 + l31 < n_kv ? j0 + l31 : n_kv - 1;
    const float* kp = K + jk * D + h * DH + 4 * g;
    f32x16 s0 = {}, s1 = {};   // two chains: shorter sums
    constexpr int KB = DH / 8 < 8 ? DH / 8 : 8;
#pragma unroll
    for (int i0 = 0; i0 < DH / 8; i0 += KB) {
      f32x4 k[KB];
#pragma unroll
      for (int i = 0; i < KB; ++i) k[i] = gload((const f32x4*)(kp + 8 * (i0 + i)));
#pragma unroll
      for (int i = 0; i < KB; i += 2) {
        s0 = mfma32f(k[i], q[i0 + i], s0);
        s1 = mfma32f(k[i + 1], q[i0 + i + 1], s1);
      }
    }
    f32x16 sc = s0 + s1;
    if (n_kv - j0 < 32) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (c_row(r, lane) >= (int)(n_kv - j0)) sc[r] = -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      // 0 on a lane's first logits; while it has none, there is nothing to scale
      const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt) acc[dt] *= alpha;
      m_run = m_new;
    }
    const float m_use = m_run == -INFINITY ? 0.f : m_run;   // every logit so far -inf: weights 0
    float ls4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sc[r] = __builtin_amdgcn_exp2f(sc[r] - m_use);
      ls4[r & 3] += sc[r];
    }
    l_run += (ls4[0] + ls4[1]) + (ls4[2] + ls4[3]);
    const float* vp = V + h * DH + l31;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) {
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t j = j0 + c_row(r, lane);
        v[r] = gload(vp + (j < n_kv ? j : n_kv - 1) * D + 32 * dt);
      }
      if (n_kv - j0 < 32) {   // a repeated key adds 0 whatever its value is
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (c_row(r, lane) >= (int)(n_kv - j0)) v[r] = 0.f;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[r], sc[r], acc[dt], 0, 0, 0);
    }
  }
  const auto ls = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
  float* xm = xo + NW * 32 * OP;
  if (g == 0) {
    xm[(wave * 32 + l31) * 2] = m_run;
    xm[(wave * 32 + l31) * 2 + 1] = __uint_as_float(ls[0]) + __uint_as_float(ls[1]);
  }
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *(f32x4*)(xo + (wave * 32 + l31) * OP + 32 * dt + 8 * q4 + 4 * g) =
          f32x4{acc[dt][4 * q4], acc[dt][4 * q4 + 1], acc[dt][4 * q4 + 2], acc[dt][4 * q4 + 3]};
  lds_barrier();
  for (int it = tid; it < 32 * (DH / 4); it += 64 * NW) {
    const int rr = it / (DH / 4), c = 4 * (it % (DH / 4)), row = row0 + rr;
    if (row >= n_q) continue;
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) M = fmaxf(M, xm[(i * 32 + rr) * 2]);
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const float mi = xm[(i * 32 + rr) * 2], li = xm[(i * 32 + rr) * 2 + 1];
      if (mi == -INFINITY && li == 0.f) continue;   // a wave without keys
      const float w = __builtin_amdgcn_exp2f(mi - M);
      L = fmaf(w, li, L);
      o += w * *(const f32x4*)(xo + (i * 32 + rr) * OP + c);
    }
    gstore((f32x4*)(O + row * D + h * DH + c), L > 0.f ? o / L : f32x4{0.f, 0.f, 0.f, 0.f});
  }
}

// The other head widths: grid n_q, block 256; per head, online softmax over
// 64-key tiles.
__global__ __launch_bounds__(256) void k_attend_f32(const float* Q, const float* K, const float* V, int n_q,
                                                    int64_t n_kv, int H, int d_h, float qscale, float* O) {
  __shared__ float q[256];
  __shared__ float pr[KT];
  __shared__ float st[4];   // running max, running sum, rescale factor
  const int r = blockIdx.x, tid = threadIdx.x, D = H * d_h;
  float* out = O + (int64_t)r * D;
  for (int h = 0; h < H; ++h) {
    for (int u = tid; u < d_h; u += 256) q[u] = Q[(int64_t)r * D + h * d_h + u] * qscale;
    if (tid == 0) {
      st[0] = -INFINITY;
      st[1] = 0.f;
    }
    float acc = 0.f;   // thread tid < d_h owns output column tid
    __syncthreads();
    for (int64_t j0 = 0; j0 < n_kv; j0 += KT) {
      if (tid < KT) {
        float s = -INFINITY;
        if (j0 + tid < n_kv) {
          const float* kr = K + ((j0 + tid) * H + h) * d_h;
          s = 0.f;
          for (int u = 0; u < d_h; ++u) s = fmaf(q[u], kr[u], s);
        }
        pr[tid] = s;
      }
      __syncthreads();
      if (tid == 0) {
        float mx = -INFINITY;
        for (int j = 0; j < KT; ++j) mx = fmaxf(mx, pr[j]);
        const float m_new = fmaxf(st[0], mx);
        const float alpha = exp2f(st[0] - m_new);
        float ps = 0.f;
        for (int j = 0; j < KT; ++j) {
          const float pj = exp2f(pr[j] - m_new);
          pr[j] = pj;
          ps += pj;
        }
        st[1] = st[1] * alpha + ps;
        st[0] = m_new;
        st[2] = alpha;
      }
      __syncthreads();
      if (tid < d_h) {
        acc *= st[2];
        const int64_t nk = n_kv - j0 < KT ? n_kv - j0 : KT;
        for (int j = 0; j < nk; ++j) acc = fmaf(pr[j], V[((j0 + j) * H + h) * d_h + tid], acc);
      }
      __syncthreads();
    }
    if (tid < d_h) out[h * d_h + tid] = st[1] > 0.f ? acc / st[1] : 0.f;
    __syncthreads();
  }
}

}  // namespace rs3

using namespace rs3;

hipError_t rs3_launch_attend_prep(const AttendPrepArgs& p, hipStream_t st) {
  const int D = p.H * p.d_h;
  const int64_t nqb = ((int64_t)p.n_q * D / 8 + 255) / 256;
  const int64_t nx = (int64_t)p.ntile * p.H > nqb ? (int64_t)p.ntile * p.H : nqb;
  if (nx == 0) {
    // nothing to lay out but the descriptor: one block writes it
    hipLaunchKernelGGL(k_attend_prep, dim3(1, 1), dim3(256), 0, st, p);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_attend_prep, dim3((unsigned)nx, 2), dim3(256), KT * (p.d_h + 2) * 2, st, p);
  return hipGetLastError();
}

hipError_t rs3_launch_attend_merge(const Rs3ReadoutArgs& a, int SA, float* O, hipStream_t st) {
  const int64_t items = (int64_t)a.max_sel * (a.D / 8);
  if (items == 0) return hipSuccess;
  hipLaunchKernelGGL(k_attend_merge, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, a, SA, O);
  return hipGetLastError();
}

hipError_t rs3_launch_attend_f32(const float* Q, const float* K, const float* V, int n_q, int64_t n_kv, int H,
                                 int d_h, float qscale, float* O, hipStream_t st) {
  if (n_q == 0) return hipSuccess;
  // The general form takes the other head widths, no keys, and more heads than
  // a grid's second dimension holds.
  if (n_kv > 0 && H <= 65535 && (d_h == 32 || d_h == 64 || d_h == 128)) {
    constexpr int NW = 8;
    const dim3 grid((n_q + 31) / 32, H), blk(64 * NW);
    const size_t lds = (size_t)NW * 32 * (d_h + 4 + 2) * 4;
    if (d_h == 32)
      hipLaunchKernelGGL((k_attend_f32_tile<32, NW>), grid, blk, lds, st, Q, K, V, n_q, n_kv, H, qscale, O);
    else if (d_h == 64)
      hipLaunchKernelGGL((k_attend_f32_tile<64, NW>), grid, blk, lds, st, Q, K, V, n_q, n_kv, H, qscale, O);
    else
      hipLaunchKernelGGL((k_attend_f32_tile<128, NW>), grid, blk, lds, st, Q, K, V, n_q, n_kv, H, qscale, O);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_attend_f32, dim3(n_q), dim3(256), 0, st, Q, K, V, n_q, n_kv, H, d_h, qscale, O);
  return hipGetLastError();
}

hipError_t rs3_attend_setup() {
  const struct {
    const void* f;
    int d_h;
  } ks[] = {{(const void*)k_attend_f32_tile<32, 8>, 32},
            {(const void*)k_attend_f32_tile<64, 8>, 64},
            {(const void*)k_attend_f32_tile<128, 8>, 128}};
  for (const auto& k : ks) {
    hipError_t e = hipFuncSetAttribute(k.f, hipFuncAttributeMaxDynamicSharedMemorySize, 8 * 32 * (k.d_h + 6) * 4);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
