// fp32 readout (Sec. 3.1, Eq. 6): y = x + softmax(q K^T / sqrt(d_h)) V W_o with
// fp32 inputs, products and sums throughout.
//   k_qproj_f32  gather + query projection (and Eq. 7's turn), 32 rows x 32
//                columns per work-group;
//   k_attn_f32   split-KV attention on the fp32 matrix cores;
//   k_merge_f32  split merge, W_o, residual, scatter (readout_f32.h).
//   k_readout_f32 the direct form, one work-group per selected row: for calls
//                without a workspace and for head widths outside {32, 64,
//                128, 256}.  (The tiled form is the faster one down to the
//                smallest: 64 selected rows, 512 keys and one head of 64 take
//                32.4 against 41.8 us per frame.)
#include "readout_f32.h"

namespace rs3 {

// grid (n_obj, ceil(max_sel/32), ceil(D/32)), block 256.
__global__ __launch_bounds__(RF_THREADS) void k_qproj_f32(Rs3ReadoutArgs a) {
  __shared__ float red[4 * 32 * RF_PITCH];
  const int o = blockIdx.x, r0 = blockIdx.y * RF_ROWS, c0 = blockIdx.z * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5;
  const int C = a.C, D = a.D;
  const int32_t* sel = a.sel_idx + (int64_t)o * a.sel_stride;
  int cnt = gload(a.sel_count + (a.sel_stride ? o : 0));   // out of range: reported by the merge
  cnt = cnt < 0 ? 0 : min(cnt, a.max_sel);
  int src = gload(sel + min(r0 + (lane & 31), a.max_sel - 1));
  int cell = gload(sel + min(r0 + (tid >> 3), a.max_sel - 1));   // of this thread's output row
  if (r0 >= cnt) return;
  // entries past the count, and bad ones, read row 0 (their queries are unused)
  src = (uint32_t)src < (uint32_t)a.mn ? src : 0;
  cell = (uint32_t)cell < (uint32_t)a.mn ? cell : 0;
  const float* xr = (const float*)a.X + (int64_t)o * a.x_stride + (int64_t)src * C + 4 * g;
  const float* wr = (const float*)a.WqT + (int64_t)(c0 + (lane & 31)) * C + 4 * g;
  f32x16 acc = {}, acc1 = {};   // two chains: shorter sums
  const int nu = C / 8, ue = (wave + 1) * nu / 4;
  for (int u0 = wave * nu / 4; u0 < ue; u0 += 8) {
    f32x4 x[8], w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int u = min(u0 + j, nu - 1);
      x[j] = gload((const f32x4*)(xr + 8 * u));
      w[j] = gload((const f32x4*)(wr + 8 * u));
    }
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      if (u0 + j < ue) acc = mfma32f(x[j], w[j], acc);
      if (u0 + j + 1 < ue) acc1 = mfma32f(x[j + 1], w[j + 1], acc1);
    }
  }
  f32x4 q = rf_reduce(acc + acc1, red);
  const int row = r0 + (tid >> 3), c = c0 + 4 * (tid & 7);
  if (row >= cnt) return;
  if (a.rope) {
    const f32x4 f = gload((const f32x4*)(a.rope + (int64_t)cell * a.d_h + (c & (a.d_h - 1))));   // two (cos, sin)
    q = f32x4{q[0] * f[0] - q[1] * f[1], q[0] * f[1] + q[1] * f[0], q[2] * f[2] - q[3] * f[3],
              q[2] * f[3] + q[3] * f[2]};
  }
  gstore((f32x4*)((float*)a.Q + ((int64_t)o * a.max_sel + row) * D + c), q * a.qscale);
}

// grid 8*n_qt*ceil(G/8) with G = n_obj*H*S key groups, block 256.  Block b ->
// key group 8*((b>>3)/n_qt) + (b&7), 32-row query tile (b>>3) % n_qt: the
// query tiles of one key group share an XCD, whose L2 then holds its keys.
// The four waves own the same 32 queries and take the 32-key half tiles
// 4s + w, 4s + w + 4S, ... of the bank (s the split); their states merge in
// LDS and one unnormalised partial (O, m, l) per query goes to the workspace.
// As in the bf16 attention the logits are computed transposed, so that a
// query's 16 logits sit in one lane, and the weights are the B operand of
// O^T += V^T P^T straight from their registers: step r of the product takes
// the key pair that accumulator register r holds in the two lane groups, and
// the V^ tile's slot order makes eight such keys 32 consecutive bytes.
// K^ and V^ rows go straight from L2 to registers: a half tile is 64 MFMAs
// (4,096 cycles) for 16 KB of loads at d_h = 64, so the matrix cores bound it.
// At 256 queries, 4,096 keys and four heads of 64 (1.1 GFLOP) the launch takes
// about 18 us; a work-group per row with VALU dot products (k_readout_f32, now
// the direct form) took 498 us.  Loading the next half tile's K^ rows during
// the V product was slower (21.4 us: 178 registers, two waves per SIMD
// instead of three).
template <int DH>
__global__ __launch_bounds__(RF_THREADS) void k_attn_f32(Rs3ReadoutArgs a, int G, Rs3AttnBanks ab) {
  extern __shared__ __attribute__((aligned(16))) float xo[];   // [4][32][DH+4], then (m, l) [4][32][2]
  constexpr int OP = DH + 4;
  const int rest = blockIdx.x >> 3;
  const int qt = rest % a.n_qt, kvg = (rest / a.n_qt) * 8 + (blockIdx.x & 7);
  if (kvg >= G) return;
  const int S = a.S, H = a.H;
  const int s = kvg % S, oh = kvg / S, h = oh % H, o = oh / H;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = qt * RF_ROWS;
  int cnt = sload(a.sel_count + (a.sel_stride ? o : 0));
  cnt = cnt < 0 ? 0 : min(cnt, a.max_sel);
  if (row0 >= cnt) return;
  const int nh = 2 * sload(ab.hdr[o] + HDR_NTILES);   // half tiles
  float* ml = a.ML + (((int64_t)o * S + s) * a.max_sel * H + h) * 2;
  if (4 * s >= nh) {   // no keys: the empty partial
    const int row = row0 + tid;
    if (tid < RF_ROWS && row < cnt) {
      gstore(ml + (int64_t)row * H * 2, -INFINITY);
      gstore(ml + (int64_t)row * H * 2 + 1, 0.f);
    }
    return;
  }
  const float* qp = (const float*)a.Q + ((int64_t)o * a.max_sel + min(row0 + (lane & 31), a.max_sel - 1)) * a.D +
                    h * DH + 4 * g;
  f32x4 q[DH / 8];
#pragma unroll
  for (int i = 0; i < DH / 8; ++i) q[i] = gload((const f32x4*)(qp + 8 * i));
  const float* Kh = (const float*)ab.kh[o];
  const float* Vh = (const float*)ab.vh[o];
  const TileEnt* tiles = ab.tiles[o];
  f32x16 acc[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt) acc[dt] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;
  for (int u = 4 * s + wave; u < nh; u += 4 * S) {
    const int tile = sload(&tiles[u >> 1].tile);
    const uint64_t mask64 = sload(&tiles[u >> 1].mask);
    const uint32_t mask = (u & 1) ? (uint32_t)(mask64 >> 32) : (uint32_t)mask64;
    if (mask == 0u) continue;
    const int64_t tb = (int64_t)tile * H + h;
    const float* kp = Kh + (tb * KT + 32 * (u & 1) + (lane & 31)) * DH + 4 * g;
    const float* vp = Vh + (tb * DH + (lane & 31)) * KT + 32 * (u & 1) + 8 * g;
    constexpr int KB = DH / 8 < 8 ? DH / 8 : 8;
    f32x16 sc = {}, sc1 = {};   // two chains: shorter sums
#pragma unroll
    for (int i0 = 0; i0 < DH / 8; i0 += KB) {
      f32x4 k[KB];
#pragma unroll
      for (int i = 0; i < KB; ++i) k[i] = gload((const f32x4*)(kp + 8 * (i0 + i)));
#pragma unroll
      for (int i = 0; i < KB; i += 2) {
        sc = mfma32f(k[i], q[i0 + i], sc);
        sc1 = mfma32f(k[i + 1], q[i0 + i + 1], sc1);
      }
    }
    sc += sc1;
    f32x4 v[DH / 32][4];
    constexpr int VB = DH / 32 < 2 ? DH / 32 : 2;   // V^ blocks in flight under the softmax
#pragma unroll
    for (int dt = 0; dt < VB; ++dt)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[dt][j] = gload((const f32x4*)(vp + (int64_t)32 * dt * KT + 16 * (j >> 1) + 4 * (j & 1)));
    if (mask != 0xffffffffu) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (!(mask >> c_row(r, lane) & 1u)) sc[r] = -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      // 0 on a lane's first logits; while all of them are -inf (products that
      // overflow), there is nothing to scale
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
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) {
      if (dt + VB < DH / 32) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[dt + VB][j] = gload((const f32x4*)(vp + (int64_t)32 * (dt + VB) * KT + 16 * (j >> 1) + 4 * (j & 1)));
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[dt][j][e], sc[4 * j + e], acc[dt], 0, 0, 0);
    }
  }
  // the four waves' (m, l, O) of each query, merged to the largest maximum
  const auto ls = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
  float* xm = xo + 4 * 32 * OP;
  if (g == 0) {
    xm[(wave * 32 + lane) * 2] = m_run;
    xm[(wave * 32 + lane) * 2 + 1] = __uint_as_float(ls[0]) + __uint_as_float(ls[1]);
  }
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *(f32x4*)(xo + (wave * 32 + (lane & 31)) * OP + 32 * dt + 8 * q4 + 4 * g) =
          f32x4{acc[dt][4 * q4], acc[dt][4 * q4 + 1], acc[dt][4 * q4 + 2], acc[dt][4 * q4 + 3]};
  lds_barrier();
  const int rr = tid >> 3, row = row0 + rr;   // eight threads per query
  if (row >= cnt) return;
  float M = -INFINITY, L = 0.f, w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) M = fmaxf(M, xm[(i * 32 + rr) * 2]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float mi = xm[(i * 32 + rr) * 2];
    w[i] = mi == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mi - M);
    L = fmaf(w[i], xm[(i * 32 + rr) * 2 + 1], L);
  }
  if ((tid & 7) == 0) {
    gstore(ml + (int64_t)row * H * 2, M);
    gstore(ml + (int64_t)row * H * 2 + 1, L);
  }
  float* op = (float*)a.Opart + (((int64_t)o * S + s) * a.max_sel + row) * a.D + h * DH;
#pragma unroll
  for (int c = 4 * (tid & 7); c < DH; c += 32) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) v += w[i] * *(const f32x4*)(xo + (i * 32 + rr) * OP + c);
    gstore((f32x4*)(op + c), v);
  }
}

// grid (n_obj, ceil(max_sel/32)), block MF_THREADS.
__global__ __launch_bounds__(MF_THREADS) void k_merge_f32(Rs3ReadoutArgs a) {
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  merge_f32_block(a, blockIdx.x, blockIdx.y, dyn);
}

// ---------------------------------------------------------------------------
// Direct form: grid (n_obj, max_sel), block 256, one selected row per
// work-group; its four waves split the resident tiles (wave w takes tiles
// w, w+4, ...) and merge their softmax states at the end.  For row i:
//   q = qscale * x W_q              threads over the attention columns
//   per head and tile of a wave:    lanes over the tile's 64 keys: logits,
//     wave max / sum (online softmax); lanes over the head's columns:
//     o = alpha*o + sum_k p_k v_k   (weights broadcast from LDS)
//   merge of the four waves' (m, l, o) per head, then
//   y = x + (o / l) W_o             threads over the output channels
// Every load that needs only the arguments (count, header, the first tile
// entries, the list entries, W_q rows) is issued first, and a wave's first
// key and value rows (heads of at most 64 columns) before the query is
// ready, so that the row's chain of dependent loads stays short.
// LDS: x [C], q [D], o [4][D], p [4][64], (m, l) [4][H] floats.
__global__ __launch_bounds__(256) void k_readout_f32(Rs3ReadoutArgs a, Rs3AttnBanks ab) {
  extern __shared__ float sm[];
  const int o = blockIdx.x, r = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int C = a.C, D = a.D, H = a.H, d_h = a.d_h;
  float* xs = sm;
  float* q = xs + C;
  float* ow = q + D + wave * D;        // this wave's o
  float* pr = q + 5 * D + wave * 64;   // this wave's weights of one tile
  float* ml = q + 5 * D + 256;         // [4][H][2]
  int32_t* hdr = (int32_t*)ab.hdr[o];
  const TileEnt* tiles = ab.tiles[o];
  const int ntcap = ab.ntcap[o];
  int cnt = gload(a.sel_count + (a.sel_stride ? o : 0));
  const int ntiles = gload(hdr + HDR_NTILES);
  // tile entries t = wave + 4*lane (a wave's first 64 tiles)
  int c_tile = 0;
  uint32_t c_lo = 0, c_hi = 0;
  if (wave + 4 * lane < ntcap) {
    c_tile = gload(&tiles[wave + 4 * lane].tile);
    const uint64_t mm = gload(&tiles[wave + 4 * lane].mask);
    c_lo = (uint32_t)mm;
    c_hi = (uint32_t)(mm >> 32);
  }
  const int32_t* sel = a.sel_idx + (int64_t)o * a.sel_stride;
  const int rc = min(r, a.max_sel - 1);
  const int i_raw = gload(sel + rc), i_prev = rc > 0 ? gload(sel + rc - 1) : -1;
  if (cnt < 0 || cnt > a.max_sel) {
    if (r == 0 && tid == 0) set_err(hdr, RS3_E_INVALID);
    cnt = cnt < 0 ? 0 : a.max_sel;
  }
  if (r >= cnt) return;
  if (!(i_raw >= 0 && i_raw < a.mn && i_prev < i_raw)) {
    if (tid == 0) set_err(hdr, RS3_E_INVALID);
    return;
  }
  const int i = i_raw;
  const float* x = (const float*)a.X + (int64_t)o * a.x_stride + (int64_t)i * C;
  float* y = (float*)a.Y + (int64_t)o * a.y_stride + (int64_t)i * C;
  if (ntiles == 0) {
    for (int c = tid; c < C; c += 256) gstore(y + c, gload(x + c));
    return;
  }
  const float* Kh = (const float*)ab.kh[o];
  const float* Vh = (const float*)ab.vh[o];
  const bool fast = d_h <= 64 && (d_h & 3) == 0 && ntiles <= 256;
  // fast path: the key row (lane = key) and value row (lane = column) of a
  // tile of this wave, first tile in flight before the query is ready
  f32x4 kc[16], vc[16];
  auto load_tile = [&](int j, int h) {   // j: the wave's j-th tile
    const int tl = __builtin_amdgcn_readlane(c_tile, j);
    const f32x4* kr = (const f32x4*)(Kh + (((int64_t)tl * H + h) * KT + lane) * d_h);
    const f32x4* vr = (const f32x4*)(Vh + (((int64_t)tl * H + h) * d_h + min(lane, d_h - 1)) * KT);
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (4 * u < d_h) kc[u] = gload(kr + u);
      vc[u] = gload(vr + u);
    }
  };
  const int nmine = ntiles > wave ? (ntiles - wave + 3) / 4 : 0;   // this wave's tiles
  if (fast && nmine > 0) load_tile(0, 0);
  for (int c = tid; c < C; c += 256) xs[c] = gload(x + c);
  __syncthreads();
  const float* WqT = (const float*)a.WqT;
  for (int d = tid; d < D; d += 256) {
    const f32x4* wr = (const f32x4*)(WqT + (int64_t)d * C);
    float s0 = 0.f, s1 = 0.f;
    for (int c4 = 0; c4 < C / 4; c4 += 2) {
      const f32x4 w0 = gload(wr + c4), x0 = *(const f32x4*)(xs + 4 * c4);
      s0 = fmaf(x0[0], w0[0], fmaf(x0[1], w0[1], fmaf(x0[2], w0[2], fmaf(x0[3], w0[3], s0))));
      if (c4 + 1 < C / 4) {
        const f32x4 w1 = gload(wr + c4 + 1), x1 = *(const f32x4*)(xs + 4 * c4 + 4);
        s1 = fmaf(x1[0], w1[0], fmaf(x1[1], w1[1], fmaf(x1[2], w1[2], fmaf(x1[3], w1[3], s1))));
      }
    }
    q[d] = (s0 + s1) * a.qscale;
  }
  __syncthreads();
  if (a.rope) {
    // Eq. 7: turn each head's channel pairs by the factors of cell i
    const float* f = a.rope + (int64_t)i * d_h;   // d_h/2 (cos, sin) pairs
    for (int pp = tid; pp < D / 2; pp += 256) {
      const int d = 2 * pp, fp = (d % d_h) & ~1;
      const float c = gload(f + fp), sn = gload(f + fp + 1), xe = q[d], xo = q[d + 1];
      q[d] = xe * c - xo * sn;
      q[d + 1] = xe * sn + xo * c;
    }
    __syncthreads();
  }
  for (int h = 0; h < H; ++h) {
    float m_run = -INFINITY, l_run = 0.f;
    const float* qh = q + h * d_h;
    for (int dd = lane; dd < d_h; dd += 64) ow[h * d_h + dd] = 0.f;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    for (int j = 0; j < nmine; ++j) {
      const int t = wave + 4 * j;
      int etile;
      uint64_t emask;
      if (fast) {
        etile = __builtin_amdgcn_readlane(c_tile, j);
        // readlane returns an int: widen its bits, not its sign
        emask = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(c_lo, j) |
                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(c_hi, j) << 32);
        if (j > 0 || h > 0) load_tile(j, h);
      } else {
        etile = gload(&tiles[t].tile);
        emask = gload(&tiles[t].mask);
      }
      const bool valid = emask >> lane & 1ull;
      float s0 = 0.f, s1 = 0.f;
      if (fast) {
#pragma unroll
        for (int u = 0; u < 16; u += 2) {
          if (4 * u < d_h) {
            const f32x4 q0 = *(const f32x4*)(qh + 4 * u);
            s0 = fmaf(q0[0], kc[u][0], fmaf(q0[1], kc[u][1], fmaf(q0[2], kc[u][2], fmaf(q0[3], kc[u][3], s0))));
          }
          if (4 * u + 4 < d_h) {
            const f32x4 q1 = *(const f32x4*)(qh + 4 * u + 4);
            s1 = fmaf(q1[0], kc[u + 1][0], fmaf(q1[1], kc[u + 1][1], fmaf(q1[2], kc[u + 1][2], fmaf(q1[3], kc[u + 1][3], s1))));
          }
        }
      } else {
        const float* krow = Kh + (((int64_t)etile * H + h) * KT + lane) * d_h;
        for (int u = 0; u < d_h; ++u) s0 = fmaf(qh[u], gload(krow + u), s0);
      }
      const float s = valid ? s0 + s1 : -INFINITY;
      const float mx = wave_max(s);
      if (mx == -INFINITY) continue;   // no resident key in the tile
      const float m_new = fmaxf(m_run, mx);
      const float alpha = exp2f(m_run - m_new);   // 0 on the wave's first keys
      const float p = valid ? exp2f(s - m_new) : 0.f;
      l_run = l_run * alpha + wave_sum(p);
      m_run = m_new;
      pr[lane] = p;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      // slot quad 4j of a V^ row holds the key quad vslot(4j) (the slot
      // permutation swaps whole quads and is its own inverse)
      if (fast) {
        if (lane < d_h) {
          float acc = ow[h * d_h + lane] * alpha;
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            const f32x4 pk = *(const f32x4*)(pr + vslot(4 * u));
            acc = fmaf(pk[0], vc[u][0], fmaf(pk[1], vc[u][1], fmaf(pk[2], vc[u][2], fmaf(pk[3], vc[u][3], acc))));
          }
          ow[h * d_h + lane] = acc;
        }
      } else {
        for (int dd = lane; dd < d_h; dd += 64) {
          const float* vr = Vh + (((int64_t)etile * H + h) * d_h + dd) * KT;
          float acc = ow[h * d_h + dd] * alpha;
          for (int k = 0; k < KT; ++k) acc = fmaf(pr[vslot(k)], gload(vr + k), acc);
          ow[h * d_h + dd] = acc;
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    if (lane == 0) {
      ml[(wave * H + h) * 2] = m_run;
      ml[(wave * H + h) * 2 + 1] = l_run;
    }
  }
  __syncthreads();
  // merge the waves' states into q's place: o = sum_w e^(m_w - M) o_w / sum_w e^(m_w - M) l_w
  float* of = q;
  for (int d = tid; d < D; d += 256) {
    const int h = d / d_h;
    float M = -INFINITY;
    for (int w = 0; w < 4; ++w) M = fmaxf(M, ml[(w * H + h) * 2]);
    float num = 0.f, den = 0.f;
    if (M != -INFINITY)
      for (int w = 0; w < 4; ++w) {
        const float mw = ml[(w * H + h) * 2];
        if (mw == -INFINITY) continue;
        const float sc = exp2f(mw - M);
        num = fmaf(sc, q[D + w * D + d], num);
        den = fmaf(sc, ml[(w * H + h) * 2 + 1], den);
      }
    of[d] = den > 0.f ? num / den : 0.f;
  }
  __syncthreads();
  const float* WoT = (const float*)a.WoT;
  for (int c = tid; c < C; c += 256) {
    const f32x4* wr = (const f32x4*)(WoT + (int64_t)c * D);
    float s0 = 0.f, s1 = 0.f;
    for (int d4 = 0; d4 < D / 4; d4 += 2) {
      const f32x4 w0 = gload(wr + d4), o0 = *(const f32x4*)(of + 4 * d4);
      s0 = fmaf(o0[0], w0[0], fmaf(o0[1], w0[1], fmaf(o0[2], w0[2], fmaf(o0[3], w0[3], s0))));
      if (d4 + 1 < D / 4) {
        const f32x4 w1 = gload(wr + d4 + 1), o1 = *(const f32x4*)(of + 4 * d4 + 4);
        s1 = fmaf(o1[0], w1[0], fmaf(o1[1], w1[1], fmaf(o1[2], w1[2], fmaf(o1[3], w1[3], s1))));
      }
    }
    gstore(y + c, xs[c] + (s0 + s1));
  }
}

}  // namespace rs3

using namespace rs3;

template <int DH>
static constexpr size_t attn_f32_lds() {
  return (size_t)(4 * 32 * (DH + 4) + 4 * 32 * 2) * 4;
}

hipError_t rs3_readout_f32_setup() {
  const struct {
    const void* f;
    size_t bytes;
  } ks[] = {{(const void*)k_attn_f32<32>, attn_f32_lds<32>()},
            {(const void*)k_attn_f32<64>, attn_f32_lds<64>()},
            {(const void*)k_attn_f32<128>, attn_f32_lds<128>()},
            {(const void*)k_attn_f32<256>, attn_f32_lds<256>()},
            {(const void*)k_merge_f32, merge_f32_lds(1024, RS3_F32_MAX_SPLITS_X_HEADS)}};
  for (const auto& k : ks) {
    hipError_t e = hipFuncSetAttribute(k.f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Projection and attention; the merge follows (rs3_launch_merge_f32 or the
// fused merge + commit).
hipError_t rs3_launch_attn_f32(const Rs3ReadoutArgs& a, const Rs3AttnBanks& ab, hipStream_t st) {
  const int n_qt = (a.max_sel + RF_ROWS - 1) / RF_ROWS;
  RS3_LAUNCH(RS3_K_QPROJ, st, k_qproj_f32, dim3(a.n_obj, n_qt, a.D / 32), dim3(RF_THREADS), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int G = a.n_obj * a.H * a.S;
  const dim3 grid(8 * n_qt * ((G + 7) / 8)), blk(RF_THREADS);
  switch (a.d_h) {
    case 32: RS3_LAUNCH(RS3_K_ATTN, st, k_attn_f32<32>, grid, blk, attn_f32_lds<32>(), st, a, G, ab); break;
    case 64: RS3_LAUNCH(RS3_K_ATTN, st, k_attn_f32<64>, grid, blk, attn_f32_lds<64>(), st, a, G, ab); break;
    case 128: RS3_LAUNCH(RS3_K_ATTN, st, k_attn_f32<128>, grid, blk, attn_f32_lds<128>(), st, a, G, ab); break;
    case 256: RS3_LAUNCH(RS3_K_ATTN, st, k_attn_f32<256>, grid, blk, attn_f32_lds<256>(), st, a, G, ab); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t rs3_launch_merge_f32(const Rs3ReadoutArgs& a, hipStream_t st) {
  RS3_LAUNCH(RS3_K_COMBINE, st, k_merge_f32, dim3(a.n_obj, (a.max_sel + RF_ROWS - 1) / RF_ROWS), dim3(MF_THREADS),
             merge_f32_lds(a.D, a.H * a.S), st, a);
  return hipGetLastError();
}

hipError_t rs3_launch_readout_f32_direct(const Rs3ReadoutArgs& a, const Rs3AttnBanks& ab, hipStream_t st) {
  const size_t lds = (size_t)(a.C + 5 * a.D + 256 + 8 * a.H) * 4;
  RS3_LAUNCH(RS3_K_READOUT_F32, st, k_readout_f32, dim3(a.n_obj, a.max_sel), dim3(256), lds, st, a, ab);
  return hipGetLastError();
}
