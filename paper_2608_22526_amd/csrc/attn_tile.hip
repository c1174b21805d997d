// Split-KV flash attention of launches with many work-groups (bf16): the
// partials of every (object, head, key split) for the readout's merge.
//
// Each of the NW waves of a work-group owns 32 queries and visits the split's
// 64-key tiles whole: logits S^T = K^ Q~^T of both halves, the weights, O^T +=
// V^ P^T; the scalar work, the wait and the barrier of a tile are paid once
// per 64 keys.  (The form this replaces took half tiles: 84 scalar
// instructions beside 64 vector ones and 4 MFMAs per half tile at d_h = 32.)
//
// Softmax.  The logit product starts from -m (m the lane's reference) as its
// accumulator input, so the exponentials need no subtraction.  m is the maximum
// of the split's first tile.  A weight 2^x above it is as good as one below (bf16
// weights and fp32 sums have the same exponent range), so the loop needs no
// maximum and no rescale per tile, only the test of a sum that it needs anyway:
// where a lane's 32 weights of a tile sum to SUM_MOVE, the reference moves to
// that tile's maximum and its weights are computed once more from the logits
// still in registers.  Whether a query's reference moves depends on that query
// alone.
//
// Precision.  Against a fixed reference a query's largest weight is one more
// rounded number, where a reference at the maximum makes it exactly 1.  Moving
// the reference whenever a tile outweighs those before it mends that, but costs
// half a tile each time, on which the other waves of the work-group wait (five
// frames of a 128x128 grid with eight heads of 32: 1,837 instead of 1,626 us).
// The larger error is that of the partials in bf16, so they are f16 at a scale of
// the row's own instead (part_sum in device_util.h).  Rounding error of weights
// and partials, relative to a reference moved per half tile in steps of at least
// 2^8 with bf16 partials (fp64 model, logits of deviation 2 to 6, 3,840 to 32,768
// keys): this form 0.43 to 0.68, with bf16 partials 1.02 to 1.10.  On the chip,
// 4,096 queries against 28,672 keys, two heads of 128: 0.00402 off here, the
// half-tile form 0.00425, the fixed reference with bf16 partials 0.00434.
//
// What bounds it: instruction issue.  Measured per SIMD (cycles at 2.4 GHz,
// four waves): v_exp_f32 8.7, other VALU 5.6, a 32x32x16 MFMA 35; one wave
// alone issues a VALU instruction every 12.  A 64-key tile of 32 queries has
// 32 exponentials, 16 conversions and 16 sums whatever the head width (about
// 510 cycles) beside 8 MFMAs (280) at d_h = 32, 32 (1,120) at 128.  So the
// form keeps the registers of one query tile per wave (four, three and two
// waves per SIMD at d_h = 32, 64 and 128).  Measured, against the half-tile
// form: 128x128 grid, eight heads of 32, 16 frames 648 -> 453 us; 64 objects,
// one head of 64 160 -> 102 us; 4,096 queries, 28,672 keys, two heads of 128 236
// -> 125 us (0.96 PFLOP/s, where a large matrix product reaches 1.24 on this
// chip); 900 queries, 6.7 k keys, one head of 256 25 -> 21 us.  Tried on one
// machine, slower: two query tiles per wave (two waves per SIMD at d_h = 32 and
// 64: 24 % and 22 %), the row sums as a product with ones (5 %), the halves one
// after the other (0-5 %).
//
// LDS: NST stages of one tile, K^ as 64 rows (keys) x DH and V^ as DH rows x
// 64 keys (slot order), without padding: 16-byte chunk c of row r lies at
// chunk c ^ f(r), so that the 16 rows of one LDS cycle fall on the 16 groups
// of four banks.  The swizzle is in the global source address of the
// direct-to-LDS loads, whose LDS destinations are consecutive.
#include "attn_util.h"

namespace rs3 {

// Sum of a lane's 32 weights of a tile from which on the reference moves.
constexpr float SUM_MOVE = 0x1p20f;
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

template <int DH>
struct TileLds {
  static constexpr int CPR = DH / 8;              // chunks per K^ row
  static constexpr int VOFF = 64 * DH * 2;        // V^ tile, bytes
  static constexpr int STAGE = 2 * VOFF;
  // swizzle of K^ row r: with CPR chunks per row, 16/CPR rows share 256 bytes
  static __device__ __forceinline__ int fk(int r) { return CPR >= 16 ? r & 15 : (r / (16 / CPR)) & (CPR - 1); }
  static __device__ __forceinline__ int fv(int d) { return (d >> 1) & 7; }
};

// grid 8*n_qt*ceil(G/8), G = n_obj*H*S key groups, block 64*NW; block b -> key
// group 8*((b>>3)/n_qt) + (b&7), query tile (b>>3) % n_qt: the query tiles of
// one key group share an XCD and its L2, and start at staggered tiles of the
// split so that they do not wait on the same misses.
template <int DH, int NW, int NST>
__global__ __launch_bounds__(64 * NW, DH <= 32 ? 4 : DH <= 64 ? 3 : DH <= 128 ? 2 : 1) void k_attn_tile(Rs3ReadoutArgs a, int G, int n_qt,
                                                                          Rs3AttnBanks ab) {
  using L = TileLds<DH>;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];   // NST * L::STAGE bytes
  constexpr int NKS = DH / 16, NDT = DH / 32;
  constexpr int NL = L::VOFF / (1024 * NW);   // K^ loads per wave and stage; as many of V^
  static_assert(NL >= 1 && NL * 1024 * NW == L::VOFF, "whole loads");
  const int rest = blockIdx.x >> 3;
  const int qt0 = rest % n_qt, kvg = (rest / n_qt) * 8 + (blockIdx.x & 7);
  if (kvg >= G) return;
  const int S = a.S, H = a.H;
  const int s = kvg % S, oh = kvg / S, h = oh % H, o = oh / H;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l31 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = (qt0 * NW + wave) * 32, row = row0 + l31;   // this wave's first query, this lane's
  int cnt = sload(a.sel_count + (a.sel_stride ? o : 0));   // out of range: reported by the merge
  cnt = cnt < 0 ? 0 : min(cnt, a.max_sel);
  if (qt0 * NW * 32 >= cnt) return;
  const int ntiles = sload(ab.hdr[o] + HDR_NTILES);
  const int tps = split_tiles(ntiles, S);
  const int tb = min(s * tps, ntiles), te = min(tb + tps, ntiles), nt = te - tb;
  float* ml = a.ML + (((int64_t)o * S + s) * a.max_sel * H + h) * 2;
  if (nt <= 0) {   // a split without tiles: the empty partial for each of its rows
    if (g == 0 && row < cnt) {
      ml[(int64_t)row * H * 2] = -INFINITY;
      ml[(int64_t)row * H * 2 + 1] = 0.f;
    }
    return;
  }
  const bf16_t* qp = (const bf16_t*)a.Q + ((int64_t)o * a.max_sel + min(row, a.max_sel - 1)) * a.D + h * DH + 8 * g;
  // rows past the count have no query in the workspace: theirs are 0, since
  // what lies there must decide nothing for the rows beside them
  u32x4 q[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) q[ks] = gload((const u32x4*)(qp + 16 * ks));
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) q[ks] = row < cnt ? q[ks] : u32x4{0, 0, 0, 0};
  const TileEnt* tiles = ab.tiles[o];
  const bf16_t* Kh = (const bf16_t*)ab.kh[o] + (int64_t)h * KT * DH;
  const bf16_t* Vh = (const bf16_t*)ab.vh[o] + (int64_t)h * KT * DH;
  // source offsets (elements) of this lane's direct-to-LDS loads: load i
  // covers chunks (i*NW + wave)*64 .. +63 of the tile, whole 16-row periods
  // of the swizzle further on (every second load at d_h = 256)
  constexpr int KP = (NW * 64 / L::CPR) % 16 == 0 ? 1 : 2;
  int koff[KP], voff;
#pragma unroll
  for (int i = 0; i < KP; ++i) {
    const int p = (i * NW + wave) * 64 + lane, r = p / L::CPR, c = p % L::CPR;
    koff[i] = (r * L::CPR + (c ^ L::fk(r))) * 8;
  }
  {
    const int p = wave * 64 + lane, r = p >> 3, c = p & 7;
    voff = r * KT + (c ^ L::fv(r)) * 8;
  }
  // The split's tile entries, one per lane (a window of 64), read back with
  // readlane: no metadata loads in the loop, which would drain the prefetch.
  // The visiting order rotates with the query tile (splits of one window).
  int cbase = tb, c_tile = 0;
  uint32_t c_mlo = 0, c_mhi = 0;
  auto window = [&]() {
    c_tile = 0;
    c_mlo = c_mhi = 0;
    if (cbase + lane < te) {
      c_tile = gload(&tiles[cbase + lane].tile);
      const uint64_t m = gload(&tiles[cbase + lane].mask);
      c_mlo = (uint32_t)m;
      c_mhi = (uint32_t)(m >> 32);
    }
    settle(c_tile, c_mlo, c_mhi);
  };
  window();
  const int rot = nt <= 64 ? ((qt0 & 7) * nt) >> 3 : 0;
  auto at = [&](int j) { const int v = j + rot; return tb + (v >= nt ? v - nt : v); };
  auto issue = [&](int j, int slot) {   // j: visited tile; its entry is in the window
    const int tile = __builtin_amdgcn_readlane(c_tile, at(j) - cbase);
    const int64_t base = (int64_t)tile * H * (KT * DH);
    const bf16_t* kg = Kh + base;
    const bf16_t* vg = Vh + base;
    uint8_t* st = lds + slot * L::STAGE + wave * 1024;
#pragma unroll
    for (int i = 0; i < NL; ++i)
      dma16(kg + (i / KP) * KP * NW * 512 + koff[i % KP], st + i * NW * 1024);
#pragma unroll
    for (int i = 0; i < NL; ++i) dma16(vg + i * NW * 512 + voff, st + L::VOFF + i * NW * 1024);
  };
  // LDS addresses of this lane's operands: K^ row l31 (+32), chunk 2 ks + g;
  // V^ row l31 (+32 dt), chunk 2 step + g
  int ka[NKS], va[4];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) ka[ks] = l31 * DH * 2 + (((2 * ks) ^ g ^ L::fk(l31)) << 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) va[i] = L::VOFF + l31 * 128 + (((2 * i) ^ g ^ L::fv(l31)) << 4);

  f32x16 acc[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt) acc[dt] = f32x16{};
  float m_run = 0.f, l_run = 0.f;
  bool unseen = true;   // no finite logit so far: the reference is still to be set
  constexpr bool BIAS = DH <= 128;   // -m kept as an accumulator input (16 registers)
  f32x16 nm = {};
#pragma unroll
  for (int j = 0; j < NST - 1; ++j)
    if (j < nt) issue(j, j);
  int slot = 0;
  for (int j = 0; j < nt; ++j) {
    wait_stages<2 * NL, NST - 2>(min(NST - 2, nt - 1 - j));   // stages that may still be in flight
    stage_barrier();
    const int idx = at(j) - cbase;
    const uint32_t mk[2] = {(uint32_t)__builtin_amdgcn_readlane(c_mlo, idx),
                            (uint32_t)__builtin_amdgcn_readlane(c_mhi, idx)};
    if (j + NST - 1 < nt) {
      if (at(j + NST - 1) - cbase >= 64) {   // (splits longer than the window) slide it to this tile
        wait_vmcnt<0>();
        cbase = at(j);
        window();
      }
      issue(j + NST - 1, slot == 0 ? NST - 1 : slot - 1);
    }
    uint8_t* st = lds + slot * L::STAGE;
    slot = slot == NST - 1 ? 0 : slot + 1;
    // logits of both halves, less the reference; -inf where not resident
    f32x16 sc[2];
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) {
      constexpr int KB = NKS < 4 ? NKS : 4;
#pragma unroll
      for (int k0 = 0; k0 < NKS; k0 += KB) {
        u32x4 kf[KB];
#pragma unroll
        for (int i = 0; i < KB; ++i) kf[i] = *(const u32x4*)(st + ka[k0 + i] + kh * 32 * DH * 2);
#pragma unroll
        for (int i = 0; i < KB; ++i) {
          if (k0 + i == 0)
            sc[kh] = mfma32(kf[i], q[0], BIAS ? nm : f32x16{});
          else
            sc[kh] = mfma32(kf[i], q[k0 + i], sc[kh]);
        }
      }
      if (mk[kh] != 0xffffffffu) {   // frame boundary
        const uint32_t m = mk[kh] >> (4 * g);
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[kh][r] = m >> (8 * (r >> 2) + (r & 3)) & 1u ? sc[kh][r] : -INFINITY;
        // a half without resident rows may hold values that are no numbers,
        // which a weight of 0 does not hide: each wave clears its V^ for itself
        // (all write the same; a branch in the product took up to 9 %)
        if (mk[kh] == 0u) {
          int l = lane;
          asm volatile("" : "+v"(l));   // the addresses are not worth registers across the loop
          for (int i = l; i < DH * 4; i += 64) {
            const int d = i >> 2, c = 4 * kh + (i & 3);
            *(u32x4*)(st + L::VOFF + d * 128 + ((c ^ L::fv(d)) << 4)) = u32x4{0, 0, 0, 0};
          }
        }
      }
    }
    // The first value operands in flight during the weights, whose test keeps the
    // compiler from loading them there: 350 -> 345 us per six frames with a head
    // of 256, 127 -> 125 at two heads of 128; at 64 their registers cost more.
    constexpr int NP = DH <= 32 ? 1 : DH <= 64 ? 0 : 4;
    u32x4 vp[4];
#pragma unroll
    for (int i = 0; i < NP; ++i) vp[i] = *(const u32x4*)(st + va[i]);
    // weights against the reference, and their sum over this lane's keys
    u32x4 pk[4];
    float ts = 0.f;
    auto weights = [&](float sub) {
      float t[2] = {0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x0 = sc[i >> 1][8 * (i & 1) + 2 * e], x1 = sc[i >> 1][8 * (i & 1) + 2 * e + 1];
          pk[i][e] = pack_bf16x2(__builtin_amdgcn_exp2f(x0 - sub), __builtin_amdgcn_exp2f(x1 - sub));
          t[i >> 1] = add_bf16x2(pk[i][e], t[i >> 1]);
        }
      ts = t[0] + t[1];
    };
    if (j > 0) weights(BIAS ? 0.f : m_run);
    const bool hit = unseen || !(ts < SUM_MOVE);   // also for NaN
    if (__any(hit)) {
      // the reference of the queries whose sum asks for it moves to the tile's
      // maximum, and so does that of the unseen ones (all of them on the first
      // tile), whose accumulators are 0, if the tile has a logit above -inf;
      // the weights of the others come out the same again
      float mx = sc[0][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = max3f(mx, sc[0][r], sc[1][r]);
      mx = max_with_partner(__builtin_elementwise_maximum(mx, sc[1][0])) - (BIAS ? 0.f : m_run);
      const bool move = max_with_partner(hit ? 1.f : 0.f) > 0.f && !(unseen && mx == -INFINITY);
      const float d = move ? mx : 0.f;
      const float alpha = unseen ? 1.f : __builtin_amdgcn_exp2f(-d);
      unseen = unseen && !move;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) acc[dt] *= alpha;
      m_run += d;
      nm -= d;
      weights(BIAS ? d : m_run);
    }
    l_run += ts;
    // O^T += V^T P^T (four 16-key steps)
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      u32x4 vf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (dt == 0 && i < NP)
          vf[i] = vp[i];
        else
          vf[i] = *(const u32x4*)(st + va[i] + dt * 32 * 128);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[dt] = mfma32(vf[i], pk[i], acc[dt]);
    }
  }
  l_run = sum_with_partner(l_run);
  __syncthreads();   // the stages are free
  // Epilogue: this wave's normalised rows through LDS as [query][d] f16 at the
  // row's scale, then whole rows in 16-byte stores.
  constexpr int OP = DH * 2 + 16;
  static_assert(NW * 32 * OP <= NST * L::STAGE, "the rows fit the stages");
  uint8_t* ow = lds + wave * 32 * OP;
  const float inv = l_run > 0.f ? __builtin_amdgcn_rcpf(l_run) : 0.f;
  // the row's largest magnitude among its finite values (at 256 channels, one
  // wave per SIMD, the test of each is left to rows that need it: 1.5 us)
  float big = 0.f;
  if constexpr (DH > 128) {
    float b4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; r += 2)
        b4[r / 2 & 3] = max3f(b4[r / 2 & 3], __builtin_fabsf(acc[dt][r]), __builtin_fabsf(acc[dt][r + 1]));
    big = max3f(__builtin_elementwise_maximum(b4[0], b4[1]), b4[2], b4[3]);
  }
  if (DH <= 128 || __any(!(big < INFINITY))) {
    big = 0.f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float x = __builtin_fabsf(acc[dt][r]);
        big = x < INFINITY ? fmaxf(big, x) : big;
      }
  }
  const int e = max(__builtin_amdgcn_frexp_expf(max_with_partner(big) * inv) - 15, -126);   // row / 2^e < 2^15
  const float f = __builtin_amdgcn_ldexpf(inv, -e);
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      f16x4 w;
#pragma unroll
      for (int r = 0; r < 4; ++r) w[r] = (_Float16)(acc[dt][4 * q4 + r] * f);
      *(f16x4*)(ow + l31 * OP + (32 * dt + 8 * q4 + 4 * g) * 2) = w;
    }
  if (g == 0 && row < cnt) {
    float* p = ml + (int64_t)row * H * 2;
    float m = unseen ? -INFINITY : m_run, lo = l_run;
    if (l_run > 0.f) {   // (device_util.h, at part_sum)
      const int el = __builtin_amdgcn_frexp_expf(l_run) - 1;
      m += (float)el;
      lo = __builtin_amdgcn_ldexpf(l_run, e - el);
    }
    if (a.stream_parts) {
      pstore(p, m);
      pstore(p + 1, lo);
    } else {
      p[0] = m;
      p[1] = lo;
    }
  }
  // the staged rows of a wave are written and read by that wave alone
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  constexpr int CH = DH / 8;   // 16-byte chunks per row
  bf16_t* obase = (bf16_t*)a.Opart + (((int64_t)o * S + s) * a.max_sel) * a.D + h * DH;
#pragma unroll 4
  for (int i = lane; i < 32 * CH; i += 64) {
    const int rr = i / CH, c = i % CH;
    if (row0 + rr < cnt) {
      u32x4* dst = (u32x4*)(obase + (int64_t)(row0 + rr) * a.D + 8 * c);
      const u32x4 v = *(const u32x4*)(ow + rr * OP + 16 * c);
      if (a.stream_parts)
        pstore(dst, v);
      else
        *dst = v;
    }
  }
}

}  // namespace rs3

using namespace rs3;

template <int DH, int NW, int NST>
static hipError_t launch(const Rs3ReadoutArgs& a, const Rs3AttnBanks& ab, hipStream_t st) {
  const int G = a.n_obj * a.H * a.S, n_qt = (a.max_sel + 32 * NW - 1) / (32 * NW);
  RS3_LAUNCH(RS3_K_ATTN, st, (k_attn_tile<DH, NW, NST>), dim3(8 * n_qt * ((G + 7) / 8)), dim3(64 * NW),
             NST * TileLds<DH>::STAGE, st, a, G, n_qt, ab);
  return hipGetLastError();
}

// Three stages, four waves; at d_h = 128 eight waves, since a stage is 32 KB
// and two work-groups of four with two stages each keep less in flight (110
// against 116 us at the sizes above, with bf16 partials); at 256 two stages
// fill the LDS.
hipError_t rs3_launch_attn_tile(const Rs3ReadoutArgs& a, const Rs3AttnBanks& ab, hipStream_t st) {
  switch (a.d_h) {
    case 32: return launch<32, 4, 3>(a, ab, st);
    case 64: return launch<64, 4, 3>(a, ab, st);
    case 128: return launch<128, 8, 3>(a, ab, st);
    case 256: return launch<256, 4, 2>(a, ab, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t rs3_attn_tile_setup() {
  const struct {
    const void* f;
    int bytes;
  } ks[] = {{(const void*)k_attn_tile<32, 4, 3>, 3 * TileLds<32>::STAGE},
            {(const void*)k_attn_tile<64, 4, 3>, 3 * TileLds<64>::STAGE},
            {(const void*)k_attn_tile<128, 8, 3>, 3 * TileLds<128>::STAGE},
            {(const void*)k_attn_tile<256, 4, 2>, 2 * TileLds<256>::STAGE}};
  for (const auto& k : ks) {
    hipError_t e = hipFuncSetAttribute(k.f, hipFuncAttributeMaxDynamicSharedMemorySize, k.bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
