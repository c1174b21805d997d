// Closure of the decoded masks and the palette argmax (Sec. 3.3; the end of
// Algorithm 1).  Each object's binary mask (logit > 0) is closed with a k x k
// square, a dilation that ignores pixels outside the image followed by an
// erosion that counts them as set; the palette then takes, per pixel, the
// object with the largest logit among those whose closed mask covers it
// (lowest index on ties), 0 where none does.
//
// One launch, one work-group per tile of 64 x (64 - 4r) pixels (k = 2r+1),
// which needs the masks of 2r pixels around it:
//   1. a wave per object (and round) reads the tile's logits with its border,
//      eight pixels per lane and load, into bits: lane y then holds row y of
//      the 96 x 64 window (16 pixels left and right, 2r above and below);
//   2. the closing runs in that wave's registers, without a barrier: along
//      rows by shifts, across rows by lane shuffles, each in doubling steps
//      (a step of at most done + 1 leaves no gap); the erosion is the dilation
//      of the complement.  The closed rows go to LDS;
//   3. after one barrier a thread takes eight pixels of every object: the
//      closed bytes, and the logits of the objects that cover any of them.
// Bound by the reads of step 1 (twice the image with the border at r = 4, from
// L2) and three memory round trips.  Eight masks of 1024 x 1024 (26 MB in and
// out): 17.6 us; three launches over bit words in memory (threshold, closing,
// palette) took 21.1 us; three masks of 480 x 854 8.9 against 13.1.
#include "device_util.h"

namespace rs3 {

constexpr int PC_TX = 64;      // tile width
constexpr int PC_HALO = 16;    // window pixels left and right of it (>= 2 * largest radius, 7)
constexpr int PC_CH = (PC_TX + 2 * PC_HALO) / 8;   // 8-pixel chunks per window row
constexpr int PC_WAVES = 8;

// Eight logits as they lie in memory (rows start at any element, so the loads
// are unaligned).  No branch: the loads of a batch go out together, where loads
// behind lane conditions wait one by one.
template <typename T>
struct Raw8;
template <>
struct Raw8<bf16_t> {
  u32x4 w;
  __device__ __forceinline__ void load(const bf16_t* p) {
    typedef u32x4 u32x4_u __attribute__((aligned(2)));
    w = *(const RS3_GLOBAL u32x4_u*)p;
  }
  // near the right border: pixels past the first n repeat pixel n - 1
  __device__ __forceinline__ void load_edge(const bf16_t* p, int n) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      w[j] = gload(p + min(2 * j, n - 1)) | (uint32_t)gload(p + min(2 * j + 1, n - 1)) << 16;
  }
  __device__ __forceinline__ float at(int j) const {
    return __uint_as_float((j & 1) ? w[j >> 1] & 0xffff0000u : w[j >> 1] << 16);
  }
};
template <>
struct Raw8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    typedef f32x4 f32x4_u __attribute__((aligned(4)));
    a = *(const RS3_GLOBAL f32x4_u*)p;
    b = *(const RS3_GLOBAL f32x4_u*)(p + 4);
  }
  __device__ __forceinline__ void load_edge(const float* p, int n) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = gload(p + min(j, n - 1));
      b[j] = gload(p + min(4 + j, n - 1));
    }
  }
  __device__ __forceinline__ float at(int j) const { return j < 4 ? a[j & 3] : b[j & 3]; }
};

// Eight bytes to p (unaligned), the first n of them at the right border.
__device__ __forceinline__ void store8(uint8_t* p, int n, uint64_t b) {
  typedef uint64_t u64_u __attribute__((aligned(1)));
  if (n >= 8)
    *(RS3_GLOBAL u64_u*)p = b;
  else
    for (int j = 0; j < n; ++j) gstore(p + j, (uint8_t)(b >> (8 * j)));
}

// One row of the window: pixels 0..63 and 64..95.
struct PcRow {
  uint64_t lo;
  uint32_t hi;
};

__device__ __forceinline__ PcRow lane_row(const PcRow& a, int src) {   // row of lane src, 0 outside the window
  const uint32_t l = (uint32_t)__shfl((int)(uint32_t)a.lo, src), m = (uint32_t)__shfl((int)(uint32_t)(a.lo >> 32), src);
  const uint32_t h = (uint32_t)__shfl((int)a.hi, src);
  const bool in = src >= 0 && src < 64;
  return PcRow{in ? (uint64_t)m << 32 | l : 0ull, in ? h : 0u};
}

// (2r+1)^2 square dilation of the window; pixels outside it are unset.
__device__ __forceinline__ PcRow dilate(PcRow a, int r) {
  const int lane = threadIdx.x & 63;
  for (int done = 0; done < r;) {
    const int s = min(done + 1, r - done);
    const uint64_t lo = a.lo, hi = a.hi;
    a.lo = lo | lo << s | lo >> s | hi << (64 - s);
    a.hi = (uint32_t)(hi | hi << s | hi >> s | lo >> (64 - s));
    done += s;
  }
  for (int done = 0; done < r;) {
    const int s = min(done + 1, r - done);
    const PcRow u = lane_row(a, lane - s), d = lane_row(a, lane + s);
    a.lo |= u.lo | d.lo;
    a.hi |= u.hi | d.hi;
    done += s;
  }
  return a;
}

// grid (ceil(W / 64), ceil(H / (64 - 4r))), block 64 * nw.  closed, palette:
// optional.  dyn: [n_obj][64] closed rows of the tile.
template <typename T>
__global__ __launch_bounds__(64 * PC_WAVES, 4) void k_post_close(const T* logits, int n_obj, int H, int W, int r,
                                                              uint8_t* closed, uint8_t* palette) {
  extern __shared__ __attribute__((aligned(16))) uint64_t rows[];   // [n_obj][64]
  __shared__ __attribute__((aligned(16))) uint8_t win[PC_WAVES][64][16];   // a wave's window: 12 bytes of each row
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int ty = 64 - 4 * r;   // tile rows: lanes 2r .. 64-2r-1
  const int x0 = blockIdx.x * PC_TX, y0 = blockIdx.y * ty;
  const int64_t plane = (int64_t)H * W;
  // this lane's row of the window and the pixels of it inside the image
  const int y = y0 - 2 * r + lane;
  PcRow inside = {0ull, 0u};
  if (y >= 0 && y < H) {
    const int n = min(W - (x0 - PC_HALO), 96);   // window pixels left of the right border
    inside.lo = n >= 64 ? ~0ull : (1ull << n) - 1ull;
    inside.hi = n >= 96 ? ~0u : n > 64 ? (1u << (n - 64)) - 1u : 0u;
    if (x0 == 0) inside.lo &= ~0ull << PC_HALO;
  }
  for (int o = wave; o < n_obj; o += nw) {
    const T* L = logits + o * plane;
    // chunk q = lane + 64 i: window row q / 12, pixels 8 (q % 12) .. +7.  Rows
    // and chunks outside the image read the nearest ones inside (their bits
    // are masked below); a chunk that crosses the right border reads the
    // row's last eight pixels and shifts them into place.
    // chunks in flight: 48 registers, fp32 32 (48 spilled eight of 128: eight
    // masks of 1024 x 1024 20.7 instead of 22.1 us)
    constexpr int NB = sizeof(T) == 2 ? PC_CH : PC_CH / 3;
#pragma unroll
    for (int i0 = 0; i0 < PC_CH; i0 += NB) {
      Raw8<T> v[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int q = lane + 64 * (i0 + i), row = q / PC_CH, c = q - row * PC_CH;
        const int yy = min(max(y0 - 2 * r + row, 0), H - 1), xx = x0 - PC_HALO + 8 * c;
        if (W >= 8)
          v[i].load(L + (int64_t)yy * W + min(max(xx, 0), W - 8));
        else
          v[i].load_edge(L + (int64_t)yy * W, W);
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int q = lane + 64 * (i0 + i), row = q / PC_CH, c = q - row * PC_CH;
        const int xx = x0 - PC_HALO + 8 * c;
        uint32_t b = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) b |= (v[i].at(j) > 0.f ? 1u : 0u) << j;
        win[wave][row][c] = (uint8_t)(b >> min(max(W >= 8 ? xx - (W - 8) : xx, 0), 8));
      }
    }
    // the window is written and read by this wave alone
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const u32x4 w = *(const u32x4*)win[wave][lane];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    PcRow a = dilate(PcRow{((uint64_t)w[1] << 32 | w[0]) & inside.lo, w[2] & inside.hi}, r);
    // erosion with the pixels outside the image set: their complement is unset
    a = dilate(PcRow{~a.lo & inside.lo, ~a.hi & inside.hi}, r);
    a.lo = ~a.lo & inside.lo;
    a.hi = ~a.hi & inside.hi;
    rows[o * 64 + lane] = a.lo >> PC_HALO | (uint64_t)a.hi << (64 - PC_HALO);   // the tile's 64 pixels
  }
  __syncthreads();
  const bool edge = x0 + PC_TX > W;   // the last tile of a row
  for (int q = tid; q < 8 * ty; q += 64 * nw) {
    const int row = q >> 3, c = q & 7, yy = y0 + row, xx = x0 + 8 * c;
    if (yy >= H || xx >= W) continue;
    const int n = W - xx;
    const int64_t px = (int64_t)yy * W + xx;
    // pos: the object with the largest positive logit, which has the pixel
    // wherever there is one (its mask, and so its closed mask, covers it);
    // any: the largest logit among the covering objects, for filled holes.
    // Objects that cover no pixel of the wave's eight rows are passed over.
    float pos[8], any[8];
    int parg[8], aarg[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      pos[j] = any[j] = 0.f;
      parg[j] = aarg[j] = -1;
    }
    for (int o = 0; o < n_obj; ++o) {
      const uint32_t b = (uint32_t)(rows[o * 64 + 2 * r + row] >> (8 * c)) & 0xffu;
      if (closed) {   // bit j -> byte j
        const uint32_t lo4 = (b & 1u) | (b & 2u) << 7 | (b & 4u) << 14 | (b & 8u) << 21;
        const uint32_t hi4 = (b >> 4 & 1u) | (b & 32u) << 3 | (b & 64u) << 10 | (b & 128u) << 17;
        store8(closed + o * plane + px, n, lo4 | (uint64_t)hi4 << 32);
      }
      if (!palette || !__any(b != 0u)) continue;
      Raw8<T> v;
      if (edge)
        v.load_edge(logits + o * plane + px, n);
      else
        v.load(logits + o * plane + px);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = v.at(j);
        parg[j] = x > pos[j] ? o : parg[j];
        pos[j] = x > pos[j] ? x : pos[j];
        const bool f = (b >> j & 1u) && (aarg[j] < 0 || x > any[j]);
        aarg[j] = f ? o : aarg[j];
        any[j] = f ? x : any[j];
      }
    }
    if (!palette) continue;
    uint64_t out = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) out |= (uint64_t)(uint32_t)((parg[j] >= 0 ? parg[j] : aarg[j]) + 1) << (8 * j);
    store8(palette + px, n, out);
  }
}

}  // namespace rs3

using namespace rs3;

// What rs3_close_masks asks of its caller's workspace (two sets of bit words
// and a byte per pixel).  The launch keeps its words in LDS and leaves the
// workspace alone; the contract stays.
size_t rs3_post_workspace_bytes(int n_obj, int H, int W) {
  const size_t WW = (size_t)(W + 63) / 64;
  const size_t words = (size_t)n_obj * H * WW * 8;
  return 2 * ((words + 255) & ~(size_t)255) + (((size_t)H * W + 255) & ~(size_t)255);
}

hipError_t rs3_launch_close_masks(int n_obj, int H, int W, const void* logits, int dtype, int k, uint8_t* closed,
                                  uint8_t* palette, hipStream_t st) {
  const int r = k / 2, ty = 64 - 4 * r;
  const int nw = n_obj < 4 ? 4 : n_obj < PC_WAVES ? n_obj : PC_WAVES;   // four for the palette's sake
  const dim3 grid((W + PC_TX - 1) / PC_TX, (H + ty - 1) / ty);
  const size_t lds = (size_t)n_obj * 64 * 8;
  if (dtype == RS3_BF16)
    hipLaunchKernelGGL(k_post_close<bf16_t>, grid, dim3(64 * nw), lds, st, (const bf16_t*)logits, n_obj, H, W, r,
                       closed, palette);
  else
    hipLaunchKernelGGL(k_post_close<float>, grid, dim3(64 * nw), lds, st, (const float*)logits, n_obj, H, W, r, closed,
                       palette);
  return hipGetLastError();
}
