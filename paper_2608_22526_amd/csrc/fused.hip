// One launch for the tail of a frame: the merge of the readout's key splits
// (output projection and residual scatter, Sec. 3.1, Eq. 6) and the commit
// of the frame's memory tokens (Sec. 3.2, Eq. 8).  The two touch disjoint
// data -- the merge reads the attention partials, X and W_o and writes Y;
// the commit reads the memory tokens and the bank state and writes the bank
// -- so their work-groups run side by side in one grid instead of one launch
// after the other.
//
// Block b < n_cb is merge block (b % n_obj, b / n_obj) of the readout; the
// others are commit blocks in the same flattened order.  The block size is
// the commit's; a merge block uses its first CB_THREADS threads and the rest
// end at once (a work-group barrier waits only for the waves still running).
#include "combine.h"
#include "commit_body.h"
#include "readout_f32.h"

namespace rs3 {

// The argument block is memory the host wrote just before the launch: every
// argument that either kind of block reads before its first data load, and
// the first entries of the bank tables (the table lines of one-object
// launches), are loaded in one batch at the start (one memory round trip),
// so that the later loads behind the block-kind test and the table index
// find them in the scalar cache.
template <typename OutT, bool F16>
__global__ __launch_bounds__(CP_THREADS) void k_merge_commit(Rs3ReadoutArgs ra, Rs3CommitArgs ca, int n_cb) {
  extern __shared__ __attribute__((aligned(16))) uint8_t dyn[];
  asm volatile("" ::"s"(n_cb), "s"(ra.n_obj), "s"(ra.D), "s"(ra.max_sel), "s"(ra.sel_idx), "s"(ra.sel_stride),
               "s"(ra.X), "s"(ra.x_stride), "s"(ra.WoT), "s"(ra.sel_count), "s"(ra.S), "s"(ra.C),
               "s"(ca.n_obj), "s"(ca.masks), "s"(ca.m), "s"(ca.n), "s"(ca.s), "s"(ca.parity), "s"(ca.t),
               "s"(ca.fall_min), "s"(ca.fall_max), "s"(ca.banks[0]), "s"(ra.banks[0]));
  const int b = blockIdx.x;
  if (b < n_cb) {
    if (threadIdx.x >= CB_THREADS) return;
    combine_block<OutT, F16>(ra, b % ra.n_obj, b / ra.n_obj, dyn);
  } else {
    const int c = b - n_cb;
    commit_block<true>(ca, c % ca.n_obj, c / ca.n_obj, (int32_t*)dyn);
  }
}

// The same for fp32 layers.
static_assert(MF_THREADS == CP_THREADS, "merge and commit blocks of one size");
__global__ __launch_bounds__(CP_THREADS) void k_merge_commit_f32(Rs3ReadoutArgs ra, Rs3CommitArgs ca, int n_cb) {
  extern __shared__ __attribute__((aligned(16))) uint8_t dyn[];
  const int b = blockIdx.x;
  if (b < n_cb) {
    merge_f32_block(ra, b % ra.n_obj, b / ra.n_obj, (float*)dyn);
  } else {
    const int c = b - n_cb;
    commit_block<false>(ca, c % ca.n_obj, c / ca.n_obj, (int32_t*)dyn);
  }
}

}  // namespace rs3

using namespace rs3;

static size_t merge_commit_f32_lds(int D, int HS, int d_kv) {
  const size_t cb = merge_f32_lds(D, HS), cp = CP_FMAX * 16 + commit_stage_bytes(RS3_F32, d_kv);
  return cb > cp ? cb : cp;
}

static size_t merge_commit_lds(int D, int d_kv) {
  const size_t cb = combine_lds_bytes(D), cp = CP_FMAX * 16 + commit_stage_bytes(RS3_BF16, d_kv);
  return cb > cp ? cb : cp;
}

hipError_t rs3_fused_setup() {
  // D <= 1024, d_kv <= 256 (checked on the host)
  size_t max_lds = 0;
  for (int D = 64; D <= 1024; D += 64) {
    const size_t b = merge_commit_lds(D, 256);
    if (b > max_lds) max_lds = b;
  }
  const void* fs[] = {(const void*)k_merge_commit<bf16_t, false>, (const void*)k_merge_commit<bf16_t, true>,
                      (const void*)k_merge_commit<float, false>, (const void*)k_merge_commit<float, true>};
  for (const void* f : fs) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds);
    if (e != hipSuccess) return e;
  }
  return hipFuncSetAttribute((const void*)k_merge_commit_f32, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)merge_commit_f32_lds(1024, RS3_F32_MAX_SPLITS_X_HEADS, 256));
}

// Work-groups of the fused launch beyond which the merge and the commit run
// as two launches: a fused work-group has the commit's 1,024 threads, whose
// register count (127) allows one per CU, while the merge's 512-thread
// blocks fit two per CU on their own.  Two rounds of work-groups are still
// faster fused (eight objects on 30x54 grids, 432 work-groups: 222 against 257
// us per six frames), four are not (eight on 64x64, 976: 357 against 340; 64
// objects 149 against 75 + 34 us a frame).
constexpr int FUSE_MAX_WGS = 768;

hipError_t rs3_launch_merge_commit(const Rs3ReadoutArgs& ra, const Rs3CommitArgs& ca, int dtype, int d_kv,
                                   hipStream_t st) {
  const bool f32 = dtype == RS3_F32;
  const int rb = f32 ? RF_ROWS : cb_rows_for(ra.D, ra.n_obj, ra.max_sel);
  const int n_cb = ra.n_obj * ((ra.max_sel + rb - 1) / rb);
  const int mn = ca.m * ca.n;
  Rs3CommitArgs c = ca;
  const int n_cp = ca.n_obj * commit_blocks(c, dtype, ra.D, mn);
  if (n_cb + n_cp > FUSE_MAX_WGS) {
    hipError_t e = f32 ? rs3_launch_merge_f32(ra, st) : rs3_launch_combine(ra, st);
    return e == hipSuccess ? rs3_launch_commit(ca, dtype, d_kv, ra.D, st) : e;
  }
  if (f32) {
    RS3_LAUNCH(RS3_K_MERGE_COMMIT, st, k_merge_commit_f32, dim3(n_cb + n_cp), dim3(CP_THREADS),
               merge_commit_f32_lds(ra.D, ra.H * ra.S, d_kv), st, ra, c, n_cb);
    return hipGetLastError();
  }
  const size_t lds = merge_commit_lds(ra.D, d_kv);
  const dim3 grid(n_cb + n_cp), blk(CP_THREADS);
  const bool f16 = !rs3_attn_projects(ra);   // the form that wrote the partials
  if (ra.y_fp32 && f16)
    RS3_LAUNCH(RS3_K_MERGE_COMMIT, st, (k_merge_commit<float, true>), grid, blk, lds, st, ra, c, n_cb);
  else if (ra.y_fp32)
    RS3_LAUNCH(RS3_K_MERGE_COMMIT, st, (k_merge_commit<float, false>), grid, blk, lds, st, ra, c, n_cb);
  else if (f16)
    RS3_LAUNCH(RS3_K_MERGE_COMMIT, st, (k_merge_commit<bf16_t, true>), grid, blk, lds, st, ra, c, n_cb);
  else
    RS3_LAUNCH(RS3_K_MERGE_COMMIT, st, (k_merge_commit<bf16_t, false>), grid, blk, lds, st, ra, c, n_cb);
  return hipGetLastError();
}
