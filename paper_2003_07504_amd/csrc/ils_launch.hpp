// Kernels and launchers for one compiled transform length L = P * Q.
// Each length gets its own translation unit (inst_<L>.hip, generated by the
// build) so the heavy register-DFT instantiations compile in parallel.
#pragma once

#include "ils_passes.hpp"

namespace ilsk {

// Work list of a launch.  A single frame travels inline in the kernel
// arguments (descs == nullptr); a batch reads frame i's descriptor from
// device memory, frame i owning blocks [starts[i], starts[i+1]).  Both use
// the same kernel, so a frame gives bitwise the same result either way.
struct WorkList {
  FrameDesc one;           // the frame when descs == nullptr
  const FrameDesc* descs;  // device array, n entries
  const int* starts;       // device array, n + 1 entries
  int n;
  int total;               // number of (frame, channel, band) items
};

__device__ __forceinline__ int find_frame(const ILS_G int* starts, int n, int b) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (starts[mid] <= b) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Workgroups are dispatched to the 8 XCDs (each with its own L2) in
// round-robin order of the block id.  Give every XCD a contiguous range of
// work items instead, so neighbouring bands (which share halo rows) and
// neighbouring column tiles (which share 128-byte lines) meet in one L2.
// Bijective on [0, total).
__device__ __forceinline__ int xcd_remap(int b, int total) {
  constexpr int X = 8;
  const int q = total / X, r = total - q * X;
  const int x = b % X, i = b / X;
  return x * q + (x < r ? x : r) + i;
}

// Resolve work item b to its frame descriptor and block-local index.
__device__ __forceinline__ FrameDesc resolve(const WorkList& wl, int b, int& local) {
  b = xcd_remap(b, wl.total);
  if (wl.descs == nullptr) {
    local = b;
    return wl.one;
  }
  const int i = __builtin_amdgcn_readfirstlane(find_frame(gm(wl.starts), wl.n, b));
  local = b - gm(wl.starts)[i];
  return gm(wl.descs)[i];
}

// Minimum waves per SIMD a kernel is compiled for: enough to keep every
// block that fits the LDS resident, but at most 4 (128 VGPRs per lane), so
// that the register DFTs of the short lengths, whose blocks need little
// LDS, are not forced into scratch spills.
constexpr int waves_per_simd(int threads, int lds_bytes) {
  return resident_waves_per_simd(threads, lds_bytes) > 4 ? 4 : resident_waves_per_simd(threads, lds_bytes);
}

template <int P, int Q, int G>
struct RowCfg {
  static constexpr int GF = G;  // rows per FINAL block (no halo; the band of the other passes)
  static constexpr int THREADS = (G + 2) * RowGeom<P, Q>::T;
  static constexpr int LDS_F = (G + 2) * RowGeom<P, Q>::SLOT_F + RowGeom<P, Q>::TAB_F;
  static constexpr int WAVES = waves_per_simd(THREADS, 4 * LDS_F);
};

template <int P, int Q, int S>
struct ColCfg {
  static constexpr int THREADS = S * ColGeom<P, Q, S>::T;
  static constexpr int LDS_F = ColGeom<P, Q, S>::LDS_F;
  static constexpr int WAVES = waves_per_simd(THREADS, 4 * LDS_F);
};

// One block per work item = (frame, channel, band of rows).
// Register budget: every block that fits the LDS must also fit the
// register file, so the kernels ask for the matching waves per SIMD.
template <int P, int Q, int G, int MODE, int PEN>
__global__ void __launch_bounds__((RowCfg<P, Q, G>::THREADS))
__attribute__((amdgpu_waves_per_eu(RowCfg<P, Q, G>::WAVES))) k_row(WorkList wl) {
  __shared__ float smem[RowCfg<P, Q, G>::LDS_F];
  constexpr int rows = (MODE == ROW_FINAL) ? RowCfg<P, Q, G>::GF : G;
  int local;
  const FrameDesc d = resolve(wl, blockIdx.x, local);
  const int nb = row_bands(d, rows);
  const int ch = local / nb;
  if constexpr (MODE == ROW_FINAL)
    row_final_body<P, Q, RowCfg<P, Q, G>::GF>(d, local - ch * nb, ch, smem);
  else
    row_body<P, Q, G, MODE, PEN>(d, local - ch * nb, ch, smem);
}

// One block per work item = (frame, channel, tile of S spectrum columns).
template <int P, int Q, int S>
__global__ void __launch_bounds__((ColCfg<P, Q, S>::THREADS))
__attribute__((amdgpu_waves_per_eu(ColCfg<P, Q, S>::WAVES))) k_col(WorkList wl) {
  __shared__ float smem[ColCfg<P, Q, S>::LDS_F];
  int local;
  const FrameDesc d = resolve(wl, blockIdx.x, local);
  const int nb = col_tiles(d, S);
  const int ch = local / nb;
  col_body<P, Q, S>(d, local - ch * nb, ch, smem);
}

// The same for the three-stage column pass (at most 128 VGPRs per lane).
template <int H, int S>
__global__ void __launch_bounds__((Col3Geom<H, S>::THREADS)) __attribute__((amdgpu_waves_per_eu(4))) k_col3(WorkList wl) {
  __shared__ float smem[Col3Geom<H, S>::LDS_F];
  int local;
  const FrameDesc d = resolve(wl, blockIdx.x, local);
  const int nb = col_tiles(d, S);
  const int ch = local / nb;
  col3_body<H, S>(d, local - ch * nb, ch, smem);
}

// Host-side table of one length's launchers (one block per work item).  Of
// its row-band and column-tile shapes the plan's tuner times the first nrow
// and ncol; the column tiles up to ncol_all are for the rule that serves
// sizes without timed alternatives.
struct RowVariant {
  int rows[3];  // output rows per block for FIRST, MID, FINAL
  int threads, lds_bytes;
  hipError_t (*launch)(int mode, int pen, const WorkList& wl, hipStream_t st);
};
struct ColVariant {
  int cols;  // spectrum columns per block
  int threads, lds_bytes;
  hipError_t (*launch)(const WorkList& wl, hipStream_t st);
};
constexpr int kMaxShapes = 6;
struct LenOps {
  int L, P, Q;
  int nrow, ncol, ncol_all;
  Split3 c3;  // split of the three-stage column pass (r1 = 0: two stages)
  RowVariant row[kMaxShapes];
  ColVariant col[kMaxShapes];
};

template <int P, int Q, int G, int PEN>
void launch_row_pen(int mode, const WorkList& wl, hipStream_t st) {
  dim3 g(wl.total), block(RowCfg<P, Q, G>::THREADS);
  if (mode == ROW_FIRST)
    hipLaunchKernelGGL((k_row<P, Q, G, ROW_FIRST, PEN>), g, block, 0, st, wl);
  else
    hipLaunchKernelGGL((k_row<P, Q, G, ROW_MID, PEN>), g, block, 0, st, wl);
}

// (A kernel per penalty: with the penalty chosen by a uniform branch inside
// one kernel the shapes of 168 VGPRs spill, 1080p MID 24 -> 30 us.)
template <int P, int Q, int G>
hipError_t launch_row(int mode, int pen, const WorkList& wl, hipStream_t st) {
  if (mode == ROW_FINAL)  // no mu in the final pass
    hipLaunchKernelGGL((k_row<P, Q, G, ROW_FINAL, PEN_CHARBONNIER>), dim3(wl.total), dim3(RowCfg<P, Q, G>::THREADS), 0,
                       st, wl);
  else if (pen == PEN_WELSCH)
    launch_row_pen<P, Q, G, PEN_WELSCH>(mode, wl, st);
  else
    launch_row_pen<P, Q, G, PEN_CHARBONNIER>(mode, wl, st);
  return hipGetLastError();
}

template <int P, int Q, int S>
hipError_t launch_col(const WorkList& wl, hipStream_t st) {
  hipLaunchKernelGGL((k_col<P, Q, S>), dim3(wl.total), dim3(ColCfg<P, Q, S>::THREADS), 0, st, wl);
  return hipGetLastError();
}

template <int P, int Q, int G>
RowVariant row_variant() {
  using C = RowCfg<P, Q, G>;
  return RowVariant{{G, G, C::GF}, C::THREADS, 4 * C::LDS_F, &launch_row<P, Q, G>};
}
template <int H, int S>
hipError_t launch_col3(const WorkList& wl, hipStream_t st) {
  hipLaunchKernelGGL((k_col3<H, S>), dim3(wl.total), dim3(Col3Geom<H, S>::THREADS), 0, st, wl);
  return hipGetLastError();
}

template <int P, int Q, int S>
ColVariant col_variant() {
  using C = ColCfg<P, Q, S>;
  return ColVariant{S, C::THREADS, 4 * C::LDS_F, &launch_col<P, Q, S>};
}

template <int P, int Q, int G>
void add_row(LenOps& o) {
  for (int i = 0; i < o.nrow; ++i)
    if (o.row[i].rows[ROW_MID] == G) return;
  o.row[o.nrow++] = row_variant<P, Q, G>();
}
template <int P, int Q, int S>
void add_col(LenOps& o) {
  for (int i = 0; i < o.ncol_all; ++i)
    if (o.col[i].cols == S) return;
  o.col[o.ncol_all++] = col_variant<P, Q, S>();
}
// Three-stage tiles in order of preference: 8 columns (half lines), 4 for
// few blocks; 12 and 2 columns are for the tuner to try.
template <int H, int S>
void add_col3(LenOps& o) {
  if constexpr (Col3Geom<H, S>::THREADS <= 1024)
    o.col[o.ncol_all++] = ColVariant{S, Col3Geom<H, S>::THREADS, 4 * Col3Geom<H, S>::LDS_F, &launch_col3<H, S>};
}

template <int P, int Q>
LenOps start_ops(int L) {
  LenOps o{};
  o.L = L;
  o.P = P;
  o.Q = Q;
  return o;
}

// The column tiles of a length; timed ones (ncol) for tuned lengths of 480
// and more, else entry 0 and narrower tiles for the rule.
template <int P, int Q>
void add_cols(LenOps& o, bool tuned) {
  if constexpr (col3_length(P * Q)) {
    o.c3 = split3(P * Q);
    add_col3<P * Q, 8>(o);
    add_col3<P * Q, 4>(o);
    o.ncol = tuned ? o.ncol_all : 1;
  } else {
    add_col<P, Q, col_tile<P, Q>()>(o);
    o.ncol = 1;
    if constexpr (P * Q >= 480) {
      if (tuned) add_col<P, Q, col_tile_alt<P, Q, 0>()>(o);
    }
    add_col<P, Q, col_tile_alt<P, Q, 1>()>(o);
    add_col<P, Q, col_tile_alt<P, Q, 2>()>(o);
    if (tuned && P * Q >= 480) o.ncol = o.ncol_all;
  }
}

// Timed alternatives are compiled only for lengths where they can matter.
// Entry 0 is the default shape (used when the tuner is off or cannot time).
template <int P, int Q>
LenOps make_ops(int L) {
  LenOps o = start_ops<P, Q>(L);
  add_row<P, Q, row_band<P, Q>()>(o);
  add_cols<P, Q>(o, true);
  if constexpr (P * Q >= 480) {
    add_row<P, Q, row_band_alt<P, Q, 0>()>(o);
    add_row<P, Q, row_band_alt<P, Q, 1>()>(o);
    add_row<P, Q, row_band_alt<P, Q, 2>()>(o);
    add_row<P, Q, row_band_alt<P, Q, 3>()>(o);
    add_row<P, Q, row_band_alt<P, Q, 4>()>(o);
    if constexpr (col3_length(P * Q)) {
      add_col3<P * Q, 12>(o);
      add_col3<P * Q, 2>(o);
      o.ncol = o.ncol_all;
    }
  }
  return o;
}

// The further lengths (lengths_more.def): one row band, column tiles for the rule.
template <int P, int Q>
LenOps make_more_ops(int L) {
  LenOps o = start_ops<P, Q>(L);
  add_row<P, Q, row_band_wide<P, Q>()>(o);
  add_cols<P, Q>(o, false);
  return o;
}

}  // namespace ilsk

#define ILS_DEFINE_LEN(L, P, Q)                            \
  const ilsk::LenOps* ilsk_ops_##L() {                     \
    static const ilsk::LenOps o = ilsk::make_ops<P, Q>(L); \
    return &o;                                             \
  }
#define ILS_DEFINE_MORE_LEN(L, P, Q)                            \
  const ilsk::LenOps* ilsk_ops_##L() {                          \
    static const ilsk::LenOps o = ilsk::make_more_ops<P, Q>(L); \
    return &o;                                                  \
  }
