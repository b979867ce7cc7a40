// Per-frame descriptor shared by the host planner and the kernels.
#pragma once

#include <cstdint>

// Global (address space 1) qualifier for device pointers.  Pointers that
// reach a kernel inside a descriptor are otherwise generic, and the compiler
// then emits FLAT memory instructions, which also count against the LDS
// wait counter: every wait for an LDS result would wait for outstanding
// image and spectrum loads too.
// (The host pass of the compiler parses the device code too; there the
// qualifier means nothing and is left out.)
#if defined(__HIP_DEVICE_COMPILE__)
#define ILS_G __attribute__((address_space(1)))
#else
#define ILS_G
#endif

namespace ilsk {

template <class T>
__host__ __device__ __forceinline__ ILS_G T* gm(T* p) {
  return (ILS_G T*)p;
}

struct cf;

// One frame (all of its channels) of one ILS call.  Layouts:
//   f, u0, out : C x H x W float32, row-major, channel stride H*W
//   specA/specB: C x H x ldS complex64, channel stride H*ldS, ldS = M + 1
//                rounded up to 16 (M = W/2).  Bins k <= M/2 of a row sit at
//                k; bins k >= M - M/2 at k + ldS - 1 - M, so that both ends
//                of a row are whole 128-byte lines and the pairs (k, M-k) of
//                the real-FFT steps are read and written line by line from
//                both ends (bin M/2 of an even M is held twice).  The
//                runtime-length passes keep bin k at k.
// The row passes read specB and write specA; the column pass reads specA
// and writes specB.
struct FrameDesc {
  const float* f;    // data term of the LS problem
  const float* u0;   // first iterate (normally == f)
  float* out;        // result u^N
  cf* specA;
  cf* specB;
  const cf* tw_row;   // exp(-2 pi i j / M), j < M          (M = W/2)
  const cf* tw2_row;  // exp(-pi i k / M),  k <= M
  const cf* twm_row;  // exp(-2 pi i t k1 / M) at [k1 * (Q|1) + t], M = P Q
  const float* sx;    // 4 sin^2(pi k / W), k <= M
  const cf* tw_col;   // exp(-2 pi i j / H), j < H
  const cf* twm_col;  // exp(-2 pi i j k1 / H) at [k1 * (Q|1) + j], H = P Q
                      // (three stages: see col3_body)
  const float* sy;    // 4 sin^2(pi l / H), l < H
  int H, W, C, ldS;
  float kappa;      // lambda * c / 2, c >= c0 = p eps^(p/2 - 1) (Welsch: c = 2)
  // Between passes the iterate is kept as s u, s = eps^(-1/2) (Welsch: s =
  // sqrt(log2(e) / 2) / gamma), so that the penalty's argument g^2 / eps is
  // the square of a difference as it stands (see set_charbonnier and
  // set_welsch).
  float u_scale;    // s
  float u_unscale;  // 1 / s, applied by the final pass
  float kappa_mu;   // kappa / s: weight of D^T mu(s u) in the right-hand side
  float a_exp;      // p/2 - 1 (Welsch: unused)
  float pen_k;      // eps s^2: 1, but at the limits of s (Welsch: unused)
  float log2_r;     // log2(c0 / c) - a_exp log2(pen_k) (Welsch: unused)
  float col_scale;  // s / (2 H W): inverse-transform normalisation (and the
                    // factor 2 the row R2C leaves in its output)
  float boost;      // final pass writes u + boost (f - u) when non-zero
                    // (detail enhancement); 0 writes u
  int nb_row;       // row bands per channel (0: as many as bands of the
                    // kernel's full height need); see row_bands
};

// Work lists of smoothings of one plane with up to kMaxLevels lambdas, which
// the kernel that makes the plane writes to the workspace header (as a batch's
// are uploaded): levels first[g] .. first[g + 1] - 1 run as group g, their
// descriptors from descs, the group's starts (row bands, then column tiles,
// kMaxLevels + 1 of each) from starts + 2 g (kMaxLevels + 1).
constexpr int kMaxLevels = 4;
struct LevelLists {
  FrameDesc d[kMaxLevels];
  int ngroups, first[3];
  int bands[2], tiles[2];  // per level of a group
  FrameDesc* descs;
  int* starts;
};

// Bands of the row passes.  A channel's H rows are split into nb bands, band
// b holding rows [b H / nb, (b + 1) H / nb) (floor or ceil of H / nb rows);
// nb is the frame's own count, kept within [ceil(H / G), H] so that no band
// exceeds the G rows a block holds.
__host__ __device__ inline int row_bands(const FrameDesc& d, int G) {
  const int lo = (d.H + G - 1) / G;
  const int nb = d.nb_row > lo ? d.nb_row : lo;
  return nb < d.H ? nb : d.H;
}

// Bin held at position pos of a spectrum row, or -1 (see FrameDesc).
__host__ __device__ inline int spec_bin(int pos, int M, int ldS) {
  const int up = pos - (ldS - 1 - M);
  return pos <= M / 2 ? pos : (up >= M - M / 2 && up <= M) ? up : -1;
}

// Column tiles of S spectrum positions per channel.
__host__ __device__ inline int col_tiles(const FrameDesc& d, int S) { return (d.ldS + S - 1) / S; }

enum RowMode : int { ROW_FIRST = 0, ROW_MID = 1, ROW_FINAL = 2 };

}  // namespace ilsk
