// The two fused passes of one ILS iteration (Algorithm 1), as device bodies.
//
// Row pass (band of G output rows of one channel):
//   MID   : spectrum rows y0-1 .. y0+G  --C2R-->  u^n rows (LDS)
//           stencil: forward differences, mu (Eq. (7)), adjoint differences
//           r = f + kappa * D^T mu                     (Eq. (9) numerator,
//                                                       one-FFT form, Sec. 3.2)
//           r rows y0 .. y0+G-1  --R2C-->  spectrum rows
//   FIRST : as MID with u^0 rows read from memory instead of the C2R
//   FINAL : spectrum rows --C2R--> u^N rows written to the output
// Column pass (tile of S spectrum columns of one channel):
//   forward column DFT, divide by 1 + kappa (Sx + Sy) (Eq. (9) denominator)
//   and the inverse normalisation, inverse column DFT.
//
// A length-M complex DFT is split M = P * Q (four-step): the element index
// n = Q n1 + t is held by lane t (register n1) in "spatial" layout; stage A
// is a P-point register DFT per lane, a twiddle exp(-+2 pi i t k1 / M), one
// LDS exchange, and stage B a Q-point register DFT per lane k1, giving
// X[k1 + P k2] in register k2.  The inverse runs the same steps backwards,
// so no digit reversal is ever materialised.
#pragma once

#include "fft_reg.hpp"
#include "ils_desc.hpp"

namespace ilsk {

constexpr int imax_c(int a, int b) { return a > b ? a : b; }

// Normalised half-quadratic variable  mu / c = g (1 - (c0/c) (1 + g^2/eps)^(p/2 - 1))
// (Eq. (7) divided by c, c0 = p eps^(p/2-1)), for a difference h = s g of the
// scaled iterate: returns s mu / c (k, l2r: see FrameDesc).  Base-2 log/exp on
// the hardware transcendental unit.
__device__ __forceinline__ float mu_ns(float h, float a_exp, float k, float l2r) {
  float t = fmaf(h, h, k);
  float pw = __builtin_amdgcn_exp2f(fmaf(a_exp, __builtin_amdgcn_logf(t), l2r));
  return fmaf(-h, pw, h);
}

// Welsch penalty (Sec. 5, Eqs. (18)-(20)): with c = c0 = 2 the normalised
// variable is mu / c = g (1 - exp(-g^2 / (2 gamma^2))).
__device__ __forceinline__ float mu_ns_welsch(float h) {
  return fmaf(-h, __builtin_amdgcn_exp2f(-h * h), h);
}

enum Penalty : int { PEN_CHARBONNIER = 0, PEN_WELSCH = 1 };

// The penalty's constants of a frame (uniform), and s mu / c of a scaled
// difference for the penalty of the kernel instance.
struct MuConst {
  float a_exp, k, l2r;
};
template <int PEN>
__device__ __forceinline__ float mu_pen(float h, const MuConst& m) {
  if constexpr (PEN == PEN_WELSCH)
    return mu_ns_welsch(h);
  else
    return mu_ns(h, m.a_exp, m.k, m.l2r);
}

// Cross-lane moves inside a wavefront (no LDS allocation): the value of the
// previous lane (a DPP wave shift), and the value of the last lane of a
// T-lane slot broadcast to the whole slot (ds_swizzle bit mode, within
// 32-lane groups; T a power of two <= 32).
__device__ __forceinline__ float from_prev_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138 /* wave_shr:1 */, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_next_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130 /* wave_shl:1 */, 0xf, 0xf, false));
}
// the value of the first lane of a T-lane slot (ds_swizzle bit mode)
template <int T>
__device__ __forceinline__ float from_slot_first_lane(float v) {
  static_assert(T <= 32 && (T & (T - 1)) == 0, "slot must be a power of two within 32 lanes");
  constexpr int pattern = 31 & ~(T - 1);  // and-mask, or-mask 0, xor-mask 0
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), pattern));
}
template <int T>
__device__ __forceinline__ float from_slot_last_lane(float v) {
  static_assert(T <= 32 && (T & (T - 1)) == 0, "slot must be a power of two within 32 lanes");
  constexpr int pattern = (31 & ~(T - 1)) | ((T - 1) << 5);  // and-mask, or-mask, xor-mask 0
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), pattern));
}

// Synchronisation inside one row slot.  When a slot lies within one
// wavefront (T divides 64) its LDS exchange needs no workgroup barrier: the
// LDS operations of a wavefront are performed in program order, so it is
// enough to keep the compiler from moving memory operations across this
// point.  Otherwise fall back to a workgroup barrier.
template <int T>
__device__ __forceinline__ void slot_sync() {
  if constexpr (64 % T == 0) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

template <int P, int Q>
struct RowGeom {
  static constexpr int M = P * Q;
  static constexpr int T = P > Q ? P : Q;    // lanes per row slot
  static constexpr int QP = Q | 1;           // padded exchange row (odd => conflict-free)
  static constexpr int SLOT_F = 2 * P * QP;  // floats of LDS per row slot (>= W)
  static constexpr int TAB_F = 2 * P * QP;   // twiddles exp(-2 pi i t k1 / M) at [k1][t]
  static constexpr int NPAIR = (M / 2 + 1 + T - 1) / T;  // (k, M-k) pairs per lane of the real-FFT pre/post-process
};

// LDS that co-resident workgroups of one kernel are planned to take in all.  A
// CU has 160 KB and gives them out in pieces of 1280 B (measured: two blocks of
// 81 920 B, three of 53 760, four of 40 960 or five of 32 000 run side by side,
// one byte more and one fewer do).  Planning with 154 560 B instead counts one
// block per CU for tiles of 77 281 to 81 920 B: with all of the 160 KB, tables
// move in and out of the LDS and kernels are compiled for more waves, which
// over 24 column heights and six workloads was up to 20 % faster (8 RGB frames
// of 225 x 640) and up to 17 % slower (4 of 256 x 1280; lone grey ones of 1728
// and 1800 x 640 8 %, while 1600 and 2400 gained 6).
constexpr int kLdsCoresident = 154560;
constexpr int resident_blocks(int lds_bytes) {
  return lds_bytes * 2 > kLdsCoresident ? 1 : kLdsCoresident / lds_bytes;
}

// Waves per SIMD that the workgroups resident on a CU (as many as fit its
// LDS, at most 8 per SIMD) need; each may then use 512 / waves VGPRs.
constexpr int resident_waves_per_simd(int threads, int lds_bytes) {
  const int blocks = resident_blocks(lds_bytes);
  const int waves = blocks * ((threads + 63) / 64);
  return (waves + 3) / 4 > 8 ? 8 : (waves + 3) / 4;
}
template <int P, int Q, int G>
constexpr int row_waves() {
  return resident_waves_per_simd((G + 2) * RowGeom<P, Q>::T, 4 * ((G + 2) * RowGeom<P, Q>::SLOT_F + RowGeom<P, Q>::TAB_F));
}

// Rows per row-pass workgroup: about half the LDS of a CU when that leaves
// bands of at least four rows, else all of it.
template <int P, int Q>
constexpr int row_band() {
  constexpr int slot = 4 * RowGeom<P, Q>::SLOT_F;
  constexpr int tab = 4 * RowGeom<P, Q>::TAB_F;
  int g = (81920 - tab) / slot - 2;
  if (g < 4) g = (163840 - tab) / slot - 2;
  if (g > 14) g = 14;
  if (g < 1) g = 1;
  return g;
}

// Alternatives offered to the tuner: one workgroup per CU with the largest
// band that fits (fewest halo rows per output row), bands of about 3/4 and
// 5/8 of it, which split a frame into fewer blocks than CUs more evenly, and
// bands of 5 and 4 rows for frames with few rows in all.
template <int P, int Q>
constexpr int row_band_max() {
  constexpr int slot = 4 * RowGeom<P, Q>::SLOT_F;
  constexpr int tab = 4 * RowGeom<P, Q>::TAB_F;
  int g = (163840 - tab) / slot - 2;
  if (g > 30) g = 30;
  while ((g + 2) * RowGeom<P, Q>::T > 1024) --g;
  if (g < 1) g = 1;
  return g;
}
template <int P, int Q, int i>
constexpr int row_band_alt() {
  constexpr int gm = row_band_max<P, Q>();
  // i = 3, 4: short bands (5 and 4 rows) that spread a one-channel frame
  // over all CUs
  return i == 0 ? gm : i == 1 ? (3 * gm + 2) / 4 : i == 2 ? (5 * gm + 4) / 8 : i == 3 ? 5 : 4;
}

// The band of a length with a single shape: one workgroup per CU with the
// largest band that fits the LDS, 1024 threads and the registers (a lane
// needs about 4 P + 28 of them in the stencil, 2 Q + 40 in the Q-point
// stages; w waves per SIMD leave 512 / w).  Single frames cut it into
// balanced shorter bands (ils_api.cpp), so a large one costs nothing when
// rows are few, and few halo rows per output row when they are many.
template <int P, int Q>
constexpr int row_band_wide() {
  constexpr int T = RowGeom<P, Q>::T;
  constexpr int need = 4 * P + 28 > 2 * Q + 40 ? 4 * P + 28 : 2 * Q + 40;
  constexpr int waves = 512 / need < 1 ? 1 : (512 / need > 4 ? 4 : 512 / need);  // per SIMD
  int g = row_band_max<P, Q>();
  while (g > 1 && (g + 2) * T > 256 * waves) --g;
  return g;
}

// Column tile of S spectrum columns.  The exchange row of one k1 is padded
// so that successive k1 groups land on different LDS banks.
constexpr int col_ks(int Q, int S) { return (S >= 16) ? Q * S : Q * S + ((S - (Q * S) % 16) + 16) % 16; }
constexpr int col_ex_f(int P, int Q, int S) { return 2 * P * col_ks(Q, S); }
constexpr bool col_fits(int P, int Q, int S, int tab_f) {
  return 4 * (col_ex_f(P, Q, S) + tab_f) <= 163840 && S * (P > Q ? P : Q) <= 1024;
}

// Tables of a column length: the twiddles as a P x (Q|1) matrix [k1][j]
// and Sy[l] = 4 sin^2(pi l / H).  A tile copies them into its LDS beside the
// exchange when that costs no resident block on a CU; otherwise (the tiles
// of the longest columns) it reads them from global memory, where every
// block of the length finds them in the cache.  Either way every tile width
// of a length computes the same bits.
template <int P, int Q, int S>
struct ColGeom {
  static constexpr int H = P * Q;
  static constexpr int T = P > Q ? P : Q;
  static constexpr int QT = Q | 1;  // row stride of the twiddle matrix
  static constexpr int KS = col_ks(Q, S);
  static constexpr int EX_F = col_ex_f(P, Q, S);
  static constexpr int TAB_F = 2 * P * QT + H;
  static constexpr bool fits = col_fits(P, Q, S, 0);
  static constexpr bool TAB_LDS =
      col_fits(P, Q, S, TAB_F) && resident_blocks(4 * (EX_F + TAB_F)) == resident_blocks(4 * EX_F);
  static constexpr int LDS_F = EX_F + (TAB_LDS ? TAB_F : 0);
};

// Default column tile: the widest whose exchange and table fit the 160 KB of
// LDS (16 columns are whole 128-byte lines of the row-major spectrum;
// narrower tiles make neighbouring blocks fetch the same lines).  The
// narrower tiles offered to the tuner trade line efficiency for a grid that
// spreads more evenly over the compute units.
template <int P, int Q>
constexpr int col_tile() {
  return ColGeom<P, Q, 16>::fits ? 16 : ColGeom<P, Q, 8>::fits ? 8 : 4;
}
template <int P, int Q, int i>
constexpr int col_tile_alt() {
  constexpr int w = col_tile<P, Q>();
  constexpr int cand[3] = {w == 16 ? 12 : 4, 8, 4};
  return ColGeom<P, Q, cand[i]>::fits && cand[i] < w ? cand[i] : w;
}

// exp(+- i pi m / n) as a compile-time complex constant.
template <long long m, long long n>
__device__ __forceinline__ cf turn_half() {
  constexpr dcs w = cossin_turn(m, 2 * n);
  return cf{float(w.c), float(w.s)};
}

// Element at byte offset `off` of a pointer that is the same for the whole
// workgroup: the pointer stays in scalar registers and the address costs one
// 32-bit register for a whole run of accesses.
template <class E>
__device__ __forceinline__ ILS_G E& at(ILS_G void* base, unsigned off) {
  return *reinterpret_cast<ILS_G E*>(reinterpret_cast<ILS_G char*>(base) + off);
}
template <class E>
__device__ __forceinline__ const ILS_G E& at(const ILS_G void* base, unsigned off) {
  return *reinterpret_cast<const ILS_G E*>(reinterpret_cast<const ILS_G char*>(base) + off);
}

// Store 8 bytes at byte offset `off` of a uniform pointer.  THROUGH: written
// through the die's L2 at once (agent scope), so that the kernel's end does
// not wait for the write-back of a pass's worth of dirty lines: 1080p RGB
// FIRST 19.9 -> 17.5 us, MID 25.4 -> 23.9, FINAL 12.0 -> 9.7, column (16
// wide) 17.4 -> 15.9; 4K MID 128 -> 123.  Only for stores that fill (nearly)
// whole lines: with column tiles of 8 or 4, half and quarter lines that the
// L2 would have gathered, the pass gets slower (4K, 8 wide: 65 -> 68 us; 4
// wide: 62 -> 77), so those stay ordinary stores.  The address must be a
// multiple of 8, which a caller's image need not be.
template <bool THROUGH>
__device__ __forceinline__ void put(ILS_G void* base, unsigned off, cf v) {
  ILS_G unsigned long long* p =
      reinterpret_cast<ILS_G unsigned long long*>(reinterpret_cast<ILS_G char*>(base) + off);
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  if constexpr (THROUGH)
    __hip_atomic_store(p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = b;
}

// ---- C2R pre-process of one row: Z[k] = E + i O with E = X[k] + conj X[M-k],
// O = (X[k] - conj X[M-k]) exp(i pi k / M), and Z[M-k] = conj E + i conj O.
// Lane `lane` of the slot's T takes the pairs (k, M-k), k = lane + T i <= M/2,
// so that each spectrum value is loaded once and a pair's sums and product
// are formed once (8 vector instructions per value less than one value per
// lane from two loads, for one more LDS round trip; with the same for r2c_post
// 1080p RGB MID 27.2 -> 25.6 us, 4K 136 -> 128); Z goes to LDS in natural order.  w1 = exp(i pi lane / M).
// base: spectrum of the channel (uniform); row: byte offset of the row; ldS
// its length.
template <int P, int Q>
__device__ __forceinline__ void c2r_pre(const ILS_G cf* base, unsigned row, int ldS, int lane, cf w1, cf* slc) {
  using Geo = RowGeom<P, Q>;
  constexpr int M = Geo::M, T = Geo::T, NP = Geo::NPAIR;
  const unsigned up = row + 8u * (unsigned)lane, dn = row + 8u * (unsigned)(ldS - 1 - lane);
  cf a[NP], b[NP];
  auto load = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    a[i] = cf(at<cf>(base + T * i, up));
    b[i] = cf(at<cf>(base - T * i, dn));
  };
  auto pair = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const int k = lane + T * i;
    if (i == 0 && lane == 0) {  // DC and Nyquist bins: real parts only
      a[i].y = 0.0f;
      b[i].y = 0.0f;
    }
    const cf e = {a[i].x + b[i].x, a[i].y - b[i].y}, df = {a[i].x - b[i].x, a[i].y + b[i].y};
    const cf wk = (i == 0) ? w1 : cmul(w1, turn_half<(long long)T * i, M>());
    const cf o = cmul(df, wk);
    slc[k] = cf{e.x - o.y, e.y + o.x};
    if (i > 0 || lane > 0) slc[M - k] = cf{e.x + o.y, o.x - e.y};
  };
  constexpr int full = M / 2 + 1 >= T * NP ? NP : NP - 1;  // pairs every lane has
  const bool tail = full < NP && lane + T * full <= M / 2;
  static_for<full>(load);
  if constexpr (full < NP) {
    if (tail) load(std::integral_constant<int, full>{});
  }
  static_for<full>(pair);
  if constexpr (full < NP) {
    if (tail) pair(std::integral_constant<int, full>{});
  }
}

// ---- C2R stage A' (lane k1 < P): the Q-point inverse DFT over k2 of
// Z[k1 + P k2]; c2r_exchange then applies the twiddle exp(2 pi i t k1 / M)
// and writes the exchange row [k1][t].
template <int P, int Q>
__device__ __forceinline__ void c2r_stage_a(const cf* slc, int k1, cf (&v)[Q]) {
  static_for<Q>([&](auto k2c) {
    constexpr int k2 = decltype(k2c)::value;
    v[k2] = slc[k1 + P * k2];
  });
  dft<Q, +1>(v);
}

// twiddle exp(2 pi i t k1 / M) from the LDS table, then the exchange row [k1][t]
// (All table reads are issued before the first exchange write: the table and
// the exchange share one LDS array, so interleaving them would serialise.)
template <int P, int Q>
__device__ __forceinline__ void c2r_exchange(const cf (&v)[Q], int k1, const cf* tws, cf* slc) {
  constexpr int QP = Q | 1;
  cf w[Q];
  const cf* wrow = tws + k1 * QP;
  static_for<Q>([&](auto tc) {
    constexpr int t = decltype(tc)::value;
    if constexpr (t > 0) w[t] = wrow[t];
  });
  static_for<Q>([&](auto tc) {
    constexpr int t = decltype(tc)::value;
    slc[k1 * QP + t] = (t == 0) ? v[t] : cmulc(v[t], w[t]);
  });
}

// ---- C2R stage B' (lane t < Q): P-point inverse DFT over k1 -> z[Q n1 + t].
template <int P, int Q>
__device__ __forceinline__ void c2r_stage_b(const cf* slc, int t, cf (&z)[P]) {
  constexpr int QP = Q | 1;
  static_for<P>([&](auto k1c) {
    constexpr int k1 = decltype(k1c)::value;
    z[k1] = slc[k1 * QP + t];
  });
  dft<P, +1>(z);
}

// ---- R2C post-process of one row held in LDS in natural order Z[0..M-1]:
// with E = Z[k] + conj Z[M-k], D = Z[k] - conj Z[M-k] and w = exp(-i pi k / M)
// the spectrum values (X' = 2 X) are X'[k] = E - i w D and X'[M-k] =
// conj(E + i w D); pairs are dealt to the lanes as in c2r_pre.
template <int P, int Q>
__device__ __forceinline__ void r2c_post(const cf* slc, int lane, cf wl, ILS_G cf* base, unsigned row, int ldS) {
  using Geo = RowGeom<P, Q>;
  constexpr int M = Geo::M, T = Geo::T, NP = Geo::NPAIR;
  const unsigned up = row + 8u * (unsigned)lane, dn = row + 8u * (unsigned)(ldS - 1 - lane);
  auto one = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const int k = lane + T * i;
    const cf A = slc[k];
    const cf B = slc[(i == 0 && lane == 0) ? 0 : M - k];
    const cf E = {A.x + B.x, A.y - B.y}, D = {A.x - B.x, A.y + B.y};
    const cf w = (i == 0) ? wl : cmul(wl, turn_half<-(long long)T * i, M>());
    const cf wD = cmul(D, w);
    put<true>(base + T * i, up, cf{E.x + wD.y, E.y - wD.x});
    put<true>(base - T * i, dn, cf{E.x - wD.y, -E.y - wD.x});
  };
  // every pair but the last of a lane is in range, so only the last one is
  // guarded and the rest stays one basic block
  constexpr int full = M / 2 + 1 >= T * NP ? NP : NP - 1;
  static_for<full>(one);
  if constexpr (full < NP) {
    if (lane + T * full <= M / 2) one(std::integral_constant<int, full>{});
  }
}

// --------------------------------------------------------------------------
// Row pass, modes FIRST and MID.  Block = (G + 2) slots x T lanes.
// Slot s holds row y0 - 1 + s (periodic), s = 0 .. Gv + 1.
// LDS: (G + 2) slots of SLOT_F floats, then the twiddle table.
// --------------------------------------------------------------------------
template <int P, int Q, int G, int MODE, int PEN>
__device__ __forceinline__ void row_body(const FrameDesc& d, int band, int ch, float* smem) {
  using Geo = RowGeom<P, Q>;
  constexpr int M = Geo::M, T = Geo::T, QP = Geo::QP, SLOT_F = Geo::SLOT_F;
  const int H = d.H;
  const int W = 2 * M;
  const int ldS = d.ldS;
  const int nb = row_bands(d, G);
  const int y0 = band * H / nb;
  const int Gv = (band + 1) * H / nb - y0;
  const int tid = threadIdx.x;
  const int slot = tid / T;
  const int lane = tid - slot * T;
  float* sl = smem + slot * SLOT_F;
  cf* slc = reinterpret_cast<cf*>(sl);
  cf* tws = reinterpret_cast<cf*>(smem + (G + 2) * SLOT_F);
  const bool in_slot = slot <= Gv + 1;
  int yrow = y0 - 1 + slot;
  yrow = yrow < 0 ? yrow + H : (yrow >= H ? yrow - H : yrow);
  if (!in_slot) yrow = 0;
  const bool out_slot = slot >= 1 && slot <= Gv;
  const int yout = out_slot ? y0 - 1 + slot : 0;
  const ILS_G float* fch = gm(d.f) + (size_t)ch * H * W;  // the channel's data term
  const unsigned foff = 4u * (unsigned)(yout * W) + 8u * (unsigned)lane;

  // per-lane factors of the real-FFT twiddles (one load each, issued first)
  const cf w2lane = gm(d.tw2_row)[lane];  // exp(-i pi lane / M)
  // twiddle table -> LDS
  for (int i = tid; i < P * Geo::QP; i += blockDim.x) tws[i] = gm(d.twm_row)[i];

  float2 fv[P];
  // When a slot is Q lanes of one wavefront (Q a power of two), mu_x is
  // passed between lanes (below).  If moreover the shape leaves 256 VGPRs
  // per lane (two waves per SIMD), each lane keeps its own pairs of u in
  // registers for the stencil and takes the right neighbour from the next
  // lane; only the row below comes from LDS.  Both read the same values.
  constexpr bool kLaneReuse = (T == Q) && (T <= 32) && ((T & (T - 1)) == 0);
  constexpr bool kRegRow = kLaneReuse && row_waves<P, Q, G>() <= 2;
  float2 ur[P];
  if constexpr (MODE == ROW_FIRST) {
    const bool f_is_u0 = d.f == d.u0;  // Algorithm 1: the data term is the slot's own u row, read once
    if (in_slot && lane < Q) {  // u^0 row of this slot, all loads in flight together
      const ILS_G float* uch = gm(d.u0) + (size_t)ch * H * W;
      const unsigned uoff = 4u * (unsigned)(yrow * W) + 8u * (unsigned)lane;
      const float us = d.u_scale;
      float2 uv[P];
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        uv[n1] = float2(at<float2>(uch + 2 * Q * n1, uoff));
      });
      if (out_slot && !f_is_u0) {
        static_for<P>([&](auto n1c) {
          constexpr int n1 = decltype(n1c)::value;
          fv[n1] = float2(at<float2>(fch + 2 * Q * n1, foff));
        });
      }
      float2* u2 = reinterpret_cast<float2*>(sl);
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        if (f_is_u0) fv[n1] = uv[n1];
        uv[n1].x *= us;
        uv[n1].y *= us;
        u2[Q * n1 + lane] = uv[n1];
        if constexpr (kRegRow) ur[n1] = uv[n1];
      });
    }
    __syncthreads();
  } else {
    // ---- C2R of this slot's row (its loads overlap the table load)
    cf v[Q];
    if (in_slot)
      c2r_pre<P, Q>(gm(d.specB) + (size_t)ch * H * ldS, 8u * (unsigned)(yrow * ldS), ldS, lane, cf{w2lane.x, -w2lane.y}, slc);
    slot_sync<T>();
    if (in_slot && lane < P) c2r_stage_a<P, Q>(slc, lane, v);
    __syncthreads();  // twiddle table ready, every read of Z done
    if (in_slot && lane < P) c2r_exchange<P, Q>(v, lane, tws, slc);
    if (out_slot && lane < Q) {  // data term, in flight during stage B'
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        fv[n1] = float2(at<float2>(fch + 2 * Q * n1, foff));
      });
    }
    slot_sync<T>();
    cf z[P];
    if (in_slot && lane < Q) c2r_stage_b<P, Q>(slc, lane, z);
    slot_sync<T>();
    if (in_slot && lane < Q) {
      float2* u2 = reinterpret_cast<float2*>(sl);
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        u2[Q * n1 + lane] = make_float2(z[n1].x, z[n1].y);
        if constexpr (kRegRow) ur[n1] = make_float2(z[n1].x, z[n1].y);
      });
    }
    __syncthreads();
  }

  // ---- stencil.  mu_y of row s (from rows s, s+1) is evaluated once by
  // slot s and handed to slot s+1 through LDS.  Slot 0 (the row above the
  // band) only supplies mu_y; it runs the whole step all the same (its r is
  // not used), since it shares a wavefront with slot 1 where slots are short.
  const int t = lane;
  cf r[P];
  float2 myd[P];
  const bool st_slot = slot <= Gv && lane < Q;  // slots 0..Gv evaluate mu_y
  if (st_slot) {
    const float2* uc = reinterpret_cast<const float2*>(sl);
    const float2* ud = reinterpret_cast<const float2*>(sl + SLOT_F);
    const MuConst mc{d.a_exp, d.pen_k, d.log2_r};
    const float kappa = d.kappa_mu;
    float mx1_prev = 0.0f;
    static_for<P>([&](auto n1c) {
      constexpr int n1 = decltype(n1c)::value;
      // mu_x left of pair j equals mu_x right of pair j - 1.  When a slot is
      // Q lanes of one wavefront, pair j - 1 sits in the previous lane (same
      // n1) or, for lane 0, in lane Q - 1 at n1 - 1: take it from there.
      // Likewise pair j + 1 (the right neighbour's first pixel) sits in the
      // next lane, or for lane Q - 1 in lane 0 at n1 + 1 (at n1 = P - 1 that
      // is pair 0, the periodic wrap).
      const int j = Q * n1 + t;
      const int jp = (j == M - 1) ? 0 : j + 1;
      float2 c;
      float right;
      if constexpr (kRegRow) {
        c = ur[n1];
        constexpr int n1n = (n1 + 1) % P;
        const float nx = from_next_lane(c.x);
        const float wx = from_slot_first_lane<T>(ur[n1n].x);
        right = (t == Q - 1) ? wx : nx;
      } else {
        c = uc[j];
        right = uc[jp].x;
      }
      const float2 dn = ud[j];
      myd[n1] = make_float2(mu_pen<PEN>(dn.x - c.x, mc), mu_pen<PEN>(dn.y - c.y, mc));
      const float mx0 = mu_pen<PEN>(c.y - c.x, mc);
      const float mx1 = mu_pen<PEN>(right - c.y, mc);
      float mxl;
      if constexpr (kLaneReuse && n1 > 0) {
        const float sh = from_prev_lane(mx1);
        const float wr = from_slot_last_lane<T>(mx1_prev);
        mxl = (t == 0) ? wr : sh;
      } else {
        const int jm = (j == 0) ? M - 1 : j - 1;
        mxl = mu_pen<PEN>(c.x - uc[jm].y, mc);
      }
      mx1_prev = mx1;
      r[n1] = {fmaf(kappa, (mxl - mx0) - myd[n1].x, fv[n1].x), fmaf(kappa, (mx0 - mx1) - myd[n1].y, fv[n1].y)};
      // batches of five positions: their LDS reads issue together, while
      // the registers of later positions are not claimed early
      if constexpr ((n1 + 1) % 5 == 0) __builtin_amdgcn_sched_barrier(0);
    });
  }
  __syncthreads();  // every read of u done
  if (st_slot && slot < Gv) {
    float2* md = reinterpret_cast<float2*>(sl);
    static_for<P>([&](auto n1c) {
      constexpr int n1 = decltype(n1c)::value;
      md[Q * n1 + t] = myd[n1];
    });
  }
  __syncthreads();
  // ---- add mu_y of the row above, then stage A (P-point forward)
  if (out_slot && lane < Q) {
    const float2* mu = reinterpret_cast<const float2*>(sl - SLOT_F);
    const float kappa = d.kappa_mu;
    static_for<P>([&](auto n1c) {
      constexpr int n1 = decltype(n1c)::value;
      const float2 m = mu[Q * n1 + t];
      r[n1] = {fmaf(kappa, m.x, r[n1].x), fmaf(kappa, m.y, r[n1].y)};
    });
    dft<P, -1>(r);
    static_for<P>([&](auto k1c) {
      constexpr int k1 = decltype(k1c)::value;
      if (k1 != 0) r[k1] = cmul(r[k1], tws[k1 * QP + t]);
    });
  }
  __syncthreads();
  if (out_slot && lane < Q) {
    static_for<P>([&](auto k1c) {
      constexpr int k1 = decltype(k1c)::value;
      slc[k1 * QP + lane] = r[k1];
    });
  }
  slot_sync<T>();
  cf zz[Q];
  if (out_slot && lane < P) {
    const int k1 = lane;
    static_for<Q>([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      zz[t] = slc[k1 * QP + t];
    });
    dft<Q, -1>(zz);
  }
  slot_sync<T>();
  if (out_slot && lane < P) {
    const int k1 = lane;
    static_for<Q>([&](auto k2c) {
      constexpr int k2 = decltype(k2c)::value;
      slc[k1 + P * k2] = zz[k2];
    });
  }
  slot_sync<T>();
  if (out_slot) r2c_post<P, Q>(slc, lane, w2lane, gm(d.specA) + (size_t)ch * H * ldS, 8u * (unsigned)(yout * ldS), ldS);
}

// --------------------------------------------------------------------------
// Row pass, mode FINAL: C2R of G rows, written to the output image.
// Block = (G + 2) slots x T lanes, the bands of the other passes; slot s holds
// row y0 + s, the last two none.
// --------------------------------------------------------------------------
template <int P, int Q, int G>
__device__ __forceinline__ void row_final_body(const FrameDesc& d, int band, int ch, float* smem) {
  using Geo = RowGeom<P, Q>;
  constexpr int M = Geo::M, T = Geo::T, SLOT_F = Geo::SLOT_F;
  const int H = d.H;
  const int W = 2 * M;
  const int ldS = d.ldS;
  const int nb = row_bands(d, G);
  const int y0 = band * H / nb;
  const int Gv = (band + 1) * H / nb - y0;
  const int tid = threadIdx.x;
  const int slot = tid / T;
  const int lane = tid - slot * T;
  cf* slc = reinterpret_cast<cf*>(smem + slot * SLOT_F);
  cf* tws = reinterpret_cast<cf*>(smem + G * SLOT_F);
  const bool in_slot = slot < Gv;
  const int yrow = in_slot ? y0 + slot : 0;
  const cf w2lane = gm(d.tw2_row)[lane];
  for (int i = tid; i < P * Geo::QP; i += blockDim.x) tws[i] = gm(d.twm_row)[i];
  cf v[Q];
  if (in_slot)
    c2r_pre<P, Q>(gm(d.specB) + (size_t)ch * H * ldS, 8u * (unsigned)(yrow * ldS), ldS, lane, cf{w2lane.x, -w2lane.y}, slc);
  slot_sync<T>();
  if (in_slot && lane < P) c2r_stage_a<P, Q>(slc, lane, v);
  __syncthreads();  // twiddle table ready, every read of Z done
  if (in_slot && lane < P) c2r_exchange<P, Q>(v, lane, tws, slc);
  slot_sync<T>();
  if (in_slot && lane < Q) {
    cf z[P];
    c2r_stage_b<P, Q>(slc, lane, z);
    ILS_G float* och = gm(d.out) + (size_t)ch * H * W;
    const unsigned off = 4u * (unsigned)(yrow * W) + 8u * (unsigned)lane;
    const float k = d.boost, us = d.u_unscale;
    static_for<P>([&](auto n1c) {
      constexpr int n1 = decltype(n1c)::value;
      z[n1] = cf{us * z[n1].x, us * z[n1].y};
    });
    if (k != 0.0f) {  // detail enhancement: u + k (f - u); each element is read before it is written
      const ILS_G float* fch = gm(d.f) + (size_t)ch * H * W;
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        const float2 fv = float2(at<float2>(fch + 2 * Q * n1, off));
        z[n1] = cf{fmaf(k, fv.x - z[n1].x, z[n1].x), fmaf(k, fv.y - z[n1].y, z[n1].y)};
      });
    }
    if (((uintptr_t)d.out & 7) == 0) {
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        put<true>(och + 2 * Q * n1, off, z[n1]);
      });
    } else {  // an image that starts at an odd float: no 8-byte store fits
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        at<float>(och + 2 * Q * n1, off) = z[n1].x;
        at<float>(och + 2 * Q * n1, off + 4u) = z[n1].y;
      });
    }
  }
}

// --------------------------------------------------------------------------
// Column pass.  Block = S columns x T lanes, lane id = s + S * j.
// LDS: exchange (P x KS complex), then the tables (twiddle matrix [k1][j],
// row stride Q|1, and Sy[l]) when they are kept in LDS.
// --------------------------------------------------------------------------
template <int P, int Q, int S_>
__device__ __forceinline__ void col_body(const FrameDesc& d, int tile, int ch, float* smem) {
  using Geo = ColGeom<P, Q, S_>;
  constexpr int H = Geo::H, S = S_, KS = Geo::KS, QT = Geo::QT;
  const int ldS = d.ldS;
  const int tid = threadIdx.x;
  const int s = tid % S;
  const int j = tid / S;
  const int bin = spec_bin(tile * S + s, d.W / 2, ldS);
  const bool col_ok = bin >= 0;
  const int cc = col_ok ? tile * S + s : 0;
  const ILS_G cf* in = gm(d.specA) + (size_t)ch * H * ldS;
  ILS_G cf* out = gm(d.specB) + (size_t)ch * H * ldS;
  const unsigned off = 8u * (unsigned)(j * ldS + cc);  // this lane's element of row group 0
  cf* ex = reinterpret_cast<cf*>(smem);
  cf* tws = reinterpret_cast<cf*>(smem + Geo::EX_F);  // LDS copy of the twiddle matrix
  float* syl = smem + Geo::EX_F + 2 * P * QT;          // LDS copy of Sy
  const ILS_G cf* gtw = gm(d.twm_col);
  const ILS_G float* gsy = gm(d.sy);
  auto tw = [&](int i) -> cf {
    if constexpr (Geo::TAB_LDS)
      return tws[i];
    else
      return cf(gtw[i]);
  };
  auto sy_at = [&](int l) -> float {
    if constexpr (Geo::TAB_LDS)
      return syl[l];
    else
      return gsy[l];
  };

  cf x[P];
  if (j < Q) {  // stage A loads first: lane n2 = j, rows Q n1 + n2
    static_for<P>([&](auto n1c) {
      constexpr int n1 = decltype(n1c)::value;
      x[n1] = col_ok ? cf(at<cf>(in + (size_t)(Q * n1) * ldS, off)) : cf{0.0f, 0.0f};
    });
  }
  const float sxk = gm(d.sx)[col_ok ? bin : 0];
  if constexpr (Geo::TAB_LDS) {
    for (int i = tid; i < P * QT; i += blockDim.x) tws[i] = gtw[i];
    for (int i = tid; i < H; i += blockDim.x) syl[i] = gsy[i];
    __syncthreads();
  }
  if (j < Q) {
    cf w[P];
    static_for<P>([&](auto k1c) {
      constexpr int k1 = decltype(k1c)::value;
      if constexpr (k1 > 0) w[k1] = tw(k1 * QT + j);
    });
    dft<P, -1>(x);
    static_for<P>([&](auto k1c) {
      constexpr int k1 = decltype(k1c)::value;
      ex[k1 * KS + j * S + s] = (k1 == 0) ? x[k1] : cmul(x[k1], w[k1]);
    });
  }
  __syncthreads();
  if (j < P) {  // stage B: lane k1 = j; forward, divide, inverse
    cf y[Q];
    static_for<Q>([&](auto n2c) {
      constexpr int n2 = decltype(n2c)::value;
      y[n2] = ex[j * KS + n2 * S + s];
    });
    dft<Q, -1>(y);
    const float kappa = d.kappa, scale = d.col_scale;
    const float ksx = fmaf(kappa, sxk, 1.0f);
    static_for<Q>([&](auto k2c) {
      constexpr int k2 = decltype(k2c)::value;
      const float den = fmaf(kappa, sy_at(j + P * k2), ksx);
      y[k2] = cscale(y[k2], scale * __builtin_amdgcn_rcpf(den));
    });
    dft<Q, +1>(y);
    // the inverse twiddle of element (k1, n2) (none for n2 = 0): here from
    // the LDS table, else in stage B', where lanes of one k1 read the global
    // table coalesced (the same products either way)
    static_for<Q>([&](auto n2c) {
      constexpr int n2 = decltype(n2c)::value;
      if constexpr (Geo::TAB_LDS)
        ex[j * KS + n2 * S + s] = (n2 == 0) ? y[n2] : cmulc(y[n2], tws[j * QT + n2]);
      else
        ex[j * KS + n2 * S + s] = y[n2];
    });
  }
  __syncthreads();
  if (j < Q) {  // stage B': lane n2 = j, P-point inverse over k1
    if constexpr (Geo::TAB_LDS) {
      static_for<P>([&](auto k1c) {
        constexpr int k1 = decltype(k1c)::value;
        x[k1] = ex[k1 * KS + j * S + s];
      });
    } else {
      cf w[P];
      static_for<P>([&](auto k1c) {
        constexpr int k1 = decltype(k1c)::value;
        w[k1] = cf(gtw[k1 * QT + j]);
      });
      static_for<P>([&](auto k1c) {
        constexpr int k1 = decltype(k1c)::value;
        x[k1] = ex[k1 * KS + j * S + s];
        if (j != 0) x[k1] = cmulc(x[k1], w[k1]);
      });
    }
    dft<P, +1>(x);
    if (col_ok) {
      static_for<P>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        put<(S_ >= 12)>(out + (size_t)(Q * n1) * ldS, off, x[n1]);
      });
    }
  }
}

// --------------------------------------------------------------------------
// Column pass of lengths 400 .. 1000 (not 625, which has no such split, nor 675
// and 750, whose smallest factor of 5 would need more than 1024 lanes) in three
// stages, H = R1 R2 R3 with factors of at most 16: a lane holds a quarter to a
// half of the two-stage pass's values, so that the chain of instructions a
// single tile waits for is short.  Whole frames, N = 4, against two stages: one
// of H x 800 grey 7 to 12 % faster at every height (480: 68.3 -> 64.0 us, 1000:
// 88.2 -> 77.8), RGB 3 to 7 %; one of H x 1600 RGB from 14 % faster (972) to 5 %
// slower (900); four of H x 800 RGB from 8 % faster to 3 % slower; four of H x
// 1600 RGB, which fill the chip, from 5 % faster (576, 640) to 5 % slower (400,
// 450, 512, 540, 864), 500 and 600, whose splits leave half the lanes idle in
// two stages, 15 and 12 % slower (245 -> 282 us, 268 -> 301).  (A length has one
// form: a batch gives the bits of its frames.)  Longer columns lose it to the
// narrower tiles (1080p RGB 16.4 -> 17.2 us a pass), shorter ones to the extra
// exchange (96 x 256 x 256: 10 -> 14).
//   n = n1 R2 R3 + n2 R3 + n3,  k = k1 + R1 k2 + R1 R2 k3:
// stage 1 over n1 (lane (n2, n3)), twiddle W_H^(k1 (n2 R3 + n3)); stage 2
// over n2 (lane (k1, n3)), twiddle W_(R2 R3)^(k2 n3); stage 3 over n3 (lane
// (k1, k2)), divide, and the same backwards.  Stages 2 and 3 exchange in
// place: a lane rewrites the values it read.
// --------------------------------------------------------------------------
struct Split3 {
  int r1, r2, r3;
};
// The split whose smallest factor is largest (fewest lanes), then whose
// largest is smallest; an odd factor last (its rows of the exchange then need
// no padding against bank conflicts).
constexpr Split3 split3(int H) {
  Split3 best{0, 0, 0};
  int least = 1, most = 17;
  for (int a = 16; a >= 2; --a)
    for (int b = a; b >= 2; --b) {
      if (H % (a * b) != 0) continue;
      const int c = H / (a * b);
      if (c > b || c < least || (c == least && a >= most)) continue;
      least = c;
      most = a;
      best = c % 2 ? Split3{a, b, c} : b % 2 ? Split3{a, c, b} : a % 2 ? Split3{b, c, a} : Split3{a, b, c};
    }
  return best;
}
constexpr bool col3_length(int H) {
  if (H < 400 || H > 1000) return false;
  const Split3 s = split3(H);
  const int least = s.r1 < s.r2 ? (s.r1 < s.r3 ? s.r1 : s.r3) : (s.r2 < s.r3 ? s.r2 : s.r3);
  return s.r1 > 0 && 8 * (H / least) <= 1024;  // eight columns of the stage with the most lanes
}

template <int H, int S>
struct Col3Geom {
  static constexpr int R1 = split3(H).r1, R2 = split3(H).r2, R3 = split3(H).r3;
  static constexpr int B1 = R2 * R3, B2 = R1 * R3, B3 = R1 * R2;  // lanes of the stages
  static constexpr int T = imax_c(B1, imax_c(B2, B3));
  static constexpr int R3P = R3 | 1;
  static constexpr int THREADS = T * S;
  static constexpr int LDS_F = 2 * R1 * R2 * R3P * S;
};

template <int H, int S>
__device__ __forceinline__ void col3_body(const FrameDesc& d, int tile, int ch, float* smem) {
  using G = Col3Geom<H, S>;
  constexpr int R1 = G::R1, R2 = G::R2, R3 = G::R3;
  cf* ex = reinterpret_cast<cf*>(smem);
  const int ldS = d.ldS;
  const int s = threadIdx.x % S, j = threadIdx.x / S;
  const int bin = spec_bin(tile * S + s, d.W / 2, ldS);
  const bool col_ok = bin >= 0;
  const int cc = col_ok ? tile * S + s : 0;
  const ILS_G cf* in = gm(d.specA) + (size_t)ch * H * ldS;
  ILS_G cf* out = gm(d.specB) + (size_t)ch * H * ldS;
  const unsigned off = 8u * (unsigned)(j * ldS + cc);
  const ILS_G cf* g1 = gm(d.twm_col);       // W_H^(k1 j) at [k1 B1 + j]
  const ILS_G cf* g2 = g1 + R1 * G::B1;     // W_(R2 R3)^(k2 n3) at [k2 R3 + n3]
  auto at3 = [&](int k1, int m2, int n3) -> cf& { return ex[((k1 * R2 + m2) * G::R3P + n3) * S + s]; };
  const int q3 = j / R3, m3 = j - q3 * R3;  // (n2, n3) in stage 1, (k1, n3) in stage 2
  const int q2 = j / R2, m2 = j - q2 * R2;  // (k1, k2) in stage 3
  cf w1[R1], w2[R2];
  if (j < G::B1) {
    cf x[R1];
    static_for<R1>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      x[i] = col_ok ? cf(at<cf>(in + (size_t)(G::B1 * i) * ldS, off)) : cf{0.0f, 0.0f};
    });
    static_for<R1>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      if constexpr (i > 0) w1[i] = cf(g1[i * G::B1 + j]);
    });
    dft<R1, -1>(x);
    static_for<R1>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      at3(i, q3, m3) = i == 0 ? x[i] : cmul(x[i], w1[i]);
    });
  }
  __syncthreads();
  if (j < G::B2) {
    cf x[R2];
    static_for<R2>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      x[i] = at3(q3, i, m3);
      if constexpr (i > 0) w2[i] = cf(g2[i * R3 + m3]);
    });
    dft<R2, -1>(x);
    static_for<R2>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      at3(q3, i, m3) = i == 0 ? x[i] : cmul(x[i], w2[i]);
    });
  }
  __syncthreads();
  if (j < G::B3) {
    cf x[R3];
    float sy[R3];
    const ILS_G float* gsy = gm(d.sy) + (q2 + R1 * m2);
    static_for<R3>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      sy[i] = gsy[R1 * R2 * i];
      x[i] = at3(q2, m2, i);
    });
    const float kappa = d.kappa, scale = d.col_scale;
    const float ksx = fmaf(kappa, gm(d.sx)[col_ok ? bin : 0], 1.0f);
    dft<R3, -1>(x);
    static_for<R3>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      x[i] = cscale(x[i], scale * __builtin_amdgcn_rcpf(fmaf(kappa, sy[i], ksx)));
    });
    dft<R3, +1>(x);
    static_for<R3>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      at3(q2, m2, i) = x[i];
    });
  }
  __syncthreads();
  if (j < G::B2) {
    cf x[R2];
    static_for<R2>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      x[i] = at3(q3, i, m3);
      if constexpr (i > 0) x[i] = cmulc(x[i], w2[i]);
    });
    dft<R2, +1>(x);
    static_for<R2>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      at3(q3, i, m3) = x[i];
    });
  }
  __syncthreads();
  if (j < G::B1) {
    cf x[R1];
    static_for<R1>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      x[i] = at3(i, q3, m3);
      if constexpr (i > 0) x[i] = cmulc(x[i], w1[i]);
    });
    dft<R1, +1>(x);
    if (col_ok) {
      static_for<R1>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        put<(S >= 12)>(out + (size_t)(G::B1 * i) * ldS, off, x[i]);
      });
    }
  }
}

}  // namespace ilsk
