// em_cell.h -- the 43 x 43 correlations of an EM iteration on the matrix cores
// with 4 x 4 output cells (arXiv:2302.05804, Sec. 2, Eqs. (1)-(3)).
//
//     out[k][l] = sum_{a,b} g[a][b] in[k - 21 + a][l - 21 + b]
//
// One product of v_mfma_f32_16x16x32 takes the 16 outputs of a 4 x 4 cell (M),
// 16 cells side by side in a row of cells (N: 64 output columns) and 32 values
// of the cells' common window (K).  The window of a cell at (R, C) holds rows
// R - 22 .. R + 25 and columns C - 22 .. C + 25: row d (0..47) and column k
// (0..47) meet output (R + p, C + q) with tap (d - 1 - p, k - 1 - q).  The table
// operand is that tap, zero outside the stamp:
//     T[4p + q][d, k] = g[d - 1 - p][k - 1 - q].
// 43 x 43 of the 46 x 48 window values that can be non-zero are taps: 84%, where a
// row of 16 outputs (a one-dimensional Toeplitz operand of 43 + 15 values in
// 64) is 67%.
//
// Window row d of cell row R is image row R - 22 + d, and cell rows are 4 apart,
// so with d = 4 j + E (class E = 0..3, j = 0..11) an image row 4 s + E serves
// every cell row s - j.  A wave owns G consecutive cell rows; in class E it walks
// over the image rows (step s reads row 4 s + E once from LDS) and multiplies
// each by the table fragments of the j = s - g that its cell rows g need.  A
// table fragment is read from LDS once per class and wave, at step j, and stays
// in registers for the G steps that use it; so LDS serves 2 (image) fragments
// per step and NB * 18 table fragments per class for 54 G (BF16 split; 37 G with its band)
// or 144 G (FP32) products.  (Plain BF16, served jobs only: 18 G.)
//
// Bound by the matrix cores (at the clock they hold under this load): 33 x 2048^2
// in FP32 issues 5.0 TFLOP of products per launch, forward 2.75 ms = 1.8 PFLOP/s,
// adjoint 2.96 ms (the r tile is staged anew for every frame); the direct FP32
// convolution took 7.35 and 7.62 ms.  BF16 split on 33 x 1999 x 2111: forward 1.41
// -> 1.18 ms, adjoint 2.17 -> 1.04 ms against one-dimensional Toeplitz operands
// (alone on the card; 272 tiles in one frame group, two rounds, took 1.77 ms).
//
// Sums on the matrix cores: a lane group's eight products are added with what is below
// 2^-24 of the largest of them cut off, then the four groups and the accumulator one
// after the other with round to nearest even.  Products of bf16 parts have 16 bits, so
// that nothing is cut off within 2^-9 of the largest; beside a bright pixel sums come
// out low by a few 1e-8.
//
// FP32 parts: a value times 2^16 is hi + mid + lo, each the bf16 nearest to what is
// left.  With that factor the last bit of every binary32 number, 2^-149, is a bf16
// (the smallest is 2^-133; the matrix cores take subnormal bf16 as they are), so every
// finite operand is held exactly.  A tile of the image with a value of 2^60 or more
// takes 2^-32 instead, so that sums do not overflow; what it then cuts off is below
// 2^-102, and sums below 2^-40 are formed another way (cell_finish).
//
// The 48 window columns of a row are one 32-wide chunk ("main") and a 16-wide
// "tail"; the tails of rows j and j + 1 of a class (image rows 4 s + E and
// 4 s + 4 + E) share one product.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "em_device.h"
#include "em_internal.h"
#include "em_mfma_common.h"

namespace em {

// f(0), f(1), ..., f(N - 1) with the index a compile-time constant
#define EM_INLINE __attribute__((always_inline))
template <class Fn, int... I>
__device__ EM_INLINE inline void static_for_seq(std::integer_sequence<int, I...>, Fn&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class Fn>
__device__ EM_INLINE inline void static_for(Fn&& f) {
  static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

constexpr int CELL_K = 43;        // kernel side
constexpr int CELL_NJ = 12;       // window rows of one class
constexpr int CELL_OFF = 22;      // window origin above / left of the cell
constexpr int CELL_EXTRA = 44;    // image rows of a tile beyond its output rows

// FP32 operands as three bf16 parts each, v = p0 + p1 + p2 exactly (24 significant
// bits in three times 8), and the eight products of weight 2^-24 and more; the one
// left out is below 2^-32 of the whole product, so a single product is as exact as an
// FP32 one (one tap over 300 x 420 pixels: largest error 5.9e-8; the six products of
// weight 2^-16 and more alone gave 8.7e-8, at 0.286 instead of 0.355 ms per iteration of
// 8 x 1024^2).  The largest product has an accumulator of its own.
template <>
struct Prec<EM_FP32> {
  using frag = bf16x8;
  static constexpr int NA = 3, NB = 3, NP = 8;
  static constexpr bool SCALED = false;
  __device__ static constexpr int pa(int s) { return s == 1 || s == 3 || s == 6 ? 1 : s == 4 || s == 7 ? 2 : 0; }
  __device__ static constexpr int pb(int s) { return s == 2 || s == 3 || s == 7 ? 1 : s == 5 || s == 6 ? 2 : 0; }
  __device__ static inline f32x4 mma(const frag& a, const frag& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// EM_FP32: the factors of the operands.
constexpr float CELL_UP = 0x1p16f;       // the taps; an image tile of values below 2^60
constexpr float CELL_UP_BIG = 0x1p-32f;  // any other image tile
__device__ inline float cell_up(bool big) { return big ? CELL_UP_BIG : CELL_UP; }
__device__ inline float cell_least(bool big) { return big ? 0x1p-40f : 0.f; }
// what undoes them in a sum of products
__device__ inline float cell_down(bool big) { return big ? 0x1p16f : 0x1p-32f; }
// |v| >= 2^60, infinite or NaN, for the largest of several `bits`
__device__ inline uint32_t cell_mag(float v) { return __float_as_uint(v) & 0x7fffffffu; }
__device__ inline bool cell_big(uint32_t bits) { return bits >= (127u + 60u) << 23; }
// True in every thread where `mine` is in one of the workgroup's NW waves; a barrier.
// flags: LDS, not written again before the next barrier.
template <int NW>
__device__ inline bool cell_any(bool mine, int w, int* flags) {
  if ((threadIdx.x & 63) == 0) flags[w] = 0;
  if (__any(mine) && (threadIdx.x & 63) == 0) flags[w] = 1;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) any |= flags[i];
  return __builtin_amdgcn_readfirstlane(any) != 0;
}

// Parts of two values (FP32: with their factor), packed bf16 pairs.
template <int PREC>
__device__ inline void cell_split2(f32x2 v, uint32_t (&q)[Prec<PREC>::NB]) {
  bf16x2 h = __builtin_convertvector(v, bf16x2);
  q[0] = __builtin_bit_cast(uint32_t, h);
#pragma unroll
  for (int p = 1; p < Prec<PREC>::NB; ++p) {
    const f32x2 f = __builtin_convertvector(h, f32x2);
    v = f32x2{v.x - f.x, v.y - f.y};
    h = __builtin_convertvector(v, bf16x2);
    q[p] = __builtin_bit_cast(uint32_t, h);
  }
}

// Which parts of the table a form holds and which products it takes.  BAND:
// the parts beyond the first enter only on the 21 kernel rows within 10 of the
// centre (window rows 12..35, j = 3..8), table rows outside them are zero.
template <int PREC_, bool BAND_>
struct CellForm {
  using P = Prec<PREC_>;
  using frag = typename P::frag;
  static constexpr int PREC = PREC_;
  static constexpr bool BAND = BAND_;
  static constexpr int NA = P::NA, NB = P::NB, NP = P::NP;
  // EM_FP32: sums in levels.  The largest product of each LEVEL rows of a class is
  // summed apart from the other products and from the other rows, then the class,
  // then the frame (adjoint: all frames, in FP64), so that the sums round less than
  // the direct convolution's 43-term chains do
  static constexpr bool LEVELS = PREC_ == EM_FP32;
  static constexpr int LEVEL = 3;
  // rows per unit (table fragments are staged in LDS one unit at a time, two
  // units in LDS), units per class
  static constexpr int JU = PREC_ == EM_FP32 ? 3 : 6;
  static constexpr int NU = CELL_NJ / JU;
  static constexpr bool has_main(int part, int j) { return part == 0 || !BAND || (j >= 3 && j <= 8); }
  // a tail fragment of part `part` for rows j and j + 1
  static constexpr bool has_tail(int part, int j) {
    return (part == 0 || !BAND) ? (j % 2 == 0) : (j == 3 || j == 5 || j == 7);
  }
  // products of image part pa with table part pb.  The image's lo part meets the
  // first table part, whose tails pair even rows: its tails cover rows 2..9.
  static constexpr bool mul_main(int pa, int pb, int j) { return has_main(pa > pb ? pa : pb, j); }
  static constexpr bool mul_tail(int pa, int pb, int j) {
    return has_tail(pb, j) && (pa == 0 || !BAND || (j >= 2 && j <= 8));
  }
  // steps (of G cell rows) at which an image part beyond the first is used
  static constexpr bool lo_step(int s, int G) { return !BAND || (s >= 2 && s <= 8 + G - 1); }
  // position of a fragment in its unit (main fragments of every part, then tails)
  static constexpr int slot(int part, int j, bool tail) {
    const int j0 = j / JU * JU;
    int s = 0;
    for (int p = 0; p < NB; ++p)
      for (int t = 0; t < 2; ++t)
        for (int i = j0; i < j0 + JU; ++i) {
          if (p == part && t == (tail ? 1 : 0) && i == j) return s;
          if (t == 0 ? has_main(p, i) : has_tail(p, i)) ++s;
        }
    return s;
  }
  static constexpr int unit_frags(int u) {
    int s = 0;
    for (int p = 0; p < NB; ++p)
      for (int i = u * JU; i < (u + 1) * JU; ++i) s += (has_main(p, i) ? 1 : 0) + (has_tail(p, i) ? 1 : 0);
    return s;
  }
  static constexpr int max_unit() {
    int m = 0;
    for (int u = 0; u < NU; ++u) m = unit_frags(u) > m ? unit_frags(u) : m;
    return m;
  }
  static constexpr int NFU = max_unit();              // fragments of a staged unit
  static constexpr int UPF = 4 * NU;                   // units per frame
  static constexpr int64_t FRAME = (int64_t)UPF * NFU * 64;   // 16-byte lanes per frame's table
};

// G cell rows per wave, WR x WC waves: (4 G WR) x (64 WC) outputs per workgroup.
template <class F_, int G_, int WR_, int WC_>
struct CellCfg {
  using F = F_;
  using frag = typename F::frag;
  static constexpr int G = G_, WR = WR_, WC = WC_;
  static constexpr int NW = WR * WC, NT = 64 * NW;
  static constexpr int TH = 4 * G * WR, TW = 64 * WC;
  static constexpr int ROWS = TH + CELL_EXTRA;   // image rows k0 - 22 .. k0 + TH + 21
  static constexpr int COLS = TW + 48;            // image columns l0 - 22 .. l0 + TW + 25
  static constexpr int PITCH = COLS;              // halves; rows start on 16-byte boundaries
  static constexpr int RS = 4;                    // rows from one cell row of a wave to its next
};

// Eight consecutive 16-bit values of a staged plane (8-byte aligned).
template <class F>
__device__ inline F cell_ld8(const unsigned short* p) {
  const uint2* q = reinterpret_cast<const uint2*>(p);
  const uint2 a = q[0], b = q[1];
  return __builtin_bit_cast(F, make_uint4(a.x, a.y, b.x, b.y));
}

// s_waitcnt vmcnt(N) lgkmcnt(0)
template <int N>
__device__ inline void cell_wait() {
  static_assert(N >= 0 && N < 16, "low field of vmcnt");
  __builtin_amdgcn_s_waitcnt(0x0070 | N);
}

// The table fragments in LDS: unit u of a class is staged in slot u & 1 (NU is
// even, so the parity is the unit's own).  The slots are separate LDS arrays,
// so that a read of one is not ordered behind the copies into the other.
template <class F>
struct CellSlots {
  static_assert(F::NU % 2 == 0, "a unit's slot is known at compile time");
  typename F::frag *s0, *s1;
};

// Copy unit `unit` (counted over the frames of the group) of a table into a slot;
// the waves share its fragments (the last fragment is copied again where they do
// not divide evenly: every wave issues the same number of copies, without a
// branch, which the wait counts below rely on).  w: this wave, wave-uniform.
template <class C>
__device__ inline void cell_issue_unit(const typename C::frag* __restrict__ tab, int unit, int w,
                                       typename C::frag* slot) {
  using F = typename C::F;
  const typename C::frag* src = tab + (int64_t)unit * F::NFU * 64 + (threadIdx.x & 63);
#pragma unroll
  for (int f = 0; f < F::NFU; f += C::NW) {
    const int i = f + C::NW <= F::NFU ? f + w : min(f + w, F::NFU - 1);
    __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)(src + i * 64),
                                     (__attribute__((address_space(3))) void*)(slot + i * 64), 16,
                                     0, 0);
  }
}

// Where a wave is in its table: units run over all frames of the group.
template <class F>
struct CellTab {
  const typename F::frag* tab;
  int unit, units, w;
  CellSlots<F> slots;
  double down;   // FP32 adjoint: what undoes the factors of the current frame's operands
};

// Work added at the unit boundaries of a frame (0 .. UPF - 1).  wait(b), before
// the barrier of boundary b: at least this wave's copies of the next unit have
// landed and its LDS reads are done.  after(b): behind the barrier, and behind
// the issue of the copies of the unit after the next.
struct CellNoHook {
  __device__ void wait(int) const { cell_wait<0>(); }
  __device__ void after(int) const {}
};

// Unit boundary: this wave's copies of the next unit have landed, every wave has
// read the current one; then the slot just freed takes the unit after the next
// (past the last one, the same unit again, so that every boundary issues the
// same copies and needs no branch).
template <class C, int U, class Hook>
__device__ inline void cell_boundary(CellTab<typename C::F>& T, int boundary, Hook& hook) {
  hook.wait(boundary);
  __builtin_amdgcn_s_barrier();
  __asm__ volatile("" ::: "memory");
  cell_issue_unit<C>(T.tab, T.unit + 2 < T.units ? T.unit + 2 : T.unit, T.w,
                     U % 2 == 0 ? T.slots.s0 : T.slots.s1);
  ++T.unit;
  hook.after(boundary);
}

// Where a frame's classes are added up.  FP32: the adjoint adds them to the sum over its
// frames, in FP64 (in FP32 the sum of 15 frames of 942 x 2100 latent pixels, one
// group, took x after two iterations from 1.14e-7, with groups of three frames in the
// direct convolution, to 1.44e-7).
typedef __attribute__((ext_vector_type(4))) double f64x4;
__device__ EM_INLINE inline void cell_add(f32x4& sum, const f32x4& v, double) { sum += v; }
__device__ EM_INLINE inline void cell_add(f64x4& sum, const f32x4& v, double down) {
  sum += __builtin_convertvector(v, f64x4) * down;
}
template <bool LEVELS>
using CellSum = std::conditional_t<LEVELS, f64x4, f32x4>;

// One class of one frame.  im, it: this lane's window start in the staged planes
// for the main and the tail chunk (plane 0, window row E of the wave's first
// cell row); plane: distance of the planes.
template <class C, int E, class Sum, class Hook>
__device__ __attribute__((always_inline)) inline void cell_class(
    const unsigned short* im, const unsigned short* it, int plane, CellTab<typename C::F>& T,
    Sum (&acc)[C::G], Hook& hook) {
  using F = typename C::F;
  using frag = typename C::frag;
  constexpr int G = C::G, NS = G + CELL_NJ - 1;
  const int lane = threadIdx.x & 63;
  frag Tm[F::NB][CELL_NJ], Tt[F::NB][CELL_NJ];
  frag Am[2][F::NA], At[2][F::NA];
  // rows 0 of class 0 and 47 of class 3 meet no tap in any output of a cell
  constexpr auto main_used = [](int p, int j) {
    return F::has_main(p, j) && !(E == 0 && j == 0) && !(E == 3 && j == CELL_NJ - 1);
  };
  auto load_T = [&](auto jc) EM_INLINE {
    constexpr int j = jc;
    const frag* sl = ((j / F::JU) % 2 == 0 ? T.slots.s0 : T.slots.s1) + lane;
    static_for<F::NB>([&](auto pc) EM_INLINE {
      constexpr int p = pc;
      if constexpr (main_used(p, j)) Tm[p][j] = sl[F::slot(p, j, false) * 64];
      if constexpr (F::has_tail(p, j)) Tt[p][j] = sl[F::slot(p, j, true) * 64];
    });
  };
  // image fragments of step s; parts beyond the first only where a product needs them
  auto load_A = [&](auto sc) EM_INLINE {
    constexpr int s = sc;
    static_for<F::NA>([&](auto pc) EM_INLINE {
      constexpr int p = pc;
      if constexpr (p == 0 || F::lo_step(s, G)) {
        Am[s & 1][p] = cell_ld8<frag>(im + p * plane + 4 * s * C::PITCH);
        if constexpr (s < NS - 1) At[s & 1][p] = cell_ld8<frag>(it + p * plane + 4 * s * C::PITCH);
      }
    });
  };
  f32x4 big[F::LEVELS ? G : 1], small[F::LEVELS ? G : 1], cls[F::LEVELS ? G : 1];
  if constexpr (F::LEVELS)
    static_for<G>([&](auto gc) EM_INLINE { big[gc] = small[gc] = f32x4{0.f, 0.f, 0.f, 0.f}; });
  load_T(std::integral_constant<int, 0>{});
  load_A(std::integral_constant<int, 0>{});
  static_for<NS>([&](auto sc) EM_INLINE {
    constexpr int s = sc;
    if constexpr (s > 0 && s % F::JU == 0 && s <= CELL_NJ)
      cell_boundary<C, s / F::JU - 1>(T, E * F::NU + s / F::JU - 1, hook);
    if constexpr (s > 0 && s < CELL_NJ && s % F::JU == 0) load_T(sc);
    if constexpr (s + 1 < CELL_NJ && (s + 1) % F::JU != 0) load_T(std::integral_constant<int, s + 1>{});
    if constexpr (s + 1 < NS) load_A(std::integral_constant<int, s + 1>{});
    // keep these loads ahead of this step's products
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (F::LEVELS)
      static_for<G>([&](auto gc) EM_INLINE {
        constexpr int j = s - gc;
        if constexpr (j > 0 && j < CELL_NJ && j % F::LEVEL == 0) {
          if constexpr (j == F::LEVEL) cls[gc] = big[gc];
          else cls[gc] += big[gc];
          big[gc] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      });
    static_for<F::NP>([&](auto kc) EM_INLINE {
      constexpr int pa = F::P::pa(kc), pb = F::P::pb(kc);
      static_for<G>([&](auto gc) EM_INLINE {
        constexpr int g = G - 1 - gc, j = s - g;
        if constexpr (j >= 0 && j < CELL_NJ) {
          auto take = [&](f32x4& sum) EM_INLINE {
            if constexpr (F::mul_main(pa, pb, j) && main_used(pb, j))
              sum = F::P::mma(Tm[pb][j], Am[s & 1][pa], sum);
            if constexpr (F::mul_tail(pa, pb, j)) sum = F::P::mma(Tt[pb][j], At[s & 1][pa], sum);
          };
          if constexpr (!F::LEVELS) take(acc[g]);
          else if constexpr (pa + pb == 0) take(big[g]);
          else take(small[g]);
        }
      });
    });
  });
  if constexpr (F::LEVELS)
    static_for<G>([&](auto gc) EM_INLINE {
      cell_add(acc[gc], cls[gc] + (big[gc] + small[gc]), T.down);
      // add now: sunk to the frame's end, the addends of every class would be spilled
      __asm__ volatile("" : "+v"(acc[gc]));
    });
}

// All classes of one frame into acc (one wave's G cell rows x 16 cells).  On
// entry the frame's first unit is in its slot (a barrier after its copy has
// been passed) and the second is in flight or landed.
template <class C, class Sum, class Hook>
__device__ __attribute__((always_inline)) inline void cell_frame(
    const unsigned short* im, const unsigned short* it, int plane, CellTab<typename C::F>& T,
    Sum (&acc)[C::G], Hook& hook) {
  cell_class<C, 0>(im, it, plane, T, acc, hook);
  cell_class<C, 1>(im + C::PITCH, it + C::PITCH, plane, T, acc, hook);
  cell_class<C, 2>(im + 2 * C::PITCH, it + 2 * C::PITCH, plane, T, acc, hook);
  cell_class<C, 3>(im + 3 * C::PITCH, it + 3 * C::PITCH, plane, T, acc, hook);
}

// Which fragment of unit u of a class stands in position `frag` (part < 0: none).
struct CellFragId {
  int part, j;
  bool tail;
};
template <class F>
__device__ inline CellFragId cell_frag_id(int u, int frag) {
  CellFragId id{-1, 0, false};
  for (int p = 0; p < F::NB; ++p)
    for (int j = u * F::JU; j < (u + 1) * F::JU; ++j) {
      if (F::has_main(p, j) && F::slot(p, j, false) == frag) id = {p, j, false};
      if (F::has_tail(p, j) && F::slot(p, j, true) == frag) id = {p, j, true};
    }
  return id;
}

// Part `part` of one tap (0 where there is none).
template <int PREC>
__device__ inline unsigned short cell_part(float v, int part) {
  uint32_t q[Prec<PREC>::NB];
  cell_split2<PREC>(f32x2{PREC == EM_FP32 ? v * CELL_UP : v, 0.f}, q);
  uint32_t out = 0;
#pragma unroll
  for (int x = 0; x < Prec<PREC>::NB; ++x) out = x == part ? q[x] : out;
  return (unsigned short)out;
}

// Position of this lane: cell row pr of its outputs, its cell's first column.
struct CellLane {
  int row0, col;   // image row of group 0's outputs of this lane, first of 4 columns
};

template <class C>
__device__ inline CellLane cell_lane(int k0, int l0) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return {k0 + (w / C::WC) * 4 * C::G + (lane >> 4), l0 + (w % C::WC) * 64 + 4 * (lane & 15)};
}

// Offsets (halves) of this lane's window in a staged plane: main and tail chunk.
template <class C>
__device__ inline int cell_main_off() {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return (w / C::WC) * 4 * C::G * C::PITCH + (w % C::WC) * 64 + 4 * (lane & 15) + 8 * (lane >> 4);
}
template <class C>
__device__ inline int cell_tail_off() {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, gq = lane >> 4;
  return (w / C::WC) * 4 * C::G * C::PITCH + (w % C::WC) * 64 + 4 * (lane & 15) +
         (gq >> 1) * 4 * C::PITCH + 32 + 8 * (gq & 1);
}

// FP32: undoes the operands' factors.  An infinity or NaN in an operand does not survive
// the split into parts (inf - inf) and meets the zeros of the table around the 43 x 43
// taps, so it makes NaN of every output whose 46 x 48 window holds it.  The outputs
// that are not finite are formed once more as the direct convolution does, one at a
// time: `value(g, i)` for element i of cell row g; so are those below `least` (in a
// tile of the lower factor, whose smallest operands are cut off).  The BF16 forms leave
// them: NaN up to three pixels outside the support (with this step their adjoint
// spilled: 33 x 1999 x 2111 1.04 -> 1.09 ms).
template <int G, class Fn>
__device__ EM_INLINE inline void cell_finish(f32x4 (&acc)[G], float down, float least, Fn&& value) {
  uint32_t bad = 0;
#pragma unroll
  for (int e = 0; e < 4 * G; ++e) {
    acc[e / 4][e % 4] *= down;
    const float m = fabsf(acc[e / 4][e % 4]);
    bad |= m >= least && m <= 3.4028235e38f ? 0u : 1u << e;
  }
  while (bad != 0) {
    const int at = __ffs(bad) - 1;
    bad &= bad - 1;
    const float v = value(at >> 2, at & 3);
#pragma unroll
    for (int e = 0; e < 4 * G; ++e) acc[e / 4][e % 4] = e == at ? v : acc[e / 4][e % 4];
  }
}

// One output of the direct sr = 1 convolution (dir 0: F_t x, 1: F_t^T r), its order of
// sums: one kernel column, then the total.  taps: the frame's coefficient table.
__device__ inline float cell_direct(const float* __restrict__ taps, const float* __restrict__ in,
                                    int H, int W, int k, int l, int dir) {
  constexpr int c = (CELL_K - 1) / 2;
  float sum = 0.f;
#pragma unroll 1
  for (int b = 0; b < CELL_K; ++b) {
    const int x = dir == 0 ? l + c - b : l - c + b;
    float part = 0.f;
#pragma unroll 4
    for (int a = 0; a < CELL_K; ++a) {
      const int y = dir == 0 ? k + c - a : k - c + a;
      const float v = y >= 0 && y < H && x >= 0 && x < W ? in[(int64_t)y * W + x] : 0.f;
      part = fmaf(taps[b * TAB_LD + a], v, part);
    }
    sum += part;
  }
  return sum;
}

__device__ inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Four consecutive values of row `row` from column `col` (clamped into the
// image; a clamped value is never used).
__device__ inline void load4(const float* __restrict__ p, int row, int col, int H, int W, bool vec,
                             float (&v)[4]) {
  const int64_t base = (int64_t)min(row, H - 1) * W;
  if (vec) {
    const float4 q = *reinterpret_cast<const float4*>(p + base + col);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = p[base + min(col + i, W - 1)];
  }
}
__device__ inline void store4(float* __restrict__ p, int row, int col, int W, bool vec,
                              const float (&v)[4]) {
  float* q = p + (int64_t)row * W + col;
  if (vec) {
    *reinterpret_cast<float4*>(q) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (col + i < W) q[i] = v[i];
  }
}

// The image tile of a workgroup on its way into the LDS planes: raw pixels in
// registers, then split and stored.  A wave takes the rows w, w + NW, ... of the
// tile, its first COLS / 4 lanes four columns each, so that the row address is
// scalar and the column arithmetic is done once.  Loads read 16 bytes from
// addresses clamped into the image (all are in flight together); values outside
// it become 0 when stored.
template <class C>
struct CellTile {
  using F = typename C::F;
  struct __attribute__((packed, aligned(4))) Quad { float v[4]; };
  static constexpr int NR = (C::ROWS + C::NW - 1) / C::NW;   // rows per wave
  static constexpr int PLANE = C::ROWS * C::PITCH;
  static_assert(C::COLS % 4 == 0 && C::COLS <= 256, "four columns per lane");
  int H, W, r0, w;
  int gx;       // image column of this lane's first value
  bool inner;   // every column of the tile is inside the image (uniform)
  f32x4 v[NR];
  __device__ CellTile(int H_, int W_, int k0, int l0, int w_)
      : H(H_), W(W_), r0(k0 - CELL_OFF), w(w_),
        gx(l0 - CELL_OFF + 4 * min((int)(threadIdx.x & 63), C::COLS / 4 - 1)),
        inner(l0 - CELL_OFF >= 0 && l0 - CELL_OFF + C::COLS <= W_) {}
  // first column read: the four columns from gx, moved inside an image of at least
  // four columns
  __device__ int first(int g) const { return min(max(g, 0), max(W - 4, 0)); }
  __device__ void load(const float* __restrict__ src) {
    int g = gx;
    __asm__ volatile("" : "+v"(g));   // keep the address arithmetic here
    const int c = first(g);
    if (W >= 4) {
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int gy = min(max(r0 + w + C::NW * i, 0), H - 1);
        const Quad q = *reinterpret_cast<const Quad*>(src + (int64_t)gy * W + c);
        v[i] = f32x4{q.v[0], q.v[1], q.v[2], q.v[3]};
      }
    } else {
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const float* rp = src + (int64_t)min(max(r0 + w + C::NW * i, 0), H - 1) * W;
        v[i] = f32x4{rp[0], rp[min(1, W - 1)], rp[min(2, W - 1)], 0.f};
      }
    }
  }
  // FP32: whether the tile takes the lower factor (a lane's share of the answer)
  __device__ bool big() const {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int x = 0; x < 4; ++x) m = max(m, cell_mag(v[i][x]));
    return cell_big(m);
  }
  // up: the factor of the values (FP32)
  __device__ void store(unsigned short* sh, float up) {
    int g = gx;
    __asm__ volatile("" : "+v"(g));
    if (!inner) {
      // move each value to its column, 0 outside the image
      const int d = g - first(g);
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const f32x4 o = v[i];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int at = x + d;
          const float val = at <= 0 ? o[0] : at == 1 ? o[1] : at == 2 ? o[2] : o[3];
          v[i][x] = (g + x >= 0 && g + x < W) ? val : 0.f;
        }
      }
    }
    if ((int)(threadIdx.x & 63) >= C::COLS / 4) return;
    unsigned short* dst = sh + w * C::PITCH + 4 * (threadIdx.x & 63);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int row = w + C::NW * i, gy = r0 + row;
      if ((i + 1) * C::NW > C::ROWS && row >= C::ROWS) break;
      const bool iny = gy >= 0 && gy < H;
      uint32_t a[F::NB], b[F::NB];
      f32x4 o = v[i];
      if constexpr (F::PREC == EM_FP32) o = f32x4{o[0] * up, o[1] * up, o[2] * up, o[3] * up};
      cell_split2<F::PREC>(iny ? f32x2{o[0], o[1]} : f32x2{0.f, 0.f}, a);
      cell_split2<F::PREC>(iny ? f32x2{o[2], o[3]} : f32x2{0.f, 0.f}, b);
#pragma unroll
      for (int p = 0; p < F::NA; ++p)
        *reinterpret_cast<uint2*>(dst + p * PLANE + C::NW * i * C::PITCH) = make_uint2(a[p], b[p]);
    }
  }
};

// Epilogue of the adjoint: Dn = acc; the fused update of Eq. (2) with its FP64
// change partials, or a store into the partial plane.  C::RS: rows from one of the
// wave's cell rows to the next.
template <class C>
__device__ inline void cell_adj_epilogue(const MfmaLaunch& a, const f32x4 (&acc)[C::G],
                                         const CellLane& p, int tile, int group, double* red) {
  const int64_t N = (int64_t)a.H * a.W;
  float* plane = a.fused ? nullptr : a.plane + (int64_t)group * N;
  const bool al = (a.W & 3) == 0 && (a.fused ? aligned16(a.x) && aligned16(a.B) : aligned16(plane));
  const bool vec = al && p.col + 3 < a.W;
  double dsq = 0.0, xsq = 0.0;
  if (!a.fused) {
#pragma unroll
    for (int g = 0; g < C::G; ++g) {
      const int k = p.row0 + C::RS * g;
      const float v[4] = {acc[g][0], acc[g][1], acc[g][2], acc[g][3]};
      if (k < a.H && p.col < a.W) store4(plane, k, p.col, a.W, vec, v);
    }
    return;
  }
  float xo[C::G][4], bv[C::G][4];
#pragma unroll
  for (int g = 0; g < C::G; ++g) {
    load4(a.x, p.row0 + C::RS * g, p.col, a.H, a.W, vec, xo[g]);
    load4(a.B, p.row0 + C::RS * g, p.col, a.H, a.W, vec, bv[g]);
  }
#pragma unroll
  for (int g = 0; g < C::G; ++g) {
    const int k = p.row0 + C::RS * g;
    if (k >= a.H || p.col >= a.W) continue;
    float xn[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      xn[i] = em_update_value(xo[g][i], bv[g][i], acc[g][i]);
      if (p.col + i < a.W) {
        const double d = (double)xn[i] - (double)xo[g][i];
        dsq += d * d;
        xsq += (double)xo[g][i] * (double)xo[g][i];
      }
    }
    store4(a.x, k, p.col, a.W, vec, xn);
  }
  if (a.part != nullptr) {
    const double s1 = block_sum<C::NT>(dsq, red);
    __syncthreads();
    const double s2 = block_sum<C::NT>(xsq, red + C::NW);
    if (threadIdx.x == 0) {
      a.part[2 * tile] = s1;
      a.part[2 * tile + 1] = s2;
    }
  }
}

}  // namespace em
