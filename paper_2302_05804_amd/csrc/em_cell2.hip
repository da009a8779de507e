// em_cell2.hip -- the convolutions of the super-resolution iteration
// (arXiv:2302.05804, Sec. 2, Eq. (3) inside Eq. (2)) on 4 x 4 latent cells of the
// matrix cores, for kernels padded to 43 x 43, in FP32 (three bf16 parts).
//
// With k = h * 1_{2x2} the 44 x 44 box-extended kernel of a frame:
//
// Forward, m[I][J] = sum_{a,b < 44} k[43 - a][43 - b] x[2I - 21 + a][2J - 21 + b]:
// the core of em_cell.h with another table.  A 4 x 4 latent cell holds 2 x 2 frame
// pixels, whose windows are 46 x 46 latent pixels, so one product takes the
// 2 x 2 pixels of four frames (M = 4 frame + 2 p + q); the x window is the same for
// all of them:
//     T[4f + 2p + q][d, k] = g_f[d - 1 - 2p][k - 1 - 2q],  g = k flipped:
// 44 x 44 of the 46 x 48 window values are taps (88%).
//
// Adjoint, s[k][l] = sum_{I,J} r[I][J] k[2I + 22 - k][2J + 22 - l]: the 16 latent
// pixels of a cell at latent (2 i0, 2 j0) share the window of r at rows
// i0 - 11 .. i0 + 12, columns j0 - 11 .. j0 + 12, with
//     T[4p + q][d, k] = k[2d - p][2k - q]   (0 outside 0..43),
// 22 x 22 of 24 x 24 window values (84%).  Cell rows are two frame rows apart, so
// with d = 2 j + E (E = 0, 1; j = 0..11) frame row 2 s + E serves the cell rows
// s - j.  A row of the window is three 8-wide pieces, and four rows of a class
// are three products: pieces 0-3, 4-7 and 8-11 of rows s .. s + 3 in order.  A
// wave owns every fourth cell row, so that the three products of rows s .. s + 3
// (read once from LDS) serve j = 0, 4 and 8 of three of its cell rows; the 9
// table fragments of a class and part stay in registers.
//
// 9 x 701 x 1022 frames: forward 0.36 -> 0.243 ms, adjoint 0.27 -> 0.180 ms against
// the direct convolution, both near 1.2 PFLOP/s of issued products (two rounds of
// tiles on 256 compute units, three of twelve frame slots empty in the forward).
#include "em_cell.h"

#include <type_traits>

namespace em {

namespace {

constexpr int CELL2_KC = 44;     // side of the box-extended kernel

// Frames of a product of the forward.
constexpr int CELL2_FQ = 4;

// k[a][b] of frame t: the 2 x 2 box extension of h (K x K, zero-padded to 43).
__device__ inline float box_kernel(const float* __restrict__ h, int K, int a, int b) {
  const int off = (CELL_K - K) / 2;
  double v = 0.0;
  for (int p = 0; p < 2; ++p)
    for (int q = 0; q < 2; ++q) {
      const int i = a - p - off, j = b - q - off;
      if (i >= 0 && i < K && j >= 0 && j < K) v += (double)h[i * K + j];
    }
  return (float)v;
}

// One output of the direct convolutions with the 44 x 44 kernel, as cell_direct.
// H, W: the frame grid; the forward's image is on the latent grid.
__device__ inline float cell2_direct_fwd(const float* __restrict__ taps, const float* __restrict__ x,
                                         int H, int W, int I, int J) {
  float sum = 0.f;
#pragma unroll 1
  for (int b = 0; b < CELL2_KC; ++b) {
    const int l = 2 * J + CELL2_KC / 2 - b;
    float part = 0.f;
#pragma unroll 4
    for (int a = 0; a < CELL2_KC; ++a) {
      const int k = 2 * I + CELL2_KC / 2 - a;
      const float v = k >= 0 && k < 2 * H && l >= 0 && l < 2 * W ? x[(int64_t)k * 2 * W + l] : 0.f;
      part = fmaf(taps[b * TAB_LD + a], v, part);
    }
    sum += part;
  }
  return sum;
}
__device__ inline float cell2_direct_adj(const float* __restrict__ taps, const float* __restrict__ r,
                                         int H, int W, int k, int l) {
  float sum = 0.f;
#pragma unroll 1
  for (int b = l & 1; b < CELL2_KC; b += 2) {
    const int J = (l + b - CELL2_KC / 2) / 2;   // even and -22 or more: -11 at least
    float part = 0.f;
#pragma unroll 2
    for (int a = k & 1; a < CELL2_KC; a += 2) {
      const int I = (k + a - CELL2_KC / 2) / 2;
      const float v = I >= 0 && I < H && J >= 0 && J < W ? r[(int64_t)I * W + J] : 0.f;
      part = fmaf(taps[b * TAB_LD + a], v, part);
    }
    sum += part;
  }
  return sum;
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------

using Fwd2 = CellCfg<CellForm<EM_FP32, false>, 4, 4, 2>;

// Two consecutive frame pixels (columns clamped into the frame when not vec).
__device__ inline f32x2 load2(const float* __restrict__ p, int row, int col, int H, int W, bool vec) {
  const int64_t base = (int64_t)min(row, H - 1) * W;
  if (vec) return *reinterpret_cast<const f32x2*>(p + base + col);
  return f32x2{p[base + min(col, W - 1)], p[base + min(col + 1, W - 1)]};
}
__device__ inline void store2(float* __restrict__ p, int row, int col, int W, bool vec, float a, float b) {
  float* q = p + (int64_t)row * W + col;
  if (vec) {
    *reinterpret_cast<f32x2*>(q) = f32x2{a, b};
  } else {
    q[0] = a;
    if (col + 1 < W) q[1] = b;
  }
}

// Forward of four frames at a time: r_t = u_t F_t x, or F_t x when u is NULL (FP64
// partials of u (y - m)^2 when asked); STUDENT: u w m and u w y.  Lane group
// lane / 16 holds one frame of the four, its element 2 p + q pixel (p, q) of the
// lane's cell.
template <class C, bool STUDENT>
__device__ inline void cell2_fwd_body(const MfmaLaunch& a, const int tile, const int group) {
  using F = typename C::F;
  using frag = typename C::frag;
  constexpr int PLANE = C::ROWS * C::PITCH;
  constexpr int TH = C::TH / 2, TW = C::TW / 2;   // frame pixels
  __shared__ __align__(16) unsigned short sh[F::NA * PLANE];
  __shared__ __align__(16) frag slot0[F::NFU * 64];
  __shared__ __align__(16) frag slot1[F::NFU * 64];
  __shared__ double red[C::NW];
  __shared__ int flags[C::NW];
  const int tiles_x = (a.W + TW - 1) / TW;
  const int I0 = (tile / tiles_x) * TH, J0 = (tile % tiles_x) * TW;
  const int t0 = group * a.fpg;
  const int t1 = min(a.n, t0 + a.fpg);
  const int quads = (t1 - t0 + CELL2_FQ - 1) / CELL2_FQ;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  CellTab<F> T{reinterpret_cast<const frag*>(a.tab) + (int64_t)(t0 / CELL2_FQ) * F::FRAME, 0,
               quads * F::UPF, w, {slot0, slot1}, 1.0};
  cell_issue_unit<C>(T.tab, 0, w, slot0);
  cell_issue_unit<C>(T.tab, 1, w, slot1);
  bool big;
  {
    CellTile<C> tl(2 * a.H, 2 * a.W, 2 * I0, 2 * J0, w);
    tl.load(a.in);
    big = cell_any<C::NW>(tl.big(), w, flags);
    tl.store(sh, cell_up(big));
  }
  cell_wait<0>();
  __syncthreads();
  const int64_t N = (int64_t)a.H * a.W;
  const unsigned short* im = sh + cell_main_off<C>();
  const unsigned short* it = sh + cell_tail_off<C>();
  const int row_l = I0 + (w / C::WC) * 2 * C::G, col_l = J0 + (w % C::WC) * 32 + 2 * (lane & 15);
  const bool ll = a.part != nullptr;
  auto al8 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7) == 0; };
  const bool vec = (a.W & 1) == 0 && col_l + 1 < a.W && al8(a.u) && al8(a.out) && al8(a.y) && al8(a.out_y);
  double llp = 0.0;
  for (int q = 0; q < quads; ++q) {
    // keep the tile's reads and the epilogue's addresses inside the loop
    int row = row_l, col = col_l;
    __asm__ volatile("" : "+v"(row), "+v"(col)::"memory");
    f32x4 acc[C::G];
#pragma unroll
    for (int g = 0; g < C::G; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    CellNoHook hook;
    cell_frame<C>(im, it, PLANE, T, acc, hook);
    const int t = t0 + CELL2_FQ * q + (lane >> 4);
    if (t >= t1 || col >= a.W) continue;
    cell_finish(acc, cell_down(big), cell_least(big), [&](int g, int e) EM_INLINE {
      const int I = row + 2 * g + (e >> 1), J = col + (e & 1);
      return I < a.H && J < a.W
                 ? cell2_direct_fwd(a.taps + (int64_t)t * CELL2_KC * TAB_LD, a.in, a.H, a.W, I, J)
                 : 0.f;
    });
    const float* ut = a.u ? a.u + (int64_t)t * N : nullptr;
    const float* yt = (STUDENT || (ll && ut)) ? a.y + (int64_t)t * N : nullptr;
    float* ot = a.out ? a.out + (int64_t)t * N : nullptr;
    f32x2 uu[C::G][2], yy[C::G][2];
#pragma unroll
    for (int g = 0; g < C::G; ++g)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        uu[g][p] = ut ? load2(ut, row + 2 * g + p, col, a.H, a.W, vec) : f32x2{1.f, 1.f};
        yy[g][p] = yt ? load2(yt, row + 2 * g + p, col, a.H, a.W, vec) : f32x2{0.f, 0.f};
      }
#pragma unroll
    for (int g = 0; g < C::G; ++g)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int I = row + 2 * g + p;
        if (I >= a.H) continue;
        float r[2], ry[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float m = acc[g][2 * p + i], u = uu[g][p][i], y = yy[g][p][i];
          const bool in = col + i < a.W;
          if constexpr (STUDENT) {
            r[i] = 0.f;
            ry[i] = 0.f;
            if (u > 0.f) {
              const float d = y - m;
              const float wt = (a.nu + 1.f) / (a.nu + u * d * d);
              r[i] = (u * wt) * m;
              ry[i] = (u * wt) * y;
              if (ll && in) {
                const double dd = (double)y - (double)m;
                llp += ((double)a.nu + 1.0) * log1p((double)u * dd * dd / (double)a.nu) - a.lcst;
              }
            }
          } else {
            r[i] = ut ? u * m : m;
            if (yt && in && u > 0.f) {
              const double d = (double)y - (double)m;
              llp += (double)u * d * d;
            }
          }
        }
        if (ot) store2(ot, I, col, a.W, vec, r[0], r[1]);
        if constexpr (STUDENT) store2(a.out_y + (int64_t)t * N, I, col, a.W, vec, ry[0], ry[1]);
      }
  }
  cell_wait<0>();   // the copies issued past the last unit
  if (a.part != nullptr) {
    const double s = block_sum<C::NT>(llp, red);
    if (threadIdx.x == 0) a.part[(int64_t)group * a.ntiles + tile] = s;
  }
}

// Forward table of four frames (blockIdx.x), one unit per blockIdx.y, four fragments
// per blockIdx.z.
template <class F>
__global__ __launch_bounds__(256) void cell2_fwd_table_kernel(const float* psf, int n, int K,
                                                              unsigned short* tab) {
  const int unit = blockIdx.y, E = unit / F::NU, u = unit % F::NU;
  const int frag = 4 * blockIdx.z + (threadIdx.x >> 6);
  if (frag >= F::NFU) return;
  const int lane = threadIdx.x & 63, m = lane & 15, gq = lane >> 4;
  const CellFragId id = cell_frag_id<F>(u, frag);
  const int t = CELL2_FQ * blockIdx.x + (m >> 2);
  const float* h = psf + (int64_t)min(t, n - 1) * K * K;
  unsigned short* dst = tab + ((((int64_t)blockIdx.x * F::UPF + unit) * F::NFU + frag) * 64 + lane) * 8;
  for (int e = 0; e < 8; ++e) {
    const int d = 4 * (id.j + (id.tail ? gq >> 1 : 0)) + E;
    const int k = id.tail ? 32 + 8 * (gq & 1) + e : 8 * gq + e;
    const int ta = d - 1 - 2 * ((m >> 1) & 1), tb = k - 1 - 2 * (m & 1);
    float gv = 0.f;
    if (id.part >= 0 && t < n && ta >= 0 && ta < CELL2_KC && tb >= 0 && tb < CELL2_KC)
      gv = box_kernel(h, K, CELL2_KC - 1 - ta, CELL2_KC - 1 - tb);
    dst[e] = cell_part<F::PREC>(gv, id.part);
  }
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------

// G cell rows per wave, every fourth one (4 waves), WC waves across.
template <int G_, int WC_>
struct Adj2Cfg {
  using P = Prec<EM_FP32>;
  using frag = typename P::frag;
  static constexpr int G = G_, WC = WC_;
  static constexpr int NA = P::NA, NB = P::NB, NP = P::NP;
  static constexpr int NW = 4 * WC, NT = 64 * NW;
  static constexpr int TH = 16 * G, TW = 64 * WC;        // latent pixels
  static constexpr int ROWS = TH / 2 + 22, COLS = TW / 2 + 22;   // frame pixels staged
  static constexpr int PITCH = (COLS + 7) / 8 * 8;
  static constexpr int PLANE = ROWS * PITCH;
  static constexpr int RS = 16;
  static constexpr int NF = 9 * NB;                       // table fragments of a class
  static constexpr int64_t FRAME = (int64_t)2 * NF * 64;  // 16-byte lanes
  static constexpr int NPT = (PLANE + NT - 1) / NT;       // staged values per thread
};

template <class C>
__device__ inline void cell2_issue(const typename C::frag* __restrict__ src, int w,
                                   typename C::frag* slot) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int f = 0; f < C::NF; f += C::NW) {
    const int i = min(f + w, C::NF - 1);
    __builtin_amdgcn_global_load_lds(
        (__attribute__((address_space(1))) void*)(src + i * 64 + lane),
        (__attribute__((address_space(3))) void*)(slot + i * 64), 16, 0, 0);
  }
}

// Eight consecutive 16-bit values (4-byte aligned).
template <class Fr>
__device__ inline Fr cell2_ld8(const unsigned short* p) {
  const uint32_t* q = reinterpret_cast<const uint32_t*>(p);
  return __builtin_bit_cast(Fr, make_uint4(q[0], q[1], q[2], q[3]));
}

// The r tile of one frame on its way to LDS: raw values (clamped addresses), split
// and stored with 0 outside the frame.
template <class C>
struct Adj2Tile {
  float v[C::NPT];
  // as CellTile::big
  __device__ bool big() const {
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < C::NPT; ++k) m = max(m, cell_mag(v[k]));
    return cell_big(m);
  }
  template <bool STORE>
  __device__ void pass(const float* __restrict__ src, int H, int W, int i0, int j0, unsigned short* sh,
                       float up) {
    int e = threadIdx.x;
    __asm__ volatile("" : "+v"(e));   // the address arithmetic stays here
#pragma unroll
    for (int k = 0; k < C::NPT; ++k, e += C::NT) {
      const int row = e / C::PITCH, cc = e - row * C::PITCH;
      const int gy = i0 + row, gx = j0 + cc;
      if constexpr (!STORE) {
        v[k] = src[(int64_t)min(max(gy, 0), H - 1) * W + min(max(gx, 0), W - 1)];
      } else if (e < C::PLANE) {
        const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
        uint32_t q[C::NB];
        cell_split2<EM_FP32>(f32x2{in ? v[k] * up : 0.f, 0.f}, q);
#pragma unroll
        for (int p = 0; p < C::NA; ++p) sh[p * C::PLANE + e] = (unsigned short)q[p];
      }
    }
  }
};

// One class: `im[P]` this lane's piece of product P at step 0 (window row E).
template <class C>
__device__ EM_INLINE inline void cell2_class(const unsigned short* const (&im)[3],
                                             const typename C::frag* slot, f64x4 (&acc)[C::G], double down) {
  using frag = typename C::frag;
  constexpr int G = C::G;
  const int lane = threadIdx.x & 63;
  frag T[C::NB][9];
  static_for<C::NB>([&](auto pc) EM_INLINE {
    static_for<9>([&](auto fc) EM_INLINE { T[pc][fc] = slot[(pc * 9 + fc) * 64 + lane]; });
  });
  f32x4 big[G], small[G];
  static_for<G>([&](auto gc) EM_INLINE { big[gc] = small[gc] = f32x4{0.f, 0.f, 0.f, 0.f}; });
  static_for<G + 2>([&](auto sc) EM_INLINE {
    constexpr int s = sc;
    frag A[C::NA][3];
    static_for<C::NA>([&](auto pc) EM_INLINE {
      static_for<3>([&](auto Pc) EM_INLINE {
        A[pc][Pc] = cell2_ld8<frag>(im[Pc] + pc * C::PLANE + 8 * s * C::PITCH);
      });
    });
    static_for<C::NP>([&](auto kc) EM_INLINE {
      constexpr int pa = C::P::pa(kc), pb = C::P::pb(kc);
      static_for<3>([&](auto uc) EM_INLINE {
        constexpr int g = s - uc;
        if constexpr (g >= 0 && g < G) {
          f32x4& sum = pa + pb == 0 ? big[g] : small[g];
          static_for<3>([&](auto Pc) EM_INLINE { sum = C::P::mma(T[pb][3 * uc + Pc], A[pa][Pc], sum); });
        }
      });
    });
  });
  static_for<G>([&](auto gc) EM_INLINE {
    cell_add(acc[gc], big[gc] + small[gc], down);
    __asm__ volatile("" : "+v"(acc[gc]));   // add now, as in cell_class
  });
}

// Adjoint: sum over the frames of this group of F_t^T r_t.  Two r tiles and two
// classes of table fragments in LDS: during a frame's first class the next
// frame's r is loaded into registers, after it stored into the other tile; a
// class's fragments are copied while the class before it runs.
template <class C>
__device__ inline void cell2_adj_body(const MfmaLaunch& a, const int tile, const int group) {
  using frag = typename C::frag;
  __shared__ __align__(16) unsigned short sh[2][C::NA * C::PLANE];
  __shared__ __align__(16) frag slot0[C::NF * 64];
  __shared__ __align__(16) frag slot1[C::NF * 64];
  __shared__ double red[2 * C::NW];
  __shared__ int flags[C::NW];
  const int tiles_x = (a.W + C::TW - 1) / C::TW;            // a.H, a.W: latent grid
  const int k0 = (tile / tiles_x) * C::TH, l0 = (tile % tiles_x) * C::TW;
  const int H = a.H / 2, W = a.W / 2;
  const int64_t Nf = (int64_t)H * W;
  const int t0 = group * a.fpg;
  const int t1 = min(a.n, t0 + a.fpg);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = w / C::WC, wc = w % C::WC;
  const frag* tab = reinterpret_cast<const frag*>(a.tab) + (int64_t)t0 * C::FRAME;
  const int units = 2 * (t1 - t0);
  cell2_issue<C>(tab, w, slot0);
  Adj2Tile<C> tl;
  const int i0 = k0 / 2 - 11, j0 = l0 / 2 - 11;
  tl.template pass<false>(a.in + (int64_t)t0 * Nf, H, W, i0, j0, nullptr, 0.f);
  bool big = cell_any<C::NW>(tl.big(), w, flags), any_big = false;
  tl.template pass<true>(nullptr, H, W, i0, j0, sh[0], cell_up(big));
  cell_wait<0>();
  __syncthreads();
  // this lane's piece x = lane / 16 of product P: piece 4 P + x of rows s .. s + 3
  int off[3];
#pragma unroll
  for (int P = 0; P < 3; ++P) {
    const int o = 4 * P + (lane >> 4);
    off[P] = 2 * (c + o / 3) * C::PITCH + wc * 32 + 2 * (lane & 15) + 8 * (o % 3);
  }
  f64x4 acc[C::G];
#pragma unroll
  for (int g = 0; g < C::G; ++g) acc[g] = f64x4{0., 0., 0., 0.};
  for (int t = t0; t < t1; ++t) {
    const unsigned short* base = sh[(t - t0) & 1];
    const int unit = 2 * (t - t0);
    cell2_issue<C>(tab + (int64_t)(unit + 1) * C::NF * 64, w, slot1);
    tl.template pass<false>(a.in + (int64_t)min(t + 1, t1 - 1) * Nf, H, W, i0, j0, nullptr, 0.f);
    const double down = cell_down(big);
    any_big |= big;
    {
      const unsigned short* const im[3] = {base + off[0], base + off[1], base + off[2]};
      cell2_class<C>(im, slot0, acc, down);
    }
    cell_wait<0>();
    big = cell_any<C::NW>(tl.big(), w, flags);   // slot 1 has landed, slot 0 and the other tile are free
    cell2_issue<C>(tab + (int64_t)min(unit + 2, units - 2) * C::NF * 64, w, slot0);
    tl.template pass<true>(nullptr, H, W, i0, j0, sh[(t - t0 + 1) & 1],
                           cell_up(big));
    {
      const unsigned short* const im[3] = {base + C::PITCH + off[0], base + C::PITCH + off[1],
                                           base + C::PITCH + off[2]};
      cell2_class<C>(im, slot1, acc, down);
    }
    cell_wait<0>();
    __syncthreads();   // the next tile and slot 0 are complete
  }
  f32x4 sum[C::G];
#pragma unroll
  for (int g = 0; g < C::G; ++g) sum[g] = __builtin_convertvector(acc[g], f32x4);
  const CellLane p{k0 + 4 * c + (lane >> 4), l0 + wc * 64 + 4 * (lane & 15)};
  cell_finish(sum, 1.f, cell_least(any_big), [&](int g, int i) EM_INLINE {
    const int k = p.row0 + C::RS * g, l = p.col + i;
    float s = 0.f;
    if (k < a.H && l < a.W)
      for (int t = t0; t < t1; ++t)
        s += cell2_direct_adj(a.taps + (int64_t)t * CELL2_KC * TAB_LD, a.in + (int64_t)t * Nf, H, W, k, l);
    return s;
  });
  cell_adj_epilogue<C>(a, sum, p, tile, group, red);
}

// Adjoint table of one frame (blockIdx.x), one class per blockIdx.y, four fragments per
// blockIdx.z.
template <class C>
__global__ __launch_bounds__(256) void cell2_adj_table_kernel(const float* psf, int K,
                                                              unsigned short* tab) {
  const int t = blockIdx.x, E = blockIdx.y, f = 4 * blockIdx.z + (threadIdx.x >> 6);
  if (f >= C::NF) return;
  const float* h = psf + (int64_t)t * K * K;
  const int lane = threadIdx.x & 63, m = lane & 15, x = lane >> 4;
  const int part = f / 9, u = f % 9 / 3, P = f % 3;
  const int o = 4 * P + x, d = 2 * (4 * u + o / 3) + E;
  unsigned short* dst = tab + ((((int64_t)t * 2 + E) * C::NF + f) * 64 + lane) * 8;
  for (int e = 0; e < 8; ++e) {
    const int ka = 2 * d - (m >> 2), kb = 2 * (8 * (o % 3) + e) - (m & 3);
    float gv = 0.f;
    if (ka >= 0 && ka < CELL2_KC && kb >= 0 && kb < CELL2_KC) gv = box_kernel(h, K, ka, kb);
    dst[e] = cell_part<EM_FP32>(gv, part);
  }
}

template <class C, bool STUDENT>
__global__ __launch_bounds__(C::NT) void cell2_fwd_kernel(MfmaLaunch a) {
  cell2_fwd_body<C, STUDENT>(a, blockIdx.x, blockIdx.y);
}
template <class C>
__global__ __launch_bounds__(C::NT) void cell2_adj_kernel(MfmaLaunch a) {
  cell2_adj_body<C>(a, blockIdx.x, blockIdx.y);
}

using Adj2 = Adj2Cfg<4, 2>;

}  // namespace

int cell2_fwd_tile_h() { return Fwd2::TH / 2; }
int cell2_fwd_tile_w() { return Fwd2::TW / 2; }
int cell2_adj_tile_h() { return Adj2::TH; }
int cell2_adj_tile_w() { return Adj2::TW; }

size_t cell2_table_bytes(int n, int dir) {
  return dir == 0 ? (size_t)((n + CELL2_FQ - 1) / CELL2_FQ) * Fwd2::F::FRAME * 16
                  : (size_t)n * Adj2::FRAME * 16;
}

hipError_t launch_cell2_tables(const Geometry& g, const float* psf, void* tab_fwd, void* tab_adj,
                               hipStream_t s) {
  if (tab_fwd != nullptr)
    hipLaunchKernelGGL(cell2_fwd_table_kernel<Fwd2::F>, dim3((g.n + CELL2_FQ - 1) / CELL2_FQ, Fwd2::F::UPF, (Fwd2::F::NFU + 3) / 4),
                       dim3(256), 0, s, psf, g.n, g.K, static_cast<unsigned short*>(tab_fwd));
  if (tab_adj != nullptr)
    hipLaunchKernelGGL(cell2_adj_table_kernel<Adj2>, dim3(g.n, 2, (Adj2::NF + 3) / 4), dim3(256), 0, s, psf, g.K,
                       static_cast<unsigned short*>(tab_adj));
  return hipGetLastError();
}

bool cell2_desc_ok(const Geometry& g, int dir, int tiles, int groups, const MfmaLaunch& a) {
  if (a.r16 != nullptr || a.taps == nullptr) return false;
  return dir == 0 ? a.H == g.Hf && a.W == g.Wf && (groups == 1 || a.fpg % CELL2_FQ == 0) &&
                        launch_grid_ok(tiles, groups, a.ntiles, a.n, a.fpg, a.H, a.W, cell2_fwd_tile_h(),
                                       cell2_fwd_tile_w())
                  : a.H == g.Hl && a.W == g.Wl &&
                        launch_grid_ok(tiles, groups, a.ntiles, a.n, a.fpg, a.H, a.W, cell2_adj_tile_h(),
                                       cell2_adj_tile_w());
}

hipError_t launch_cell2(const Geometry& g, int dir, int tiles, int groups, const MfmaLaunch& a, hipStream_t s) {
  if (!cell2_desc_ok(g, dir, tiles, groups, a)) return hipErrorInvalidValue;
  const dim3 grid(tiles, groups);
  if (dir == 1) hipLaunchKernelGGL(cell2_adj_kernel<Adj2>, grid, dim3(Adj2::NT), 0, s, a);
  else if (a.out_y) hipLaunchKernelGGL((cell2_fwd_kernel<Fwd2, true>), grid, dim3(Fwd2::NT), 0, s, a);
  else hipLaunchKernelGGL((cell2_fwd_kernel<Fwd2, false>), grid, dim3(Fwd2::NT), 0, s, a);
  return hipGetLastError();
}

}  // namespace em
