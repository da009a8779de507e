// em_cell.hip -- kernels of one EM iteration on the 4 x 4 cell core of em_cell.h:
// forward model, weighting and adjoint of Eq. (2) (arXiv:2302.05804, Sec. 2) for
// sr = 1 and kernels padded to 43 x 43, in FP32, the BF16 split form and, served, plain
// BF16.
#include "em_cell.h"

#include <type_traits>

namespace em {

namespace {

// 128 x 128 outputs per workgroup, 8 waves of 8 cell rows x 16 cells; 64 x 128 and
// 4 cell rows per wave in FP32, whose three image planes take half the LDS more
template <int PREC, bool BAND>
using CellOf = CellCfg<CellForm<PREC, BAND>, PREC == EM_FP32 ? 4 : 8, 4, 2>;

// The forward's weights of this lane's outputs, loaded while the last class of
// the frame runs, so that the epilogue does not wait for HBM.
template <class C>
struct CellWeights {
  const float* ut;   // frame base, nullptr: nothing to load
  int H, W;
  CellLane p;
  bool vec;
  float4 uu[C::G];
  __device__ void wait(int) const { cell_wait<0>(); }
  __device__ void after(int b) {
    if (b == C::F::UPF - 2 && ut != nullptr && vec) {
#pragma unroll
      for (int g = 0; g < C::G; ++g)
        uu[g] = *reinterpret_cast<const float4*>(ut + (int64_t)min(p.row0 + 4 * g, H - 1) * W + p.col);
    }
  }
};

// Forward: r_t = u_t (f_t * x) for the frames of this group, or m when u is NULL
// (FP64 partials of u (y - m)^2 when asked); STUDENT: the E-step weights, u w m
// and u w y.  The x tile is staged once.
template <class C, bool STUDENT>
__device__ inline void cell_fwd_body(const MfmaLaunch& a, const int tile, const int group) {
  using F = typename C::F;
  using frag = typename C::frag;
  constexpr int PLANE = C::ROWS * C::PITCH;
  __shared__ __align__(16) unsigned short sh[F::NA * PLANE];
  __shared__ __align__(16) frag slot0[F::NFU * 64];
  __shared__ __align__(16) frag slot1[F::NFU * 64];
  __shared__ double red[C::NW];
  __shared__ int flags[C::NW];
  const int tiles_x = (a.W + C::TW - 1) / C::TW;
  const int k0 = (tile / tiles_x) * C::TH, l0 = (tile % tiles_x) * C::TW;
  const int t0 = group * a.fpg;
  const int t1 = min(a.n, t0 + a.fpg);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  CellTab<F> T{reinterpret_cast<const frag*>(a.tab) + (int64_t)t0 * F::FRAME, 0,
               (t1 - t0) * F::UPF, w, {slot0, slot1}, 1.0};
  cell_issue_unit<C>(T.tab, 0, w, slot0);
  cell_issue_unit<C>(T.tab, 1, w, slot1);
  bool big = false;
  {
    CellTile<C> tl(a.H, a.W, k0, l0, w);
    tl.load(a.in);
    if constexpr (F::PREC == EM_FP32) big = cell_any<C::NW>(tl.big(), w, flags);
    tl.store(sh, cell_up(big));
  }
  cell_wait<0>();
  __syncthreads();

  const int64_t N = (int64_t)a.H * a.W;
  const CellLane lane_pos = cell_lane<C>(k0, l0);
  const unsigned short* im = sh + cell_main_off<C>();
  const unsigned short* it = sh + cell_tail_off<C>();
  const bool ll = a.part != nullptr;
  const bool al = (a.W & 3) == 0 && aligned16(a.u) && (a.out == nullptr || aligned16(a.out)) &&
                  (!(STUDENT || ll) || aligned16(a.y)) &&
                  (!STUDENT || aligned16(a.out_y));
  const bool vec = al && lane_pos.col + 3 < a.W;
  double llp = 0.0;
  for (int t = t0; t < t1; ++t) {
    // the staged tile does not change between frames: keep its reads inside the
    // loop, and the epilogue's address arithmetic (held in registers over the
    // products, it would spill)
    CellLane p = lane_pos;
    __asm__ volatile("" : "+v"(p.row0), "+v"(p.col)::"memory");
    f32x4 acc[C::G];
#pragma unroll
    for (int g = 0; g < C::G; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* ut = a.u ? a.u + (int64_t)t * N : nullptr;
    CellWeights<C> hook{ut, a.H, a.W, p, vec, {}};
    cell_frame<C>(im, it, PLANE, T, acc, hook);
    if constexpr (F::PREC == EM_FP32)
      cell_finish(acc, cell_down(big), cell_least(big), [&](int g, int i) EM_INLINE {
        const int k = p.row0 + 4 * g, l = p.col + i;
        return k < a.H && l < a.W ? cell_direct(a.taps + (int64_t)t * CELL_K * TAB_LD, a.in, a.H, a.W, k, l, 0)
                                  : 0.f;
      });
    const float* yt = (STUDENT || (ll && ut)) ? a.y + (int64_t)t * N : nullptr;
    float* ot = a.out ? a.out + (int64_t)t * N : nullptr;
#pragma unroll
    for (int g = 0; g < C::G; ++g) {
      const int k = p.row0 + 4 * g;
      const float m[4] = {acc[g][0], acc[g][1], acc[g][2], acc[g][3]};
      float u[4] = {1.f, 1.f, 1.f, 1.f}, y[4] = {0.f, 0.f, 0.f, 0.f};
      if (ut) {
        if (vec) {
          u[0] = hook.uu[g].x; u[1] = hook.uu[g].y; u[2] = hook.uu[g].z; u[3] = hook.uu[g].w;
        } else {
          load4(ut, k, p.col, a.H, a.W, false, u);
        }
      }
      if (yt) load4(yt, k, p.col, a.H, a.W, vec, y);
      if (k >= a.H || p.col >= a.W) continue;
      float r[4], ry[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = p.col + i < a.W;
        if constexpr (STUDENT) {
          r[i] = 0.f;
          ry[i] = 0.f;
          if (u[i] > 0.f) {
            const float d = y[i] - m[i];
            const float w = (a.nu + 1.f) / (a.nu + u[i] * d * d);
            r[i] = (u[i] * w) * m[i];
            ry[i] = (u[i] * w) * y[i];
            if (ll && in) {
              const double dd = (double)y[i] - (double)m[i];
              llp += ((double)a.nu + 1.0) * log1p((double)u[i] * dd * dd / (double)a.nu) - a.lcst;
            }
          }
        } else {
          r[i] = ut ? u[i] * m[i] : m[i];
          if (yt && in && u[i] > 0.f) {
            const double d = (double)y[i] - (double)m[i];
            llp += (double)u[i] * d * d;
          }
        }
      }
      if (ot) store4(ot, k, p.col, a.W, vec, r);
      if constexpr (STUDENT) store4(a.out_y + (int64_t)t * N, k, p.col, a.W, vec, ry);
    }
  }
  cell_wait<0>();   // the copies issued past the last unit
  if (a.part != nullptr) {
    const double s = block_sum<C::NT>(llp, red);
    if (threadIdx.x == 0) a.part[(int64_t)group * a.ntiles + tile] = s;
  }
}

// The next frame's r tile, loaded into registers while the last rows of the
// current frame's last class run (loaded a boundary earlier, it spilled: 2.72
// instead of 2.48 ms on 33 x 2048^2 in FP32).
template <class C>
struct CellTileHook {
  CellTile<C> tl;
  const float* next;
  __device__ void wait(int) const { cell_wait<0>(); }
  __device__ void after(int b) {
    if (b == C::F::UPF - 1) tl.load(next);
  }
};

// Adjoint: sum over the frames of this group of F_t^T r_t; the r_t tile is staged
// per frame.
template <class C>
__device__ inline void cell_adj_body(const MfmaLaunch& a, const int tile, const int group) {
  using F = typename C::F;
  using frag = typename C::frag;
  using Hook = CellTileHook<C>;
  constexpr int PLANE = C::ROWS * C::PITCH;
  __shared__ __align__(16) unsigned short sh[F::NA * PLANE];
  __shared__ __align__(16) frag slot0[F::NFU * 64];
  __shared__ __align__(16) frag slot1[F::NFU * 64];
  __shared__ double red[2 * C::NW];
  __shared__ int flags[C::NW];
  const int tiles_x = (a.W + C::TW - 1) / C::TW;
  const int k0 = (tile / tiles_x) * C::TH, l0 = (tile % tiles_x) * C::TW;
  const int64_t N = (int64_t)a.H * a.W;
  const int t0 = group * a.fpg;
  const int t1 = min(a.n, t0 + a.fpg);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  CellTab<F> T{reinterpret_cast<const frag*>(a.tab) + (int64_t)t0 * F::FRAME, 0,
               (t1 - t0) * F::UPF, w, {slot0, slot1}, 1.0};
  cell_issue_unit<C>(T.tab, 0, w, slot0);
  cell_issue_unit<C>(T.tab, 1, w, slot1);
  const CellLane p = cell_lane<C>(k0, l0);
  const unsigned short* im = sh + cell_main_off<C>();
  const unsigned short* it = sh + cell_tail_off<C>();
  using Sum = CellSum<F::LEVELS>;
  Sum acc[C::G];
#pragma unroll
  for (int g = 0; g < C::G; ++g) acc[g] = Sum{0, 0, 0, 0};
  Hook hook{CellTile<C>(a.H, a.W, k0, l0, w), a.in + (int64_t)t0 * N};
  hook.tl.load(hook.next);
  bool any_big = false;
  for (int t = t0; t < t1; ++t) {
    float up = 1.f;
    if constexpr (F::PREC == EM_FP32) {
      const bool big = cell_any<C::NW>(hook.tl.big(), w, flags);   // every wave is done with the tile
      up = cell_up(big);
      T.down = cell_down(big);
      any_big |= big;
    }
    hook.tl.store(sh, up);
    cell_wait<0>();
    __syncthreads();
    hook.next = a.in + (int64_t)min(t + 1, t1 - 1) * N;
    if constexpr (F::LEVELS) {
      cell_frame<C>(im, it, PLANE, T, acc, hook);
    } else {
      // each frame is summed by itself and then added to the total
      f32x4 accf[C::G];
#pragma unroll
      for (int g = 0; g < C::G; ++g) accf[g] = f32x4{0.f, 0.f, 0.f, 0.f};
      cell_frame<C>(im, it, PLANE, T, accf, hook);
#pragma unroll
      for (int g = 0; g < C::G; ++g) acc[g] += accf[g];
    }
    if constexpr (F::PREC != EM_FP32) __syncthreads();   // every wave is done with the tile
  }
  cell_wait<0>();   // the copies issued past the last unit
  f32x4 sum[C::G];
#pragma unroll
  for (int g = 0; g < C::G; ++g) sum[g] = __builtin_convertvector(acc[g], f32x4);
  if constexpr (F::PREC == EM_FP32)
    cell_finish(sum, 1.f, cell_least(any_big), [&](int g, int i) EM_INLINE {
      const int k = p.row0 + 4 * g, l = p.col + i;
      float s = 0.f;
      if (k < a.H && l < a.W)
        for (int t = t0; t < t1; ++t)
          s += cell_direct(a.taps + (int64_t)t * CELL_K * TAB_LD, a.in + (int64_t)t * N, a.H, a.W, k, l, 1);
      return s;
    });
  cell_adj_epilogue<C>(a, sum, p, tile, group, red);
}

// One job per launch, grid (tiles, frame groups), or the (job, tile, group) items
// of several jobs strided over by the workgroups.
enum { K_FWD = 0, K_FWD_T = 1, K_ADJ = 2 };

template <class C, int KIND>
__device__ inline void cell_body(const MfmaLaunch& a, int tile, int group) {
  if constexpr (KIND == K_ADJ) cell_adj_body<C>(a, tile, group);
  else cell_fwd_body<C, KIND == K_FWD_T>(a, tile, group);
}

template <class C, int KIND>
__global__ __launch_bounds__(C::NT) void cell_kernel(MfmaLaunch a) {
  cell_body<C, KIND>(a, blockIdx.x, blockIdx.y);
}

template <class C, int KIND>
__global__ __launch_bounds__(C::NT) void cell_batched(const MfmaLaunch* __restrict__ descs,
                                                      const int4* __restrict__ items, int n_items) {
  for (int i = blockIdx.x; i < n_items; i += gridDim.x) {
    const int4 w = items[i];
    const MfmaLaunch d = descs[w.x];
    cell_body<C, KIND>(d, w.y, w.z);
    __syncthreads();
  }
}

// Tables of one frame (blockIdx.x), one unit per blockIdx.y, the directions that have a
// table and four fragments to a block in blockIdx.z (with one block per unit and direction the 12
// frames of a 700 x 800 job took 28 us in FP32, 64 us in the banded form): lane
// (m, gq) of a fragment holds T[m][window row, column 8 gq + e] of its part (see
// em_cell.h); direction 0: g = f flipped (forward), 1: g = f; f zero-padded from K
// to 43.
template <class F>
__global__ __launch_bounds__(256) void cell_table_kernel(const float* psf, int K,
                                                         unsigned short* tab_fwd,
                                                         unsigned short* tab_adj) {
  const int t = blockIdx.x, unit = blockIdx.y, E = unit / F::NU, u = unit % F::NU;
  const bool both = tab_fwd != nullptr && tab_adj != nullptr;
  const int dir = both ? blockIdx.z & 1 : tab_fwd == nullptr;
  const int frag = 4 * (both ? blockIdx.z >> 1 : blockIdx.z) + (threadIdx.x >> 6);
  if (frag >= F::NFU) return;
  unsigned short* tab = dir == 0 ? tab_fwd : tab_adj;
  const int off = (CELL_K - K) / 2;
  const float* f = psf + (int64_t)t * K * K;
  const int lane = threadIdx.x & 63, m = lane & 15, gq = lane >> 4;
  const CellFragId id = cell_frag_id<F>(u, frag);
  unsigned short* dst = tab + ((((int64_t)t * F::UPF + unit) * F::NFU + frag) * 64 + lane) * 8;
  for (int e = 0; e < 8; ++e) {
    // window row and column of this K position
    const int d = 4 * (id.j + (id.tail ? gq >> 1 : 0)) + E;
    const int k = id.tail ? 32 + 8 * (gq & 1) + e : 8 * gq + e;
    const int ta = d - 1 - (m >> 2), tb = k - 1 - (m & 3);
    float gv = 0.f;
    if (id.part >= 0 && ta >= 0 && ta < CELL_K && tb >= 0 && tb < CELL_K &&
        (id.part == 0 || !F::BAND || (ta >= 11 && ta <= 31))) {
      const int fa = (dir == 0 ? CELL_K - 1 - ta : ta) - off;
      const int fb = (dir == 0 ? CELL_K - 1 - tb : tb) - off;
      if (fa >= 0 && fa < K && fb >= 0 && fb < K) gv = f[fa * K + fb];
    }
    dst[e] = cell_part<F::PREC>(gv, id.part);
  }
}

template <int PREC, bool BAND>
hipError_t launch_one(int kind, dim3 grid, const MfmaLaunch& a, hipStream_t s) {
  using C = CellOf<PREC, BAND>;
  const dim3 block(C::NT);
  if (kind == K_FWD) hipLaunchKernelGGL((cell_kernel<C, K_FWD>), grid, block, 0, s, a);
  else if (kind == K_FWD_T) hipLaunchKernelGGL((cell_kernel<C, K_FWD_T>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((cell_kernel<C, K_ADJ>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int PREC, bool BAND>
hipError_t launch_many(int kind, int grid, const MfmaLaunch* d, const int4* it, int n, hipStream_t s) {
  using C = CellOf<PREC, BAND>;
  const dim3 block(C::NT);
  if (kind == K_FWD) hipLaunchKernelGGL((cell_batched<C, K_FWD>), dim3(grid), block, 0, s, d, it, n);
  else if (kind == K_FWD_T) hipLaunchKernelGGL((cell_batched<C, K_FWD_T>), dim3(grid), block, 0, s, d, it, n);
  else hipLaunchKernelGGL((cell_batched<C, K_ADJ>), dim3(grid), block, 0, s, d, it, n);
  return hipGetLastError();
}

}  // namespace

int cell_tile_h(int precision) {
  return precision == EM_FP32 ? CellOf<EM_FP32, false>::TH : CellOf<EM_BF16_SPLIT, false>::TH;
}
static_assert(CellOf<EM_FP32, false>::TW == CELL_TILE_W && CellOf<EM_BF16_SPLIT, false>::TW == CELL_TILE_W, "tile");

size_t cell_table_bytes(int n) { return (size_t)n * CellForm<EM_FP32, false>::FRAME * 16; }
template <class F>
constexpr bool cell_table_fits = F::FRAME * 16 <= (int64_t)mfma_table_frame(KT_LARGE);
static_assert(cell_table_fits<CellForm<EM_BF16_SPLIT, false>> && cell_table_fits<CellForm<EM_BF16_SPLIT, true>> &&
                  cell_table_fits<CellForm<EM_BF16, false>>,
              "the BF16 forms' tables within mfma_table_bytes");

// The BF16 split form takes its band for jobs whose PSFs passed the band check,
// and not in serving.
hipError_t launch_cell(int precision, int dir, dim3 grid, const MfmaLaunch& a, hipStream_t s) {
  if (a.r16 != nullptr || (precision == EM_FP32 && a.taps == nullptr)) return hipErrorInvalidValue;
  const int kind = dir == 1 ? K_ADJ : a.out_y ? K_FWD_T : K_FWD;
  switch (precision) {
    case EM_FP32: return launch_one<EM_FP32, false>(kind, grid, a, s);
    case EM_BF16_SPLIT:
      return a.lo_band ? launch_one<EM_BF16_SPLIT, true>(kind, grid, a, s)
                       : launch_one<EM_BF16_SPLIT, false>(kind, grid, a, s);
    case EM_BF16: return launch_one<EM_BF16, false>(kind, grid, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_cell_batched(int precision, int dir, const MfmaLaunch* descs, const int4* items,
                               int n_items, int grid, hipStream_t s, bool robust) {
  const int kind = dir == 1 ? K_ADJ : robust ? K_FWD_T : K_FWD;
  switch (precision) {
    case EM_BF16_SPLIT: return launch_many<EM_BF16_SPLIT, false>(kind, grid, descs, items, n_items, s);
    case EM_BF16: return launch_many<EM_BF16, false>(kind, grid, descs, items, n_items, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_cell_tables(const Geometry& g, const float* psf, void* tab_fwd, void* tab_adj,
                              bool lo_band, hipStream_t s) {
  auto go = [&](auto form) {
    using F = decltype(form);
    const int dirs = (tab_fwd != nullptr) + (tab_adj != nullptr);
    hipLaunchKernelGGL(cell_table_kernel<F>, dim3(g.n, F::UPF, dirs * ((F::NFU + 3) / 4)), dim3(256), 0, s, psf,
                       g.K, static_cast<unsigned short*>(tab_fwd), static_cast<unsigned short*>(tab_adj));
  };
  if (g.precision == EM_FP32) go(CellForm<EM_FP32, false>{});
  else if (g.precision == EM_BF16) go(CellForm<EM_BF16, false>{});
  else if (lo_band) go(CellForm<EM_BF16_SPLIT, true>{});
  else go(CellForm<EM_BF16_SPLIT, false>{});
  return hipGetLastError();
}

}  // namespace em
