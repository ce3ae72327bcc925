// 2D sweep of small grids for gfx950 (device code + launcher): a workgroup
// keeps a whole tile in registers and advances it bt time steps per launch.
//
// The streaming kernels (sweep2d.h) walk a tile along axis 0, so a launch
// lasts at least (rows of a stream block + 2 bt r) row steps of bt dependent
// levels each, however small the grid: a 512^2 round of ten float64 steps
// takes 23 us there, most of it with one wave per SIMD.  Here every wave
// holds M consecutive rows of the tile, all rows advance together, and a
// launch lasts the load, bt short steps and the store.  What bounds it is the
// latency of a step (one LDS exchange and one barrier, and the arithmetic of M
// rows) and, on larger grids, the redundant cells of the overlap.
//
// MI355X mapping: a workgroup of NW waves is one tile of NW*M rows by 64*CPL
// columns; lane l owns CPL consecutive columns of its wave's rows.  In-row
// neighbours in another lane come from DPP whole-wave shifts (chained where R
// exceeds CPL); the rows above and below a wave come from a double-buffered
// LDS exchange of its first and last R rows, one barrier per step.  The valid
// region shrinks by R cells per side and step; waves whose rows have left it
// (or lie outside the grid) skip the arithmetic.  Every cell sums its terms in
// the canonical order with the accumulation of the other kernels, so the bits
// are the same.  bt is a run-time argument: the time loop is not unrolled.
#pragma once

#include "gradient.h"
#include "kcommon.h"
#include "tile.h"

namespace s5d {

// Geometry of one launch (one grid, bt steps).
struct Tile2DArgs {
  const void* src;
  void* dst;
  int32_t I0, I1;
  int32_t bt;
  int32_t lo;       // overlap columns on the left (16-byte phase, >= bt * R)
  int32_t c0, c1;   // compute region of a tile: rows, columns
  int32_t n1;       // tiles along axis 1
  int32_t nblocks;  // tiles of the launch
};

// The first and last R rows of every wave, double-buffered by step parity.
template <typename T, int R, int CPL, int NW>
struct alignas(16) TileHalo {
  T rows[2][NW][2 * R][64][CPL];
};

template <typename T, int ACC, int EXPR, int R, bool BOX, int CPL, int M, int NW, bool EDGE>
__device__ __forceinline__ void tile2d_body(const Tile2DArgs& a, const CoefPack<T, ncoef(2, R, BOX, EXPR)>& cf, int lb,
                                            TileHalo<T, R, CPL, NW>& halo) {
  static_assert(R <= M, "the row exchange reaches one neighbouring wave only");
  constexpr int B0 = NW * M;
  constexpr int XL = CPL + 2 * R;
  constexpr int LK = R % CPL;  // a.lo = R modulo 16 bytes, a multiple of the lane's cells
  static_assert(16 / sizeof(T) % CPL == 0, "a lane holds at most 16 bytes of a row");
  constexpr uint32_t WB = sizeof(T);
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  const int I0 = a.I0, I1 = a.I1, P0 = I0 + 2 * R, P1 = I1 + 2 * R;
  const int r_first = R + (lb / a.n1) * a.c0, c_first = R + (lb % a.n1) * a.c1;
  const int tr0 = r_first - a.bt * R;  // first row of the tile
  const int row0 = tr0 + w * M;        // first row of this wave
  const int colL = c_first - a.lo + lane * CPL;
  const T* __restrict__ src = static_cast<const T*>(a.src);
  T* __restrict__ dst = static_cast<T*>(a.dst);

  using RowV = T __attribute__((ext_vector_type(CPL)));
  RowV cur[M];
  sfor<M>([&](auto MI) S5D_INL {
    const int i = row0 + MI;
    const bool in = i >= 0 && i < P0;
    const auto rs = make_rsrc(src + static_cast<int64_t>(in ? i : 0) * P1, in ? static_cast<uint32_t>(P1) * WB : 0u);
    T v[CPL];
    buf_load_lane(v, rs, static_cast<uint32_t>(colL) * WB);
    sfor<CPL>([&](auto K) S5D_INL { cur[MI][+K] = v[K]; });
  });
  bool fix[CPL];  // columns that keep their value: the boundary and beyond
  if constexpr (EDGE) sfor<CPL>([&](auto K) S5D_INL { fix[K] = colL + K < R || colL + K >= I1 + R; });
  const bool grid_rows = row0 + M > R && row0 < I0 + R;  // does this wave hold interior rows?
  const int wu = w > 0 ? w - 1 : w, wd = w + 1 < NW ? w + 1 : w;

  Finish<EXPR, T, CoefPack<T, ncoef(2, R, BOX, EXPR)>> fin(cf);
  // scalar registers are short here (13 points: 242 reads of spilled ones in the
  // float32 step, 76 with the bound in a vector register)
  if constexpr (EXPR == EXPR_DIV) fin.least = to_vgpr(fin.least);
  // row MI takes its new values, except the cells that keep theirs
  auto keep = [&](auto MI, const T (&out)[CPL]) S5D_INL {
    if constexpr (EDGE) {
      const bool rowb = row0 + MI < R || row0 + MI >= I0 + R;
      sfor<CPL>([&](auto K) S5D_INL { cur[MI][+K] = (rowb || fix[K]) ? cur[MI][+K] : out[K]; });
    } else {
      sfor<CPL>([&](auto K) S5D_INL { cur[MI][+K] = out[K]; });
    }
  };

  for (int t = 1; t <= a.bt; ++t) {
    auto& hb = halo.rows[t & 1];
    sfor<R>([&](auto J) S5D_INL {
      sfor<CPL>([&](auto K) S5D_INL {
        hb[w][J][lane][K] = cur[J][+K];
        hb[w][R + J][lane][K] = cur[M - R + J][+K];
      });
    });
    __syncthreads();
    // rows of the tile that are valid after t steps: [t R, B0 - t R)
    if (!grid_rows || w * M + M <= t * R || w * M >= B0 - t * R) continue;
    // extended rows: R from the wave above, own M, R from the wave below; the
    // columns beyond the lane's own only where a term reads them
    T X[M + 2 * R][XL];
    sfor<R>([&](auto J) S5D_INL {
      const LaneVec<T, CPL> up = *reinterpret_cast<const LaneVec<T, CPL>*>(hb[wu][R + J][lane]);
      const LaneVec<T, CPL> dn = *reinterpret_cast<const LaneVec<T, CPL>*>(hb[wd][J][lane]);
      sfor<CPL>([&](auto K) S5D_INL {
        X[J][R + K] = up.v[K];
        X[R + M + J][R + K] = dn.v[K];
      });
    });
    sfor<M>([&](auto MI) S5D_INL { sfor<CPL>([&](auto K) S5D_INL { X[R + MI][R + K] = cur[MI][+K]; }); });
    sfor<M + 2 * R>([&](auto XI) S5D_INL {
      if constexpr (BOX || (XI >= R && XI < R + M)) {
        sfor<R>([&](auto J) S5D_INL {  // distance J + 1 from the lane's cells
          constexpr int d = J + 1;
          X[XI][R - d] = lane_from_lower(X[XI][R - d + CPL]);
          X[XI][R + CPL - 1 + d] = lane_from_upper(X[XI][R - 1 + d]);
        });
      }
    });
    T sums[EXPR == EXPR_DIV ? M : 1][CPL];
    sfor<M>([&](auto MI) S5D_INL {
      T out[CPL];
      sfor<CPL>([&](auto K) S5D_INL {
        if constexpr (EXPR == EXPR_GRADIENT) {
          out[K] = gradient_cell(cf.c[0], cf.c[1], X[1 + MI][1 + K], X[MI][1 + K], X[1 + MI][K], X[1 + MI][2 + K],
                                 X[2 + MI][1 + K]);
        } else {
          Accum<T, ACC> acc;
          sfor<2 * R + 1>([&](auto D0) S5D_INL {
            sfor<2 * R + 1>([&](auto D1) S5D_INL {
              constexpr int d0 = D0 - R, d1 = D1 - R;
              if constexpr (BOX || d0 == 0 || d1 == 0) {
                constexpr int ci = BOX ? D0 * (2 * R + 1) + D1 : (d0 < 0 ? D0 : (d0 > 0 ? 3 * R + d0 : R + D1));
                if constexpr (ci == 0) acc.first(cf.c[0], X[MI + D0][K + D1]);
                else acc.add(cf.c[ci], X[MI + D0][K + D1]);
              }
            });
          });
          out[K] = acc.value();
        }
      });
      if constexpr (EXPR == EXPR_DIV) {  // the sums of all rows first: one check of their range
        sfor<CPL>([&](auto K) S5D_INL { sums[MI][K] = out[K]; });
        if constexpr (MI == M - 1) fin(sums);
      }
      if constexpr (EXPR != EXPR_DIV) keep(MI, out);
    });
    if constexpr (EXPR == EXPR_DIV) sfor<M>([&](auto MI) S5D_INL { keep(MI, sums[MI]); });
  }

  // store the compute region: lanes from c_first on as vectors cut off by the
  // descriptor at the region's end, the lane it starts in its last CPL - LK cells
  const uint32_t st_bytes = static_cast<uint32_t>(min(c_first + a.c1, I1 + R)) * WB;
  const uint32_t vstore = colL >= c_first ? static_cast<uint32_t>(colL) * WB : kOutOfRange;
  const uint32_t lstore = colL == c_first - LK ? static_cast<uint32_t>(c_first) * WB : kOutOfRange;
  const int row_end = min(r_first + a.c0, I0 + R);
  sfor<M>([&](auto MI) S5D_INL {
    const int i = row0 + MI;
    const bool keep = i >= r_first && i < row_end;
    const auto rs = make_rsrc(dst + static_cast<int64_t>(keep ? i : r_first) * P1, keep ? st_bytes : 0u);
    T v[CPL];
    sfor<CPL>([&](auto K) S5D_INL { v[K] = cur[MI][+K]; });
    buf_store_cells<0>(v, rs, vstore);
    if constexpr (LK != 0) buf_store_cells<LK>(v, rs, lstore);
  });
}

template <typename T, int ACC, int EXPR, int R, bool BOX, int CPL, int M, int NW>
__device__ __forceinline__ void tile2d_block(const Tile2DArgs& a, const CoefPack<T, ncoef(2, R, BOX, EXPR)>& cf, int lb,
                                             TileHalo<T, R, CPL, NW>& halo) {
  // does the tile hold cells that keep their value?
  const int tr0 = R + (lb / a.n1) * a.c0 - a.bt * R, tc0 = R + (lb % a.n1) * a.c1 - a.lo;
  const bool edge = tr0 < R || tr0 + NW * M > a.I0 + R || tc0 < R || tc0 + 64 * CPL > a.I1 + R;
  if (edge)
    tile2d_body<T, ACC, EXPR, R, BOX, CPL, M, NW, true>(a, cf, lb, halo);
  else
    tile2d_body<T, ACC, EXPR, R, BOX, CPL, M, NW, false>(a, cf, lb, halo);
}

template <typename T, int ACC, int EXPR, int R, bool BOX, int CPL, int M, int NW>
__global__ __launch_bounds__(64 * NW) void tile2d_kernel(Tile2DArgs a, CoefPack<T, ncoef(2, R, BOX, EXPR)> cf) {
  __shared__ TileHalo<T, R, CPL, NW> halo;
  tile2d_block<T, ACC, EXPR, R, BOX, CPL, M, NW>(a, cf, xcd_logical_block(blockIdx.x, gridDim.x), halo);
}

// One grid of a batched launch: its geometry and coefficients.
template <typename T, int NP>
struct alignas(16) TileItem2D {
  Tile2DArgs a;
  CoefPack<T, NP> cf;
};

// Batched launch: workgroup b runs tile map[b].block of grid map[b].item; the
// grids may advance different numbers of steps.
template <typename T, int ACC, int EXPR, int R, bool BOX, int CPL, int M, int NW>
__global__ __launch_bounds__(64 * NW) void tile2d_batch_kernel(
    const TileItem2D<T, ncoef(2, R, BOX, EXPR)>* __restrict__ items, const BlockMap* __restrict__ map) {
  __shared__ TileHalo<T, R, CPL, NW> halo;
  const BlockMap m = map[xcd_logical_block(blockIdx.x, gridDim.x)];
  const TileItem2D<T, ncoef(2, R, BOX, EXPR)>& it = items[__builtin_amdgcn_readfirstlane(m.item)];
  const Tile2DArgs a = uniform_copy(it.a);
  const CoefPack<T, ncoef(2, R, BOX, EXPR)> cf = uniform_copy(it.cf);
  tile2d_block<T, ACC, EXPR, R, BOX, CPL, M, NW>(a, cf, __builtin_amdgcn_readfirstlane(m.block), halo);
}

// Geometry of a grid's launch of bt steps; nblocks = 0 if bt does not fit the
// tile or the launch does not fit 32 bits.
template <typename T, int EXPR, int R, bool BOX, int CPL, int M, int NW>
Tile2DArgs make_tile2d(const Round2D& rd, int bt, CoefPack<T, ncoef(2, R, BOX, EXPR)>& cf) {
  // gradient2d carries two coefficients (cc, c0) in the pack of five
  constexpr int NC = EXPR == EXPR_GRADIENT ? 2 : ncoef(2, R, BOX, EXPR);
  for (int k = 0; k < ncoef(2, R, BOX, EXPR); ++k) cf.c[k] = k < NC ? static_cast<T>(rd.coeffs[k]) : T(0);
  Tile2DArgs a{};
  a.src = rd.src;
  a.dst = rd.dst;
  a.I0 = rd.I0;
  a.I1 = rd.I1;
  a.bt = bt;
  a.lo = overlap_left(bt, R, sizeof(T));
  a.c0 = NW * M - 2 * bt * R;
  a.c1 = compute_width(64 * CPL, bt, R, sizeof(T));
  if (a.c0 < 1 || a.c1 < 1) return a;
  a.n1 = (rd.I1 + a.c1 - 1) / a.c1;
  const int64_t n = static_cast<int64_t>((rd.I0 + a.c0 - 1) / a.c0) * a.n1;
  a.nblocks = n > INT32_MAX ? 0 : static_cast<int32_t>(n);
  return a;
}

template <typename T, int ACC, int EXPR, int R, bool BOX, int CPL, int M, int NW>
hipError_t launch_tile2d(const Round2D& rd, int bt) {
  CoefPack<T, ncoef(2, R, BOX, EXPR)> cf;
  const Tile2DArgs a = make_tile2d<T, EXPR, R, BOX, CPL, M, NW>(rd, bt, cf);
  if (a.nblocks == 0) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((tile2d_kernel<T, ACC, EXPR, R, BOX, CPL, M, NW>), dim3(a.nblocks), dim3(64 * NW), 0, rd.stream, a,
                     cf);
  return hipGetLastError();
}

template <typename T, int EXPR, int R, bool BOX, int CPL, int M, int NW>
int fill_tile2d(void* item, const Round2D& rd, int bt) {
  TileItem2D<T, ncoef(2, R, BOX, EXPR)> it;
  it.a = make_tile2d<T, EXPR, R, BOX, CPL, M, NW>(rd, bt, it.cf);
  __builtin_memcpy(item, &it, sizeof(it));
  return it.a.nblocks;
}

template <typename T, int ACC, int EXPR, int R, bool BOX, int CPL, int M, int NW>
hipError_t launch_tile2d_batch(const void* items, const BlockMap* map, int nblocks, hipStream_t stream) {
  hipLaunchKernelGGL((tile2d_batch_kernel<T, ACC, EXPR, R, BOX, CPL, M, NW>), dim3(nblocks), dim3(64 * NW), 0, stream,
                     static_cast<const TileItem2D<T, ncoef(2, R, BOX, EXPR)>*>(items), map);
  return hipGetLastError();
}

}  // namespace s5d
