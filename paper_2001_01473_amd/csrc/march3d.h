// Direct 3D kernel for high-order stars: one time step per launch, marching
// along axis 0.
//
// The row-streaming kernel (stream3d.h) loads 2r + 1 + 2r / M rows for every
// row it writes; at radius 2 and more those loads, which hit in L2, bound it.
// Here a workgroup owns a tile of NW*M rows by 64*CPL columns and walks along
// axis 0 over a block of planes.  Every plane of the tile is loaded once; it
// is pushed at once into the 2r + 1 output planes it feeds, of which 2r are
// pending in registers, so what remains per cell is one load, one store, the
// 6r + 1 terms and the exchange of the waves' edge rows.  Bound by HBM and by
// vector issue.
//
// MI355X mapping (as in sweep3d.h): wave w holds rows w*M .. w*M+M-1, lane l
// CPL consecutive columns of them.  Neighbours along axis 2 come from DPP
// whole-wave shifts, chained where r exceeds CPL; neighbours along axis 1 in
// another wave through a double-buffered LDS exchange of r rows a side, one
// barrier per plane.  The barrier is late: the output plane the arriving one
// completes needs no neighbour, so it is finished and stored first.  Every
// output sums its terms in the canonical (d0, d1, d2) order with the same
// accumulation as the other kernels: same bits.
//
// Loads and stores go through one descriptor per plane; a lane's offset into
// it is fixed per row.  Rows outside the grid are out of its range; columns
// outside it read a neighbouring row's cells, which feed no stored cell.  So
// there is no branch and no address arithmetic but the plane's base, at any
// pitch: ragged rows cost nothing extra.
#pragma once

#include "kcommon.h"

namespace s5d {

struct March3DArgs {
  const void* src;
  void* dst;
  int32_t I0, I1, I2;
  int32_t n1, n2;   // tiles along axes 1 and 2
  int32_t planes;   // output planes per block
};

template <typename T, int ACC, int R, int CPL, int M, int NW>
__device__ __forceinline__ void march3d_block(const March3DArgs& a, const CoefPack<T, npts(3, R, false)>& cf, int lb,
                                              T (&xbuf)[2][NW][2 * R][64][CPL]) {
  static_assert(R <= M, "the row exchange reaches one neighbouring wave only");
  constexpr int NA = 2 * R;           // pending output planes
  constexpr int NR = R == 3 ? 3 : 4;  // planes in the load ring: a divisor of 2R, so 2 or 3 planes are in flight
  constexpr int NS = lcm_i(NA, NR);   // steps per unrolled iteration
  constexpr int LO = overlap_left(1, R, sizeof(T));
  constexpr int C1 = NW * M - 2 * R, C2 = compute_width(64 * CPL, 1, R, sizeof(T));
  static_assert(CPL <= 2, "a cut lane stores one cell");
  constexpr int XR = M + 2 * R, XL = CPL + 2 * R;
  constexpr uint32_t WB = sizeof(T);
  static_assert(C1 >= 1 && C2 >= 1, "tile narrower than its overlap");
  using RowV = T __attribute__((ext_vector_type(CPL)));
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  const int t2 = lb % a.n2, t1 = (lb / a.n2) % a.n1, blk = lb / (a.n2 * a.n1);
  const int I0 = a.I0, I1 = a.I1, I2 = a.I2;
  const int P0 = I0 + 2 * R, P1 = I1 + 2 * R, P2 = I2 + 2 * R;
  const int r_first = R + t1 * C1, c_first = R + t2 * C2;
  const int row0 = r_first - R + w * M;
  const int colL = c_first - LO + lane * CPL;
  const int pl_a = R + blk * a.planes, pl_b = min(pl_a + a.planes, I0 + R);
  const int row_end = min(r_first + C1, I1 + R);
  const int col_end = min(c_first + C2, I2 + R);
  const uint32_t plane_bytes = static_cast<uint32_t>(P1) * static_cast<uint32_t>(P2) * WB;
  // byte offsets into a plane: loads, whole-lane stores, and the store of the
  // one cell of a lane that the compute columns' first or last column cuts
  uint32_t loff[M], voff[M], poff[M];
  const bool cut_left = CPL == 2 && colL == c_first - 1, cut_right = CPL == 2 && colL == col_end - 1;
  sfor<M>([&](auto MI) S5D_INL {
    const int i = row0 + MI;
    const uint32_t off = (static_cast<uint32_t>(i) * static_cast<uint32_t>(P2) + static_cast<uint32_t>(colL)) * WB;
    loff[MI] = i >= 0 && i < P1 ? off : kOutOfRange;
    const bool st = i >= r_first && i < row_end;
    voff[MI] = st && colL >= c_first && colL + CPL <= col_end ? off : kOutOfRange;
    poff[MI] = st && (cut_left || cut_right) ? off + (cut_left ? WB : 0u) : kOutOfRange;
  });
  const T* __restrict__ src = static_cast<const T*>(a.src);
  T* __restrict__ dst = static_cast<T*>(a.dst);
  const int wu = w > 0 ? w - 1 : w, wd = w + 1 < NW ? w + 1 : w;

  auto load_plane = [&](RowV (&v)[M], int p) S5D_INL {
    const bool in = p < P0;
    const auto rs = make_rsrc(src + static_cast<int64_t>(in ? p : 0) * P1 * P2, in ? plane_bytes : 0u);
    sfor<M>([&](auto MI) S5D_INL {
      T t[CPL];
      buf_load_lane(t, rs, loff[MI]);
      sfor<CPL>([&](auto K) S5D_INL { v[MI][+K] = t[K]; });
    });
  };

  Accum<T, ACC> acc[NA][M][CPL];
  RowV ring[NR][M];
  sfor<NA>([&](auto S) S5D_INL {
    sfor<M>([&](auto MI) S5D_INL { sfor<CPL>([&](auto K) S5D_INL { acc[S][MI][K].zero(); }); });
  });

  // plane s arrives at step s - s0 and completes output plane s - R; slots are
  // fixed by the step's phase
  const int s0 = pl_a - R;
  const int niter = (pl_b + R - s0 + NS - 1) / NS;
  sfor<NR - 1>([&](auto J) S5D_INL {
    load_plane(ring[J], s0 + J);
    __builtin_amdgcn_sched_barrier(0);
  });

  for (int it = 0; it < niter; ++it) {
    sfor<NS>([&](auto PH) S5D_INL {
      const int s = s0 + it * NS + PH;
      constexpr int so = pmod(PH + R, NA);  // slot of output planes s-R and s+R
      load_plane(ring[(PH + NR - 1) % NR], s + NR - 1);
      __builtin_amdgcn_sched_barrier(0);
      const RowV(&cur)[M] = ring[PH % NR];

      // publish the edge rows
      auto& hb = xbuf[PH & 1];
      sfor<R>([&](auto J) S5D_INL {
        sfor<CPL>([&](auto K) S5D_INL {
          hb[w][J][lane][K] = cur[J][+K];
          hb[w][R + J][lane][K] = cur[M - R + J][+K];
        });
      });

      // output plane s-R receives its last term, (R, 0, 0), and leaves; s+R
      // starts in its slot with (-R, 0, 0)
      const int o = s - R;
      const bool keep = o >= pl_a && o < pl_b;
      const auto rs = make_rsrc(dst + static_cast<int64_t>(keep ? o : pl_a) * P1 * P2, keep ? plane_bytes : 0u);
      sfor<M>([&](auto MI) S5D_INL {
        T out[CPL];
        sfor<CPL>([&](auto K) S5D_INL {
          acc[so][MI][K].add(cf.c[6 * R], cur[MI][+K]);
          out[K] = acc[so][MI][K].value();
          acc[so][MI][K].first(cf.c[0], cur[MI][+K]);
        });
        buf_store_cells<0>(out, rs, voff[MI]);
        if constexpr (CPL == 2) buf_store(cut_left ? out[1] : out[0], rs, poff[MI]);
      });
      // the other off-centre planes: (d0, 0, 0), d0 = -R+1 .. -1 and 1 .. R-1
      sfor<2 * R - 1>([&](auto J) S5D_INL {
        constexpr int d0 = -R + 1 + J;
        if constexpr (d0 != 0) {
          constexpr int sl = pmod(PH - d0, NA);
          constexpr int ci = d0 < 0 ? d0 + R : 5 * R + d0;
          sfor<M>([&](auto MI) S5D_INL {
            sfor<CPL>([&](auto K) S5D_INL { acc[sl][MI][K].add(cf.c[ci], cur[MI][+K]); });
          });
        }
      });
      // the centre plane: rows above and below from the neighbouring waves
      __syncthreads();
      constexpr int sc = pmod(PH, NA);
      T X[XR][CPL];  // extended rows
      sfor<R>([&](auto J) S5D_INL {
        const LaneVec<T, CPL> up = *reinterpret_cast<const LaneVec<T, CPL>*>(hb[wu][R + J][lane]);
        const LaneVec<T, CPL> dn = *reinterpret_cast<const LaneVec<T, CPL>*>(hb[wd][J][lane]);
        sfor<CPL>([&](auto K) S5D_INL {
          X[J][K] = up.v[K];
          X[R + M + J][K] = dn.v[K];
        });
      });
      sfor<M>([&](auto MI) S5D_INL { sfor<CPL>([&](auto K) S5D_INL { X[R + MI][K] = cur[MI][+K]; }); });
      sfor<M>([&](auto MI) S5D_INL {
        T E[XL];  // the row with r columns more on either side
        sfor<CPL>([&](auto K) S5D_INL { E[R + K] = cur[MI][+K]; });
        sfor<R>([&](auto J) S5D_INL {
          constexpr int d = J + 1;
          E[R - d] = lane_from_lower(E[R - d + CPL]);
          E[R + CPL - 1 + d] = lane_from_upper(E[R - 1 + d]);
        });
        sfor<CPL>([&](auto K) S5D_INL {
          auto& ak = acc[sc][MI][K];
          sfor<R>([&](auto J) S5D_INL { ak.add(cf.c[R + J], X[MI + J][K]); });
          sfor<2 * R + 1>([&](auto D2) S5D_INL { ak.add(cf.c[2 * R + D2], E[K + D2]); });
          sfor<R>([&](auto J) S5D_INL { ak.add(cf.c[4 * R + 1 + J], X[MI + R + 1 + J][K]); });
        });
      });
    });
  }
}

template <typename T, int ACC, int R, int CPL, int M, int NW>
__global__ __launch_bounds__(64 * NW) void march3d_kernel(March3DArgs a, CoefPack<T, npts(3, R, false)> cf) {
  __shared__ __attribute__((aligned(16))) T xbuf[2][NW][2 * R][64][CPL];
  march3d_block<T, ACC, R, CPL, M, NW>(a, cf, xcd_logical_block(blockIdx.x, gridDim.x), xbuf);
}

// One grid of a batched launch: its geometry and coefficients.
template <typename T, int NP>
struct alignas(16) MarchItem3D {
  March3DArgs a;
  CoefPack<T, NP> cf;
};

template <typename T, int ACC, int R, int CPL, int M, int NW>
__global__ __launch_bounds__(64 * NW) void march3d_batch_kernel(const MarchItem3D<T, npts(3, R, false)>* __restrict__ items,
                                                                const BlockMap* __restrict__ map) {
  __shared__ __attribute__((aligned(16))) T xbuf[2][NW][2 * R][64][CPL];
  const BlockMap m = map[xcd_logical_block(blockIdx.x, gridDim.x)];
  const MarchItem3D<T, npts(3, R, false)>& it = items[__builtin_amdgcn_readfirstlane(m.item)];
  const March3DArgs a = uniform_copy(it.a);
  const CoefPack<T, npts(3, R, false)> cf = uniform_copy(it.cf);
  march3d_block<T, ACC, R, CPL, M, NW>(a, cf, __builtin_amdgcn_readfirstlane(m.block), xbuf);
}

template <typename T, int ACC, int R, int CPL, int M, int NW>
int occupancy_march3d() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, march3d_kernel<T, ACC, R, CPL, M, NW>, 64 * NW, 0) != hipSuccess)
    return 0;
  return nb;
}

// Geometry of a grid's launch in blocks of rd.chunk planes; returns its
// workgroups (0: too large).
template <typename T, int ACC, int R, int CPL, int M, int NW>
int64_t march3d_args(March3DArgs& a, CoefPack<T, npts(3, R, false)>& cf, const Round3D& rd) {
  constexpr int C1 = NW * M - 2 * R, C2 = compute_width(64 * CPL, 1, R, sizeof(T));
  for (int k = 0; k < npts(3, R, false); ++k) cf.c[k] = static_cast<T>(rd.coeffs[k]);
  a.src = rd.src;
  a.dst = rd.dst;
  a.I0 = rd.I0;
  a.I1 = rd.I1;
  a.I2 = rd.I2;
  a.n1 = (rd.I1 + C1 - 1) / C1;
  a.n2 = (rd.I2 + C2 - 1) / C2;
  a.planes = rd.chunk;
  if (a.planes < 1) return 0;
  const int64_t nblk = static_cast<int64_t>(a.n1) * a.n2 * ((rd.I0 + a.planes - 1) / a.planes);
  return nblk > INT32_MAX ? 0 : nblk;
}

template <typename T, int ACC, int R, int CPL, int M, int NW>
hipError_t launch_march3d(const Round3D& rd) {
  March3DArgs a;
  CoefPack<T, npts(3, R, false)> cf;
  const int64_t nblk = march3d_args<T, ACC, R, CPL, M, NW>(a, cf, rd);
  if (nblk == 0) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((march3d_kernel<T, ACC, R, CPL, M, NW>), dim3(static_cast<unsigned>(nblk)), dim3(64 * NW), 0,
                     rd.stream, a, cf);
  return hipGetLastError();
}

template <typename T, int ACC, int R, int CPL, int M, int NW>
int fill_march3d(void* item, const Round3D& rd) {
  MarchItem3D<T, npts(3, R, false)> it;
  const int64_t nblk = march3d_args<T, ACC, R, CPL, M, NW>(it.a, it.cf, rd);
  __builtin_memcpy(item, &it, sizeof(it));
  return static_cast<int>(nblk);
}

template <typename T, int ACC, int R, int CPL, int M, int NW>
hipError_t launch_march3d_batch(const void* items, const BlockMap* map, int nblocks, hipStream_t stream) {
  hipLaunchKernelGGL((march3d_batch_kernel<T, ACC, R, CPL, M, NW>), dim3(nblocks), dim3(64 * NW), 0, stream,
                     static_cast<const MarchItem3D<T, npts(3, R, false)>*>(items), map);
  return hipGetLastError();
}

}  // namespace s5d
