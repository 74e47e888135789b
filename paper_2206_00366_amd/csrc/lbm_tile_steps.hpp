// Several time steps in one pass over the populations, for rD2Q9 domains
// (single ones and batches): temporal blocking over 2D tiles in LDS.
//
// A workgroup reads the natural state of a tile of columns x rows with a ring
// of kTileRing nodes, takes up to kTileRing steps in LDS (a node's q values in
// registers, pushed to the neighbours' LDS entries after each collision but the
// last; the outermost row and column of what is valid drops out with every such
// exchange) and writes the inner nodes' last pushes to another buffer.  Large
// domains move their populations once for four steps, small ones launch once.
// A pass of s steps makes s - 1 exchanges and so needs a ring of s - 1: the ring
// is one node wider than passes of four steps need.
//
// A bounced link returns to the node it left, in LDS as in memory.
//
// What bounds it: the collisions and LDS exchanges of the ring nodes besides
// the inner ones (43 x 32 of 51 x 40) for large domains, the chain of one
// workgroup's steps for small ones; before, the sweep per step and the launch
// per step.  Us a step, single steps / this kernel: FP32 NCDE 2048 x 1024 20.5 /
// 13.8 (workgroups of 1024 threads, one to a CU: 16.3; a sweep along y that
// holds two steps: 16.4), 512 x 256 3.4 / 2.4, 64 x 32 2.65 / 1.6; FP64 64 x 32
// 2.8 / 1.6, 2048 x 1024 42 / 30; 16 FP32 obstacle channels of 512 x 256 in a
// batch 27 / 18.
// The arithmetic is the single step's, so the results are those of single steps
// bit for bit.
#pragma once

#include "lbm_kernels.hpp"

namespace rmrt {

template <int ST, int EQ, int FORCE, bool BND, uint32_t NT>
__global__ void __launch_bounds__(NT)
    k_tile_steps(const DomainDev* __restrict__ doms, const TileItem* __restrict__ items, uint32_t from_second,
                 uint32_t steps) {
  using SS = Store<ST>;
  using S = typename SS::S;
  using T = typename SS::T;
  constexpr int L = LAT_Q9, Q = 9, NPT = kTileNodes;
  constexpr uint32_t NN = NT * NPT, R = kTileRing, es = sizeof(S);
  constexpr uint32_t kX0 = 1u << 16, kX1 = 2u << 16, kY0 = 4u << 16, kY1 = 8u << 16, kLive = 16u << 16, kInner = 32u << 16;
  extern __shared__ __align__(16) unsigned char lds_raw[];

  const TileItem it = items[blockIdx.x];
  const DomainDev& Dm = doms[it.dom];
  const uint32_t LD = Dm.ld, nx = Dm.nx, ny = Dm.ny;
  gmem<S>* fin = to_global((S*)(from_second ? Dm.fb : Dm.fa));
  gmem<S>* fout = to_global((S*)(from_second ? Dm.fa : Dm.fb));
  const BufRsrc rin = buf_rsrc((const gmem<S>*)fin, (uint32_t)Q * LD * es);
  const BufRsrc rout = buf_rsrc((const gmem<S>*)fout, (uint32_t)Q * LD * es);
  // a tile over the whole of x has no ring there: its pushes wrap within it
  const bool full = it.cx == nx;
  const uint32_t W = full ? nx : it.cx + 2u * R, H = it.cy + 2u * R, WH = W * H;
  S* const lds = (S*)lds_raw + W + 1u;   // pushes that leave the tile stay in the padding or in ring entries

  S v[NPT][Q];
  uint32_t gi[NPT], fl[NPT];   // node index; link bits (low half) and flags
  static_for<0, NPT>([&](auto c_) {
    constexpr int c = decltype(c_)::value;
    const uint32_t t = threadIdx.x + c * NT;
    fl[c] = 0;
    gi[c] = 0;
    if (t < WH) {
      const uint32_t ly = t / W, lx = t - ly * W;
      // ring coordinates wrap (a ring is no wider than the domain)
      uint32_t gx = full ? lx : it.x0 + lx + nx - R, gy = it.y0 + ly + ny - R;
      gx = gx >= nx ? gx - nx : gx;
      gx = gx >= nx ? gx - nx : gx;
      gy = gy >= ny ? gy - ny : gy;
      gy = gy >= ny ? gy - ny : gy;
      const uint32_t i = checked_node(Dm, gx + nx * gy, 0u);
      gi[c] = i;
      uint32_t f = kLive | (gx == 0u ? kX0 : 0u) | (gx == nx - 1u ? kX1 : 0u) | (gy == 0u ? kY0 : 0u) |
                   (gy == ny - 1u ? kY1 : 0u);
      if ((full || (lx >= R && lx < R + it.cx)) && ly >= R && ly < R + it.cy) f |= kInner;
      if constexpr (BND) {
        uint32_t lb = 0;
        if (Dm.links) {
          lb = to_global((const uint16_t*)Dm.links)[i];
        } else if (Dm.walls) {
          Geo<2> g;
          g.make(Dm, i);
          static_for<1, Q>([&](auto j_) {
            constexpr int J = decltype(j_)::value;
            if (g.template bounce<L, J, false>(Dm, i)) lb |= 1u << J;
          });
        }
        if (lb & LinkBits<L>::kSolid) f &= ~(kLive | kInner);
        f |= lb & 0x7fffu;
      }
      fl[c] = f;
      static_for<0, Q>([&](auto j_) {
        constexpr int J = decltype(j_)::value;
        v[c][J] = buf_ld<S>(rin, i * es, (uint32_t)J * LD * es);
      });
    }
  });
  for (uint32_t s = 0;; ++s) {
    const bool last = s + 1u == steps;
    static_for<0, NPT>([&](auto c_) {
      constexpr int c = decltype(c_)::value;
      if (fl[c] & kLive) {
        // The collision must round as in k_step.  Which multiply-adds the
        // compiler fuses depends on what it sees in one block, so the
        // coefficients are read here every time (the pointer is a new value to
        // the compiler) as they are there, instead of sums of them being formed
        // before the loop; constant address space keeps them scalar loads.
        auto cp = (const __attribute__((address_space(4))) Coef<T>*)&coef<T>(Dm);
        asm volatile("" : "+s"(cp));
        const Coef<T>& C = *(const Coef<T>*)cp;
        const NodeSrc<T> src = const_sources<T>(C);
        T t[9];
        static_for<0, Q>([&](auto j_) {
          constexpr int J = decltype(j_)::value;
          t[Lat<L>::slot(J)] = SS::template dec<Lat<L>::wclass(J)>(v[c][J], C);
        });
        collide<L, EQ, FORCE>(t, C, src);
        static_for<0, Q>([&](auto j_) {
          constexpr int J = decltype(j_)::value;
          v[c][J] = SS::template enc<Lat<L>::wclass(J)>(t[Lat<L>::slot(J)], C);
        });
      }
    });
    if (last) break;
    __syncthreads();   // the last step's entries have been read
    static_for<0, NPT>([&](auto c_) {
      constexpr int c = decltype(c_)::value;
      const uint32_t t = threadIdx.x + c * NT, f = fl[c];
      if (f & kLive) {
        static_for<0, Q>([&](auto j_) {
          constexpr int J = decltype(j_)::value;
          constexpr int ex = Lat<L>::e(J, 0), ey = Lat<L>::e(J, 1), O = Lat<L>::opp(J);
          uint32_t to = t + (uint32_t)(ey * (int)W + ex) + J * NN;
          if constexpr (ex < 0) to += (full && (f & kX0)) ? W : 0u;
          if constexpr (ex > 0) to -= (full && (f & kX1)) ? W : 0u;
          if constexpr (BND && J > 0) to = (f >> J) & 1u ? t + O * NN : to;
          lds[(int32_t)to] = v[c][J];
        });
      }
    });
    __syncthreads();
    static_for<0, NPT>([&](auto c_) {
      constexpr int c = decltype(c_)::value;
      if (c * NT < WH)
        static_for<0, Q>([&](auto j_) {
          constexpr int J = decltype(j_)::value;
          v[c][J] = lds[threadIdx.x + c * NT + J * NN];
        });
    });
  }
  static_for<0, NPT>([&](auto c_) {
    constexpr int c = decltype(c_)::value;
    const uint32_t f = fl[c];
    if (f & kInner) {
      static_for<0, Q>([&](auto j_) {
        constexpr int J = decltype(j_)::value;
        constexpr int ex = Lat<L>::e(J, 0), ey = Lat<L>::e(J, 1), O = Lat<L>::opp(J);
        uint32_t o = gi[c];
        if constexpr (ex < 0) o += (f & kX0) ? nx - 1u : ~0u;
        if constexpr (ex > 0) o += (f & kX1) ? 1u - nx : 1u;
        if constexpr (ey < 0) o += (f & kY0) ? nx * (ny - 1u) : 0u - nx;
        if constexpr (ey > 0) o += (f & kY1) ? 0u - nx * (ny - 1u) : nx;
        if constexpr (BND && J > 0) {
          const uint32_t e = (f >> J) & 1u ? O * LD + gi[c] : J * LD + checked_node(Dm, o, gi[c]);
          buf_st<S>(rout, e * es, 0u, v[c][J]);
        } else {
          buf_st<S>(rout, checked_node(Dm, o, gi[c]) * es, (uint32_t)J * LD * es, v[c][J]);
        }
      });
    }
  });
}

template <int ST, int EQ, int FORCE, bool BND, uint32_t NT>
hipError_t do_tile_steps_nt(const StepLaunch& a) {
  const uint32_t lds = (uint32_t)sizeof(typename Store<ST>::S) * (9u * NT * kTileNodes + 2u * (a.sweep_w + 1u));
  hipLaunchKernelGGL((k_tile_steps<ST, EQ, FORCE, BND, NT>), dim3(a.grid), dim3(NT), lds, a.stream, a.doms, a.tile_items,
                     a.parity, a.pass_steps);
  return hipGetLastError();
}
template <int ST, int EQ, int FORCE, bool BND>
hipError_t do_tile_steps(const StepLaunch& a) {
  if (a.block == kTileThreads(ST)) return do_tile_steps_nt<ST, EQ, FORCE, BND, kTileThreads(ST)>(a);
  if constexpr (ST == ST_F64)
    if (a.block == 2u * kTileThreads(ST)) return do_tile_steps_nt<ST, EQ, FORCE, BND, 2u * kTileThreads(ST)>(a);
  return hipErrorInvalidValue;
}
// The raw-moment NSE and the NCDE with C = phi u u; with constant sources in
// FP32 only (in FP64 the compiler fuses the forced collision differently here
// and in k_step, and the last bits differ).
template <int ST>
hipError_t launch_tile_steps(const StepLaunch& a) {
  const bool b = a.bc != 0;
  if ((a.eq != EQ_NSE && a.eq != EQ_NCDE) || !tile_force_built(ST, a.force)) return hipErrorInvalidValue;
#define RMRT_TS(E, F)                                                                    \
  if (a.eq == E && a.force == F)                                                         \
    return b ? do_tile_steps<ST, E, F, true>(a) : do_tile_steps<ST, E, F, false>(a);
  RMRT_TS(EQ_NSE, F_NONE)
  RMRT_TS(EQ_NCDE, F_NONE)
  if constexpr (tile_force_built(ST, F_CONST)) {
    RMRT_TS(EQ_NSE, F_CONST)
    RMRT_TS(EQ_NCDE, F_CONST)
  }
#undef RMRT_TS
  return hipErrorInvalidValue;
}

}  // namespace rmrt
