// Two time steps in one pass over the populations (temporal blocking), for
// periodic 3D domains of the raw-moment NSE without sources.
//
// What bounds the single step is one read and one write of every population
// per step.  This kernel reads the natural state of one buffer, takes both
// steps and writes the natural state two steps later into another buffer, so
// a pass of the same traffic advances two steps.
//
// A workgroup owns a patch of lattice columns along z plus a ring of one column
// on each side, one or two columns per thread, and walks a chunk of planes:
//   stage 1  plane p: read the own slots, collide, push the q values into LDS
//            (slot j of the column at e_j's offset within the patch)
//   stage 2  plane p - 1 of the inner columns: its q values are what stage 1
//            pushed from planes p - 2, p - 1 and p; collide, push to memory
// A value pushed up (e_z = 1) waits two planes and one pushed level one plane
// for its stage 2; both wait in registers of the column's thread, so LDS
// holds one plane of q values only.  The next plane's loads are issued before
// the current plane's exchange and land behind it.
//
// What bounds this kernel is how many cache lines its rows touch and the
// accesses a CU can have in flight, then HBM: with patches of 32 x 13 inner
// columns (34 x 15 threads) the L1 asked the L2 for 4 times the populations'
// bytes and a step took 208-225 us (rD3Q19 FP32, 256 x 256 x 128; single
// step 196.5), with 64 x 13 it took 171, with patches that span x (no ring
// along x, whole rows end to end in memory: 256 x 4 inner columns) 140, and
// with waves that hold ring columns only skipping stage 2 135 us.  The ring
// and the two extra planes of a chunk are collided by more than one workgroup;
// their reads mostly hit the L2.  rD3Q27 FP32 256 x 256 x 128: 293 -> 192 us a
// step; rD3Q19 FP64: 449 -> 303 us.  FP16 storage in the patches of FP32 gained
// nothing (106 -> 111 us; patches sized for its entries are not tried) and rD3Q27
// FP64 lost (its rows of 27 doubles leave patches of 512 columns), so neither is built.
//
// The arithmetic is the single step's (collide_nse, and the storage type
// between the steps), so the results are those of two single steps bit for
// bit.
#pragma once

#include "lbm_kernels.hpp"

namespace rmrt {

// Waits for this wave's LDS accesses and synchronises the workgroup.  Unlike
// __syncthreads it leaves global loads and stores in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int L, int ST>
__global__ void __launch_bounds__((TwoStep<L, ST>::kThreads))
    k_two_step(const DomainDev* __restrict__ dom, const SweepItem* __restrict__ items, uint32_t from_second) {
  using SS = Store<ST>;
  using S = typename SS::S;
  using T = typename SS::T;
  constexpr int Q = Lat<L>::Q, NS = Lat<L>::NS;
  constexpr int NPT = TwoStep<L, ST>::kColumns;
  constexpr uint32_t NT = TwoStep<L, ST>::kThreads, NC = NT * NPT;
  constexpr uint32_t es = sizeof(S);
  extern __shared__ __align__(16) unsigned char lds_raw[];
  S* const lds = (S*)lds_raw;

  const SweepItem it = items[blockIdx.x];
  const DomainDev& Dm = *dom;
  // the parameter block never changes while a kernel runs: constant address
  // space, so that the barriers do not make the loop read it again
  const Coef<T>& C = *(const Coef<T>*)(const __attribute__((address_space(4))) Coef<T>*)&coef<T>(Dm);
  const uint32_t LD = Dm.ld;
  gmem<S>* fin = to_global((S*)(from_second ? Dm.fb : Dm.fa));
  gmem<S>* fout = to_global((S*)(from_second ? Dm.fa : Dm.fb));
  const BufRsrc rin = buf_rsrc((const gmem<S>*)fin, (uint32_t)Q * LD * es);
  const BufRsrc rout = buf_rsrc((const gmem<S>*)fout, (uint32_t)Q * LD * es);

  const uint32_t nx = Dm.nx, ny = Dm.ny, SN = Dm.nz, PS = Dm.nxny;   // SN planes of PS nodes
  // patch: W x H columns; a patch over the whole of x has no ring there (its
  // pushes wrap within the patch)
  const bool full = it.cx == nx;
  const uint32_t W = full ? nx : it.cx + 2u, H = it.cy + 2u;

  struct Column {
    uint32_t col;          // node index in plane 0
    uint32_t at;           // LDS entry of slot 0
    uint32_t flags;        // kCore and the domain faces the column touches
  };
  constexpr uint32_t kX0 = 1u, kX1 = 2u, kY0 = 4u, kY1 = 8u, kCore = 16u;
  Column cl[NPT];
  static_for<0, NPT>([&](auto c_) {
    constexpr int c = decltype(c_)::value;
    const uint32_t t = threadIdx.x + c * NT;
    const uint32_t ly = t / W, lx = t - ly * W;
    const bool active = t < W * H;
    uint32_t gx;
    if (full) {
      gx = lx;
    } else {   // wrapped coordinates of the ring
      gx = it.x0 + lx;
      gx = gx == 0u ? nx - 1u : (gx > nx ? 0u : gx - 1u);
    }
    uint32_t gy = it.y0 + ly;
    gy = gy == 0u ? ny - 1u : (gy > ny ? 0u : gy - 1u);
    const bool core = active && (full || (lx >= 1u && lx <= it.cx)) && ly >= 1u && ly <= it.cy;
    cl[c].col = active ? gx + nx * gy : 0u;
    // A thread beyond the patch collides column 0.  Its entry is the second one
    // past the patch (the plan leaves none or at least three): its pushes then
    // reach back to the last row and forward to the next array's first, which
    // are ring.
    cl[c].at = W + 1u + (active ? t : W * H + 1u);
    cl[c].flags = !active ? 0u : (core ? kCore : 0u) | (gx == 0u ? kX0 : 0u) | (gx == nx - 1u ? kX1 : 0u) |
                  (gy == 0u ? kY0 : 0u) | (gy == ny - 1u ? kY1 : 0u);
  });
  // node offset of the neighbouring column along e_J
  auto nbr_off = [&](auto j_, uint32_t fl) -> uint32_t {
    constexpr int J = decltype(j_)::value;
    constexpr int ex = Lat<L>::e(J, 0), ey = Lat<L>::e(J, 1);
    uint32_t o = 0;
    if constexpr (ex < 0) o += (fl & kX0) ? nx - 1u : ~0u;
    if constexpr (ex > 0) o += (fl & kX1) ? 1u - nx : 1u;
    if constexpr (ey < 0) o += (fl & kY0) ? nx * (ny - 1u) : 0u - nx;
    if constexpr (ey > 0) o += (fl & kY1) ? 0u - nx * (ny - 1u) : nx;
    return o;
  };
  // LDS offset of the neighbouring column along e_J.  Pushes that leave the
  // patch land on ring entries of a neighbouring row or slot array, or on the
  // padding of W + 1 entries at both ends; nothing reads those.
  auto lds_off = [&](auto j_, uint32_t fl) -> uint32_t {
    constexpr int J = decltype(j_)::value;
    constexpr int ex = Lat<L>::e(J, 0), ey = Lat<L>::e(J, 1);
    uint32_t o = (uint32_t)ey * W + (uint32_t)ex;
    if constexpr (ex < 0) o += (full && (fl & kX0)) ? W : 0u;
    if constexpr (ex > 0) o -= (full && (fl & kX1)) ? W : 0u;
    return o;
  };

  const uint32_t planes = it.cz + 2u;
  auto sweep = [&](auto inner_) {
    constexpr int INNER = decltype(inner_)::value;
    S v[NPT][Q];   // the next plane's populations, as stored
    auto fetch = [&](auto c_, uint32_t z) {
      constexpr int c = decltype(c_)::value;
      const uint32_t at = PS * z;
      static_for<0, Q>([&](auto j_) {
        constexpr int J = decltype(j_)::value;
        if constexpr (RMRT_CHECKED != 0)
          v[c][J] = buf_ld<S>(rin, checked_node(Dm, cl[c].col + at, 0u) * es, (uint32_t)J * LD * es);
        else
          v[c][J] = buf_ld<S>(rin, cl[c].col * es, ((uint32_t)J * LD + at) * es);
      });
    };
    // values waiting in the thread: pushed up one and two planes ago, level one
    // plane ago
    S up1[NPT][Q], up2[NPT][Q], lev[NPT][Q];
    uint32_t z = it.z0 == 0u ? SN - 1u : it.z0 - 1u;   // plane p of stage 1, wrapped
    uint32_t zprev = z;
    static_for<0, NPT>([&](auto c_) {
      constexpr int c = decltype(c_)::value;
      static_for<0, Q>([&](auto j_) {
        constexpr int J = decltype(j_)::value;
        up1[c][J] = up2[c][J] = lev[c][J] = S(0);
      });
      fetch(c_, z);
    });
    // the loop's waits count the accesses issued after a plane's loads; landing
    // the first plane here keeps them from being merged with this entry's count,
    // which would drain the stores in every iteration
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    for (uint32_t k = 0; k < planes; ++k) {
      const uint32_t znext = z + 1u == SN ? 0u : z + 1u;
      static_for<0, NPT>([&](auto c_) {
        constexpr int c = decltype(c_)::value;
        T t[NS];
        static_for<0, NS>([&](auto s_) {
          constexpr int s = decltype(s_)::value;
          if constexpr (Lat<L>::absent(s)) t[s] = T(0);
        });
        static_for<0, Q>([&](auto j_) {
          constexpr int J = decltype(j_)::value;
          t[Lat<L>::slot(J)] = SS::template dec<Lat<L>::wclass(J)>(v[c][J], C);
        });
        fetch(c_, znext);
        collide_nse<L>(t, C);
        uint32_t fl = cl[c].flags;
        asm("" : "+v"(fl));   // the offsets are formed here each time, not held across the loop
        static_for<0, Q>([&](auto j_) {
          constexpr int J = decltype(j_)::value;
          const S e = SS::template enc<Lat<L>::wclass(J)>(t[Lat<L>::slot(J)], C);
          lds[cl[c].at + lds_off(j_, fl) + J * NC] = e;
        });
      });
      lds_barrier();
      static_for<0, NPT>([&](auto c_) {
        constexpr int c = decltype(c_)::value;
        if constexpr ((INNER >> c) & 1) {
          S n[Q];
          static_for<0, Q>([&](auto j_) {
            constexpr int J = decltype(j_)::value;
            n[J] = lds[cl[c].at + J * NC];
          });
          T t[NS];
          static_for<0, NS>([&](auto s_) {
            constexpr int s = decltype(s_)::value;
            if constexpr (Lat<L>::absent(s)) t[s] = T(0);
          });
          static_for<0, Q>([&](auto j_) {
            constexpr int J = decltype(j_)::value;
            constexpr int ez = Lat<L>::e(J, 2);
            t[Lat<L>::slot(J)] =
                SS::template dec<Lat<L>::wclass(J)>(ez < 0 ? n[J] : (ez == 0 ? lev[c][J] : up2[c][J]), C);
            if constexpr (ez > 0) {
              up2[c][J] = up1[c][J];
              up1[c][J] = n[J];
            } else if constexpr (ez == 0) {
              lev[c][J] = n[J];
            }
          });
          collide_nse<L>(t, C);
          // Lanes with nothing to write store beyond the buffer, where the hardware
          // drops the store: a branch around the stores would make the compiler
          // wait for them before the next plane's loads (it cannot count accesses
          // that may not have been issued).
          uint32_t fl = cl[c].flags;
          asm("" : "+v"(fl));
          const bool run2 = (fl & kCore) && k >= 2u;
          const uint32_t base = run2 ? cl[c].col * es : kBeyond;
          // planes zprev - 1, zprev, zprev + 1 of the pushes (zprev + 1 = z)
          const uint32_t zlow = zprev == 0u ? SN - 1u : zprev - 1u;
          static_for<0, Q>([&](auto j_) {
            constexpr int J = decltype(j_)::value;
            constexpr int ez = Lat<L>::e(J, 2);
            const S r = SS::template enc<Lat<L>::wclass(J)>(t[Lat<L>::slot(J)], C);
            const uint32_t zt = ez < 0 ? zlow : (ez == 0 ? zprev : z);
            const uint32_t off = nbr_off(j_, fl);
            if constexpr (RMRT_CHECKED != 0)
              if (run2) checked_node(Dm, cl[c].col + off + PS * zt, 0u);
            buf_st<S>(rout, base + off * es, ((uint32_t)J * LD + PS * zt) * es, r);
          });
        }
      });
      lds_barrier();
      zprev = z;
      z = znext;
    }
  };
  // bit c: this wave has inner columns among its c-th ones.  Columns that are
  // all on the ring (or beyond the patch) have no stage 2; the wave runs the
  // form of the loop without it.
  uint32_t inner = 0;
  static_for<0, NPT>([&](auto c_) {
    constexpr int c = decltype(c_)::value;
    if (__builtin_amdgcn_ballot_w64((cl[c].flags & kCore) != 0u) != 0) inner |= 1u << c;
  });

  inner = __builtin_amdgcn_readfirstlane(inner);
  static_for<0, (1 << NPT)>([&](auto m_) {
    if (inner == (uint32_t)decltype(m_)::value) sweep(m_);
  });
}

// Launch, or (occupancy set) report the columns of a workgroup and how many
// workgroups fit a CU with the widest patch (three rows).
template <int L, int ST>
hipError_t do_two_step(const StepLaunch& a) {
  constexpr int threads = TwoStep<L, ST>::kThreads, columns = threads * TwoStep<L, ST>::kColumns;
  const uint32_t w = a.occupancy ? (uint32_t)columns / 3u : a.sweep_w;
  const uint32_t lds = (uint32_t)sizeof(typename Store<ST>::S) * (Lat<L>::Q * columns + 2u * (w + 1u));
  if (a.occupancy) {
    *a.columns = columns;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(a.occupancy, k_two_step<L, ST>, threads, lds);
  }
  hipLaunchKernelGGL((k_two_step<L, ST>), dim3(a.grid), dim3(threads), lds, a.stream, a.doms, a.sweep, a.parity);
  return hipGetLastError();
}

}  // namespace rmrt
