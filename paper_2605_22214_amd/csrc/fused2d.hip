// Several time steps of a periodic D2Q9 lattice in one launch, for the node
// records (moment form of g with the record form of f, or diffusive-only
// runs).  A workgroup loads the records of its tile and a halo of 2 T nodes
// into LDS and takes T steps there, both halves of each (the reconstruction of
// C, E_B and the f moments, then the update), over a region that shrinks by
// one node a side per half: the halo is recomputed instead of exchanged.
// Every value is formed as k_conc_m and k_update form it, in the same order,
// and records are rounded to their storage type after every step, so a run
// does not depend on how its steps are split over the two paths.
//
// Float runs that fill the chip are bound by vector-ALU issue (75% of its peak
// and LDS busy 48% of the time over 32 lenses of 3.0 M nodes, N = 3: 602
// instructions a node and step with those of the halo and of the lanes beyond
// a shrinking row), FP64 at N = 6 by latency at 2.2 wavefronts a SIMD (VALU
// 32%, LDS 23%), small lattices by the latency of the launch and of its phases.
// Per step, two kernels against this one: 64 x 64 FP64 N = 3 7.8 -> 3.0 us, nine
// 300 x 150 lenses FP64 N = 6 61 -> 39 us, those 32 lenses 97 -> 61 us, 512 x
// 512 FP32 N = 4 10.1 -> 8.7 us, 2048 x 2048 FP32 N = 4 without the flow 88 ->
// 32 us.  From N = 5 on the halo's arithmetic can cost more than the launches
// and the memory round trips it saves: fused_plan (api.cpp) draws that line.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "fused2d.h"

namespace nflbm {

// LDS, row by row of W positions: the fields C, next C, mu~ and, with the
// flow, vx, vy, -3/2 v.v, fB, Fx, Fy, E_B and the moments of the streamed f.
// One lane per position reads consecutive words of a field, so no banks
// collide.  (Records of 16-byte words a position, as k_conc_m keeps them in
// float, were no faster: the wider reads cost the LDS more than the address
// additions they save the vector ALU.)

template <class S>
__device__ __forceinline__ typename S::T rec_round(typename S::T v, typename S::T scale) {
  using T = typename S::T;
  if constexpr (sizeof(typename S::RS) == sizeof(T)) {
    (void)scale;
    return v;
  } else {
    return static_cast<T>(static_cast<typename S::RS>(v * scale)) * (T(1) / scale);
  }
}

template <int NC, int ST, bool FR, int WL, int NT>
__device__ __forceinline__ void fused_tile(const FusedArgs& a, const DevParams<typename StoreT<ST>::T>* __restrict__ Pp,
                                           int b, int nsteps, uint32_t nanmask, unsigned char* smem_raw) {
  using L = D2Q9;
  using S = StoreT<ST>;
  using T = typename S::T;
  constexpr int Q = 9, NE = NC - 1, W = 1 << WL;
  constexpr int NF = 3 * NE + (FR ? 10 : 0);
  constexpr int oM = 2 * NE, oV = 3 * NE, oF = oV + 3, oE = oV + 6, oJ = oV + 7;
  constexpr int RS = NF * W;                       // LDS row stride
  constexpr int RPP = NT / W;                      // rows a pass takes
  // FP64 reads of LDS are volatile, which keeps them from being paired: a
  // paired read reaches 255 values beyond its address, so that every few
  // fields cost an address addition, a single one 64 KB (N = 6: 45.2 -> 41.2
  // us a step over 637 x 637).  In float the halved number of LDS
  // instructions is worth more than the additions (N = 3, 1740 x 1740: 52.7
  // against 56.0 us).
  using LV = __attribute__((address_space(3))) T;
  using LT = std::conditional_t<sizeof(T) == 8, volatile LV, LV>;
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int lx = threadIdx.x & (W - 1), lr = threadIdx.x >> WL;
  const int tile_x = b % a.tiles_x, tile_y = b / a.tiles_x;
  const int x0 = tile_x * a.tile_w, y0 = tile_y * a.tile_h;
  const int tw = min(a.tile_w, a.nx - x0), th = min(a.tile_h, a.ny - y0);
  const int H = 2 * nsteps;
  const uint32_t nx = a.nx;
  const DevParams<T>* P0 = gptr<const DevParams<T>>(Pp);

  // ---- records of the tile and its halo into LDS, U rows a thread in flight
  {
    const int rows = th + 2 * H;
    const bool xin = lx < tw + 2 * H;
    const bool near = H <= a.nx && H <= a.ny;      // at most one wrap
    auto wrapped = [&](int v, int n) { return near ? v + (v < 0 ? n : (v >= n ? -n : 0)) : wrap(v, n); };
    const int gx = xin ? wrapped(x0 - H + lx, a.nx) : 0;
    constexpr int U = sizeof(T) == 8 ? (NT == 768 ? 1 : 2) : 3;
    for (int row = lr; row < rows; row += U * RPP) {
      T cc[U][NE], mm[U][NE], vv[U][4], ff[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!xin || row + u * RPP >= rows) continue;
        const uint32_t node = uint32_t(gx) + nx * uint32_t(wrapped(y0 - H + row + u * RPP, a.ny));
        vld<T, NE>(at(gptr<const T>(a.csrc), node * NE), cc[u]);
        rec_load<S, NE>(const_cast<NFLBM_GLOBAL void*>(a.mu_src), node * NE, mm[u], T(S::mu_scale));
        if constexpr (FR) {
          rec_load<S, 4>(const_cast<NFLBM_GLOBAL void*>(a.vel_src), node * 4, vv[u], T(S::vel_scale));
          rec_load<S, 4>(const_cast<NFLBM_GLOBAL void*>(a.frec_src), node * 4, ff[u], T(S::vel_scale));
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!xin || row + u * RPP >= rows) continue;
        T* p = sm + (row + u * RPP) * RS + lx;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          p[e * W] = cc[u][e];
          p[(oM + e) * W] = mm[u][e];
        }
        if constexpr (FR) {
          p[oV * W] = vv[u][0];
          p[(oV + 1) * W] = vv[u][1];
          p[(oV + 2) * W] = vv[u][3];
#pragma unroll
          for (int d = 0; d < 3; ++d) p[(oF + d) * W] = ff[u][d];
        }
      }
    }
  }
  __syncthreads();

  int oC = 0;     // the current C; the next one goes to NE - oC
  // One position's record: C, mu~, (vx, vy, -3/2 v.v), (fB, Fx, Fy)
  struct Rec {
    T c[NE], m[NE], v[3], f[3];
  };
  auto read_rec = [&](const LT* p, Rec& R) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      if constexpr (FR) R.c[e] = p[(oC + e) * W];
      R.m[e] = p[(oM + e) * W];
    }
    if constexpr (FR) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        R.v[d] = p[(oV + d) * W];
        R.f[d] = p[(oF + d) * W];
      }
    }
  };
  for (int t = 0; t < nsteps; ++t) {
    // ---- reconstruction over the tile and 2 (T - t) - 1 nodes around it
    {
      const int m0r = 2 * t + 1;                   // margin to the region's edge
      const int rows = th + 2 * (H - m0r);
      const bool xin = lx >= m0r && lx < tw + 2 * H - m0r;
      for (int row = lr; row < rows; row += RPP) {
        if (!xin) continue;
        const NFLBM_CONST DevParams<T>& P = *fresh_const(P0);
        const T negm = -P.m;
        T* own = sm + (row + m0r) * RS + lx;
        const LT* cor = (const LT*)(own - RS - 1);              // lowest corner of the 3 x 3 neighbourhood
        T c0[NE], s[NE], sd[NE], d0[NE];
        T fm = T(0), jm[3] = {T(0), T(0), T(0)};
        constexpr bool CLASS = sizeof(T) == 4 && !FR;
        {
          Rec R;
          read_rec((const LT*)own, R);
          if constexpr (!FR) {
#pragma unroll
            for (int e = 0; e < NE; ++e) R.c[e] = own[(oC + e) * W];
          }
          const T s0 = FR ? static_cast<T>(L::w[0]) * R.v[2] : T(0);
          const T m0 = moving_weight_sum<L, T>() * P.m;
#pragma unroll
          for (int e = 0; e < NE; ++e) {
            c0[e] = R.c[e];
            const T dd = FR ? fma(c0[e], s0, m0 * R.m[e]) : m0 * R.m[e];
            s[e] = CLASS ? T(0) : T(0) + dd;
            sd[e] = T(0);
            d0[e] = dd;
          }
        }
#pragma unroll
        for (int k = 1; k < Q; ++k) {
          Rec R;
          read_rec(cor + (1 - L::e[k][1]) * RS + (1 - L::e[k][0]), R);
          const T wk = static_cast<T>(L::w[k]);
          if constexpr (!FR) {
            // v = 0: what arrives is -w_k m mu~
            const T mw = negm * wk;
#pragma unroll
            for (int e = 0; e < NE; ++e) {
              if constexpr (CLASS) {
                if (k <= 4) s[e] = fma(negm, R.m[e], s[e]);
                else sd[e] = fma(negm, R.m[e], sd[e]);
              } else {
                s[e] = fma(mw, R.m[e], s[e]);
              }
            }
          } else {
            const int kp = (k & 1) ? k : k - 1;
            const T vs[3] = {R.v[0], R.v[1], T(0)};
            const T ev = proj<L>(kp, vs);
            const T u = fma(ev, fma(T(4.5), ev, (k & 1) ? T(3) : -T(3)), R.v[2]);
            const T wu = wk * u, mw = negm * wk;
#pragma unroll
            for (int e = 0; e < NE; ++e) s[e] = fma(R.c[e], wu, fma(mw, R.m[e], s[e]));
            const T F[3] = {R.f[1], R.f[2], T(0)};
            const T eF = proj<L>(kp, F);
            const T tt = fma(eF, fma(T(4.5), ev, (k & 1) ? T(1.5) : -T(1.5)), R.f[0]);
            const T fk = fma(wk, tt, wu);
            fm += fk;
#pragma unroll
            for (int d = 0; d < 2; ++d)
              if (L::e[k][d] != 0) jm[d] += (L::e[k][d] > 0) ? fk : -fk;
          }
        }
        T cn[NC];
        T rest = T(0);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          T d = s[e];
          if constexpr (CLASS) d = d0[e] + fma(static_cast<T>(L::w[1]), s[e], static_cast<T>(L::w[Q - 1]) * sd[e]);
          cn[e] = c0[e] + d;
          rest += cn[e];
        }
        T En = T(0);
        if constexpr (FR) {
          cn[NE] = T(1) - rest;
          En = bulk_energy<NC, T>(cn, P);
          fm = rec_round<S>(fm, T(S::vel_scale));
          jm[0] = rec_round<S>(jm[0], T(S::vel_scale));
          jm[1] = rec_round<S>(jm[1], T(S::vel_scale));
        }
        const int oN = NE - oC;
#pragma unroll
        for (int e = 0; e < NE; ++e) own[(oN + e) * W] = cn[e];
        if constexpr (FR) {
          own[oE * W] = En;
          own[oJ * W] = fm;
          own[(oJ + 1) * W] = jm[0];
          own[(oJ + 2) * W] = jm[1];
        }
      }
    }
    __syncthreads();
    oC = NE - oC;
    // ---- update over one node less; the last step's goes to memory
    const bool last = t == nsteps - 1;
    const bool check = (nanmask >> t) & 1u;
    auto update = [&](auto PL) {
      constexpr bool PLAIN = decltype(PL)::value;
      const bool omega = !PLAIN && (a.flags & kFlagOmega);
      const bool potential = !PLAIN && (a.flags & kFlagPotential);
      const int m0r = 2 * t + 2;
      const int rows = th + 2 * (H - m0r);
      const bool xin = lx >= m0r && lx < tw + 2 * H - m0r;
      for (int row = lr; row < rows; row += RPP) {
        if (!xin) continue;
        const NFLBM_CONST DevParams<T>& P = *fresh_const(P0);
        T* own = sm + (row + m0r) * RS + lx;
        const LT* cor = (const LT*)(own - RS - 1);
        // C (evolved) and E_B of the neighbour at e
        auto read_ce = [&](int ex, int ey, T (&ce)[NC]) {
          const LT* p = cor + (1 + ey) * RS + (1 + ex);
#pragma unroll
          for (int e = 0; e < NE; ++e) ce[e] = p[(oC + e) * W];
          if constexpr (FR) ce[NE] = p[oE * W];
        };
        T c[NC];
        {
          T ce[NC];
          read_ce(0, 0, ce);
          T rest = ce[0];
          c[0] = rest;
#pragma unroll
          for (int e = 1; e < NE; ++e) {
            c[e] = ce[e];
            rest += c[e];
          }
          c[NE] = T(1) - rest;
        }
        T gC[NC][2], lap[NC], gE[2] = {T(0), T(0)};
#pragma unroll
        for (int i = 0; i < NC; ++i) lap[i] = gC[i][0] = gC[i][1] = T(0);
#pragma unroll
        for (int k = 1; k < Q; k += 2) {
          const int ex = L::e[k][0], ey = L::e[k][1];
          const T wk = static_cast<T>(L::w[k]);
          T pp[NC], pm[NC];
          read_ce(ex, ey, pp);
          read_ce(-ex, -ey, pm);
#pragma unroll
          for (int i = 0; i < NE; ++i) {
            const T vp = pp[i], vm = pm[i];
            lap[i] = fma(wk, vp + vm, lap[i]);
            if constexpr (FR) {
              const T dd = vp - vm;
              if (ex != 0) gC[i][0] = fma((ex > 0) ? wk : -wk, dd, gC[i][0]);
              if (ey != 0) gC[i][1] = fma((ey > 0) ? wk : -wk, dd, gC[i][1]);
            }
          }
          if constexpr (FR) {
            const T dE = pp[NE] - pm[NE];
            if (ex != 0) gE[0] = fma((ex > 0) ? wk : -wk, dE, gE[0]);
            if (ey != 0) gE[1] = fma((ey > 0) ? wk : -wk, dE, gE[1]);
          }
        }
        constexpr T wsum = moving_weight_sum<L, T>();
#pragma unroll
        for (int i = 0; i < NE; ++i) lap[i] = fma(-wsum, c[i], lap[i]);
#pragma unroll
        for (int i = 0; i < NE; ++i) {
          lap[NE] -= lap[i];
#pragma unroll
          for (int d = 0; d < 2; ++d) gC[NE][d] -= gC[i][d];
        }
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          lap[i] *= T(6);
#pragma unroll
          for (int d = 0; d < 2; ++d) gC[i][d] *= T(3);
        }
        gE[0] *= T(3);
        gE[1] *= T(3);

        // flux potential mu~ (factored form)
        T mu[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) {
          T br = -(T(1) - T(3) * c[i] + T(2) * c[i] * c[i]);
#pragma unroll
          for (int l = 0; l < NC; ++l) {
            if (l == i) continue;
            T rw = T(0);
            bool any = false;
#pragma unroll
            for (int m = l + 1; m < NC; ++m)
              if (m != i) {
                rw = any ? fma(P.psi[i][l][m], c[m], rw) : P.psi[i][l][m] * c[m];
                any = true;
              }
            if (any) br = fma(rw, c[l], br);
          }
          T val = fma(P.k34D, lap[i], (P.k12D * c[i]) * br);
          if (omega) {
            T sx = T(0);
#pragma unroll
            for (int k2 = 0; k2 < NC; ++k2)
#pragma unroll
              for (int l = k2 + 1; l < NC; ++l)
                if (k2 != i && l != i) sx = fma(P.xt[i][k2][l], (c[k2] * c[k2]) * (c[l] * c[l]), sx);
            T sy = T(0);
#pragma unroll
            for (int l = 0; l < NC; ++l) {
              if (l == i) continue;
              T inner = T(0);
#pragma unroll
              for (int m = 0; m < NC; ++m)
                if (m != i && m != l) inner = fma(P.zt[i][l][m], c[m], inner);
              sy = fma(c[l] * c[l], inner, sy);
            }
            val = fma((P.k12D * P.omega_stab) * c[i], fma(c[i], sy, sx), val);
          }
          mu[i] = val;
        }
        bool bad = false;
        if (check) {
          T q = T(0);
#pragma unroll
          for (int i = 0; i < NE; ++i) q += c[i] + mu[i];
          bad = !(q - q == T(0));
        }
        const uint32_t node = uint32_t(x0 + lx - H) + nx * uint32_t(y0 + row);   // of the last step
        if (last) {
          vst<T, NE>(at(gptr<T>(a.cdst), node * NE), reinterpret_cast<const T(&)[NE]>(c));
          rec_store<S, NE, false>(a.mu_dst, node * NE, mu, T(S::mu_scale));
        } else {
#pragma unroll
          for (int e = 0; e < NE; ++e) own[(oM + e) * W] = rec_round<S>(mu[e], T(S::mu_scale));
        }
        if constexpr (!FR) {
          if (check && bad) *a.nanflag = 1;
        } else {
          // surface tension force (Eq. Fsnew, or Eq. ststand) + body force
          T F[3];
          if (potential) {
            F[0] = F[1] = T(0);
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              T mraw = T(0);
#pragma unroll
              for (int k2 = 0; k2 < NC; ++k2)
                if (k2 != i)
                  mraw += fma(P.kappa[i][k2], lap[k2], P.beta[i][k2] * (fprime(c[i]) - fprime(c[i] + c[k2])));
#pragma unroll
              for (int d = 0; d < 2; ++d) F[d] = fma(mraw, gC[i][d], F[d]);
            }
          } else {
            F[0] = gE[0];
            F[1] = gE[1];
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              T kl = T(0);
#pragma unroll
              for (int j = 0; j < NC; ++j)
                if (j != i) kl = fma(P.kappa[i][j], lap[j], kl);
#pragma unroll
              for (int d = 0; d < 2; ++d) F[d] = fma(kl, gC[i][d], F[d]);
            }
          }
          F[0] += P.fb[0];
          F[1] += P.fb[1];
          F[2] = T(0) + P.fb[2];
          const T fsum = own[oJ * W];
          const T jm[3] = {own[(oJ + 1) * W], own[(oJ + 2) * W], T(0)};
          T v[3];
#pragma unroll
          for (int d = 0; d < 3; ++d) v[d] = fma(T(0.5), F[d], jm[d]);
          const T vv = fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0]));
          const T s0 = static_cast<T>(L::w[0]) * (-T(1.5) * vv);
          const T Pn = static_cast<T>((1.0 / 3.0) / (1.0 - L::w[0])) * (fsum + s0);
          if (check) {
            const T q = vv + Pn;
            if (bad || !(q - q == T(0))) *a.nanflag = 1;
          }
          const T base_s = -T(1.5) * vv;
          const T vF = fma(v[2], F[2], fma(v[1], F[1], v[0] * F[0]));
          const T cP = T(3) * Pn;
          const T fB = static_cast<T>(fma(-T(1.5), vF, cP));
          if (last) {
            // a resting node's -3/2 v.v is -0, which the update's conversion to
            // binary16 (a fused multiply-add onto 0) stores as +0
            constexpr bool HALF = sizeof(typename S::RS) != sizeof(T);
            const T vel[4] = {v[0], v[1], v[2], HALF ? base_s + T(0) : base_s};
            const T fr[4] = {fB, F[0], F[1], F[2]};
            rec_store<S, 4, false>(a.vel_dst, node * 4, vel, T(S::vel_scale));
            rec_store<S, 4, false>(a.frec_dst, node * 4, fr, T(S::vel_scale));
          } else {
            const T r6[6] = {rec_round<S>(v[0], T(S::vel_scale)),  rec_round<S>(v[1], T(S::vel_scale)),
                             rec_round<S>(base_s, T(S::vel_scale)), rec_round<S>(fB, T(S::vel_scale)),
                             rec_round<S>(F[0], T(S::vel_scale)),  rec_round<S>(F[1], T(S::vel_scale))};
#pragma unroll
            for (int d = 0; d < 6; ++d) own[(oV + d) * W] = r6[d];
          }
        }
      }
    };
    if (a.flags & (kFlagOmega | kFlagPotential)) update(std::false_type{});
    else update(std::true_type{});
    if (!last) __syncthreads();
  }
}

template <int NC, int ST, bool FR, int WL, int NT>
__global__ void __launch_bounds__(NT)
k_fused2d(FusedArgs a, const DevParams<typename StoreT<ST>::T>* __restrict__ Pp, int nsteps, uint32_t nanmask) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  fused_tile<NC, ST, FR, WL, NT>(a, Pp, xcd_remap(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x)), nsteps,
                                 nanmask, smem_raw);
}

template <int NC, int ST, bool FR, int WL, int NT>
__global__ void __launch_bounds__(NT)
k_fused2d_batch(const FusedArgs* __restrict__ args, const DevParams<typename StoreT<ST>::T>* __restrict__ params,
                const int2* __restrict__ work, int nsteps, uint32_t nanmask) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int2 w = work[xcd_remap(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x))];
  const FusedArgs a = args[w.x];
  fused_tile<NC, ST, FR, WL, NT>(a, params + w.x, w.y, nsteps, nanmask, smem_raw);
}

namespace {

template <int NC, int ST, bool FR, int WL, int NT>
hipError_t launch_shape(const FusedLaunch& f, hipStream_t s) {
  using T = typename StoreT<ST>::T;
  const auto* P = static_cast<const DevParams<T>*>(f.params);
  if (f.batch)
    hipLaunchKernelGGL((k_fused2d_batch<NC, ST, FR, WL, NT>), dim3(f.blocks), dim3(NT), f.lds, s, f.batch, P, f.work,
                       f.nsteps, f.nanmask);
  else
    hipLaunchKernelGGL((k_fused2d<NC, ST, FR, WL, NT>), dim3(f.blocks), dim3(NT), f.lds, s, *f.one, P, f.nsteps,
                       f.nanmask);
  return hipGetLastError();
}

template <int NC, int ST>
hipError_t launch_nc(const FusedLaunch& f, hipStream_t s) {
  // the shapes fused_plan chooses from; 1024 threads leave 128 VGPRs each, 768
  // leave 168
  constexpr bool few = !(ST == kStoreF64 && NC >= 5);
  if (f.frecord && f.wlog2 == 5) {
    if (f.threads == 512) return launch_shape<NC, ST, true, 5, 512>(f, s);
    if constexpr (ST == kStoreF64 && (NC == 5 || NC == 6)) {
      if (f.threads == 768) return launch_shape<NC, ST, true, 5, 768>(f, s);
    }
    if constexpr (few) {
      if (f.threads == 1024) return launch_shape<NC, ST, true, 5, 1024>(f, s);
    }
  } else if (f.wlog2 == 5) {
    if (f.threads == 512) return launch_shape<NC, ST, false, 5, 512>(f, s);
    if constexpr (few) {
      if (f.threads == 1024) return launch_shape<NC, ST, false, 5, 1024>(f, s);
    }
  } else if (!f.frecord && f.wlog2 == 6 && f.threads == 1024) {
    return launch_shape<NC, ST, false, 6, 1024>(f, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

#define FUSED_CAT2(a, b) a##b
#define FUSED_CAT(a, b) FUSED_CAT2(a, b)
// One translation unit per storage precision (NFLBM_UNIT_STORE).
hipError_t FUSED_CAT(launch_fused2d_, NFLBM_UNIT_STORE)(int nc, const FusedLaunch& f, hipStream_t s) {
  constexpr int ST = NFLBM_UNIT_STORE;
  switch (nc) {
    case 2: return launch_nc<2, ST>(f, s);
    case 3: return launch_nc<3, ST>(f, s);
    case 4: return launch_nc<4, ST>(f, s);
    case 5: return launch_nc<5, ST>(f, s);
    case 6: return launch_nc<6, ST>(f, s);
    case 7: return launch_nc<7, ST>(f, s);
    case 8: return launch_nc<8, ST>(f, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace nflbm
