// Time steps of a periodic D2Q9 lattice with the concentration-dependent
// mobility (Appendix C), diffusive-only and every tau_g = 1, one or two in a
// launch.  There the collision leaves exactly the source terms, g*_k = w_k
// e_k.G (1 - 1/2) m* and the rest population C less their sum, so a step is
//   C    = sum of the streamed populations      (k_conc)
//   Phi  = mu + phi + xi from C and its Laplacian (k_mob_potentials)
//   G    = sum_j alpha_ij grad Phi_j             (k_mob_source)
// and the four launches of the general path (whose update only copies) pass
// everything through memory between them: 26 us a step of the 400 x 400 run
// in FP32, of which each launch's latency is most.  Here a workgroup forms C
// over its tile and a halo of 3 T - 1 nodes, from the populations in memory
// before the first step and from G and the rest populations in LDS after it,
// then Phi over one node less, then G over another; the last step writes the
// populations.  Every value is formed as the general path forms it, in the
// same order, populations rounded to their storage type.
#include <hip/hip_runtime.h>

#include "device.h"
#include "fused2d.h"

namespace nflbm {

template <int NC, int ST>
__global__ void __launch_bounds__(512) k_fused_mob(FusedMobArgs ma, int nsteps, uint32_t nanmask) {
  using L = D2Q9;
  using S = StoreT<ST>;
  using T = typename S::T;
  using FS = typename S::FS;
  using G0S = typename S::G0S;
  constexpr int Q = 9, NE = NC - 1, W = 32, RPP = 512 / W;
  // LDS, row by row: C and Phi of every component, G and the rest population
  // of the evolved ones
  constexpr int oP = NC, oG = 2 * NC, oR = oG + 2 * NE, NF = oR + NE, RS = NF * W;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int lx = threadIdx.x & (W - 1), lr = threadIdx.x / W;
  const int b = xcd_remap(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
  const int x0 = (b % ma.tiles_x) * ma.tile_w, y0 = (b / ma.tiles_x) * ma.tile_h;
  const int tw = min(ma.tile_w, ma.nx - x0), th = min(ma.tile_h, ma.ny - y0);
  const int H = 3 * nsteps - 1;
  const uint32_t nx = ma.nx;
  const size_t gst = static_cast<size_t>(ma.gstride);
  const DevParams<T>* P0 = gptr<const DevParams<T>>(static_cast<const DevParams<T>*>(ma.params));
  const MobParams<T>* M0 = gptr<const MobParams<T>>(static_cast<const MobParams<T>*>(ma.mob));
  const bool omega = (ma.flags & kFlagOmega) != 0;

  for (int t = 0; t < nsteps; ++t) {
    const bool last = t == nsteps - 1;
    const bool check = (nanmask >> t) & 1u;
    // ---- C, a margin of 3 t nodes to the region's edge
    {
      const int mg = 3 * t, rows = th + 2 * (H - mg);
      const bool xin = lx >= mg && lx < tw + 2 * H - mg;
      for (int row = lr; row < rows; row += RPP) {
        if (!xin) continue;
        T* own = sm + (row + mg) * RS + lx;
        T s[NE], r[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) s[e] = T(0);
        if (t == 0) {
          const int x = wrap(x0 - H + lx, ma.nx), y = wrap(y0 - H + row, ma.ny);
          const uint32_t xo[3] = {uint32_t(x == 0 ? ma.nx - 1 : x - 1), uint32_t(x), uint32_t(x == ma.nx - 1 ? 0 : x + 1)};
          const uint32_t yo[3] = {nx * uint32_t(y == 0 ? ma.ny - 1 : y - 1), nx * uint32_t(y),
                                  nx * uint32_t(y == ma.ny - 1 ? 0 : y + 1)};
          const FS* gk = static_cast<const FS*>(ma.gk_src);
#pragma unroll
          for (int k = 1; k < Q; ++k) {
            FS v[NE];
            vld<FS, NE>(at(gk + size_t(k - 1) * gst, (xo[1 - L::e[k][0]] + yo[1 - L::e[k][1]]) * NE), v);
#pragma unroll
            for (int e = 0; e < NE; ++e) s[e] += S::unpack(v[e]);
          }
          G0S r0[NE];
          vld<G0S, NE>(at(static_cast<const G0S*>(ma.g0_src), (xo[1] + yo[1]) * NE), r0);
#pragma unroll
          for (int e = 0; e < NE; ++e) r[e] = static_cast<T>(r0[e]);
        } else {
#pragma unroll
          for (int k = 1; k < Q; ++k) {
            const T* src = own - L::e[k][1] * RS - L::e[k][0];
            const T wk = static_cast<T>(L::w[k]);
#pragma unroll
            for (int e = 0; e < NE; ++e) {
              const T G[3] = {src[(oG + 2 * e) * W], src[(oG + 2 * e + 1) * W], T(0)};
              s[e] += S::unpack(S::pack(wk * proj<L>(k, G)));
            }
          }
#pragma unroll
          for (int e = 0; e < NE; ++e) r[e] = own[(oR + e) * W];
        }
        T rest = T(0);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          s[e] = r[e] + s[e];
          rest += s[e];
          own[e * W] = s[e];
        }
        own[NE * W] = T(1) - rest;
      }
    }
    __syncthreads();
    // ---- Phi over one node less
    {
      const int mg = 3 * t + 1, rows = th + 2 * (H - mg);
      const bool xin = lx >= mg && lx < tw + 2 * H - mg;
      for (int row = lr; row < rows; row += RPP) {
        if (!xin) continue;
        const NFLBM_CONST DevParams<T>& P = *fresh_const(P0);
        const NFLBM_CONST MobParams<T>& M = *fresh_const(M0);
        T* own = sm + (row + mg) * RS + lx;
        T c[NC], lap[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
          c[j] = own[j * W];
          lap[j] = T(0);
        }
#pragma unroll
        for (int k = 1; k < Q; ++k) {
          const T* src = own + L::e[k][1] * RS + L::e[k][0];
          const T wk = static_cast<T>(L::w[k]);
#pragma unroll
          for (int j = 0; j < NC; ++j) lap[j] = fma(wk, src[j * W] - c[j], lap[j]);
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) lap[j] *= T(6);
        T probe = T(0);
#pragma unroll
        for (int j = 0; j < NC; ++j) {
          T mu = T(0);
#pragma unroll
          for (int k = 0; k < NC; ++k)
            if (k != j) mu = fma(P.beta[j][k], fprime(c[j]) - fprime(c[j] + c[k]), mu);
#pragma unroll
          for (int k = 0; k < NC; ++k)
            if (k != j) mu = fma(P.kappa[j][k], lap[k], mu);
          T ph = T(0);
#pragma unroll
          for (int k = 0; k < NC; ++k)
#pragma unroll
            for (int l = k + 1; l < NC; ++l)
#pragma unroll
              for (int m = l + 1; m < NC; ++m)
                if (k != j && l != j && m != j) ph = fma(M.lam[j][k][l][m], c[k] * c[l] * c[m], ph);
          T xi = T(0);
          if (omega) {
#pragma unroll
            for (int k = 0; k < NC; ++k)
#pragma unroll
              for (int l = k + 1; l < NC; ++l) {
                if (k == j || l == j) continue;
                T inner = T(2) * c[j];
#pragma unroll
                for (int m = 0; m < NC; ++m)
                  if (m != j && m != k && m != l) inner = fma(-M.theta[k][l][j][m], c[m], inner);
                xi = fma((c[k] * c[k]) * (c[l] * c[l]), inner, xi);
              }
            xi *= P.k12D * P.omega_stab;
          }
          const T phi = fma(P.k12D, ph, mu) + xi;
          own[(oP + j) * W] = phi;
          probe += c[j] + phi;
        }
        // a non-finite C or Phi makes probe - probe NaN
        if (check && !(probe - probe == T(0))) *ma.nanflag = 1;
      }
    }
    __syncthreads();
    // ---- G over another; the last step's populations go to memory
    {
      const int mg = 3 * t + 2, rows = th + 2 * (H - mg);
      const bool xin = lx >= mg && lx < tw + 2 * H - mg;
      for (int row = lr; row < rows; row += RPP) {
        if (!xin) continue;
        const NFLBM_CONST MobParams<T>& M = *fresh_const(M0);
        T* own = sm + (row + mg) * RS + lx;
        T p0[NC], grad[NC][2], c[NC], c2[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
          p0[j] = own[(oP + j) * W];
          c[j] = own[j * W];
          c2[j] = c[j] * c[j];
          grad[j][0] = grad[j][1] = T(0);
        }
#pragma unroll
        for (int k = 1; k < Q; ++k) {
          const T* src = own + L::e[k][1] * RS + L::e[k][0];
          const T wk = static_cast<T>(L::w[k]);
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const T d = wk * (src[(oP + j) * W] - p0[j]);
#pragma unroll
            for (int e = 0; e < 2; ++e)
              if (L::e[k][e] != 0) grad[j][e] = (L::e[k][e] > 0) ? grad[j][e] + d : grad[j][e] - d;
          }
        }
#pragma unroll
        for (int j = 0; j < NC; ++j)
#pragma unroll
          for (int e = 0; e < 2; ++e) grad[j][e] *= T(3);
        T G[NE][3];
#pragma unroll
        for (int i = 0; i < NE; ++i) {
          T aii = T(0), acc[2] = {T(0), T(0)};
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            if (j == i) continue;
            const T aij = c2[i] * c2[j];
            aii -= aij;
#pragma unroll
            for (int e = 0; e < 2; ++e) acc[e] = fma(aij, grad[j][e], acc[e]);
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) G[i][e] = M.pre[i] * fma(aii, grad[i][e], acc[e]);
          G[i][2] = T(0);
        }
        T moved[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) moved[i] = T(0);
        const uint32_t node = uint32_t(x0 + lx - H) + nx * uint32_t(y0 + row);   // of the last step
#pragma unroll
        for (int k = 1; k < Q; ++k) {
          const T wk = static_cast<T>(L::w[k]);
          FS v[NE];
#pragma unroll
          for (int i = 0; i < NE; ++i) {
            // the general path adds the source to the population its update
            // left, a zero: a source of -0 is stored as +0
            v[i] = S::pack(T(0) + wk * proj<L>(k, G[i]));
            moved[i] += S::unpack(v[i]);
          }
          if (last) vst<FS, NE>(at(static_cast<FS*>(ma.gk_dst) + size_t(k - 1) * gst, node * NE), v);
        }
        G0S r0[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) r0[i] = static_cast<G0S>(c[i] - moved[i]);
        if (last) {
          vst<G0S, NE>(at(static_cast<G0S*>(ma.g0_dst), node * NE), r0);
        } else {
#pragma unroll
          for (int i = 0; i < NE; ++i) {
            own[(oG + 2 * i) * W] = G[i][0];
            own[(oG + 2 * i + 1) * W] = G[i][1];
            own[(oR + i) * W] = static_cast<T>(r0[i]);
          }
        }
      }
    }
    if (!last) __syncthreads();
  }
}

#define FUSED_CAT2(a, b) a##b
#define FUSED_CAT(a, b) FUSED_CAT2(a, b)
// One translation unit per storage precision (NFLBM_UNIT_STORE).
hipError_t FUSED_CAT(launch_fused_mob_, NFLBM_UNIT_STORE)(int nc, const FusedMobArgs& a, int blocks, int nsteps,
                                                          uint32_t nanmask, size_t lds, hipStream_t s) {
  constexpr int ST = NFLBM_UNIT_STORE;
#define FUSED_MOB(N_) \
  case N_: hipLaunchKernelGGL((k_fused_mob<N_, ST>), dim3(blocks), dim3(512), lds, s, a, nsteps, nanmask); break;
  switch (nc) {
    FUSED_MOB(2)
    FUSED_MOB(3)
    FUSED_MOB(4)
    FUSED_MOB(5)
    FUSED_MOB(6)
    FUSED_MOB(7)
    FUSED_MOB(8)
    default: return hipErrorInvalidValue;
  }
#undef FUSED_MOB
  return hipGetLastError();
}

}  // namespace nflbm
