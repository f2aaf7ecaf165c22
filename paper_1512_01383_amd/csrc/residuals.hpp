// residuals.hpp -- device bodies of the residual pass (steps.hip), also run as a part of the
// check's launches (aux.hip)
#pragma once

#include "device_math.hpp"
#include "internal.hpp"

namespace {

constexpr int RB = 256;

template <typename DT>
__device__ __forceinline__ void residuals_body(const ResPtrs &R, const IterArgs &A, long long blk, long long nblk) {
  __shared__ double sp_[RB], sd_[RB], sx_[RB], sy_[RB];
  const DT *v = (const DT *)R.v, *z = (const DT *)R.z, *vo = (const DT *)R.vo, *zo = (const DT *)R.zo;
  const DT *p = (const DT *)R.p, *po = (const DT *)R.po;
  const int H = A.H, W = A.W, k = A.k;
  const long long ps = A.ps, N = (long long)H * W;
  double accp = 0.0, accd = 0.0, acckx = 0.0, accky = 0.0;
  // steps enter as reciprocals: one division per step instead of one per residual entry
  const float isig_p = 1.f / A.sig_p;
  for (long long x = blk * RB + threadIdx.x; x < N; x += nblk * RB) {
    const int r = (int)(x / W), c = (int)(x - (long long)r * W);
    const bool hr = c < W - 1, hl = c > 0, hd = r < H - 1, hu = r > 0;
    const int deg = hr + hl + hd + hu;
    const float itau_u = (1.f + (float)deg) / A.tau_c;
    float T = 0.f;
    for (int i = 0; i < k; i++) {
      const size_t o = (size_t)i * ps;
      T += A.h[i] * (R.sp[o + x] - R.s[o + x]);
    }
    const float dq = R.qo[x] - R.q[x];
    float suf = T, pre = 0.f;
    for (int i = 0; i < k; i++) {
      const size_t o = (size_t)i * ps, oy = (size_t)(k + i) * ps;
      const float du = R.up[o + x] - R.u[o + x];
      const float ds = R.sp[o + x] - R.s[o + x];
      const float dv = ldv(vo, o + x) - ldv(v, o + x);
      const float dz = ldv(zo, o + x) - ldv(z, o + x);
      const float dpx = ldv(po, o + x) - ldv(p, o + x);
      const float dpy = ldv(po, oy + x) - ldv(p, oy + x);
      float div = 0.f;
      if (hr) div += dpx;
      if (hl) div -= ldv(po, o + x - 1) - ldv(p, o + x - 1);
      if (hd) div += dpy;
      if (hu) div -= ldv(po, oy + x - W) - ldv(p, oy + x - W);
      const float gx = hr ? (R.up[o + x + 1] - R.u[o + x + 1]) - du : 0.f;
      const float gy = hd ? (R.up[o + x + W] - R.u[o + x + W]) - du : 0.f;
      suf -= A.h[i] * ds;
      const float itaus = 1.f / A.taus[i], isig = 1.f / A.sig[i];
      const float rpu = du * itau_u - (dv - div);
      const float rps = ds * itaus - (dz - A.h[i] * dq + A.h[i] * pre - A.gam[i] * dv);
      pre += dv;
      const float rdv = dv * isig - (du - A.gam[i] * ds + suf);
      const float rdz = dz * isig - ds;
      const float rdx = dpx * isig_p - gx, rdy = dpy * isig_p - gy;
      accp += (double)fabsf(rpu) + (double)fabsf(rps);
      accd += (double)fabsf(rdv) + (double)fabsf(rdz) + (double)fabsf(rdx) + (double)fabsf(rdy);
      // the variables at the new iterate: x = (u, s), y = (v, z, p, q)
      acckx += (double)fabsf(R.u[o + x]) + (double)fabsf(R.s[o + x]);
      accky += (double)fabsf(ldv(v, o + x)) + (double)fabsf(ldv(z, o + x)) + (double)fabsf(ldv(p, o + x)) +
               (double)fabsf(ldv(p, oy + x));
    }
    accd += (double)fabsf(dq * (1.f / A.sig_q) + T);
    accky += (double)fabsf(R.q[x]);
  }
  sp_[threadIdx.x] = accp;
  sd_[threadIdx.x] = accd;
  sx_[threadIdx.x] = acckx;
  sy_[threadIdx.x] = accky;
  __syncthreads();
  for (int s = RB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sp_[threadIdx.x] += sp_[threadIdx.x + s];
      sd_[threadIdx.x] += sd_[threadIdx.x + s];
      sx_[threadIdx.x] += sx_[threadIdx.x + s];
      sy_[threadIdx.x] += sy_[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    R.part[4 * blk] = sp_[0];
    R.part[4 * blk + 1] = sd_[0];
    R.part[4 * blk + 2] = sy_[0];   // |y|, the scale of the primal residual
    R.part[4 * blk + 3] = sx_[0];   // |x|, the scale of the dual residual
  }
}

// block q (0..3) adds column q of the per-block quadruples, in block order
__device__ __forceinline__ void sum_quads_body(const double *part, int nb, double *out, int q) {
  __shared__ double a[RB];
  double x = 0.0;
  for (int j = threadIdx.x; j < nb; j += RB) x += part[4 * j + q];
  a[threadIdx.x] = x;
  __syncthreads();
  for (int s = RB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) a[threadIdx.x] += a[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[q] = a[0];
}
}  // namespace
