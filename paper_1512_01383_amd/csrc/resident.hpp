// resident.hpp -- many iterations of the fused primal-dual step (pdhg_iter.hip) in one
// launch, with the whole state on chip.
//
// A problem whose state fits the registers and LDS of the chip does not have to stream it
// through memory once per iteration: every block owns one tile of 64 x TH pixels for the
// whole launch, every thread CH labels of one pixel, and only the rim of each tile travels
// between blocks. That takes away the launch, the loads and stores of 14 planes per label
// and the waits on them. Measured, us per iteration, one launch per iteration -> on chip:
// ROF 64 x 64, L = 2: 5.0 -> 1.7; truncated quadratic 256 x 256, L = 5: 9.1 -> 4.2, L = 20:
// 17.8 -> 8.0; phase 256 x 256, L = 8: 8.5 -> 3.8; stereo 288 x 384, L = 8: 21.5 -> 13.6;
// ROF-like 512 x 500, L = 8, bf16 duals: 18.1 -> 9.3. What is left is bound by the vector
// unit (and on the smallest problems by the serial chain of one iteration: 1.1 us of it is
// the round trip of the rim, measured with no work around it).
//
// What a block needs from its neighbours is ubar on the rows above and below its tile, on
// the columns left and right of it and on two corners: p of the row above and of the column
// to the left is kept twice (by its owner and by the neighbour that needs it in div p) and
// advanced with the same expression, so it never travels. ubar of the rim goes through
// memory as 64-bit words (value, tag) with the tag naming the iteration: one relaxed
// device-scope store and load per value, no fence and no flag, and a word is either the
// wanted iteration's or it is polled again. Two slots per value in turn are enough: a block
// writes slot n + 2 after it has read its neighbours' n + 1, which they wrote after they
// had read its n. The pointwise part of an iteration (the epigraph projections, most of the
// arithmetic) comes first and hides the exchange; the neighbours' values enter with p.
//
// The wait ends because all blocks are on the chip at the same time (a cooperative launch)
// and each publishes before it waits; should it last longer than kWaitTicks all the same,
// the wave stops waiting for the rest of the launch and raises the error word.
//
// Labels are walked, summed and rounded as the one-pass kernel does with G label groups
// (G = LG groups per thread times the groups of the block), so the iterates are bitwise
// those of the one-pass kernel in the problem's tiling.
#pragma once

#include "device_math.hpp"
#include "internal.hpp"

namespace resident {

constexpr unsigned long long kWaitTicks = 2000000000ull;   // 20 s of the 100 MHz clock

__device__ __forceinline__ float rdlane(float x, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
// x of the next lane (lane 63 takes `last`), x of the previous lane (lane 0 takes `first`)
__device__ __forceinline__ float from_right(float x, float last) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, last),
                                                               __builtin_bit_cast(int, x), 0x130, 0xF, 0xF, false));
}
__device__ __forceinline__ float from_left(float x, float first) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, first),
                                                               __builtin_bit_cast(int, x), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ float round_bf16(float x) { return __uint_as_float((uint32_t)f2bf(x) << 16); }

typedef unsigned long long u64;
// a rim word at a wave-uniform address plus a lane's byte offset
__device__ __forceinline__ void put(char *base, unsigned off, float x, unsigned tag) {
  __hip_atomic_store((u64 *)(base + off), ((u64)tag << 32) | __float_as_uint(x), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 get(const char *base, unsigned off) {
  return __hip_atomic_load((const u64 *)(base + off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS: fixed strides, so that a label's place is an instruction offset from one address
constexpr int LS = 1024;   // threads of the largest block: stride of a label's own values
// one row of 64 pixels for each group of threads (4 / LG at most: there are at most 4 label groups)
constexpr int row_stride(int lg) { return 256 / lg; }
// LDS of a block: ubar, sbar, p_y (with the row above the tile), p of the row above, group
// sums; for truncated quadratics also w, centres, straddle words and the two lists
constexpr size_t lds_bytes(int piece, int ch, int lg, int G, int TH) {
  return sizeof(float) * ((size_t)ch * (3 * LS + 3 * row_stride(lg)) + (size_t)2 * G * 64 * TH +
                          (piece == SLI_TRUNC ? (size_t)ch * LS + 2 * LS + (size_t)ch * LS / 2 + LS : 0));
}

// barrier that orders LDS only: rim words and loads in flight stay in flight across it (the
// plain barrier waits for every store's acknowledgement from memory)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ float uniform(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

// PIECE, ADD: as in the one-pass kernel. CH labels per thread in LG label groups of CH / LG.
//
// An iteration of a thread, with its barriers:
//   s from the partial update and the earlier groups' v, sbar, sums of h sbar       | 1
//   q, the data-term duals' points before their projection
//   (truncated quadratics: into LDS | 2, the points in the band and on its edges from lists | 3)
//   projections, partial s, sums of v; p                                             | 4
//   div p, u, ubar, rim out
// For truncated quadratics p comes between 2 and 3, and 4 follows u.
//
// Truncated quadratics: of a pixel's labels a few lie in the band (quadratic pieces) and at
// most two straddle its edges (hulls of samples); the rest is the constant piece. Which is
// which never changes, so a block lists its quadratic and its straddling (label, pixel) pairs
// once, and its wavefronts walk the lists 64 pairs at a time. Walked label by label instead,
// nearly every wavefront has some lane in every class and pays for all three (256 x 256, L =
// 20: 11.5 us per iteration label by label and with plain barriers, 8.0 with the lists and
// barriers for LDS alone).
template <int PIECE, bool ADD, int CH, int LG>
__global__ __launch_bounds__(1024) void pdhg_resident_kernel(ResidentArgs R) {
  static_assert(CH % LG == 0 && CH <= 16, "labels per thread");
  constexpr int CN = CH / LG;   // labels of a label group
  constexpr int LH = row_stride(LG), LP = LS + LH;
  constexpr bool LIST = PIECE == SLI_TRUNC;
  // the rim is requested before the projections where its words in flight fit the registers
  constexpr bool EARLY = CH <= 2;
  extern __shared__ float lds[];
  __shared__ int lcount[2];                        // lengths of the lists
  __shared__ float4 ltab[LIST ? SLI_MAXK : 1];     // g0, g1, 1/(1+g0^2), 1/(1+g1^2) per label
  const int H = R.H, W = R.W, k = R.k, TH = R.TH, NP = 64 * TH, G = R.G;
  const long long ps = R.ps;
  const int tx = (int)threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // label groups of this wave, its row of the tile: rows turned by the group, so that the
  // tile's first rows (which have two rows' p to do) are not all on the same SIMD
  const int gp = wave / TH, ty = (wave + gp) % TH;
  const int tid = gp * NP + ty * 64 + tx;
  const int i0 = gp * CH, n = min(CH, k - i0);     // the thread's labels i0 .. i0 + n - 1 (n may be <= 0)

  float *const lub = lds + tid;                    // [CH][LS] ubar of the thread's labels
  float *const lsb = lub + CH * LS;                // [CH][LS] sbar; then y of the listed points; then the partial s
  float *const lpy = lds + 2 * CH * LS + gp * (NP + 64) + 64 + ty * 64 + tx;   // [CH][LP] new py; 64 before it the row above's
  float *const lhx = lds + 2 * CH * LS + CH * LP + gp * 64 + tx;               // [CH][LH] px, py of the row above the tile
  float *const lhy = lhx + CH * LH;
  float *const exa = lds + 2 * CH * LS + CH * LP + 2 * CH * LH + ty * 64 + tx;   // [G][NP] sums of h sbar, [G][NP] sums of v
  float *const exb = exa + G * NP;
  float *const lists = lds + 2 * CH * LS + CH * LP + 2 * CH * LH + 2 * G * NP;   // LIST only:
  float *const lw = lists + tid;                               // [CH][LS] w of the listed points
  float *const lfc = lists + CH * LS;                          // [LS] data centre of each thread's pixel
  unsigned *const lin = (unsigned *)(lfc + LS);                // [LS] its straddle word, gp in the top bits
  uint16_t *const lq = (uint16_t *)(lin + LS);                 // [CH][LS] quadratic points: label of the thread * LS + thread
  uint16_t *const lc = lq + CH * LS;                           // [2][LS] straddling points

  const int ntc = (W + 63) / 64;
  const int tile = (int)blockIdx.x, tr = tile / ntc, tc = tile - tr * ntc;
  const int r0 = tr * TH, c0 = tc * 64;
  const int r = r0 + ty, c = c0 + tx;
  const bool on = r < H && n > 0;                  // uniform in the wave: it has work
  const bool in = r < H && c < W;
  const unsigned x = in ? (unsigned)(r * W + c) : 0u, xb = x * 4u;
  const bool top = on && ty == 0 && r0 > 0, bottom = on && ty == TH - 1 && r < H - 1;
  const bool halo = top || bottom;                 // a row of ubar beyond the tile enters
  const int deg = (c < W - 1) + (c > 0) + (r < H - 1) + (r > 0);
  const float tau_u = R.tau_c / (1.f + (float)deg);
  // differences across the image's border are zero: the factor 0 or 1 goes into the step
  const float mr_ = c < W - 1 ? 1.f : 0.f, ml_ = c > 0 ? 1.f : 0.f, md_ = r < H - 1 ? 1.f : 0.f, mu_ = r > 0 ? 1.f : 0.f;
  const bool aniso = R.aniso != 0, bf16 = R.bf16 != 0;

  // exchange: per tile and label 64 words of the first row, 64 of the last, TH of the first
  // and TH of the last column
  const int exw = 128 + 2 * TH;
  const unsigned exs = 8u * gridDim.x * k * exw;   // bytes of a slot
  auto at = [&](int trr, int tcc, int i, int word) { return 8u * (unsigned)(((trr * ntc + tcc) * k + i) * exw + word); };
  // one word per lane for the edges: lanes 0-15 ubar(r, c0-1), 16-31 ubar(r+1, c0-1), 32-47
  // ubar(r, c0+64), 48-63 ubar(r0-1, c0+64), each of label i0 + (lane & 15)
  const int el = tx & 15, es = tx >> 4;
  bool ev = on && el < n;
  unsigned eo = 0;
  if (ev) {
    const int i = i0 + el;
    if (es == 0) {
      ev = c0 > 0;
      if (ev) eo = at(tr, tc - 1, i, 128 + TH + ty);
    } else if (es == 1) {
      ev = c0 > 0 && r + 1 < H;
      if (ev) eo = ty + 1 < TH ? at(tr, tc - 1, i, 128 + TH + ty + 1) : at(tr + 1, tc - 1, i, 128 + TH);
    } else if (es == 2) {
      ev = c0 + 64 < W;
      if (ev) eo = at(tr, tc + 1, i, 128 + ty);
    } else {
      ev = top && c0 + 64 < W;
      if (ev) eo = at(tr - 1, tc + 1, i, 128 + TH - 1);
    }
  }
  const unsigned hrow = top ? at(tr - 1, tc, i0, 64) : bottom ? at(tr + 1, tc, i0, 0) : 0u;   // row beyond the tile
  char *const mine = (char *)R.ex + at(tr, tc, on ? i0 : 0, 0);
  const unsigned txo = 8u * (unsigned)tx;
  const unsigned hxo = 8u * (unsigned)min(tx, W - 1 - c0);   // lanes past the image wait for its last pixel's

  // ---- the state
  float u[CH], s[CH], v[CH], z[CH], px[CH];
  const float *vf = (const float *)R.v, *zf = (const float *)R.z, *pf = (const float *)R.p;
  const uint16_t *vh = (const uint16_t *)R.v, *zh = (const uint16_t *)R.z, *ph = (const uint16_t *)R.p;
  auto ldp = [&](long long o) { return bf16 ? ldv(ph, o) : pf[o]; };
#pragma unroll
  for (int j = 0; j < CH; j++) {
    u[j] = s[j] = v[j] = z[j] = px[j] = 0.f;
    float ub = 0.f, sb = 0.f, py = 0.f, hx = 0.f, hy = 0.f;
    const long long o = (long long)(i0 + j) * ps + x, oy = (long long)(k + i0 + j) * ps + x;
    if (in && j < n) {
      u[j] = R.u[o];
      ub = 2.f * u[j] - R.up[o];
      s[j] = R.s[o];
      sb = 2.f * s[j] - R.sp[o];
      v[j] = bf16 ? ldv(vh, o) : vf[o];
      z[j] = bf16 ? ldv(zh, o) : zf[o];
      px[j] = ldp(o);
      py = ldp(oy);
      if (top) {
        hx = ldp(o - W);
        hy = ldp(oy - W);
      }
    }
    lub[j * LS] = ub;
    lsb[j * LS] = sb;
    lpy[j * LP] = py;
    if (ty == 0) {
      lpy[j * LP - 64] = 0.f;   // above the image: times zero in div p
      lhx[j * LH] = hx;
      lhy[j * LH] = hy;
    }
  }
  float q = in ? R.q[x] : 0.f;
  float fc = PIECE != SLI_SAMPLED && in ? R.fn[x] : 0.f, lam = uniform(R.lam);
  // p left of the tile, label i0 + lane
  float pxL = 0.f, pyL = 0.f, radL = 0.f;
  const bool left = on && c0 > 0;
  if (left && tx < n) {
    const long long o = (long long)(i0 + tx) * ps + (long long)r * W + c0 - 1;
    pxL = ldp(o);
    pyL = ldp(o + (long long)k * ps);
    radL = R.lam * R.lab[i0 + tx].h;
  }
  bool listed[CH];
  if (LIST) {
    if (threadIdx.x < 2) lcount[threadIdx.x] = 0;
    if ((int)threadIdx.x < k) {
      const ResidentLabel &B = R.lab[threadIdx.x];
      ltab[threadIdx.x] = make_float4(B.g0, B.g1, B.ig0, B.ig1);
    }
    const unsigned info = in ? R.sinfo[x] : 31u | (31u << 13);
    lfc[tid] = fc;
    lin[tid] = (info & 0x3FFFFFFu) | ((unsigned)gp << 26);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < CH; j++) {
      const int i = i0 + j;
      const bool str = in && j < n && (i == (int)(info & 31u) || i == (int)((info >> 13) & 31u));
      const bool quad = in && j < n && !str && fc - R.del <= R.lab[i].g0 && R.lab[i].g1 <= fc + R.del;
      listed[j] = str || quad;
      for (int l = 0; l < 2; l++) {
        const bool mem = l == 0 ? quad : str;
        const u64 m = __ballot(mem);
        if (m == 0) continue;
        int base = 0;
        if (tx == 0) base = atomicAdd(&lcount[l], __popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
        if (mem) (l == 0 ? lq : lc)[base + __popcll(m & ((1ull << tx) - 1ull))] = (uint16_t)(j * LS + tid);
      }
    }
  }

  // the rim's ubar out: the row's words if it is the tile's first or last, and by lanes 0 and
  // 63 the first and last column's
  const bool pe = in && ((tx == 0 && c0 > 0) || (tx == 63 && c < W - 1));
  const bool pe_any = on && (c0 > 0 || c0 + 64 < W);
  const unsigned peo = 8u * (unsigned)(128 + (tx == 0 ? 0 : TH) + ty);
  auto publish = [&](unsigned tag) {
    char *const slot = mine + (tag & 1u) * exs;
    if (halo) {
      if (in) {
#pragma unroll
        for (int j = 0; j < CH; j++)
          if (j < n) put(slot + (top ? 0u : 512u) + 8u * (unsigned)(j * exw), txo, lub[j * LS], tag);
      }
    }
    if (pe_any) {
      if (pe) {
#pragma unroll
        for (int j = 0; j < CH; j++)
          if (j < n) put(slot + 8u * (unsigned)(j * exw), peo, lub[j * LS], tag);
      }
    }
  };
  __syncthreads();   // every value of the neighbours' state has been read before the first word goes out
  const int nq = LIST ? __builtin_amdgcn_readfirstlane(lcount[0]) : 0;
  const int nc = LIST ? __builtin_amdgcn_readfirstlane(lcount[1]) : 0;
  const int bc = (nc + 63) / 64, batches = bc + (nq + 63) / 64, waves = (int)blockDim.x >> 6;
  publish(R.tag);

  bool dead = false;
#pragma unroll 1
  for (int it = 1; it <= R.iters; it++) {
    // values of one label or pixel that no iteration changes are formed where they are used:
    // hoisted out of the loop by the compiler they would take a register each and spill
    int ii = i0;
    asm volatile("" : "+v"(fc), "+s"(lam), "+s"(ii));
    // past the last label (j >= n) a thread works on zeros: h and the steps are 0 there, and
    // so every sum's share, and nothing is stored
    const ResidentLabel *const lab = R.lab + ii;
    // ---- sums of h sbar per label group
#pragma unroll
    for (int g = 0; g < LG; g++) {
      float Tc = 0.f;
#pragma unroll
      for (int jj = 0; jj < CN; jj++) Tc += lab[g * CN + jj].h * lsb[(g * CN + jj) * LS];
      exa[(gp * LG + g) * NP] = Tc;
    }
    lds_barrier();
    // the rim of the previous iteration: requested here, looked at when p is due
    const unsigned tag = R.tag + (unsigned)(it - 1);
    const char *const slot = (const char *)R.ex + (tag & 1u) * exs;
    u64 hw[CH], ew = 0;
    auto request = [&]() {
      if (ev) ew = get(slot, eo);
      if (halo) {
#pragma unroll
        for (int j = 0; j < CH; j++) hw[j] = get(slot + hrow + 8u * (unsigned)(min(j, n - 1) * exw), hxo);
      }
    };
    if (EARLY) request();
    float pl = 0.f;   // new px left of the tile, label i0 + lane
    auto p_update = [&]() {
      u64 t0 = 0;
      if (!EARLY) request();
      while (true) {
        unsigned wrong = ev ? (unsigned)(ew >> 32) ^ tag : 0u;
        if (halo) {
#pragma unroll
          for (int j = 0; j < CH; j++) wrong |= (unsigned)(hw[j] >> 32) ^ tag;
        }
        if (dead || !__any(wrong != 0u)) break;
        const u64 now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 > kWaitTicks) {
          dead = true;
          *R.err = 1u;
        }
        request();
      }
      const float eub = __uint_as_float((unsigned)ew);
      // p: own, of the row above the tile and of the column left of it
      if (left) {
        const float own = tx < n ? lub[tx * LS - tx] : 0.f;
        const float dn = __shfl(eub, (tx & 15) + 16);
        pl = pxL;
        float py = pyL;
        p_step(pl, py, R.sig_p, own - eub, (r < H - 1) ? dn - eub : 0.f, radL, aniso);
        pxL = bf16 ? round_bf16(pl) : pl;
        pyL = bf16 ? round_bf16(py) : py;
      }
      if (bf16) {   // p_y as it is stored; div p of the previous iteration took it unrounded
#pragma unroll
        for (int j = 0; j < CH; j++) lpy[j * LP] = round_bf16(lpy[j * LP]);
      }
      const float spx = R.sig_p * mr_, spy = R.sig_p * md_;
#pragma unroll
      for (int j = 0; j < CH; j++) {
        const float rad = lam * lab[j].h, hub = halo && j < n ? __uint_as_float((unsigned)hw[j]) : 0.f;
        const float ub = lub[j * LS];
        const float ubr = from_right(ub, rdlane(eub, 32 + j));
        const float ubd = ty + 1 < TH ? lub[j * LS + 64] : hub;
        float py = lpy[j * LP];
        px[j] = px[j] + spx * (ubr - ub);
        py = py + spy * (ubd - ub);
        proj_K(px[j], py, rad, aniso);
        lpy[j * LP] = py;
        if (top) {
          const float ubur = from_right(hub, rdlane(eub, 48 + j));
          float hx = lhx[j * LH], hy = lhy[j * LH];
          hx = hx + spx * (ubur - hub);
          hy = hy + R.sig_p * (ub - hub);
          proj_K(hx, hy, rad, aniso);
          lpy[j * LP - 64] = hy;
          lhx[j * LH] = hx;
          lhy[j * LH] = hy;
        }
      }
      if (bf16 && top) {
#pragma unroll
        for (int j = 0; j < CH; j++) {
          lhx[j * LH] = round_bf16(lhx[j * LH]);
          lhy[j * LH] = round_bf16(lhy[j * LH]);
        }
      }
    };
    float wlo[ADD ? CH + 1 : 1];   // additive values at the thread's labels
    if (on) {
      float T = 0.f;
      for (int g = 0; g < G; g++) T += exa[g * NP];
      q = q - R.sig_q * (1.f + T);
      if (ADD) {
#pragma unroll
        for (int j = 0; j <= CH; j++) wlo[ADD ? j : 0] = in ? ldb(R.wadd + (long long)min(i0 + j, k) * ps, xb) : 0.f;
      }
      // ---- data-term duals before their projection, over h
#pragma unroll
      for (int g = 0; g < LG; g++) {
        float base = 0.f;
        for (int gg = gp * LG + g + 1; gg < G; gg++) base += exa[gg * NP];
        float suf = base + exa[(gp * LG + g) * NP];
#pragma unroll
        for (int jj = 0; jj < CN; jj++) {
          const int j = g * CN + jj;
          const float sb = lsb[j * LS], ub = lub[j * LS];
          suf -= lab[j].h * sb;
          const float ve = v[j] + lab[j].sig * (ub + suf - lab[j].g0 * sb);
          const float ze = z[j] + lab[j].sig * sb;
          float y = ve * lab[j].ih, w = ze * lab[j].ih;
          if (ADD) {
            const float bs = (wlo[ADD ? j + 1 : 0] - wlo[ADD ? j : 0]) * lab[j].ih;
            y -= bs;
            w -= -wlo[ADD ? j : 0] + bs * lab[j].g0;
          }
          if (LIST) {
            lsb[j * LS] = y;
            lw[j * LS] = w;
            proj_flat(R.nu, lab[j].g0, lab[j].g1, lab[j].ig0, lab[j].ig1, y, w);
          }
          v[j] = y;
          z[j] = w;
        }
      }
    }
    if (LIST) {
      lds_barrier();
      for (int b = wave; b < batches; b += waves) {
        const bool hull = b < bc;
        const int e = (hull ? b : b - bc) * 64 + tx;
        if (e < (hull ? nc : nq)) {
          const int at = (int)(hull ? lc : lq)[e], who = at & (LS - 1);
          const unsigned info = lin[who];
          const int i = (int)(info >> 26) * CH + at / LS;
          const float4 g = ltab[i];
          const float f = lfc[who];
          float *const py = lds + CH * LS + at, *const pw = lists + at;
          float y = *py, w = *pw;
          if (hull) {
            const unsigned m = info >> ((int)(info & 31u) == i ? 0 : 13);
            proj_tq_chain(R.a, f, R.nu, g.x, g.y, (int)((m >> 5) & 15u), (int)((m >> 9) & 15u), y, w);
          } else {
            proj_quad(R.a, R.ia, f, g.x, g.y, g.z, g.w, y, w);
          }
          *py = y;
          *pw = w;
        }
      }
      if (on) p_update();
      lds_barrier();
    }
    if (on) {
      // ---- projections, partial s
      float pre = 0.f, rlast = 0.f;
#pragma unroll
      for (int j = 0; j < CH; j++) {
        if (LG > 1 && j > 0 && j % CN == 0) {
          exb[(gp * LG + j / CN - 1) * NP] = pre;
          pre = 0.f;
        }
        float y = v[j], w = z[j];
        if (PIECE == SLI_QUAD) {
          proj_quad(R.a, R.ia, piece_centre(fc, lab[j].g0, lab[j].g1, R.per, R.iper), lab[j].g0, lab[j].g1, lab[j].ig0,
                    lab[j].ig1, y, w);
        } else if (LIST) {
          const float yl = lsb[j * LS], wl = lw[j * LS];
          y = listed[j] ? yl : y;
          w = listed[j] ? wl : w;
        } else if (j < n) {
          const int m0 = __builtin_amdgcn_readfirstlane(R.sidx[i0 + j]);
          const int m1 = __builtin_amdgcn_readfirstlane(R.sidx[i0 + j + 1]);
          auto cost = [&](int m) { return ldb(R.cost + (long long)m * ps, xb); };
          PLScan pl;
          pl.init(y, w);
          pl.push(ldtab(R.tau, m0), j > 0 ? rlast : cost(m0));
          for (int mb = m0 + 1; mb <= m1; mb += 8) {
            float rr[8];
            float4 tq[8];
#pragma unroll
            for (int e = 0; e < 8; e++) {
              rr[e] = cost(min(mb + e, m1));
              tq[e] = ldtab(R.tau, min(mb + e, m1));
            }
#pragma unroll
            for (int e = 0; e < 8; e++)
              if (mb + e <= m1) pl.push(tq[e], rr[e]);
          }
          rlast = pl.cp;
          if (pl.finish(y, w)) {   // rare: no region holds the point (rounding)
            PLNear nn;
            nn.init(y, w);
            for (int m = m0; m <= m1; m++) nn.push(ldtab(R.tau, m), cost(m));
            nn.finish(y, w);
          }
        }
        if (ADD) {
          const float bs = (wlo[ADD ? j + 1 : 0] - wlo[ADD ? j : 0]) * lab[j].ih;
          y += bs;
          w += -wlo[ADD ? j : 0] + bs * lab[j].g0;
        }
        v[j] = lab[j].h * y;
        z[j] = lab[j].h * w;
        lsb[j * LS] = s[j] - lab[j].taus * (z[j] - lab[j].h * q + lab[j].h * pre - lab[j].g0 * v[j]);
        pre += v[j];
      }
      exb[(gp * LG + LG - 1) * NP] = pre;
      if (!LIST) p_update();
    }
    if (!LIST) lds_barrier();
    const bool last = it == R.iters;
    if (on) {
      // ---- u and ubar (after the last iteration u_prev in ubar's place, for the way out)
#pragma unroll
      for (int j = 0; j < CH; j++) {
        const float pxl = from_left(px[j], rdlane(pl, j));
        float dv = mr_ * px[j];
        dv -= ml_ * pxl;
        dv += md_ * lpy[j * LP];
        dv -= mu_ * lpy[j * LP - 64];
        const float un = u[j] - tau_u * (v[j] - dv);
        lub[j * LS] = last ? u[j] : 2.f * un - u[j];
        u[j] = un;
      }
      if (!last) publish(R.tag + (unsigned)it);
      if (bf16) {
#pragma unroll
        for (int j = 0; j < CH; j++) {
          v[j] = round_bf16(v[j]);
          z[j] = round_bf16(z[j]);
          px[j] = round_bf16(px[j]);
        }
      }
    }
    if (LIST) lds_barrier();
    if (on) {
      // ---- s with the earlier groups' v, and sbar
#pragma unroll
      for (int g = 0; g < LG; g++) {
        float vb = 0.f;
        for (int gg = 0; gg < gp * LG + g; gg++) vb += exb[gg * NP];
#pragma unroll
        for (int jj = 0; jj < CN; jj++) {
          const int j = g * CN + jj;
          float sn = lsb[j * LS];
          if (G > 1) sn = sn - lab[j].taus * (lab[j].h * vb);
          lsb[j * LS] = last ? s[j] : 2.f * sn - s[j];
          s[j] = sn;
        }
      }
    }
  }

  // ---- the state back to memory (after a wait that was given up: no state, but NaN)
  if (dead) {
#pragma unroll
    for (int j = 0; j < CH; j++) u[j] = __builtin_nanf("");
  }
  if (in) {
    float *vo = (float *)R.vo, *zo = (float *)R.zo, *po = (float *)R.po;
    uint16_t *voh = (uint16_t *)R.vo, *zoh = (uint16_t *)R.zo, *poh = (uint16_t *)R.po;
#pragma unroll
    for (int j = 0; j < CH; j++) {
      if (j >= n) continue;
      const long long o = (long long)(i0 + j) * ps + x, oy = (long long)(k + i0 + j) * ps + x;
      const float py = lpy[j * LP];
      R.uo[o] = u[j];
      R.upo[o] = lub[j * LS];
      R.so[o] = s[j];
      R.spo[o] = lsb[j * LS];
      if (bf16) {
        stv(voh, o, v[j]);
        stv(zoh, o, z[j]);
        stv(poh, o, px[j]);
        stv(poh, oy, py);
      } else {
        vo[o] = v[j];
        zo[o] = z[j];
        po[o] = px[j];
        po[oy] = py;
      }
    }
    if (gp == 0) R.qo[x] = q;
  }
}

// labels per thread and label groups per thread that are built: every chunk length up to 9
// with one group per thread, and the chunks of two or four groups that a thread takes
// together when the image has too many tiles for a wavefront per group
template <int PIECE, bool ADD>
inline const void *kernel_of(int ch, int lg) {
#define SLI_RES(C, L) \
  if (ch == C && lg == L) return (const void *)pdhg_resident_kernel<PIECE, ADD, C, L>
  SLI_RES(1, 1);
  SLI_RES(2, 1);
  SLI_RES(3, 1);
  SLI_RES(4, 1);
  SLI_RES(5, 1);
  SLI_RES(6, 1);
  SLI_RES(7, 1);
  SLI_RES(8, 1);
  SLI_RES(9, 1);
  SLI_RES(2, 2);
  SLI_RES(4, 2);
  SLI_RES(6, 2);
  SLI_RES(8, 2);
  SLI_RES(10, 2);
  SLI_RES(4, 4);
  SLI_RES(8, 4);
#undef SLI_RES
  return nullptr;
}

}  // namespace resident
