// resident.hpp -- many iterations of the fused primal-dual step (pdhg_iter.hip) in one
// launch, with the whole state on chip.
//
// A problem whose state fits the registers and LDS of the chip does not have to stream it
// through memory once per iteration: every block owns one tile of 64 x TH pixels for the
// whole launch, every thread CH labels of one pixel, and only the rim of each tile travels
// between blocks. That takes away the launch, the loads and stores of 14 planes per label
// and the waits on them. Measured, us per iteration, one launch per iteration -> on chip:
// ROF 64 x 64, L = 2: 5.0 -> 1.5, 1531 x 2039: 37 -> 19 (12 rows per thread); truncated
// quadratic 256 x 256, L = 5: 9.1 -> 3.3, L = 20: 17.8 -> 7.7, 353 x 517, L = 10 (anisotropic):
// 30 -> 16; phase 256 x 256, L = 8: 8.5 -> 3.6; stereo 288 x 384, L = 8: 21.5 -> 9.3. Of the time
// of these launches the vector unit is busy 74 % (256 x 256, L = 20), 59 % (353 x 517), 82 %
// (1531 x 2039) and 64 % (stereo); on the smallest problems it is the serial chain of one
// iteration (ROF 64 x 64: 24 %), of which 1.1 us is the round trip of the rim, measured with no
// work around it.
//
// A cooperative launch goes through a queue of its own: the first of a process takes 10 ms more,
// and launches of several streams run one after another. With many small problems on many
// streams that can be slower than single launches side by side (64 x 64, L = 20, us per
// iteration and problem: one stream 15.3 -> 6.2, eight streams 4.3 -> 6.0); a batch is the
// better way then. Plain launches would not do: two that each held part of the chip would wait
// for each other's blocks.
//
// 16 wavefronts a block leave 128 registers a lane. Whatever is not needed at once is kept out
// of them: planes go in and out one element after another, rim words are waited for four labels
// at a time, per-label constants are loaded in each section. With them held in registers the
// state spilled from 6 labels per thread on, and 10 labels (353 x 517, L = 10) ran at 30 us.
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
// and each publishes before it waits; should a wave have looked R.limit times in vain all the
// same, it raises the error word and stops waiting for the rest of the launch. (Looks, not
// time, so that a wave does not give up over time in which it was off the chip itself.) What
// it and its neighbours compute from then on is void: every reader of the state looks at the
// error word.
//
// Labels are walked, summed and rounded as the one-pass kernel does with G label groups
// (G = LG groups per thread times the groups of the block), so the iterates are bitwise
// those of the one-pass kernel in the problem's tiling.
#pragma once

#include "device_math.hpp"
#include "internal.hpp"

namespace resident {

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
// one row of 64 pixels for each of the `ph` groups of threads that a kernel is built for
constexpr int row_stride(int ph) { return 64 * ph; }
// LDS of a block of `phys` groups of threads: ubar, sbar, p_y (with the row above the tile), p of
// the row above, the label groups' sums where they are of several threads; for truncated
// quadratics the w of a pixel's `slots` listed labels, centres, straddle words and the lists
constexpr size_t lds_bytes(int piece, int ch, int lg, int rp, int ph, int G, int TH, int qmax, int slots) {
  const size_t e = (size_t)ch * rp, np = (size_t)64 * TH, lh = row_stride(ph);
  const size_t hulls = slots < 2 ? slots : 2;
  return sizeof(float) * (e * (3 * LS + lh) + 2 * ch * lh + (G > lg ? 2 * G * np : 0)) +
         (piece == SLI_TRUNC ? rp * (slots * np * 4 + LS * 8 + (qmax + hulls) * np * 2) + 16 : 0);
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
// For truncated quadratics p comes between 2 and 3, and 4 follows u. With one group of threads
// the sums stay with the thread: then 1 and 4 are not needed there.
//
// Truncated quadratics: of a pixel's labels a few lie in the band (quadratic pieces) and at
// most two straddle its edges (hulls of samples); the rest is the constant piece. Which is
// which never changes, so a block lists its quadratic and its straddling (label, pixel) pairs
// once, and its wavefronts walk the lists 64 pairs at a time. Walked label by label instead,
// nearly every wavefront has some lane in every class and pays for all three (353 x 517, L =
// 10: 29.5 us per iteration label by label, 16 with the lists). y of a listed point waits in
// its sbar's place, w in the slot of its place among the pixel's listed labels.
//
// RP > 1 (few labels, large images): a thread has its column's pixels in RP rows one below the
// other, all labels of each; element e = row * CH + label of the thread. One label group only.
// PH: most groups of threads in a block (the LDS strides follow it).
// KEEP: every state goes to memory as it is reached (the replay of the reverse pass). The stores
// follow the rim's, so the neighbours do not wait for them. 256x256, 7 labels: 5.3 us a state (5.0
// without the stores), 11.4 by the one-pass kernel.
template <int PIECE, bool ADD, int CH, int LG, int RP, int PH, bool KEEP = false>
__global__ __launch_bounds__(1024) void pdhg_resident_kernel(ResidentArgs R) {
  static_assert(CH % LG == 0 && CH * RP <= 16, "labels per thread");
  static_assert(RP == 1 || (LG == 1 && PH == 1 && !ADD && PIECE != SLI_SAMPLED), "rows per thread");
  constexpr int CN = CH / LG;   // labels of a label group
  constexpr int E = CH * RP;
  constexpr int LH = row_stride(PH), LP = LS + LH;
  constexpr bool LIST = PIECE == SLI_TRUNC;
  // the rim is requested before the projections where its words in flight fit the registers
  constexpr bool EARLY = CH <= 2 && E <= 4;
  // and in turns of HB labels where the words of all would not fit them
  constexpr int HB = CH <= 6 ? CH : 4;
  extern __shared__ float lds[];
  __shared__ int lcount[2];                        // lengths of the lists
  __shared__ float4 ltab[LIST ? SLI_MAXK : 1];     // g0, g1, 1/(1+g0^2), 1/(1+g1^2) per label
  const int H = R.H, W = R.W, k = R.k, TH = R.TH, TR = TH * RP, NP = 64 * TH, G = RP > 1 ? 1 : R.G;
  const long long ps = R.ps;
  const int tx = (int)threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // label groups of this wave, its row (its RP rows) of the tile: rows turned by the group, so that the
  // tile's first rows (which have two rows' p to do) are not all on the same SIMD
  const int gp = wave / TH, ty = (wave + gp) % TH;
  const int tid = gp * NP + ty * 64 + tx;
  const int i0 = gp * CH, n = min(CH, k - i0);     // the thread's labels i0 .. i0 + n - 1 (n may be <= 0)

  constexpr int OP = 2 * E * LS, OH = OP + E * LP, OX = OH + 2 * CH * LH;
  float *const lub = lds + tid;                    // [E][LS] ubar of the thread's elements
  float *const lsb = lub + E * LS;                 // [E][LS] sbar; then y of the listed points; then the partial s
  float *const lpy = lds + OP + gp * (NP + 64) + 64 + ty * 64 + tx;   // [E][LP] new py; 64 before it the row above's
  float *const lhx = lds + OH + gp * 64 + tx;      // [CH][LH] px, py of the row above the tile
  float *const lhy = lhx + CH * LH;
  const bool one = PH == 1 || G == LG;                        // one group of threads: the sums stay with the thread
  float *const exa = lds + OX + ty * 64 + tx;      // !one: [G][NP] sums of h sbar, [G][NP] sums of v
  float *const exb = exa + G * NP;
  // LIST only: per pixel of the tile (row rp of a thread: RP times as many)
  const int slots = R.slots, qmax = R.qmax;
  float *const lists = lds + OX + (one ? 0 : 2 * G * NP);
  float *const lw = lists + ty * 64 + tx;                      // [RP][slots][NP] w of a pixel's listed labels, in their order
  float *const lfc = lists + RP * slots * NP;                  // [RP][LS] data centre of each thread's pixels
  unsigned *const lin = (unsigned *)(lfc + RP * LS);           // [RP][LS] their hulls, see pack below
  uint16_t *const lq = (uint16_t *)(lin + RP * LS);            // [RP][qmax][NP] quadratic points: element * LS + thread
  uint16_t *const lc = lq + RP * qmax * NP;                    // [RP][min(2, slots)][NP] straddling points

  const int ntc = (W + 63) / 64;
  const int tile = (int)blockIdx.x, tr = tile / ntc, tc = tile - tr * ntc;
  const int r0 = tr * TR, c0 = tc * 64;
  const int r = r0 + ty * RP, c = c0 + tx;         // the thread's (first) row, its column
  const bool on = r < H && n > 0;                  // uniform in the wave: it has work
  const bool col = c < W, in = r < H && col;
  const unsigned x = in ? (unsigned)(r * W + c) : 0u, xb = x * 4u;
  // row rp of the thread is in the image: uniform in the wave, so that with `col` one lane mask
  // serves all rows (a mask per row, kept in spilled scalar registers, came back wrong once)
  auto row_in = [&](int rp) { return r + rp < H; };
  auto row_off = [&](int rp) { return RP == 1 ? xb : xb + 4u * (unsigned)(rp * W); };
  const bool top = on && ty == 0 && r0 > 0, bottom = on && ty == TH - 1 && r0 + TR < H;
  const bool halo = top || bottom;                 // a row of ubar beyond the tile enters
  const float dc = (float)((c < W - 1) + (c > 0));
  const float tau_mid = R.tau_c / (1.f + (dc + 2.f));                                     // rows inside the image
  const float tau_rim = RP == 1 ? R.tau_c / (1.f + (dc + (float)((r < H - 1) + (r > 0))))   // this one row
                                : R.tau_c / (1.f + (dc + 1.f));                             // first and last row
  // differences across the image's border are zero: the factor 0 or 1 goes into the step
  const float mr_ = c < W - 1 ? 1.f : 0.f, ml_ = c > 0 ? 1.f : 0.f;
  const bool aniso = R.aniso != 0, bf16 = R.bf16 != 0;

  // exchange: per tile and label 64 words of the first row, 64 of the last, TR of the first
  // and TR of the last column
  const int exw = 128 + 2 * TR;
  const unsigned exs = 8u * gridDim.x * k * exw;   // bytes of a slot
  auto at = [&](int trr, int tcc, int i, int word) { return 8u * (unsigned)(((trr * ntc + tcc) * k + i) * exw + word); };
  // one word per lane for the edges: lanes 0-15 ubar(r, c0-1), 16-31 ubar(r+1, c0-1), 32-47
  // ubar(r, c0+64), 48-63 ubar(r0-1, c0+64), each of element lane & 15
  const int el = tx & 15, es = tx >> 4;
  const int ej = RP == 1 ? el : el % CH, er = RP == 1 ? 0 : el / CH, et = ty * RP + er;   // label, row, row of the tile
  bool ev = on && (RP == 1 ? el < n : el < E && r + er < H);
  unsigned eo = 0;
  if (ev) {
    const int i = i0 + ej;
    if (es == 0) {
      ev = c0 > 0;
      if (ev) eo = at(tr, tc - 1, i, 128 + TR + et);
    } else if (es == 1) {
      ev = c0 > 0 && r + er + 1 < H;
      if (ev) eo = et + 1 < TR ? at(tr, tc - 1, i, 128 + TR + et + 1) : at(tr + 1, tc - 1, i, 128 + TR);
    } else if (es == 2) {
      ev = c0 + 64 < W;
      if (ev) eo = at(tr, tc + 1, i, 128 + et);
    } else {
      ev = top && er == 0 && c0 + 64 < W;
      if (ev) eo = at(tr - 1, tc + 1, i, 128 + TR - 1);
    }
  }
  const unsigned hrow = top ? at(tr - 1, tc, i0, 64) : bottom ? at(tr + 1, tc, i0, 0) : 0u;   // row beyond the tile
  char *const mine = (char *)R.ex + at(tr, tc, on ? i0 : 0, 0);
  const unsigned txo = 8u * (unsigned)tx;
  const unsigned hxo = 8u * (unsigned)min(tx, W - 1 - c0);   // lanes past the image wait for its last pixel's

  // one element after another: on the way in and out the compiler would otherwise hold every
  // plane of every element in registers at once; and with several rows per thread their rows,
  // their values read from LDS again by every section (registers are what limits the rows)
  auto in_turn = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto row_by_row = [&] {
    if (RP > 1) in_turn();
  };
  auto label_by_label = [&] {
    if (RP == 1 && CH >= 7) in_turn();
  };

  const unsigned lost = scalar_word(R.err);   // the error word when the launch began
  // ---- the state
  float u[E], s[E], v[E], z[E], px[E], q[RP], fc[RP], lam = uniform(R.lam);
  // a dual's value in plane i of `base` at byte offset off of a float plane
  auto ldd = [&](const void *base, int i, unsigned off) {
    return bf16 ? ldvb((const uint16_t *)base + (long long)i * ps, off / 2)
                : ldvb((const float *)base + (long long)i * ps, off);
  };
#pragma unroll
  for (int rp = 0; rp < RP; rp++) {
    const unsigned xr = row_off(rp);
    q[rp] = fc[rp] = 0.f;
    if (row_in(rp)) {
      if (col) {
        q[rp] = ldb(R.q, xr);
        if (PIECE != SLI_SAMPLED) fc[rp] = ldb(R.fn, xr);
      }
    }
#pragma unroll
    for (int j = 0; j < CH; j++) {
      if (E > 4) in_turn();
      const int e = rp * CH + j, i = i0 + j;
      u[e] = s[e] = v[e] = z[e] = px[e] = 0.f;
      float ub = 0.f, sb = 0.f, py = 0.f, hx = 0.f, hy = 0.f;
      if (row_in(rp) && j < n) {
        if (col) {
          const long long o = (long long)i * ps;
          u[e] = ldb(R.u + o, xr);
          ub = 2.f * u[e] - ldb(R.up + o, xr);
          s[e] = ldb(R.s + o, xr);
          sb = 2.f * s[e] - ldb(R.sp + o, xr);
          v[e] = ldd(R.v, i, xr);
          z[e] = ldd(R.z, i, xr);
          px[e] = ldd(R.p, i, xr);
          py = ldd(R.p, k + i, xr);
          if (rp == 0 && top) {
            hx = ldd(R.p, i, xr - 4u * (unsigned)W);
            hy = ldd(R.p, k + i, xr - 4u * (unsigned)W);
          }
        }
      }
      lub[e * LS] = ub;
      lsb[e * LS] = sb;
      lpy[e * LP] = py;
      if (ty == 0 && rp == 0) {
        lpy[((RP - 1) * CH + j) * LP - 64] = 0.f;   // above the image: times zero in div p
        lhx[j * LH] = hx;
        lhy[j * LH] = hy;
      }
    }
  }
  // p left of the tile, of element `lane`
  float pxL = 0.f, pyL = 0.f, radL = 0.f;
  const bool left = on && c0 > 0;
  const int lj = RP == 1 ? tx : tx % CH, lr = RP == 1 ? 0 : tx / CH;
  const bool mdL = r + lr < H - 1;
  const bool ownL = RP == 1 ? tx < n : tx < E && r + lr < H;
  if (left && ownL) {
    const unsigned xl = 4u * (unsigned)((r + lr) * W + c0 - 1);
    pxL = ldd(R.p, i0 + lj, xl);
    pyL = ldd(R.p, k + i0 + lj, xl);
    radL = R.lam * R.lab[i0 + lj].h;
  }
  bool listed[E];
  int lfirst[RP];   // the pixel's first listed label: they are neighbours, so label i has slot i - lfirst
  if (LIST) {
    if (threadIdx.x < 2) lcount[threadIdx.x] = 0;
    if ((int)threadIdx.x < k) {
      const ResidentLabel &B = R.lab[threadIdx.x];
      ltab[threadIdx.x] = make_float4(B.g0, B.g1, B.ig0, B.ig1);
    }
    __syncthreads();
#pragma unroll
    for (int rp = 0; rp < RP; rp++) {
      const bool inr = col && row_in(rp);
      unsigned info = 31u | (31u << 13);
      if (row_in(rp)) {
        if (col) info = ldb(R.sinfo, row_off(rp));
      }
      const int s0 = (int)(info & 31u), s1 = (int)((info >> 13) & 31u);
      const float lo = fc[rp] - R.del, hb = fc[rp] + R.del;
      int first = k;
      for (int i = k - 1; i >= 0; i--)
        if (i == s0 || i == s1 || (lo <= R.lab[i].g0 && R.lab[i].g1 <= hb)) first = i;
      lfirst[rp] = first;
      lfc[rp * LS + tid] = fc[rp];
      // hull ranges of the two straddles (16 bits), label of the first, first listed label, gp
      lin[rp * LS + tid] = ((info >> 5) & 0xFFu) | ((info >> 10) & 0xFF00u) | ((unsigned)s0 << 16) |
                           ((unsigned)(first & 31) << 21) | ((unsigned)gp << 26);
#pragma unroll
      for (int j = 0; j < CH; j++) {
        const int e = rp * CH + j, i = i0 + j;
        const bool str = inr && j < n && (i == s0 || i == s1);
        const bool quad = inr && j < n && !str && lo <= R.lab[i].g0 && R.lab[i].g1 <= hb;
        listed[e] = str || quad;
        for (int l = 0; l < 2; l++) {
          const bool mem = l == 0 ? quad : str;
          const u64 m = __ballot(mem);
          if (m == 0) continue;
          int base = 0;
          if (tx == 0) base = atomicAdd(&lcount[l], __popcll(m));
          base = __builtin_amdgcn_readfirstlane(base);
          if (mem) (l == 0 ? lq : lc)[base + __popcll(m & ((1ull << tx) - 1ull))] = (uint16_t)(e * LS + tid);
        }
      }
    }
  }

  // the rim's ubar out: the row's words if it is the tile's first or last, and by lanes 0 and
  // 63 the first and last column's
  const bool pe = in && ((tx == 0 && c0 > 0) || (tx == 63 && c < W - 1));
  const bool pe_any = on && (c0 > 0 || c0 + 64 < W);
  const unsigned peo = 8u * (unsigned)(128 + (tx == 0 ? 0 : TR) + ty * RP);
  auto publish = [&](unsigned tag) {
    char *const slot = mine + (tag & 1u) * exs;
    if (halo) {
      if (in) {
        const int first = top ? 0 : (RP - 1) * CH * LS;
#pragma unroll
        for (int j = 0; j < CH; j++) {
          label_by_label();
          if (j < n) put(slot + (top ? 0u : 512u) + 8u * (unsigned)(j * exw), txo, lub[first + j * LS], tag);
        }
      }
    }
    if (pe_any) {
      if (pe) {
#pragma unroll
        for (int rp = 0; rp < RP; rp++)
#pragma unroll
          for (int j = 0; j < CH; j++) {
            label_by_label();
            if (j < n && (RP == 1 || r + rp < H))
              put(slot + 8u * (unsigned)(j * exw + rp), peo, lub[(rp * CH + j) * LS], tag);
          }
      }
    }
  };
  __syncthreads();   // every value of the neighbours' state has been read before the first word goes out
  const int nq = LIST ? __builtin_amdgcn_readfirstlane(lcount[0]) : 0;
  const int nc = LIST ? __builtin_amdgcn_readfirstlane(lcount[1]) : 0;
  const int bc = (nc + 63) / 64, batches = bc + (nq + 63) / 64, waves = (int)blockDim.x >> 6;
  publish(R.tag);
  // Nothing to do for a state that an earlier launch has lost: no second wait of that length.
  // (Here and not earlier: spills ahead of the loop are put where this block starts, with all
  // lanes on, and not at the end of publish's divergent part.)
  if (lost != 0u) return;

  // a dual into plane i of `base`, at byte offset off of a float plane
  auto std_ = [&](void *base, int i, unsigned off, float val) {
    if (bf16)
      stvb((uint16_t *)base + (long long)i * ps, off / 2, val);
    else
      stvb((float *)base + (long long)i * ps, off, val);
  };
  // what the residuals of the last iteration compare with: the duals before it
  auto save_duals = [&] {
    int is = i0;   // addresses formed here, not ahead of all iterations
    unsigned xs = xb;
    asm volatile("" : "+s"(is), "+v"(xs));
#pragma unroll
    for (int rp = 0; rp < RP; rp++) {
      if (!row_in(rp)) continue;
      const unsigned xr = RP == 1 ? xs : xs + 4u * (unsigned)(rp * W);
      if (col) {
#pragma unroll
        for (int j = 0; j < CH; j++) {
          if (j >= n) continue;
          in_turn();
          const int e = rp * CH + j, i = is + j;
          std_(R.vsave, i, xr, v[e]);
          std_(R.zsave, i, xr, z[e]);
          std_(R.psave, i, xr, px[e]);
          std_(R.psave, k + i, xr, lpy[e * LP]);
        }
        if (gp == 0) stb(R.qsave, xr, q[rp]);
      }
    }
  };
  bool dead = false;
  int it = 1, stop = R.vsave ? R.iters - 1 : R.iters;
  // samples: the prologue's loads end here; left pending, the compiler would wait, in every
  // iteration, at the first use of these for whatever else is in flight
  if constexpr (PIECE == SLI_SAMPLED) {
#pragma unroll
    for (int e = 0; e < E; e++) asm volatile("" : "+v"(v[e]), "+v"(z[e]), "+v"(px[e]));
    asm volatile("" : "+v"(q[0]), "+v"(pxL), "+v"(pyL), "+v"(radL));
  }
  while (true) {
#pragma unroll 1
  for (; it <= stop; it++) {
    // values of one label or pixel that no iteration changes are formed where they are used:
    // hoisted out of the loop by the compiler they would take a register each and spill
    int ii = i0;
    asm volatile("" : "+s"(lam), "+s"(ii));
    if (RP == 1 && !LIST) asm volatile("" : "+v"(fc[0]));
    // past the last label (j >= n) a thread works on zeros: h and the steps are 0 there, and
    // so every sum's share, and nothing is stored
    const ResidentLabel *const lab = R.lab + ii;
    const unsigned nb4 = 4u * (unsigned)(H * W);
    int rr = r;
    unsigned xo = xb;
    if (RP > 1) {   // (one statement each: with a vector operand the scalar one would count as divergent)
      asm volatile("" : "+s"(rr));
      asm volatile("" : "+v"(xo));
    }
    auto md_ = [&](int rp) { return rr + rp < H - 1 ? 1.f : 0.f; };
    auto mu_ = [&](int rp) { return rr + rp > 0 ? 1.f : 0.f; };
    // ---- sums of h sbar per label group
    float Tc[LG];
    if constexpr (RP == 1) {
#pragma unroll
      for (int g = 0; g < LG; g++) {
        Tc[g] = 0.f;
#pragma unroll
        for (int jj = 0; jj < CN; jj++) Tc[g] += lab[g * CN + jj].h * lsb[(g * CN + jj) * LS];
        if (!one) exa[(gp * LG + g) * NP] = Tc[g];
      }
    }
    if (!LIST || !one) lds_barrier();
    // the rim of the previous iteration: requested here, looked at when p is due
    const unsigned tag = R.tag + (unsigned)(it - 1);
    const char *const slot = (const char *)R.ex + (tag & 1u) * exs;
    u64 hw[HB], ew = 0;
    auto request = [&](int b0) {
      if (b0 == 0 && ev) ew = get(slot, eo);
      if (halo) {
#pragma unroll
        for (int j = 0; j < HB; j++) hw[j] = get(slot + hrow + 8u * (unsigned)(min(b0 + j, n - 1) * exw), hxo);
      }
    };
    if (EARLY) request(0);
    float pl = 0.f;   // new px left of the tile, label i0 + lane
    unsigned looks = 0;   // in vain
    auto wait = [&](int b0) {
      if (!EARLY || b0 > 0) request(b0);
      while (true) {
        unsigned wrong = b0 == 0 && ev ? (unsigned)(ew >> 32) ^ tag : 0u;
        if (halo) {
#pragma unroll
          for (int j = 0; j < HB; j++) wrong |= (unsigned)(hw[j] >> 32) ^ tag;
        }
        if (dead || !__any(wrong != 0u)) break;
        if (looks++ == R.limit) {
          dead = true;
          *R.err = 1u;
        }
        __builtin_amdgcn_s_sleep(1);   // 64 clocks between looks: without, up to 1 % slower (256x256, L = 20)
        request(b0);   // (also after giving up: a second way out of this loop costs spills)
      }
    };
    auto p_update = [&]() {
      wait(0);
      const float eub = __uint_as_float((unsigned)ew);
      // p: own, of the row above the tile and of the column left of it
      if (left) {
        const float own = ownL ? lub[tx * LS - tx] : 0.f;
        const float dn = __shfl(eub, (tx & 15) + 16);
        pl = pxL;
        float py = pyL;
        p_step(pl, py, R.sig_p, own - eub, mdL ? dn - eub : 0.f, radL, aniso);
        pxL = bf16 ? round_bf16(pl) : pl;
        pyL = bf16 ? round_bf16(py) : py;
      }
      if (bf16) {   // p_y as it is stored; div p of the previous iteration took it unrounded
#pragma unroll
        for (int e = 0; e < E; e++) {
          label_by_label();
          lpy[e * LP] = round_bf16(lpy[e * LP]);
        }
      }
      const float spx = R.sig_p * mr_;
#pragma unroll
      for (int b0 = 0; b0 < CH; b0 += HB)
#pragma unroll
      for (int rp = 0; rp < RP; rp++) {
        if (b0 > 0) {
          in_turn();
          wait(b0);
        }
        row_by_row();
        const float spy = R.sig_p * md_(rp);
#pragma unroll
        for (int j = b0; j < (b0 + HB < CH ? b0 + HB : CH); j++) {
          const int e = rp * CH + j;
          const float rad = lam * lab[j].h, hub = halo && j < n ? __uint_as_float((unsigned)hw[j - b0]) : 0.f;
          const float ub = lub[e * LS];
          const float ubr = from_right(ub, rdlane(eub, 32 + e));
          const float ubd = rp + 1 < RP ? lub[(e + CH) * LS] : ty + 1 < TH ? lub[j * LS + 64] : hub;
          float py = lpy[e * LP];
          px[e] = px[e] + spx * (ubr - ub);
          py = py + spy * (ubd - ub);
          proj_K(px[e], py, rad, aniso);
          lpy[e * LP] = py;
          if (rp == 0 && top) {
            const float ubur = from_right(hub, rdlane(eub, 48 + j));
            float hx = lhx[j * LH], hy = lhy[j * LH];
            hx = hx + spx * (ubur - hub);
            hy = hy + R.sig_p * (ub - hub);
            proj_K(hx, hy, rad, aniso);
            lpy[((RP - 1) * CH + j) * LP - 64] = hy;
            lhx[j * LH] = hx;
            lhy[j * LH] = hy;
          }
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
    float pre_[LG];   // sums of the new v per label group
    float wlo[ADD ? CH + 1 : 1];   // additive values at the thread's labels
    // samples: those of the label at work and, a batch of NS ahead of their use, the next ones
    // (mb on, up to the last one `most`); a label starts with the last sample of the one before
    constexpr int NS = 5;
    float rnext[NS], rfirst = 0.f;
    int mb = 0;
    auto cost = [&](int m) {
      return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(plane_rsrc(R.cost, 0x7fffffffu), (int)xb,
                                                                            (int)(4u * (unsigned)ps * (unsigned)m), 0));
    };
    auto samples = [&](int most) {
#pragma unroll
      for (int m = 0; m < NS; m++) rnext[m] = cost(min(mb + m, most));
    };
    auto last_sample = [&](int i) { return __builtin_amdgcn_readfirstlane(R.sidx[i + 1]); };
    if (PIECE == SLI_SAMPLED && on && n > 0) {
      mb = __builtin_amdgcn_readfirstlane(R.sidx[i0]);
      rfirst = cost(mb);
      mb++;
      samples(last_sample(i0));
      __builtin_amdgcn_sched_barrier(0);
    }
    if (on) {
      if (ADD) {
#pragma unroll
        for (int j = 0; j <= CH; j++) wlo[ADD ? j : 0] = in ? ldb(R.wadd + (long long)min(i0 + j, k) * ps, xb) : 0.f;
      }
      // ---- data-term duals before their projection, over h
#pragma unroll
      for (int rg = 0; rg < RP * LG; rg++) {   // rows, or label groups
        const int rp = RP == 1 ? 0 : rg, g = RP == 1 ? rg : 0;
        row_by_row();
        float T = 0.f, suf;
        if constexpr (RP == 1) {
          float base = 0.f;   // sums of the label groups after this one
          if (one) {
#pragma unroll
            for (int gg = 0; gg < LG; gg++) {
              T += Tc[gg];
              if (gg > g) base += Tc[gg];
            }
          } else {
            if (g == 0)
              for (int gg = 0; gg < G; gg++) T += exa[gg * NP];
            for (int gg = gp * LG + g + 1; gg < G; gg++) base += exa[gg * NP];
          }
          suf = base + Tc[g];
        } else {
#pragma unroll
          for (int j = 0; j < CH; j++) T += lab[j].h * lsb[(rp * CH + j) * LS];
          suf = T;
        }
        if (g == 0) q[rp] = q[rp] - R.sig_q * (1.f + T);
#pragma unroll
        for (int jj = 0; jj < CN; jj++) {
          label_by_label();
          const int j = g * CN + jj, e = rp * CH + j;
          const float sb = lsb[e * LS], ub = lub[e * LS];
          suf -= lab[j].h * sb;
          const float ve = v[e] + lab[j].sig * (ub + suf - lab[j].g0 * sb);
          const float ze = z[e] + lab[j].sig * sb;
          float y = ve * lab[j].ih, w = ze * lab[j].ih;
          if (ADD) {
            const float bs = (wlo[ADD ? j + 1 : 0] - wlo[ADD ? j : 0]) * lab[j].ih;
            y -= bs;
            w -= -wlo[ADD ? j : 0] + bs * lab[j].g0;
          }
          if (LIST) {
            lsb[e * LS] = y;
            if (listed[e]) lw[(rp * slots + i0 + j - lfirst[rp]) * NP] = w;
            proj_flat(R.nu, lab[j].g0, lab[j].g1, lab[j].ig0, lab[j].ig1, y, w);
          }
          v[e] = y;
          z[e] = w;
        }
      }
    }
    if (LIST) {
      lds_barrier();
      for (int b = wave; b < batches; b += waves) {
        const bool hull = b < bc;
        const int e = (hull ? b : b - bc) * 64 + tx;
        if (e < (hull ? nc : nq)) {
          const int at = (int)(hull ? lc : lq)[e], el_ = at / LS, who = at & (LS - 1), row = RP == 1 ? 0 : el_ / CH;
          const unsigned info = lin[row * LS + who];
          const int g_ = RP == 1 ? (int)(info >> 26) : 0;
          const int i = RP == 1 ? g_ * CH + el_ : el_ % CH;
          const float4 g = ltab[i];
          const float f = lfc[row * LS + who];
          float *const py = lds + E * LS + at;
          float *const pw = lists + (row * slots + i - (int)((info >> 21) & 31u)) * NP + who - g_ * NP;
          float y = *py, w = *pw;
          if (hull) {
            const unsigned m = info >> ((int)((info >> 16) & 31u) == i ? 0 : 8);
            proj_tq_chain(R.a, f, R.nu, g.x, g.y, (int)(m & 15u), (int)((m >> 4) & 15u), y, w);
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
      auto fload = [&](int rp) { return bld(R.fn, nb4, xo + 4u * (unsigned)(rp * W)); };
      float fnext = 0.f;
      if (PIECE == SLI_QUAD && RP > 1) {
        fnext = fload(0);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int g = 0; g < LG; g++) pre_[g] = 0.f;
#pragma unroll
      for (int rp = 0; rp < RP; rp++) {
        row_by_row();
        float pre = 0.f;   // sum of the new v of the label group so far
        // the data centre: kept, or with several rows loaded again, a row ahead (registers are
        // dearer; rows past the image read 0). 1531x2039, 12 rows a thread: 21.2 us an iteration
        // with each row's load waited for, 19.4 with it a row ahead.
        float f = fc[0];
        if (PIECE == SLI_QUAD && RP > 1) {
          f = fnext;
          if (rp + 1 < RP) fnext = fload(rp + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < CH; j++) {
          const int e = rp * CH + j;
          if (LG > 1 && j > 0 && j % CN == 0) {
            pre_[j / CN - 1] = pre;
            pre = 0.f;
          }
          float y = v[e], w = z[e];
          if (PIECE == SLI_QUAD) {
            proj_quad(R.a, R.ia, piece_centre(f, lab[j].g0, lab[j].g1, R.per, R.iper), lab[j].g0, lab[j].g1,
                      lab[j].ig0, lab[j].ig1, y, w);
          } else if (LIST) {
            if (listed[e]) {
              y = lsb[e * LS];
              w = lw[(rp * slots + i0 + j - lfirst[rp]) * NP];
            }
          } else if (j < n) {
            // a batch's places past the label's last sample repeat it; the kink of the sample with
            // itself is put at 0 times infinity, which lies right of no point
            const int m1 = last_sample(i0 + j), m2 = last_sample(min(i0 + j + 1, k - 1));
            PLScan pl;
            pl.first(y, w, ldtab(R.tau, mb - 1), rfirst);
            while (mb <= m1) {
              float rr[NS];
              float4 tq[NS];
#pragma unroll
              for (int m = 0; m < NS; m++) {
                rr[m] = rnext[m];
                tq[m] = ldtab(R.tau, min(mb + m, m1));
                if (mb + m > m1) tq[m].z = SL_INF;
              }
              mb = min(mb + NS, m1 + 1);
              samples(mb <= m1 ? m1 : m2);
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int m = 0; m < NS; m++) pl.push(tq[m], rr[m]);
              rfirst = rr[NS - 1];
            }
            pl.finish(y, w);
          }
          if (ADD) {
            const float bs = (wlo[ADD ? j + 1 : 0] - wlo[ADD ? j : 0]) * lab[j].ih;
            y += bs;
            w += -wlo[ADD ? j : 0] + bs * lab[j].g0;
          }
          v[e] = lab[j].h * y;
          z[e] = lab[j].h * w;
          lsb[e * LS] = s[e] - lab[j].taus * (z[e] - lab[j].h * q[rp] + lab[j].h * pre - lab[j].g0 * v[e]);
          pre += v[e];
        }
        if (RP == 1) pre_[LG - 1] = pre;
      }
      if (RP == 1 && !one) {
#pragma unroll
        for (int g = 0; g < LG; g++) exb[(gp * LG + g) * NP] = pre_[g];
      }
      if (!LIST) p_update();
    }
    if (!LIST) lds_barrier();
    const bool last = it == R.iters;
    if (on) {
      // ---- u and ubar (after the last iteration u_prev in ubar's place, for the way out)
#pragma unroll
      for (int rp = 0; rp < RP; rp++) {
        row_by_row();
        const float tau_u = RP == 1 || rr + rp == 0 || rr + rp >= H - 1 ? tau_rim : tau_mid;
#pragma unroll
        for (int j = 0; j < CH; j++) {
          label_by_label();
          const int e = rp * CH + j;
          const float pxl = from_left(px[e], rdlane(pl, e));
          const float pyu = rp > 0 ? lpy[(e - (rp > 0 ? CH : 0)) * LP] : lpy[((RP - 1) * CH + j) * LP - 64];
          float dv = mr_ * px[e];
          dv -= ml_ * pxl;
          dv += md_(rp) * lpy[e * LP];
          dv -= mu_(rp) * pyu;
          const float un = u[e] - tau_u * (v[e] - dv);
          lub[e * LS] = last ? u[e] : 2.f * un - u[e];
          u[e] = un;
        }
      }
      if (!last) publish(R.tag + (unsigned)it);
      if (bf16) {
#pragma unroll
        for (int e = 0; e < E; e++) {
          v[e] = round_bf16(v[e]);
          z[e] = round_bf16(z[e]);
          px[e] = round_bf16(px[e]);
        }
      }
    }
    if (LIST && !one) lds_barrier();
    if (on) {
      // ---- s with the earlier groups' v, and sbar
#pragma unroll
      for (int rg = 0; rg < RP * LG; rg++) {
        const int rp = RP == 1 ? 0 : rg, g = RP == 1 ? rg : 0;
        float vb = 0.f;
        if constexpr (RP == 1) {
          if (one) {
#pragma unroll
            for (int gg = 0; gg < LG; gg++)
              if (gg < g) vb += pre_[gg];
          } else {
            for (int gg = 0; gg < gp * LG + g; gg++) vb += exb[gg * NP];
          }
        }
#pragma unroll
        for (int jj = 0; jj < CN; jj++) {
          const int j = g * CN + jj, e = rp * CH + j;
          float sn = lsb[e * LS];
          if (RP == 1 && G > 1) sn = sn - lab[j].taus * (lab[j].h * vb);
          lsb[e * LS] = last ? s[e] : 2.f * sn - s[e];
          s[e] = sn;
        }
      }
      if constexpr (KEEP) {
        static_assert(RP == 1, "one row");
        if (!last && row_in(0)) {
          const long long at = (long long)it * R.kstep;
          float *const ky = R.ky + (long long)it * R.ystep;
          if (col) {
#pragma unroll
            for (int j = 0; j < CH; j++) {
              if (j >= n) continue;
              const long long o = (long long)(i0 + j) * ps;
              stb(R.ku + at + o, xb, u[j]);
              stb(R.ks + at + o, xb, s[j]);
              stb(ky + o, xb, v[j]);
              stb(ky + k * ps + o, xb, z[j]);
              stb(ky + (2 * k + 1) * ps + o, xb, px[j]);
              stb(ky + (3 * k + 1) * ps + o, xb, lpy[j * LP]);
            }
            if (gp == 0) stb(ky + 2 * k * ps, xb, q[0]);
          }
        }
      }
    }
  }

  if (it > R.iters) break;
  save_duals();
  stop = R.iters;
  }

  // ---- the state back to memory (of a wave that gave up: NaN)
  if (dead) {
#pragma unroll
    for (int e = 0; e < E; e++) u[e] = __builtin_nanf("");
  }
#pragma unroll
  for (int rp = 0; rp < RP; rp++) {
    if (!row_in(rp)) continue;
    const unsigned xr = row_off(rp);
    if (col) {
#pragma unroll
      for (int j = 0; j < CH; j++) {
        if (j >= n) continue;
        if (E > 4) in_turn();
        const int e = rp * CH + j, i = i0 + j;
        const long long o = (long long)i * ps;
        stb(R.uo + o, xr, u[e]);
        stb(R.upo + o, xr, lub[e * LS]);
        stb(R.so + o, xr, s[e]);
        stb(R.spo + o, xr, lsb[e * LS]);
        std_(R.vo, i, xr, v[e]);
        std_(R.zo, i, xr, z[e]);
        std_(R.po, i, xr, px[e]);
        std_(R.po, k + i, xr, lpy[e * LP]);
      }
      if (gp == 0) stb(R.qo, xr, q[rp]);
    }
  }
}

// What is built: chunks of up to 8 labels per thread, with a wavefront per label group in blocks
// of up to 4 groups, and of 9 in blocks of one; the chunks of two or four label groups that a
// thread takes together when the image has too many tiles for a wavefront per group; for long
// chunks (whose LDS is scarce) blocks of one group of threads apart from those of several; several
// rows per thread for few labels. Not built, because one launch per iteration is as fast: two rows
// of 6 quadratic labels (1501x192: 19.6 us on chip, 19.1 off it) and two groups of 5 quadratic
// labels with additive values (701x256: 21.8 and 21.7, with bf16 duals 22.4 and 20.7). Returns the
// kernel for `phys` groups of threads and its PH.
template <int PIECE, bool ADD>
inline const void *kernel_of(int ch, int lg, int rp, int phys, int *ph, bool keep) {
  if (keep) {   // the shapes of the images that are differentiated through
    if constexpr (PIECE != SLI_SAMPLED) {
      *ph = 4;
      if (lg == 1 && rp == 1 && phys <= 4) {
        if (ch == 1) return (const void *)pdhg_resident_kernel<PIECE, ADD, 1, 1, 1, 4, true>;
        if (ch == 2) return (const void *)pdhg_resident_kernel<PIECE, ADD, 2, 1, 1, 4, true>;
        if (ch == 3) return (const void *)pdhg_resident_kernel<PIECE, ADD, 3, 1, 1, 4, true>;
        if (ch == 4) return (const void *)pdhg_resident_kernel<PIECE, ADD, 4, 1, 1, 4, true>;
      }
    }
    return nullptr;
  }
#define SLI_RES(C, L, P, H)                                                       \
  if (ch == C && lg == L && rp == P && phys <= H) {                               \
    *ph = H;                                                                      \
    return (const void *)pdhg_resident_kernel<PIECE, ADD, C, L, P, H>;            \
  }
  SLI_RES(1, 1, 1, 4)
  SLI_RES(2, 1, 1, 4)
  SLI_RES(3, 1, 1, 4)
  SLI_RES(4, 1, 1, 4)
  SLI_RES(5, 1, 1, 4)
  SLI_RES(6, 1, 1, 4)
  SLI_RES(7, 1, 1, 1)
  SLI_RES(8, 1, 1, 1)
  SLI_RES(9, 1, 1, 1)
  SLI_RES(7, 1, 1, 4)
  SLI_RES(8, 1, 1, 4)
  SLI_RES(2, 2, 1, 2)
  SLI_RES(4, 2, 1, 2)
  SLI_RES(6, 2, 1, 2)
  SLI_RES(8, 2, 1, 1)
  if constexpr (!(PIECE == SLI_QUAD && ADD)) SLI_RES(10, 2, 1, 1)
  SLI_RES(8, 2, 1, 2)
  SLI_RES(4, 4, 1, 1)
  SLI_RES(8, 4, 1, 1)
  if constexpr (PIECE != SLI_SAMPLED && !ADD) {
    SLI_RES(1, 1, 2, 1)
    SLI_RES(1, 1, 3, 1)
    SLI_RES(1, 1, 4, 1)
    SLI_RES(1, 1, 6, 1)
    SLI_RES(2, 1, 2, 1)
    SLI_RES(2, 1, 3, 1)
    SLI_RES(3, 1, 2, 1)
  }
  if constexpr (PIECE == SLI_QUAD && !ADD) {
    SLI_RES(1, 1, 8, 1)
    SLI_RES(1, 1, 12, 1)
    SLI_RES(2, 1, 4, 1)
    SLI_RES(2, 1, 6, 1)
    SLI_RES(3, 1, 3, 1)
    SLI_RES(3, 1, 4, 1)
    SLI_RES(4, 1, 2, 1)
    SLI_RES(4, 1, 3, 1)
    SLI_RES(5, 1, 2, 1)
  }
#undef SLI_RES
  return nullptr;
}

}  // namespace resident
