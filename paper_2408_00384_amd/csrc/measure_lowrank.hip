// Z-measurement of a list of qubits in blocks of 64, each block one low-rank
// update of the tableau in memory; kernel boundaries are the only grid-wide
// sync (two launches per block, no waiting between workgroups).
//
// Method: paper Sec. 2 (Aaronson & Gottesman 2004 tableau rules); outcomes,
// tableau bits and signs are those of the step-by-step rule.
//
//  * A random measurement of qubit a with pivot p (smallest stabilizer row
//    with x = 1 on column a) multiplies every other row with x = 1 on column
//    a by row p, copies row p into row p - n and sets row p to +-Z_a.  On the
//    bits of a column this is one linear map of the rows, the same for every
//    column.  Over a block with pivots p_0, p_1, .. every row i that is not
//    a pivot row ends as
//        new_i = [i not replaced] old_i  XOR  sum_t U[i][t] old_{p_t}
//    (old: at the block's start; the replaced rows are p_t - n), and p_t ends
//    as Z_{a_t}.  So every column takes x ^= sum over t with x[p_t] = 1 of
//    U_t, and the same for z.
//  * The bits of the block's own columns, row by row (64 bits a row, "row
//    form"), determine everything: step t finds the smallest stabilizer row
//    with bit t, and every row with bit t XORs that row's bits into its own.
//    Only the few smallest rows have to be followed step by step to find the
//    pivots (the planner); every other row replays the steps on its own.
//  * A measurement without a pivot is deterministic and changes nothing.
//    Z_a is then in the stabilizer group, and measurements of other Z's leave
//    it there with its sign, so the outcome is read from the tableau at the
//    end of the pass: the sign of the product of the stabilizers n + i with
//    x_ia = 1.
//  * Signs.  Every product formed is of commuting Pauli rows, so a final row
//    is the product of its factors (old_i if kept, and the pivot rows in
//    U[i]) in any order, with sign
//        sum of the factors' signs + (sum of the factors' Y counts
//        - Y count of the result) / 2 + sum over factor pairs a < b of
//        z(a).x(b)   (mod 2).
//    With old_i first the pair sum is z(old_i).(x_new_i ^ x_old_i), summed in
//    the sweep, plus the pivot rows' Gram matrix z(p_a).x(p_b) over the pairs
//    in U[i].
//
// Launches for block b (b = -1 starts the pipeline, b = nb ends it):
//   k_lr_prep   rows:    U of block b from the plan and the row form; the next
//                        block's row form, brought past block b
//               columns: x and z of every column at the pivot rows; the
//                        pivots' Y counts and Gram rows
//               signs:   block b - 1's sign flips H per row word; per shot its
//                        pivots' signs and the outcome bits
//   k_lr_sweep  planner (one workgroup) of block b + 1; the sweep of block b
//               over all columns; the signs of block b - 1 for every shot
// and k_lr_det_terms, k_lr_det, the deterministic outcomes, at the end of the pass.
//
// Bound: the sweep reads and writes the tableau once per 64 measurements and
// takes 32 table reads per two words of x and z.  n = 10,000: 21 us a launch,
// vector instructions 72 % of the busy cycles, LDS 36 %, the tableau in the
// last-level cache at 0.57 of a plain copy's rate; n = 25,000: 123 us, memory, at
// 0.96 of a plain copy's rate (the launches before the first and after the last
// block, which touch no tableau, 22 and 17 us); below n = 6,000 the planner's chain of 64 dependent steps (0.11 us each;
// 11 us a sweep launch at n = 1,024) and the prep launch's chain of loads (7
// to 8 us).  Against one rowsum sweep per measurement (register-resident up to
// n = 10,240, one kernel per measurement above), circuit and measure-all:
// n = 64, 16 shots 0.114 against 0.389 ms; n = 1,024, 128 shots 0.44 against
// 2.68 ms; n = 3,001 after 2 layers, a third of the outcomes deterministic,
// 1.21 against 7.28 ms; n = 5,003 1.84 against 8.23 ms; n = 10,000 4.9 against
// 16.4 ms (blocks of 32 in registers); 128 of n = 25,000 2.30 against 12.3 ms.
// Blocks of 64: twice the work per launch of 32 at the same number of tableau
// passes, and a row's bits are one 64-bit word.
#include <algorithm>

#include "internal.h"
#include "philox.h"

namespace cliff {

namespace {

constexpr uint32_t kK = kLrK;              // measurements per block
constexpr uint32_t kPrepThreads = 256;
constexpr uint32_t kSweepThreads = 1024;
constexpr uint32_t kSweepWaves = kSweepThreads / 64;
constexpr uint32_t kPrepCols = 8;          // columns per wave of the prep kernel, all in flight
constexpr uint32_t kWindow = 512;          // rows the planner can follow step by step

__device__ __forceinline__ uint64_t lbit(uint32_t b) { return 1ull << (b & 63); }
__device__ __forceinline__ uint64_t pair64(uint32_t lo, uint32_t hi) { return (uint64_t(hi) << 32) | lo; }
__device__ __forceinline__ uint32_t rdlane(uint32_t v, uint32_t l) {
  return uint32_t(__builtin_amdgcn_readlane(int(v), int(l)));
}
__device__ __forceinline__ uint64_t rdlane64(uint64_t v, uint32_t l) {
  return pair64(rdlane(uint32_t(v), l), rdlane(uint32_t(v >> 32), l));
}

template <uint32_t J>
__device__ __forceinline__ uint32_t swz_xor(uint32_t v) {
  return uint32_t(__builtin_amdgcn_ds_swizzle(int(v), int((J << 10) | 0x1f)));
}
template <uint32_t J>
__device__ __forceinline__ uint32_t transpose_step(uint32_t v, uint32_t lane) {
  constexpr uint32_t m = J == 16 ? 0x0000ffffu : J == 8 ? 0x00ff00ffu : J == 4 ? 0x0f0f0f0fu
                       : J == 2 ? 0x33333333u : 0x55555555u;
  const uint32_t y = swz_xor<J>(v);
  return (lane & J) ? ((v & ~m) | ((y & ~m) >> J)) : ((v & m) | ((y & m) << J));
}
// 64 x 64 bit transpose across a wave: bit j of lane i <-> bit i of lane j.
__device__ __forceinline__ uint64_t transpose64(uint64_t v, uint32_t lane) {
  uint32_t lo = uint32_t(v), hi = uint32_t(v >> 32);
  const uint32_t give = lane < 32 ? hi : lo;
  const uint32_t got = uint32_t(__shfl_xor(int(give), 32));
  if (lane < 32) hi = got;
  else lo = got;
  lo = transpose_step<16>(lo, lane); hi = transpose_step<16>(hi, lane);
  lo = transpose_step<8>(lo, lane);  hi = transpose_step<8>(hi, lane);
  lo = transpose_step<4>(lo, lane);  hi = transpose_step<4>(hi, lane);
  lo = transpose_step<2>(lo, lane);  hi = transpose_step<2>(hi, lane);
  lo = transpose_step<1>(lo, lane);  hi = transpose_step<1>(hi, lane);
  return pair64(lo, hi);
}

// a ^= v where bit `on` (0 or 1) is set
__device__ __forceinline__ uint64_t xor_if(uint64_t a, uint64_t v, uint32_t mask) {
  return pair64(bop3<LUT_AND_XOR>(uint32_t(v), mask, uint32_t(a)),
                bop3<LUT_AND_XOR>(uint32_t(v >> 32), mask, uint32_t(a >> 32)));
}
__device__ __forceinline__ uint32_t bit_mask(uint64_t v, uint32_t t) {   // all ones where bit t of v is set
  return 0u - (uint32_t(v >> t) & 1u);
}

}  // namespace

struct LrArgs {
  const uint32_t *q;      // device: the pass's measured qubits
  uint32_t k, b;          // measurements of the pass; block (int32: -1 .. nb)
  uint32_t nR, nC, nH, nS, nF;   // prep: workgroups per part
  uint32_t CG, T, lp;     // sweep: column groups, row tiles, log2 of the lanes per column
  uint32_t nA;            // sweep: sign workgroups
  uint64_t seed, circuit, shot0, m0;
};

// ------------------------------------------------------------------ prep ---
// One wave per 64 rows: lane = row.
__device__ __forceinline__ void prep_rows(const TabDev &t, const LrDev &s, const LrArgs &a, uint32_t wg,
                                          uint64_t *sV, uint32_t *sP, uint32_t *spec) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t b = int32_t(a.b);
  const bool cur = b >= 0;                                   // block b has a plan
  const uint32_t base = uint32_t(b + 1) * kK;                // the next block's first measurement
  const uint32_t kn = base < a.k ? min(kK, a.k - base) : 0u;
  if (!cur && kn == 0) return;
  const uint32_t row0 = wg * kPrepThreads, w = wg * 4 + wave;
  const bool have = w < t.W;
  const LrPlan *pl = s.plan + (uint32_t(b) & 3u);
  const uint32_t myq = lane < kn ? a.q[base + lane] : 0u;
  // this wave's word of the next block's columns (lane j: column j)
  uint64_t nw = lane < kn && have ? t.X[size_t(myq) * t.Wp + w] : 0ull;
  uint64_t e = cur && have ? s.Bt[size_t(w) * 64 + lane] : 0ull;
  spec[tid] = 0;
  if (cur && tid < kK) sP[tid] = pl->P[tid];
  const uint64_t rx = cur ? pl->RX[lane] : 0ull, rand = cur ? pl->rand : 0ull;
  __syncthreads();
  // V_t: the next block's columns at pivot row t, as they stand before block
  // b; loaded under the rows' replay
  uint32_t p[16];
  uint64_t xv[16];
  if (cur && kn) {
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) {
      p[i] = __builtin_amdgcn_readfirstlane(sP[wave * 16 + i]);
      xv[i] = t.X[size_t(myq) * t.Wp + (p[i] != kNone ? p[i] >> 6 : 0)];
    }
  }
  if (cur && tid < kK && sP[tid] != kNone) {
    const uint32_t r = sP[tid] - row0, r2 = sP[tid] - t.n - row0;
    if (r < kPrepThreads) spec[r] = 255;          // pivot row
    if (r2 < kPrepThreads) spec[r2] = tid + 1;    // replaced row
  }
  uint64_t v = transpose64(nw, lane);
  __syncthreads();
  uint64_t u = 0;
  if (cur) {
    // the row replays the block's steps: after step t bit t holds U[row][t].
    // Replaced row p_s - n takes row p_s's bits at step s and goes on from
    // there: the steps after s act on its later bits alone, and what they
    // add below is added to the bits it took.
    const uint32_t sp = spec[tid];
    uint64_t low = 0;
    if (sp) {
      const uint32_t st = sp - 1;
      e = sp == 255 ? 0ull : pl->RX[st] | lbit(st);
      const uint64_t upto = sp == 255 ? 0ull : lbit(st) | (lbit(st) - 1);
      low = e & upto;
      e &= ~upto;
      v = 0;
    }
#pragma unroll
    for (uint32_t i = 0; i < kK; ++i) e = xor_if(e, rdlane64(rx, i), bit_mask(e, i));
    u = (e ^ low) & rand;
    if (kn) {
#pragma unroll
      for (uint32_t i = 0; i < 16; ++i) {
        const uint64_t bits = __ballot(lane < kn && p[i] != kNone && ((xv[i] >> (p[i] & 63)) & 1u));
        if (lane == 0) sV[wave * 16 + i] = bits;
      }
    }
  }
  __syncthreads();
  if (!have) return;
  if (cur) {
    if (kn) {
      const uint64_t vt = sV[lane];
#pragma unroll
      for (uint32_t i = 0; i < kK; ++i) v = xor_if(v, rdlane64(vt, i), bit_mask(u, i));
    }
    s.U[(uint32_t(b) & 1u)][size_t(w) * kK + lane] = transpose64(u, lane);
  }
  if (kn) s.Bt[size_t(w) * 64 + lane] = v;
}

// One wave per column at a time: lane = pivot.
__device__ __forceinline__ void prep_cols(const TabDev &t, const LrDev &s, const LrArgs &a, uint32_t wg,
                                          unsigned long long *sG, uint32_t *sY) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const LrPlan *pl = s.plan + (a.b & 3u);
  const uint64_t rand = pl->rand;
  if (rand == 0) return;
  const uint32_t p = pl->P[lane], base = a.b * kK, n = t.n;
  const bool mine = (rand >> lane) & 1u;
  const uint32_t wp = mine ? p >> 6 : 0u, sh = p & 63;
  const uint64_t ru = mine ? pl->RX[lane] & rand & (lbit(lane) - 1) : 0ull;   // pivots row p absorbed before its step
  const uint32_t q = mine ? a.q[base + lane] : kNone;
  if (tid <= kK) sG[tid] = 0;   // [kK]: the pivot rows' support
  if (tid < kK) sY[tid] = 0;
  __syncthreads();
  uint64_t g = 0;
  uint32_t y = 0;
  unsigned long long sup = 0;
  const uint32_t wv = wg * 4 + wave, nwv = a.nC * 4;
  constexpr uint32_t B = kPrepCols;
  for (uint32_t c0 = wv; c0 < n; c0 += nwv * B) {
    uint64_t xw[B], zw[B];
#pragma unroll
    for (uint32_t i = 0; i < B; ++i) {
      const uint32_t c = c0 + i * nwv;
      const size_t at = c < n ? size_t(c) * t.Wp + wp : 0;
      xw[i] = t.X[at];
      zw[i] = t.Z[at];
    }
#pragma unroll
    for (uint32_t i = 0; i < B; ++i) {
      const uint32_t c = c0 + i * nwv;
      if (c >= n) break;
      const uint32_t xb = mine ? uint32_t(xw[i] >> sh) & 1u : 0u, zb = mine ? uint32_t(zw[i] >> sh) & 1u : 0u;
      const uint64_t bx = __ballot(xb), bz = __ballot(zb), me = __ballot(q == c);
      if (lane == 0) {
        s.BX[c] = bx;
        s.BZ[c] = bz;
        s.ME[c] = me ? uint32_t(__builtin_ctzll(me)) + 1u : 0u;
      }
      g = xor_if(g, bx, 0u - zb);
      y += xb & zb;
      // the pivot row at its step: row p plus the pivots it had absorbed
      const uint32_t xs = (xb ^ uint32_t(__popcll(bx & ru))) & 1u, zs = (zb ^ uint32_t(__popcll(bz & ru))) & 1u;
      if (mine) sup += 2 * (xs | zs) + xs + zs;
    }
  }
  atomicXor(&sG[lane], (unsigned long long)g);
  atomicAdd(&sY[lane], y);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sup += __shfl_xor(sup, off);
  if (lane == 0) atomicAdd(&sG[kK], sup);
  __syncthreads();
  if (tid == 0) s.Sp[wg] = sG[kK];
  if (tid < kK) {
    s.Gp[size_t(wg) * kK + tid] = sG[tid];
    s.Yp[size_t(wg) * kK + tid] = sY[tid];
  }
}

// Sign flips of block b - 1, one wave per row word: lane = pivot (and a
// share of the column groups' partials).
__device__ __forceinline__ void prep_flips(const TabDev &t, const LrDev &s, const LrArgs &a, uint32_t wg) {
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t bp = a.b - 1, w = wg * 4 + wave;
  const LrPlan *pl = s.plan + (bp & 3u);
  if (w >= t.W || pl->rand == 0) return;
  const uint64_t u = s.U[bp & 1u][size_t(w) * kK + lane];
  const uint64_t gr = s.G[lane] & ~(lbit(lane) | (lbit(lane) - 1));   // pairs (lane, b > lane)
  const uint32_t yc = s.Y[lane], p = pl->P[lane];
  uint64_t c0 = 0, c1 = 0, x = 0;   // (Y_old - Y_new) mod 4 in two planes; flips
#pragma unroll 2
  for (uint32_t cg = lane; cg < a.CG; cg += 64) {
    const uint64_t *part = s.part + size_t(cg) * 3 * t.Wp + w;
    const uint64_t v0 = part[0], v1 = part[t.Wp], v2 = part[2 * size_t(t.Wp)];
    c1 ^= v1 ^ (c0 & v0);
    c0 ^= v0;
    x ^= v2;
  }
  // this word's rows among the pivot and the replaced rows
  const bool isp = p != kNone && (p >> 6) == w, isq = p != kNone && ((p - t.n) >> 6) == w;
  uint64_t cons = isp ? lbit(p) : 0ull, kill = cons | (isq ? lbit(p - t.n) : 0ull);
  // the absorbed pivots' Y counts, and their Gram pairs
  const uint64_t uy = (yc & 1u) ? u : 0ull;
  c1 ^= c0 & uy;
  c0 ^= uy;
  if (yc & 2u) c1 ^= u;
  uint64_t acc = 0;
#pragma unroll
  for (uint32_t i = 1; i < kK; ++i) acc = xor_if(acc, rdlane64(u, i), bit_mask(gr, i));
  x ^= u & acc;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t b0 = __shfl_xor(c0, off), b1 = __shfl_xor(c1, off);
    c1 ^= b1 ^ (c0 & b0);
    c0 ^= b0;
    x ^= __shfl_xor(x, off);
  }
  if (__ballot(isp || isq)) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      cons |= __shfl_xor(cons, off);
      kill |= __shfl_xor(kill, off);
    }
  }
  if (lane == 0) {
    const uint64_t odd = c0 & ~cons;
    if (odd) atomicAdd(&t.state[ST_ANOMALY], uint32_t(__popcll(odd)));
    s.H[w] = (c1 ^ x) & ~cons;
    s.KW[w] = kill;
    s.CW[w] = cons;
  }
}

// Block b - 1, one wave per shot: lane = pivot.  Its sign before the block,
// and the outcome bit.
__device__ __forceinline__ void prep_shots(const TabDev &t, const LrDev &s, const LrArgs &a, uint32_t wg) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t bp = a.b - 1, S = t.S;
  const LrPlan *pl = s.plan + (bp & 3u);
  const uint64_t rand = pl->rand;
  if (rand == 0) return;
  const bool mine = (rand >> lane) & 1u;
  const uint32_t p = mine ? pl->P[lane] : 0u;
  const size_t slot = size_t(bp) * kK + lane;
  for (uint32_t sh = wg * 4 + wave; sh < S; sh += a.nS * 4) {
    const uint64_t r = t.R[size_t(p >> 6) * S + sh];
    uint32_t o = 0;
    if (mine) {
      o = outcome_bit(a.seed, a.circuit, a.shot0 + sh, a.m0 + slot);
      t.out[slot * S + sh] = uint8_t(o);
    }
    const uint64_t rp = __ballot(mine && ((r >> (p & 63)) & 1u)), ob = __ballot(o != 0);
    if (lane == 0) {
      s.RP[sh] = rp;
      s.OB[sh] = ob;
    }
  }
}

__global__ void __launch_bounds__(kPrepThreads) k_lr_prep(TabDev t, LrDev s, LrArgs a) {
  __shared__ uint64_t s_mem[kK + 1];
  __shared__ uint32_t s_a[kPrepThreads], s_b[kK];
  uint32_t wg = blockIdx.x;
  if (wg < a.nR) return prep_rows(t, s, a, wg, s_mem, s_b, s_a);
  wg -= a.nR;
  if (wg < a.nC) return prep_cols(t, s, a, wg, reinterpret_cast<unsigned long long *>(s_mem), s_b);
  wg -= a.nC;
  if (wg < a.nH) return prep_flips(t, s, a, wg);
  wg -= a.nH;
  if (wg < a.nS) return prep_shots(t, s, a, wg);
  wg -= a.nS;
  // start of the pass: pending gate signs into every shot's signs (the sweep
  // launch after this one clears them), the pass's counters
  const size_t nr = size_t(t.Wp) * t.S;
  for (size_t i = size_t(wg) * blockDim.x + threadIdx.x; i < nr; i += size_t(a.nF) * blockDim.x) {
    const uint64_t p = t.P[i / t.S];
    if (p) t.R[i] ^= p;
  }
  for (size_t i = size_t(wg) * blockDim.x + threadIdx.x; i < a.k; i += size_t(a.nF) * blockDim.x)
    t.detpar[i] = t.detY[i] = 0;
  if (wg == 0 && threadIdx.x < 2) s.cnt[threadIdx.x] = 0;
}

// --------------------------------------------------------------- planner ---
// One workgroup finds block b + 1's pivots from the row form of the
// stabilizer rows.  Wave 0 follows the smallest rows that have a bit at all
// (128 of them, or all when there are at most 512) step by step, a row a
// lane: a ballot finds the pivot, a lane read gives its bits.  The other rows
// are needed only when none of those has the step's bit and there are more
// rows: then every wave replays the steps so far on its rows (in registers,
// from where its last search left them) and searches them.
struct PlanShared {
  uint64_t we[kWindow], rx[kK], sv[kSweepWaves];
  uint32_t wi[kWindow], cnt[kSweepWaves], sr[kSweepWaves], cmd;
};

template <int RW>
struct PlanRows {
  uint64_t e[RW > 0 ? RW : 1];
  uint32_t done;   // steps already replayed
  uint32_t i0, i1; // this wave's stabilizer words
};

__device__ __forceinline__ uint64_t plan_load(const TabDev &t, const LrDev &s, uint32_t i, uint32_t lane) {
  const uint32_t w = (t.n >> 6) + i;
  const uint64_t v = s.Bt[size_t(w) * 64 + lane];
  return (w * 64 + lane >= t.n) ? v : 0ull;   // the first word may hold destabilizer rows too
}

// Smallest row of this wave with bit tt after steps 0 .. tt - 1, into sr / sv.
template <int RW>
__device__ __forceinline__ void plan_search(const TabDev &t, const LrDev &s, PlanRows<RW> &r, PlanShared &sh,
                                            uint32_t tt, uint32_t wave, uint32_t lane) {
  uint32_t row = kNone;
  uint64_t val = 0;
  if constexpr (RW > 0) {
    for (uint32_t d = r.done; d < tt; ++d) {
      const uint64_t rx = rdlane64(sh.rx[d], 0);
      if (rx == 0) continue;
#pragma unroll
      for (int k = 0; k < RW; ++k) r.e[k] = xor_if(r.e[k], rx, bit_mask(r.e[k], d));
    }
    r.done = tt;
#pragma unroll
    for (int k = 0; k < RW; ++k) {
      const uint64_t bal = __ballot((r.e[k] >> tt) & 1u);
      if (bal && row == kNone) {
        const uint32_t l = uint32_t(__builtin_ctzll(bal));
        row = ((t.n >> 6) + r.i0 + k) * 64 + l;
        val = rdlane64(r.e[k], l);
      }
    }
  } else {
    for (uint32_t i = r.i0; i < r.i1 && row == kNone; ++i) {
      uint64_t e = plan_load(t, s, i, lane);
      for (uint32_t d = 0; d < tt; ++d) e = xor_if(e, rdlane64(sh.rx[d], 0), bit_mask(e, d));
      const uint64_t bal = __ballot((e >> tt) & 1u);
      if (bal) {
        const uint32_t l = uint32_t(__builtin_ctzll(bal));
        row = ((t.n >> 6) + i) * 64 + l;
        val = rdlane64(e, l);
      }
    }
  }
  if (lane == 0) {
    sh.sr[wave] = row;
    sh.sv[wave] = val;
  }
}

// Wave 0's state: the followed rows' bits in halves, and per lane t step t's
// results (pos: window position of the pivot, or its row | 1 << 31).
template <int R>
struct PlanWindow {
  uint32_t el[R], eh[R];
};
struct PlanSteps {
  uint32_t pos, rxl, rxh;
};

__device__ __forceinline__ uint32_t sbit(uint32_t v, uint32_t t) {   // all ones where bit t (< 32) is set
  return uint32_t(__builtin_amdgcn_sbfe(int(v), t, 1));
}

// Steps t0 .. of half H (bits 32 H ..) while a window row has the step's bit;
// returns the first step without one, or t1.  A step is one chain of
// dependent instructions: bit test, ballot, first lane, its bits by lane
// read, XOR.
template <int R, int H>
__device__ __forceinline__ uint32_t plan_run(PlanWindow<R> &w, PlanSteps &st, uint32_t t0, uint32_t t1,
                                             uint32_t lane) {
  uint32_t t = t0;
  auto apply = [&](uint32_t tb, uint32_t rl, uint32_t rh, uint32_t pos) {
    const uint32_t xl = H ? rl : rl & ~(1u << tb), xh = H ? rh & ~(1u << tb) : rh;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const uint32_t m = sbit(H ? w.eh[i] : w.el[i], tb);
      w.el[i] = bop3<LUT_AND_XOR>(xl, m, w.el[i]);
      w.eh[i] = bop3<LUT_AND_XOR>(xh, m, w.eh[i]);
    }
    const bool me = lane == t;
    st.rxl = me ? xl : st.rxl;
    st.rxh = me ? xh : st.rxh;
    st.pos = me ? pos : st.pos;
  };
  for (;;) {
    // the usual case alone in a loop of its own (taken branches are dear here)
    uint64_t bal;
    while ((bal = __ballot(sbit(H ? w.eh[0] : w.el[0], t & 31) != 0)) != 0) {
      const uint32_t l = uint32_t(__builtin_ctzll(bal));
      apply(t & 31, rdlane(w.el[0], l), rdlane(w.eh[0], l), l);
      if (++t >= t1) return t;
    }
    uint32_t l = 0, pos = 0, rl = 0, rh = 0;
#pragma unroll
    for (int i = 1; i < R; ++i) {
      if (bal) break;   // wave-uniform
      bal = __ballot(sbit(H ? w.eh[i] : w.el[i], t & 31) != 0);
      l = uint32_t(__builtin_ctzll(bal | (1ull << 63)));
      rl = rdlane(w.el[i], l);
      rh = rdlane(w.eh[i], l);
      pos = uint32_t(i) * 64 + l;
    }
    if (bal == 0) return t;
    apply(t & 31, rl, rh, pos);
    if (++t >= t1) return t;
  }
}

// A pivot found outside the window: the same updates.
template <int R>
__device__ __forceinline__ void plan_apply(PlanWindow<R> &w, PlanSteps &st, uint32_t t, uint32_t row, uint64_t rb,
                                           uint32_t lane) {
  const uint64_t rx = rb & ~lbit(t);
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint64_t v = xor_if(pair64(w.el[i], w.eh[i]), rx, bit_mask(pair64(w.el[i], w.eh[i]), t));
    w.el[i] = uint32_t(v);
    w.eh[i] = uint32_t(v >> 32);
  }
  if (lane == t) {
    st.rxl = uint32_t(rx);
    st.rxh = uint32_t(rx >> 32);
    st.pos = row | 0x80000000u;
  }
}

// Steps t0 .. kb - 1 following the first 64 R rows (replaying the steps before
// t0).  Returns kb, or the step at which a larger window of `total` rows
// would do without a search.
template <int RW, int R>
__device__ __forceinline__ uint32_t plan_steps(const TabDev &t, const LrDev &s, PlanRows<RW> &r, PlanShared &sh,
                                               uint32_t t0, uint32_t kb, uint32_t total, uint32_t lane,
                                               PlanSteps &st) {
  PlanWindow<R> w;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint64_t e = uint32_t(i) * 64 + lane < total ? sh.we[i * 64 + lane] : 0ull;
    w.el[i] = uint32_t(e);
    w.eh[i] = uint32_t(e >> 32);
  }
  for (uint32_t d = 0; d < t0; ++d) {
    const uint64_t rx = pair64(rdlane(st.rxl, d), rdlane(st.rxh, d));
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const uint64_t e = pair64(w.el[i], w.eh[i]), v = xor_if(e, rx, bit_mask(e, d));
      w.el[i] = uint32_t(v);
      w.eh[i] = uint32_t(v >> 32);
    }
  }
  uint32_t tt = t0;
  while (tt < kb) {
    if (tt < 32) tt = plan_run<R, 0>(w, st, tt, min(kb, 32u), lane);
    if (tt >= 32 && tt < kb) tt = plan_run<R, 1>(w, st, tt, kb, lane);
    if (tt == kb) break;
    // no window row has the bit
    if (total > uint32_t(R) * 64) {
      if (total <= kWindow) return tt;
      sh.rx[lane] = pair64(st.rxl, st.rxh);
      if (lane == 0) sh.cmd = tt + 1;
      __syncthreads();
      plan_search<RW>(t, s, r, sh, tt, 0, lane);
      __syncthreads();
      const uint32_t cr = lane < kSweepWaves ? sh.sr[lane] : kNone;
      const uint64_t cv = lane < kSweepWaves ? sh.sv[lane] : 0ull;
      const uint64_t bal = __ballot(cr != kNone);   // waves hold ascending rows
      if (bal) {
        const uint32_t l = uint32_t(__builtin_ctzll(bal));
        plan_apply<R>(w, st, tt, rdlane(cr, l), rdlane64(cv, l), lane);
      }
    }
    ++tt;   // without a pivot: deterministic
  }
  return kb;
}

template <int RW>
__device__ __forceinline__ void plan_block(const TabDev &t, const LrDev &s, const LrArgs &a, PlanShared &sh) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t bn = a.b + 1, base = bn * kK, kb = min(kK, a.k - base);
  const uint32_t nsw = t.W - (t.n >> 6), per = (nsw + kSweepWaves - 1) / kSweepWaves;
  PlanRows<RW> r;
  r.done = 0;
  r.i0 = min(nsw, wave * per);
  r.i1 = min(nsw, r.i0 + per);
  uint32_t mycnt = 0;
  if constexpr (RW > 0) {
#pragma unroll
    for (int k = 0; k < RW; ++k) r.e[k] = r.i0 + k < r.i1 ? plan_load(t, s, r.i0 + k, lane) : 0ull;
#pragma unroll
    for (int k = 0; k < RW; ++k) mycnt += uint32_t(__popcll(__ballot(r.e[k] != 0)));
  } else {
    for (uint32_t i = r.i0; i < r.i1; ++i) mycnt += uint32_t(__popcll(__ballot(plan_load(t, s, i, lane) != 0)));
  }
  if (lane == 0) sh.cnt[wave] = mycnt;
  if (tid == 0) sh.cmd = 0;
  __syncthreads();
  uint32_t at = 0, total = 0;
  for (uint32_t v = 0; v < kSweepWaves; ++v) {
    if (v < wave) at += sh.cnt[v];
    total += sh.cnt[v];
  }
  at = __builtin_amdgcn_readfirstlane(at);
  total = __builtin_amdgcn_readfirstlane(total);
  // the first rows with a bit, in order
  auto fill = [&](uint64_t e, uint32_t i) {
    const uint64_t bal = __ballot(e != 0);
    const uint32_t pos = at + uint32_t(__popcll(bal & (lbit(lane) - 1)));
    if (e != 0 && pos < kWindow) {
      sh.we[pos] = e;
      sh.wi[pos] = ((t.n >> 6) + i) * 64 + lane;
    }
    at += uint32_t(__popcll(bal));
  };
  if constexpr (RW > 0) {
#pragma unroll
    for (int k = 0; k < RW; ++k)
      if (at < kWindow) fill(r.e[k], r.i0 + k);
  } else {
    for (uint32_t i = r.i0; i < r.i1 && at < kWindow; ++i) fill(plan_load(t, s, i, lane), i);
  }
  __syncthreads();
  if (wave != 0) {   // searches on request
    for (;;) {
      __syncthreads();
      const uint32_t cmd = __builtin_amdgcn_readfirstlane(sh.cmd);
      if (cmd == 0) return;
      plan_search<RW>(t, s, r, sh, cmd - 1, wave, lane);
      __syncthreads();
    }
  }
  PlanSteps st{kNone, 0, 0};
  // 128 rows do in a dense tableau (64 random bits each); where they fall
  // short and there are at most 512, all of them are followed
  const uint32_t tt = plan_steps<RW, 2>(t, s, r, sh, 0, kb, total, lane, st);
  if (tt < kb) plan_steps<RW, kWindow / 64>(t, s, r, sh, tt, kb, total, lane, st);
  const uint32_t P = st.pos == kNone ? kNone : (st.pos & 0x80000000u) ? st.pos & 0x7fffffffu : sh.wi[st.pos];
  const uint64_t RX = pair64(st.rxl, st.rxh);
  if (lane == 0) sh.cmd = 0;
  __syncthreads();
  LrPlan *pl = s.plan + (bn & 3u);
  const uint64_t rand = __ballot(P != kNone);
  pl->P[lane] = P;
  pl->RX[lane] = RX;
  if (lane < kb) {
    t.kind[base + lane] = P != kNone ? 1 : 0;
    if (P == kNone) s.dets[s.cnt[0] + uint32_t(__popcll(~rand & (lbit(lane) - 1)))] = base + lane;
  }
  if (lane == 0) {
    pl->rand = rand;
    const uint32_t nr = uint32_t(__popcll(rand));
    if (nr) atomicAdd(&t.state[ST_RANDOM_CNT], nr);
    if (kb > nr) {
      atomicAdd(&t.state[ST_DET_CNT], kb - nr);
      s.cnt[0] += kb - nr;
    }
  }
}

// ----------------------------------------------------------------- sweep ---
// A workgroup updates a tile of up to 64 row words in a share of the columns.
// Its 64 U columns are laid out as tables in LDS, all 16 sums of each group
// of 4, so that a column takes one 16-byte read per group, plane and two
// words instead of four masked XORs a word.  A column is held by LP lanes (two
// words each; LP = 32, so two columns a wave, from 64 words on), each with
// that column's pivot-row bits, so there is no scalar work per column.  (The
// masked form, bits as scalar masks, spent two scalar instructions per mask,
// one scalar unit for the four SIMDs: 51 us a launch at n = 10,000, now 21.)
struct SweepShared {
  uint64_t tab[16][16][64];                  // [group][sum][word]
  uint64_t kill[64];                         // rows p_t and p_t - n
  unsigned long long e0[64], e1[64], zx[64];
  uint32_t P[kK], any;
};

__device__ __forceinline__ void xor3(uint4 &a, const uint4 b, const uint4 c) {
  a.x = bop3<LUT_XOR3>(a.x, b.x, c.x);
  a.y = bop3<LUT_XOR3>(a.y, b.y, c.y);
  a.z = bop3<LUT_XOR3>(a.z, b.z, c.z);
  a.w = bop3<LUT_XOR3>(a.w, b.w, c.w);
}
__device__ __forceinline__ uint4 as4(uint64_t a, uint64_t b) {
  return make_uint4(uint32_t(a), uint32_t(a >> 32), uint32_t(b), uint32_t(b >> 32));
}

__device__ __forceinline__ void lr_sweep(const TabDev &t, const LrDev &s, const LrArgs &a, uint32_t wg, SweepShared &sh) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const LrPlan *pl = s.plan + (a.b & 3u);
  if (pl->rand == 0) return;   // nothing random in this block
  const uint32_t tile = wg % a.T, cg = wg / a.T, n = t.n, W = t.W, w0 = tile * 64;
  if (tid < 64) {
    sh.kill[tid] = 0;
    sh.e0[tid] = sh.e1[tid] = sh.zx[tid] = 0;
    sh.P[tid] = pl->P[tid];
  }
  if (tid == 0) sh.any = 0;
  __syncthreads();
  {
    // thread (word, group): the 16 sums of its four U words
    const uint32_t wl = lane, g = wave;
    uint64_t c[16];
    c[0] = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i)
      c[1u << i] = w0 + wl < W ? s.U[a.b & 1u][size_t(w0 + wl) * kK + 4 * g + i] : 0ull;
    uint64_t any = c[1] | c[2] | c[4] | c[8];
#pragma unroll
    for (uint32_t v = 1; v < 16; ++v) c[v] = c[v & (v - 1)] ^ c[v & (0u - v)];
#pragma unroll
    for (uint32_t v = 0; v < 16; ++v) sh.tab[g][v][wl] = c[v];
    if (tid < kK && sh.P[tid] != kNone) {
      const uint32_t p = sh.P[tid], r = (p >> 6) - w0, r2 = ((p - n) >> 6) - w0;
      if (r < 64) atomicOr(reinterpret_cast<unsigned long long *>(&sh.kill[r]), (unsigned long long)lbit(p));
      if (r2 < 64) atomicOr(reinterpret_cast<unsigned long long *>(&sh.kill[r2]), (unsigned long long)lbit(p - n));
      any |= uint64_t(r < 64 || r2 < 64);
    }
    if (__ballot(any != 0) && lane == 0) sh.any = 1;
  }
  __syncthreads();
  if (sh.any) {   // (otherwise no row of this tile changes)
    const uint32_t wl = 2 * (lane & ((1u << a.lp) - 1u)), cl = lane >> a.lp;   // this lane's words wl, wl + 1; column slot
    const bool live = w0 + wl < W;   // (an odd W's second word is padding: zero, and stays so)
    const uint32_t step = kSweepWaves << (6 - a.lp);   // columns the workgroup takes at a time
    const uint32_t c0 = uint32_t(uint64_t(cg) * n / a.CG), c1 = uint32_t(uint64_t(cg + 1) * n / a.CG);
    const uint4 kl = as4(sh.kill[wl], sh.kill[wl + 1]);
    const unsigned char *tb = reinterpret_cast<const unsigned char *>(&sh.tab[0][0][wl]);
    constexpr uint32_t B = 2;   // columns in flight ahead of the one at hand
    struct Col {
      uint4 x, z;
      uint64_t bx, bz;
      uint32_t me;
    } nx[B];
    auto fetch = [&](Col &d, uint32_t c) {
      const bool ok = c < c1 && live;
      const size_t at = ok ? size_t(c) * t.Wp + w0 + wl : 0, ac = ok ? c : 0;
      d.x = *reinterpret_cast<const uint4 *>(t.X + at);
      d.z = *reinterpret_cast<const uint4 *>(t.Z + at);
      d.bx = s.BX[ac];
      d.bz = s.BZ[ac];
      d.me = s.ME[ac];
      if (!ok) d.bx = d.bz = 0;
    };
    uint4 e0 = make_uint4(0, 0, 0, 0), e1 = e0, zx = e0;
    const uint32_t cw = c0 + (wave << (6 - a.lp)) + cl;
#pragma unroll
    for (uint32_t i = 0; i < B; ++i) fetch(nx[i], cw + i * step);
    for (uint32_t cb = c0; cb < c1; cb += B * step) {
#pragma unroll
      for (uint32_t i = 0; i < B; ++i) {
        const uint32_t c = cw + (cb - c0) + i * step;
        const Col d = nx[i];
        fetch(nx[i], c + B * step);
        uint4 dx = make_uint4(0, 0, 0, 0), dz = dx;
        if (__ballot((d.bx | d.bz) != 0)) {
#pragma unroll
          for (uint32_t g = 0; g < 16; g += 2) {
            const uint32_t xs = uint32_t(d.bx >> (4 * g)), zs = uint32_t(d.bz >> (4 * g));
            auto get = [&](uint32_t gg, uint32_t nib) {
              return *reinterpret_cast<const uint4 *>(tb + gg * (16 * 64 * 8) + nib * (64 * 8));
            };
            xor3(dx, get(g, xs & 15u), get(g + 1, (xs >> 4) & 15u));
            xor3(dz, get(g, zs & 15u), get(g + 1, (zs >> 4) & 15u));
          }
        }
        if (c < c1 && live) {
          uint32_t ox[4] = {d.x.x, d.x.y, d.x.z, d.x.w}, oz[4] = {d.z.x, d.z.y, d.z.z, d.z.w};
          uint32_t px[4] = {dx.x, dx.y, dx.z, dx.w}, pz[4] = {dz.x, dz.y, dz.z, dz.w};
          uint32_t *f0 = &e0.x, *f1 = &e1.x, *fz = &zx.x;
          const uint32_t kw[4] = {kl.x, kl.y, kl.z, kl.w};
          uint32_t chx = 0, chz = 0, pz_bit[4] = {0, 0, 0, 0};
          if (d.me) {   // this column was measured: its pivot row becomes Z on it
            const uint32_t p = sh.P[d.me - 1], h = (p >> 5) - 2 * (w0 + wl);
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
              if (h == q) pz_bit[q] = 1u << (p & 31);
          }
#pragma unroll
          for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t kx = ox[q] & ~kw[q], kz = oz[q] & ~kw[q];
            px[q] = (kx ^ px[q]);
            const uint32_t dq = px[q] ^ kx;
            pz[q] = (kz ^ pz[q]) | pz_bit[q];
            // (Y_old - Y_new) mod 4 in two planes, and z_old.(x_new ^ x_old)
            const uint32_t yn = px[q] & pz[q], anti = (kx & kz) ^ yn;
            f1[q] = bop3<LUT_AND_XOR>(anti, f0[q] ^ yn, f1[q]);
            f0[q] ^= anti;
            fz[q] = bop3<LUT_AND_XOR>(kz, dq, fz[q]);
            chx |= px[q] ^ ox[q];
            chz |= pz[q] ^ oz[q];
          }
          const size_t at = size_t(c) * t.Wp + w0 + wl;
          if (chx) *reinterpret_cast<uint4 *>(t.X + at) = make_uint4(px[0], px[1], px[2], px[3]);
          if (chz) *reinterpret_cast<uint4 *>(t.Z + at) = make_uint4(pz[0], pz[1], pz[2], pz[3]);
        }
      }
    }
    // the lanes' counters summed in LDS: mod-4 addition with the low plane's
    // carry taken from the atomic XOR's old value
    auto add = [&](uint32_t w, uint64_t v0, uint64_t v1, uint64_t vz) {
      const unsigned long long old = atomicXor(&sh.e0[w], (unsigned long long)v0);
      atomicXor(&sh.e1[w], (unsigned long long)(v1 ^ (old & v0)));
      atomicXor(&sh.zx[w], (unsigned long long)vz);
    };
    add(wl, pair64(e0.x, e0.y), pair64(e1.x, e1.y), pair64(zx.x, zx.y));
    add(wl + 1, pair64(e0.z, e0.w), pair64(e1.z, e1.w), pair64(zx.z, zx.w));
  }
  __syncthreads();
  if (tid < 64 && w0 + tid < W) {
    uint64_t *part = s.part + size_t(cg) * 3 * t.Wp + w0 + tid;
    part[0] = sh.e0[tid];
    part[t.Wp] = sh.e1[tid];
    part[2 * size_t(t.Wp)] = sh.zx[tid];
  }
}

// The signs of block b - 1: r = [kept] r ^ H ^ sum over pivots with r = 1 of
// U_t, the pivot rows take the outcomes.
__device__ __forceinline__ void lr_signs(const TabDev &t, const LrDev &s, const LrArgs &a, uint32_t wg, uint32_t *sP) {
  const uint32_t bp = a.b - 1, S = t.S;
  const LrPlan *pl = s.plan + (bp & 3u);
  if (pl->rand == 0) return;
  if (threadIdx.x < kK) sP[threadIdx.x] = pl->P[threadIdx.x];
  __syncthreads();
  const size_t total = size_t(t.W) * S;
  for (size_t i = size_t(wg) * kSweepThreads + threadIdx.x; i < total; i += size_t(a.nA) * kSweepThreads) {
    const uint32_t w = uint32_t(i / S), sh = uint32_t(i % S);
    const uint64_t rp = s.RP[sh], cons = s.CW[w];
    const ulonglong2 *U = reinterpret_cast<const ulonglong2 *>(s.U[bp & 1u] + size_t(w) * kK);
    uint64_t v = (t.R[i] & ~s.KW[w]) ^ s.H[w];
#pragma unroll 8
    for (uint32_t st = 0; st < kK / 2; ++st) {
      const ulonglong2 u = U[st];
      v = xor_if(v, u.x, bit_mask(rp, 2 * st));
      v = xor_if(v, u.y, bit_mask(rp, 2 * st + 1));
    }
    if (cons) {
      const uint64_t ob = s.OB[sh];
      for (uint32_t st = 0; st < kK; ++st) {
        const uint32_t p = sP[st];
        if (p != kNone && (p >> 6) == w && ((ob >> st) & 1u)) v |= lbit(p);
      }
    }
    t.R[i] = v;
  }
}

// Gram rows and Y counts of block b over the prep kernel's workgroups.
__device__ __forceinline__ void lr_gram(const TabDev &t, const LrDev &s, const LrArgs &a, uint64_t *sg, uint32_t *sy) {
  const uint32_t tid = threadIdx.x, st = tid & 63, sl = tid >> 6;
  if (s.plan[a.b & 3u].rand == 0) return;
  if (tid < kK) {
    sg[tid] = 0;
    sy[tid] = 0;
  }
  __syncthreads();
  uint64_t g = 0;
  uint32_t y = 0;
#pragma unroll 4
  for (uint32_t q = sl; q < a.nC; q += kSweepWaves) {
    g ^= s.Gp[size_t(q) * kK + st];
    y += s.Yp[size_t(q) * kK + st];
  }
  atomicXor(reinterpret_cast<unsigned long long *>(&sg[st]), (unsigned long long)g);
  atomicAdd(&sy[st], y);
  if (sl == 0) {   // the pivot rows' support
    unsigned long long sup = 0;
    for (uint32_t q = st; q < a.nC; q += 64) sup += s.Sp[q];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sup += __shfl_xor(sup, off);
    if (st == 0) atomicAdd(reinterpret_cast<unsigned long long *>(t.state + ST_SUPPORT), sup);
  }
  __syncthreads();
  if (tid < kK) {
    s.G[tid] = sg[tid];
    s.Y[tid] = sy[tid] & 3u;
  }
}

// Columns with an x bit in a stabilizer row, for the deterministic outcomes.
__device__ __forceinline__ void lr_columns(const TabDev &t, const LrDev &s, const LrArgs &a, uint32_t wg) {
  if (s.cnt[0] == 0) return;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t c = wg * kSweepWaves + wave; c < t.n; c += a.CG * kSweepWaves) {
    uint64_t any = 0;
    for (uint32_t w = (t.n >> 6) + lane; w < t.W; w += 64) {
      uint64_t v = t.X[size_t(c) * t.Wp + w];
      if (w == (t.n >> 6)) v &= ~0ull << (t.n & 63);
      any |= v;
    }
    if (__ballot(any != 0) && lane == 0) s.list[atomicAdd(&s.cnt[1], 1u)] = c;
  }
}

template <int RW>
__global__ void __launch_bounds__(kSweepThreads) k_lr_sweep(TabDev t, LrDev s, LrArgs a) {
  __shared__ union {
    SweepShared sweep;
    PlanShared plan;
    struct {
      uint64_t g[kK];
      uint32_t y[kK];
    } gram;
    uint32_t P[kK];
  } sh;
  const int32_t b = int32_t(a.b), nb = int32_t((a.k + kK - 1) / kK);
  uint32_t wg = blockIdx.x;
  if (wg == 0) {
    if (b + 1 < nb) plan_block<RW>(t, s, a, sh.plan);
    return;
  }
  if (wg == 1) {
    if (b >= 0 && b < nb) return lr_gram(t, s, a, sh.gram.g, sh.gram.y);
    if (b < 0)   // the pending signs were folded by the launch before this one
      for (uint32_t i = threadIdx.x; i < t.Wp; i += kSweepThreads) t.P[i] = 0;
    return;
  }
  wg -= 2;
  if (wg < a.nA) return lr_signs(t, s, a, wg, sh.P);
  wg -= a.nA;
  if (b < nb) lr_sweep(t, s, a, wg, sh.sweep);
  else lr_columns(t, s, a, wg);
}

// --------------------------------------------------- deterministic outcomes ---
// Measurement m's product rows in word w: the destabilizer half of its
// column, shifted up by n rows.
__device__ __forceinline__ uint64_t det_rows(const TabDev &t, const uint64_t *col, uint32_t w) {
  const uint32_t w0 = t.n >> 6, sh = t.n & 63, i = w - w0;
  auto src = [&](uint32_t j) -> uint64_t {
    if (j >= t.NW) return 0ull;
    uint64_t v = col[j];
    if (j == w0 && sh) v &= lbit(sh) - 1;
    return v;
  };
  uint64_t v = src(i) << sh;
  if (sh && i) v |= src(i - 1) >> (64 - sh);
  return v;
}

// The x/z terms of the ordered product of the rows (-1)^r i^(x.z) X^x Z^z: the
// pairs s < t with z_s x_t, and the Y count.  They come from the columns with
// x bits in stabilizer rows (none after a measure-all), which the grid's x
// dimension shares out; its y dimension shares out the measurements.  A wave
// takes as many columns at a time as their row words fill lanes (n = 97: 16.5
// us a launch with one at a time, now 3.9).
__global__ void __launch_bounds__(256) k_lr_det_terms(TabDev t, LrDev s, LrArgs a) {
  const uint32_t nd = s.cnt[0], ncol = s.cnt[1];
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t w0 = t.n >> 6, W = t.W;
  // a column's words w0 .. W in 2^lg neighbouring lanes, and in turns of 64
  const uint32_t lg = W - w0 >= 64 ? 6u : 32u - uint32_t(__builtin_clz(max(W - w0, 2u) - 1));
  const uint32_t grp = lane >> lg, lw = lane & ((1u << lg) - 1), per = 64u >> lg;
  const uint64_t mine = lg == 6 ? ~0ull : (lbit(1u << lg) - 1) << (grp << lg);   // this column's lanes
  const uint32_t wv = (blockIdx.x * 4 + wave) * per, nwv = gridDim.x * 4 * per;
  if (wv >= ncol) return;
  for (uint32_t d = blockIdx.y; d < nd; d += gridDim.y) {
    const uint32_t m = s.dets[d];
    const uint64_t *col = t.X + size_t(a.q[m]) * t.Wp;
    uint32_t y = 0, par = 0;
    for (uint32_t ic = wv + grp; ic - grp < ncol; ic += nwv) {
      const bool on = ic < ncol;
      const size_t at = size_t(s.list[on ? ic : 0]) * t.Wp;
      uint32_t carry = 0;   // z parity of the product rows in earlier words
#pragma unroll 2
      for (uint32_t wb = w0; wb < W; wb += 64) {
        const uint32_t w = wb + lw;
        const uint64_t tm = on && w < W ? det_rows(t, col, w) : 0ull;
        const uint64_t xt = tm ? t.X[at + w] & tm : 0ull, zt = tm ? t.Z[at + w] & tm : 0ull;
        y += uint32_t(__popcll(xt & zt));
        uint64_t pre = zt << 1;   // exclusive prefix parity inside the word
        pre ^= pre << 1; pre ^= pre << 2; pre ^= pre << 4;
        pre ^= pre << 8; pre ^= pre << 16; pre ^= pre << 32;
        const uint64_t zb = __ballot(__popcll(zt) & 1) & mine;
        const uint32_t cin = (carry ^ uint32_t(__popcll(zb & (lbit(lane) - 1)))) & 1u;
        par ^= (uint32_t(__popcll(xt & pre)) & 1u) ^ (cin & uint32_t(__popcll(xt)) & 1u);
        carry ^= uint32_t(__popcll(zb)) & 1u;
      }
    }
    const uint64_t pb = __ballot(par & 1u);
    for (int off = 32; off > 0; off >>= 1) y += __shfl_xor(y, off);
    if (lane == 0) {
      if (y) atomicAdd(&t.detY[m], y);
      if (__popcll(pb) & 1) atomicXor(&t.detpar[m], 1u);
    }
  }
}

// One workgroup per deterministic measurement (of those it meets at its
// stride): outcome = XOR of the product rows' signs ^ the x/z terms.
__global__ void __launch_bounds__(256) k_lr_det(TabDev t, LrDev s, LrArgs a) {
  __shared__ uint32_t s_out[256];
  const uint32_t nd = s.cnt[0], tid = threadIdx.x, W = t.W, S = t.S, w0 = t.n >> 6;
  for (uint32_t d = blockIdx.x; d < nd; d += gridDim.x) {
    const uint32_t m = s.dets[d];
    const uint64_t *col = t.X + size_t(a.q[m]) * t.Wp;
    const uint32_t y = t.detY[m], terms = t.detpar[m] ^ (y >> 1);
    // 256 threads over the shots, several threads a shot when there are fewer
    const uint32_t ss = min(S, 256u), per = 256 / ss, my = tid / ss;
    for (uint32_t s0 = 0; s0 < S; s0 += ss) {
      const uint32_t si = s0 + tid % ss;
      s_out[tid] = 0;
      __syncthreads();
      if (my < per && si < S) {
        uint32_t rt = 0;
        for (uint32_t w = w0 + my; w < W; w += per)
          rt ^= uint32_t(__popcll(det_rows(t, col, w) & t.R[size_t(w) * S + si])) & 1u;
        if (rt) atomicXor(&s_out[tid % ss], 1u);
      }
      __syncthreads();
      if (tid < ss && si < S) t.out[size_t(m) * S + si] = uint8_t((s_out[tid] ^ terms) & 1u);
      __syncthreads();
    }
    if (tid == 0 && (y & 1u)) atomicAdd(&t.state[ST_ANOMALY], 1u);   // odd Y count
  }
}

// ------------------------------------------------------------------ host ---
static uint32_t div_up(size_t a, size_t b) { return uint32_t((a + b - 1) / b); }

// Sweep shape: row tiles of 64 words, or the whole column by fewer lanes, and
// one workgroup per compute unit (the tables take most of its LDS), the
// planner and the sign work aside; at least two rounds of columns each.
struct LrShape {
  uint32_t T, lp, CG, nC, nA;
};
static LrShape lr_shape(uint32_t n, uint32_t S, uint32_t num_cus) {
  LrShape r;
  const uint32_t W = (2 * n + 63) / 64;
  r.T = div_up(W, 64);
  r.lp = 0;
  while (r.lp < 5 && (2u << r.lp) < W) ++r.lp;
  r.nA = std::min(div_up(size_t(W) * S, kSweepThreads), std::max(1u, num_cus / 8));
  const uint32_t wgs = num_cus > 2 + r.nA ? num_cus - 2 - r.nA : 1;
  const uint32_t most = div_up(n, 2 * (kSweepWaves << (6 - r.lp)));
  r.CG = std::max(1u, std::min(wgs / r.T, most));
  r.nC = std::min(div_up(n, 4 * kPrepCols), 512u);
  return r;
}

size_t lr_scratch_bytes(const Dims &d, uint32_t num_cus) {
  LrDev s;
  return lr_scratch_bind(d, num_cus, nullptr, s);
}

size_t lr_scratch_bind(const Dims &d, uint32_t num_cus, uint8_t *base, LrDev &s) {
  const LrShape h = lr_shape(d.n, d.S, num_cus);
  size_t cur = 0;
  auto take = [&](size_t bytes) {
    uint8_t *at = base + cur;
    cur = align256(cur + bytes);
    return at;
  };
  s.plan = reinterpret_cast<LrPlan *>(take(4 * sizeof(LrPlan)));
  s.Bt = reinterpret_cast<uint64_t *>(take(size_t(d.W) * 64 * 8));
  s.U[0] = reinterpret_cast<uint64_t *>(take(size_t(d.W) * kK * 8));
  s.U[1] = reinterpret_cast<uint64_t *>(take(size_t(d.W) * kK * 8));
  s.BX = reinterpret_cast<uint64_t *>(take(size_t(d.n) * 8));
  s.BZ = reinterpret_cast<uint64_t *>(take(size_t(d.n) * 8));
  s.ME = reinterpret_cast<uint32_t *>(take(size_t(d.n) * 4));
  s.Gp = reinterpret_cast<uint64_t *>(take(size_t(h.nC) * kK * 8));
  s.Sp = reinterpret_cast<unsigned long long *>(take(size_t(h.nC) * 8));
  s.Yp = reinterpret_cast<uint32_t *>(take(size_t(h.nC) * kK * 4));
  s.G = reinterpret_cast<uint64_t *>(take(kK * 8));
  s.Y = reinterpret_cast<uint32_t *>(take(kK * 4));
  s.part = reinterpret_cast<uint64_t *>(take(size_t(h.CG) * 3 * d.Wp * 8));
  s.H = reinterpret_cast<uint64_t *>(take(size_t(d.Wp) * 8));
  s.KW = reinterpret_cast<uint64_t *>(take(size_t(d.Wp) * 8));
  s.CW = reinterpret_cast<uint64_t *>(take(size_t(d.Wp) * 8));
  s.RP = reinterpret_cast<uint64_t *>(take(size_t(d.S) * 8));
  s.OB = reinterpret_cast<uint64_t *>(take(size_t(d.S) * 8));
  s.list = reinterpret_cast<uint32_t *>(take(size_t(d.n) * 4));
  s.dets = reinterpret_cast<uint32_t *>(take(size_t(d.n) * 4));
  s.cnt = reinterpret_cast<uint32_t *>(take(2 * 4));
  return cur;
}

hipError_t launch_measure_lr(const TabDev &t, const LrDev &s, const uint32_t *dev_qubits, uint32_t k, uint64_t seed,
                             uint64_t circuit, uint64_t shot0, uint64_t m0, int num_cus, hipStream_t st,
                             Profiler *prof) {
  if (k == 0) return hipSuccess;
  const LrShape h = lr_shape(t.n, t.S, uint32_t(num_cus));
  const int32_t nb = int32_t((k + kK - 1) / kK);
  // stabilizer words per planner wave: registers for up to 32 of them
  const uint32_t per = div_up(t.W - (t.n >> 6), kSweepWaves);
  LrArgs a{};
  a.q = dev_qubits;
  a.k = k;
  a.CG = h.CG;
  a.T = h.T;
  a.lp = h.lp;
  a.seed = seed;
  a.circuit = circuit;
  a.shot0 = shot0;
  a.m0 = m0;
  hipError_t e;
  for (int32_t b = -1; b <= nb; ++b) {
    a.b = uint32_t(b);
    a.nR = b < nb ? div_up(t.W, 4) : 0;
    a.nC = b >= 0 && b < nb ? h.nC : 0;
    a.nH = b > 0 ? div_up(t.W, 4) : 0;
    a.nS = b > 0 ? std::min(div_up(t.S, 4), 256u) : 0;
    a.nF = b < 0 ? std::min(div_up(size_t(t.Wp) * t.S, kPrepThreads), 256u) : 0;
    if (prof) prof->begin(PK_SELECT, st);
    k_lr_prep<<<a.nR + a.nC + a.nH + a.nS + a.nF, kPrepThreads, 0, st>>>(t, s, a);
    if (prof) prof->end(PK_SELECT, st);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    a.nC = h.nC;
    a.nA = b > 0 ? h.nA : 0;
    const uint32_t sweep = b < 0 ? 0 : b < nb ? h.T * h.CG : h.CG;
    const dim3 grid(2 + a.nA + sweep);
    const ProfKind kind = b >= 0 && b < nb ? PK_BLOCKED : PK_FINAL;
    if (prof) prof->begin(kind, st);
    if (per <= 2) k_lr_sweep<2><<<grid, kSweepThreads, 0, st>>>(t, s, a);
    else if (per <= 11) k_lr_sweep<11><<<grid, kSweepThreads, 0, st>>>(t, s, a);
    else if (per <= 32) k_lr_sweep<32><<<grid, kSweepThreads, 0, st>>>(t, s, a);
    else k_lr_sweep<0><<<grid, kSweepThreads, 0, st>>>(t, s, a);
    if (prof) prof->end(kind, st);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (prof) prof->begin(PK_FINAL, st);
  const uint32_t dx = std::min(div_up(t.n, 32), 256u);
  k_lr_det_terms<<<dim3(dx, std::min(k, std::max(4u, 256u / dx))), 256, 0, st>>>(t, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_lr_det<<<std::min(k, 1024u), 256, 0, st>>>(t, s, a);
  if (prof) prof->end(PK_FINAL, st);
  return hipGetLastError();
}

}  // namespace cliff
