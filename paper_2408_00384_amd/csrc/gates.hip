// Tableau initialisation and gate sweeps (column updates).
//
// Gate rules of the phase-space method (paper Sec. 2, after Aaronson &
// Gottesman 2004), applied to 64 rows at once with word-wise bit logic:
//   H(a):        r ^= x_a & z_a;  swap(x_a, z_a)
//   S(a):        r ^= x_a & z_a;  z_a ^= x_a
//   CNOT(a->b):  r ^= x_a & z_b & ~(x_b ^ z_a);  x_b ^= x_a;  z_a ^= z_b
// and the rest of the Clifford gate set (S^dagger, X, Y, Z, CZ, SWAP) in the
// same form; an op word carries one single-qubit Clifford per qubit and one
// two-qubit gate (the encoding and rules are in gate_ops.h).
// Gates on disjoint qubits touch disjoint columns and their sign terms read
// only their own columns, so every op of a layer can run concurrently; the
// sign contributions are XOR-accumulated per thread and flushed once.
#include <string.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "internal.h"

namespace cliff {

// |0...0>: X[j] has bit j (destabilizer j = X_j), Z[j] has bit n+j
// (stabilizer n+j = Z_j); signs, pending flips and the measurement state zero.
// One pass, no memset, so the launch is safe inside a captured graph; at small
// n a launch of its own for the state would cost as much again (100 tableaux
// of n = 500: 414 -> 200 us).
__global__ void __launch_bounds__(256) k_init_zero(TabDev t) {
  const size_t ncol = size_t(t.n) * t.Wp;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < ncol; i += stride) {
    const uint32_t j = uint32_t(i / t.Wp), w = uint32_t(i % t.Wp);
    const uint32_t zr = t.n + j;
    t.X[i] = (w == (j >> 6)) ? (1ull << (j & 63)) : 0ull;
    t.Z[i] = (w == (zr >> 6)) ? (1ull << (zr & 63)) : 0ull;
  }
  const size_t nr = size_t(t.Wp) * t.S;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < nr; i += stride) t.R[i] = 0;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < t.Wp; i += stride) t.P[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < kStateWords) t.state[threadIdx.x] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *t.abort_flag = 0;
}

// R[w][s] ^= P[w] for every shot (pending gate sign flips become real).
__global__ void __launch_bounds__(256) k_fold_pending(TabDev t) {
  const size_t nr = size_t(t.Wp) * t.S;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < nr; i += stride) {
    const uint64_t p = t.P[i / t.S];
    if (p) t.R[i] ^= p;
  }
}

__global__ void __launch_bounds__(256) k_clear_pending(TabDev t) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < t.Wp; i += gridDim.x * blockDim.x)
    t.P[i] = 0;
}

__global__ void __launch_bounds__(64) k_clear_state(TabDev t) {
  if (threadIdx.x < kStateWords) t.state[threadIdx.x] = 0;
}

// One layer of ops on row words w0 .. w1.  Block = 4 waves; lane <-> row word
// (coalesced along the column), wave <-> kLayerOps neighbouring ops at a time,
// whose columns (all distinct) are loaded together.  Bound: memory, or the
// last-level cache where the caller keeps to as many row words as it holds.
// n = 25,000 (312 MB of X and Z, read and written): 120 us a layer with one op
// at a time, 107 with four (5.8 TB/s), 95 in two halves of the row words
// (thirds: 102, quarters: 112; each launch ramps up and drains).
constexpr uint32_t kLayerOps = 4;
__global__ void __launch_bounds__(256) k_gate_layer(TabDev t, const uint64_t *__restrict__ ops, uint32_t nops,
                                                    uint32_t ops_per_block, uint32_t w0, uint32_t w1) {
  __shared__ uint64_t s_r[4][64];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t w = w0 + blockIdx.x * 64 + lane;
  const uint32_t o0 = blockIdx.y * ops_per_block;
  const uint32_t o1 = min(nops, o0 + ops_per_block);
  const size_t Wp = t.Wp;
  uint64_t racc = 0;
  if (w < w1) {
    for (uint32_t o = o0 + wave * kLayerOps; o < o1; o += 4 * kLayerOps) {
      uint64_t op[kLayerOps], xa[kLayerOps], za[kLayerOps], xb[kLayerOps], zb[kLayerOps];
      bool ok[kLayerOps], two[kLayerOps];
#pragma unroll
      for (uint32_t i = 0; i < kLayerOps; ++i) {
        op[i] = o + i < o1 ? ops[o + i] : ~0ull;
        ok[i] = op_valid(op[i], t.n);   // (malformed ops are skipped)
        two[i] = ok[i] && op_pair(op[i]) != PAIR_NONE;
      }
#pragma unroll
      for (uint32_t i = 0; i < kLayerOps; ++i) {
        // (a column that the op has not is read as column 0)
        const size_t a = ok[i] ? op_a(op[i]) : 0, b = two[i] ? op_b(op[i]) : 0;
        xa[i] = t.X[a * Wp + w];
        za[i] = t.Z[a * Wp + w];
        xb[i] = t.X[b * Wp + w];
        zb[i] = t.Z[b * Wp + w];
      }
#pragma unroll
      for (uint32_t i = 0; i < kLayerOps; ++i) {
        if (!ok[i]) continue;
        const size_t a = op_a(op[i]) * Wp + w;
        if (op_ca(op[i])) sq_apply(op_ca(op[i]), xa[i], za[i], racc);
        if (two[i]) {
          const size_t b = op_b(op[i]) * Wp + w;
          if (op_cb(op[i])) sq_apply(op_cb(op[i]), xb[i], zb[i], racc);
          pair_apply(op_pair(op[i]), xa[i], za[i], xb[i], zb[i], racc);
          t.X[b] = xb[i];
          t.Z[b] = zb[i];
        }
        t.X[a] = xa[i];
        t.Z[a] = za[i];
      }
    }
  }
  s_r[wave][lane] = racc;
  __syncthreads();
  if (wave == 0 && w < w1) {
    racc = s_r[0][lane] ^ s_r[1][lane] ^ s_r[2][lane] ^ s_r[3][lane];
    if (racc) atomicXor(reinterpret_cast<unsigned long long *>(t.P + w), (unsigned long long)racc);
  }
}

typedef __attribute__((address_space(1))) const uint64_t GlobalU64;
typedef __attribute__((address_space(1))) const uint32_t GlobalU32;

__device__ __forceinline__ void lds_xor(uint32_t *p, uint32_t v) { atomicXor(p, v); }
__device__ __forceinline__ void lds_xor(uint64_t *p, uint64_t v) {
  atomicXor(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}
__device__ __forceinline__ void lds_xor(U128 *p, U128 v) {
  lds_xor(&p->lo, v.lo);
  lds_xor(&p->hi, v.hi);
}
__device__ __forceinline__ bool nonzero(uint32_t v) { return v != 0; }
__device__ __forceinline__ bool nonzero(uint64_t v) { return v != 0; }
__device__ __forceinline__ bool nonzero(U128 v) { return (v.lo | v.hi) != 0; }

// All layers of a gate stream in one launch.  Gates act row by row, so a
// workgroup that owns a group of rows (32 or 64: the bits of T) of every
// column can apply every layer to them without talking to any other
// workgroup: it loads its row group of X and Z into LDS (2 n sizeof(T)
// bytes), runs the layers with a workgroup barrier between consecutive
// layers, and writes them back once.  Its sign flips stay in registers and
// land in its own part of P.
template <typename T>
__device__ __forceinline__ void apply_op_lds(uint64_t op, uint32_t n, T *sx, T *sz, T &racc) {
  if (!op_valid(op, n)) return;   // malformed op
  const uint32_t a = op_a(op), pair = op_pair(op);
  T xa = sx[a], za = sz[a];
  if (op_ca(op)) sq_apply(op_ca(op), xa, za, racc);
  if (pair != PAIR_NONE) {
    const uint32_t b = op_b(op);
    T xb = sx[b], zb = sz[b];
    if (op_cb(op)) sq_apply(op_cb(op), xb, zb, racc);
    pair_apply(pair, xa, za, xb, zb, racc);
    sx[b] = xb;
    sz[b] = zb;
  }
  sx[a] = xa;
  sz[a] = za;
}

template <typename T>
__device__ __forceinline__ void fused_body(uint64_t *X, uint64_t *Z, uint64_t *P, uint32_t n, uint32_t Wp,
                                           const uint64_t *__restrict__ ops,
                                           const uint32_t *__restrict__ offs, uint32_t depth,
                                           uint32_t unit, T *sx, T *sz, T *s_r) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const size_t cs = size_t(Wp) * 8 / sizeof(T);  // column stride in T words (Wp is a multiple of 8)
  const T *XT = reinterpret_cast<const T *>(X);
  const T *ZT = reinterpret_cast<const T *>(Z);
  for (uint32_t j = tid; j < n; j += nthr) {
    sx[j] = XT[j * cs + unit];
    sz[j] = ZT[j * cs + unit];
  }
  if (tid == 0) *s_r = T{};
  __syncthreads();
  // The op stream and the offsets are read through global-address-space
  // pointers: global (not flat) loads count only in vmcnt, so the LDS waits
  // of a layer do not wait for them.
  const GlobalU64 *gops = (const GlobalU64 *)ops;
  const GlobalU32 *goffs = (const GlobalU32 *)offs;
  // Layer boundaries: lane i of every wave holds offs[base + i] of the
  // current block of 64 (one load per 64 layers); a layer reads its two
  // bounds with readlane.  The first op of the next layer is loaded while
  // the current layer runs, so its latency hides behind the LDS work.
  uint32_t base = 0, offv = lane <= depth ? goffs[lane] : 0u;
  auto bound = [&](uint32_t i) -> uint32_t {   // offs[i], i uniform, i <= depth
    if ((i & ~63u) != base) {
      base = i & ~63u;
      offv = base + lane <= depth ? goffs[base + lane] : 0u;
    }
    return uint32_t(__builtin_amdgcn_readlane(int(offv), int(i & 63u)));
  };
  T racc{};
  uint32_t lo = bound(0), hi = depth ? bound(1) : lo;
  uint64_t nxt = lo + tid < hi ? gops[lo + tid] : 0ull;
  for (uint32_t l = 0; l < depth; ++l) {
    const uint32_t a0 = lo, a1 = hi;
    const uint64_t cur = nxt;
    if (l + 1 < depth) {
      lo = a1;
      hi = bound(l + 2);
      nxt = lo + tid < hi ? gops[lo + tid] : 0ull;
    }
    if (a0 + tid < a1) apply_op_lds(cur, n, sx, sz, racc);
    for (uint32_t k = a0 + tid + nthr; k < a1; k += nthr) apply_op_lds(uint64_t(gops[k]), n, sx, sz, racc);
    lds_barrier();
  }
  if (nonzero(racc)) lds_xor(s_r, racc);
  T *XW = reinterpret_cast<T *>(X);
  T *ZW = reinterpret_cast<T *>(Z);
  for (uint32_t j = tid; j < n; j += nthr) {
    XW[j * cs + unit] = sx[j];
    ZW[j * cs + unit] = sz[j];
  }
  __syncthreads();
  if (tid == 0 && nonzero(*s_r)) reinterpret_cast<T *>(P)[unit] ^= *s_r;   // this part of P is ours alone
}

// ---- decoded streams --------------------------------------------------------
// For longer streams the op words are first decoded, once for all row groups,
// into what a lane needs to work on LDS, each layer padded to whole waves:
//   word 0: LDS address of column a (bits 0..17) | code of a (bits 18..24) | step flags
//   word 1: LDS address of column b (bits 0..17) | code of b (bits 18..24) | two-qubit gate, one of kDec*
// The step flags say what any op of the step needs, so that a wave branches on
// a scalar.  Padding, malformed ops and the missing second qubit of a
// single-qubit op refer to spare columns past the tableau's (zero, so that
// they add no sign), and a step of the gate kernel has no test per lane.
//
// Bound: instruction issue and the LDS accesses at random columns, which
// hardly overlap in a layer of one round: n = 1,500 (750 ops a layer), per
// layer and CU, 470 of 840 clocks issue VALU instructions (38 a step) and 456
// serve LDS (4 x 9.5 a step, 3 each without bank conflicts).  From op words a
// step took about 200 instructions with its branches (decode, range checks,
// masks).  From op words -> decoded: n = 1,500, 3,000 layers 1,858 -> 1,041 us
// (+ 13 to decode); n = 500 x 100 tableaux, 2,000 layers 1,382 -> 936 (+ 150);
// n = 64, 64 layers 34 -> 16; n = 1,024, 100 layers 60 -> 37; n = 10,000, 20 layers
// 302 -> 212 (50 of it by the XCD order of the row groups).
constexpr uint32_t kSpareCols = 16;
constexpr uint32_t kDecBits = (1u << 18) - 1;
constexpr uint32_t kDecCnot = 25, kDecCz = 26, kDecSwap = 27;        // bits of word 1
constexpr uint32_t kStepCodes = 25, kStepPauli = 26, kStepSwap = 27;   // bits of word 0
static_assert(kFusedGateLds + kSpareCols * 32 <= kDecBits, "column addresses fit the decoded words");

// Decodes the layers of tableau blockIdx.y for columns of `cb` bytes of LDS: a
// wave a layer, blockIdx.z shares out a layer's steps.  poffs: padded layer
// starts in steps of 64.
__device__ __forceinline__ void decode_layers(const uint64_t *__restrict__ ops, const uint32_t *__restrict__ offs,
                                              const uint32_t *__restrict__ poffs, uint32_t depth, uint32_t n,
                                              uint32_t cb, uint2 *__restrict__ out) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t spare = cb * (n + (lane & (kSpareCols - 1)));
  for (uint32_t l = blockIdx.x * 4 + wave; l < depth; l += gridDim.x * 4) {
    const uint32_t lo = offs[l], cnt = offs[l + 1] - lo, p0 = poffs[l];
    for (uint32_t st = blockIdx.z; st * 64 < cnt; st += gridDim.z) {
      const uint32_t i = st * 64 + lane;
      const uint64_t op = i < cnt ? ops[lo + i] : ~0ull;
      const uint32_t pair = op_pair(op);
      uint2 d = make_uint2(spare, spare);
      uint32_t codes = 0;
      bool swap = false;
      if (op_valid(op, n)) {   // (~0 is not)
        codes = op_ca(op);
        d.x = cb * op_a(op) | codes << 18;
        if (pair != PAIR_NONE) {
          codes |= op_cb(op);
          d.y = cb * op_b(op) | op_cb(op) << 18 | 1u << (kDecCnot + pair - PAIR_CNOT);
          swap = pair == PAIR_SWAP;
        }
      }
      if (__ballot(codes != 0)) d.x |= 1u << kStepCodes;
      if (__ballot((codes & kSqPauli) != 0)) d.x |= 1u << kStepPauli;
      if (__ballot(swap)) d.x |= 1u << kStepSwap;
      out[size_t(p0 + st) * 64 + lane] = d;
    }
  }
}
__global__ void __launch_bounds__(256) k_decode_ops(const uint64_t *__restrict__ ops, const uint32_t *__restrict__ offs,
                                                    const uint32_t *__restrict__ poffs, uint32_t depth, uint32_t n,
                                                    uint2 *__restrict__ out) {
  decode_layers(ops, offs, poffs, depth, n, 8, out);
}
// Steps and rounds (decoded_body) of every tableau's layers, one workgroup a
// tableau: each thread a run of layers, run totals scanned over the workgroup.
__global__ void __launch_bounds__(1024) k_plan_many(const ManyDesc *__restrict__ descs, uint32_t waves) {
  __shared__ uint32_t s_st[1024], s_rd[1024];
  const ManyDesc d = descs[blockIdx.x];
  const uint32_t tid = threadIdx.x, per = (d.depth + 1023) / 1024;
  const uint32_t l0 = min(d.depth, tid * per), l1 = min(d.depth, l0 + per);
  auto steps_of = [&](uint32_t l) -> uint32_t { return (d.offs[l + 1] - d.offs[l] + 63) / 64; };
  uint32_t st = 0, rd = 0;
  for (uint32_t l = l0; l < l1; ++l) {
    const uint32_t c = steps_of(l);
    st += c;
    rd += (c + waves - 1) / waves;
  }
  s_st[tid] = st;
  s_rd[tid] = rd;
  __syncthreads();
  for (uint32_t off = 1; off < 1024; off <<= 1) {
    const uint32_t a = tid >= off ? s_st[tid - off] : 0u, b = tid >= off ? s_rd[tid - off] : 0u;
    __syncthreads();
    s_st[tid] += a;
    s_rd[tid] += b;
    __syncthreads();
  }
  uint32_t at = s_st[tid] - st, r = s_rd[tid] - rd;
  for (uint32_t l = l0; l < l1; ++l) {
    const uint32_t c = steps_of(l);
    d.poffs[l] = at;
    for (uint32_t k = 0; k < c; k += waves) {
      const uint32_t cnt = min(waves, c - k);
      d.sched[r++] = cnt | (k + cnt == c ? kRoundEnds : 0u);
    }
    at += c;
  }
  if (tid == 1023) d.poffs[d.depth] = s_rd[1023];   // the number of rounds
}
__global__ void __launch_bounds__(256) k_decode_many(const ManyDesc *__restrict__ descs, uint32_t cb) {
  const ManyDesc d = descs[blockIdx.y];
  decode_layers(d.ops, d.offs, d.poffs, d.depth, d.n, cb, d.dec);
}

// x and z of a column's rows side by side at its LDS address.  (The kernels
// below have no other LDS than what they are launched with, which begins at
// address 0; a decoded address is used as it is.)
template <typename T>
struct alignas(2 * sizeof(T) < 16 ? 2 * sizeof(T) : 16) XZ {
  T x, z;
};
template <typename T>
__device__ __forceinline__ T *lds_at(uint32_t addr) {
  return (T *)(__attribute__((address_space(3))) T *)uintptr_t(addr);
}

// (word by word: a struct copied between memories would pass through a stack
// slot, which the compiler may place in LDS, at address 0)
template <typename T>
__device__ __forceinline__ void copy_word(T &d, const T &s) { d = s; }
__device__ __forceinline__ void copy_word(U128 &d, const U128 &s) {
  const uint64_t lo = s.lo, hi = s.hi;
  d.lo = lo;
  d.hi = hi;
}

// One store of a column's x and z.  (The empty asm keeps the value in
// neighbouring registers: from others the compiler makes two stores of half
// the width, at twice the bank conflicts.)
__device__ __forceinline__ void put_col(XZ<uint32_t> *c, uint32_t x, uint32_t z) {
  uint64_t v = uint64_t(z) << 32 | x;
  asm volatile("" : "+v"(v));
  *reinterpret_cast<uint64_t *>(c) = v;
}
typedef uint64_t U64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void put_col(XZ<uint64_t> *c, uint64_t x, uint64_t z) {
  U64x2 v = {x, z};
  asm volatile("" : "+v"(v));
  *reinterpret_cast<U64x2 *>(c) = v;
}
__device__ __forceinline__ void put_col(XZ<U128> *c, U128 x, U128 z) {
  put_col(reinterpret_cast<XZ<uint64_t> *>(&c->x), x.lo, x.hi);
  put_col(reinterpret_cast<XZ<uint64_t> *>(&c->z), z.lo, z.hi);
}
// And its load, of the same type: one wave has no barrier between layers, and
// accesses of different types the compiler may reorder.
__device__ __forceinline__ void get_col(const XZ<uint32_t> *c, uint32_t &x, uint32_t &z) {
  const uint64_t v = *reinterpret_cast<const uint64_t *>(c);
  x = uint32_t(v);
  z = uint32_t(v >> 32);
}
__device__ __forceinline__ void get_col(const XZ<uint64_t> *c, uint64_t &x, uint64_t &z) {
  const U64x2 v = *reinterpret_cast<const U64x2 *>(c);
  x = v.x;
  z = v.y;
}
__device__ __forceinline__ void get_col(const XZ<U128> *c, U128 &x, U128 &z) {
  get_col(reinterpret_cast<const XZ<uint64_t> *>(&c->x), x.lo, x.hi);
  get_col(reinterpret_cast<const XZ<uint64_t> *>(&c->z), z.lo, z.hi);
}

// The 64 ops of a step, one a lane.
template <typename T>
__device__ __forceinline__ void apply_decoded(uint2 d, T &racc) {
  const uint32_t flags = uint32_t(__builtin_amdgcn_readfirstlane(int(d.x)));
  XZ<T> *pa = lds_at<XZ<T>>(d.x & kDecBits), *pb = lds_at<XZ<T>>(d.y & kDecBits);
  T xa, za, xb, zb;
  get_col(pa, xa, za);
  get_col(pb, xb, zb);
  auto mask = [](uint32_t w, uint32_t bit) { return mask_if<T>((w >> bit) & 1u); };
  if (flags & (1u << kStepCodes)) {   // (layers of two-qubit gates alone have none)
    if (flags & (1u << kStepPauli)) racc = bop3<LUT_XOR3>(sq_pauli<18>(d.x, xa, za), sq_pauli<18>(d.y, xb, zb), racc);
    racc = bop3<LUT_XOR3>(sq_rest<18>(d.x, xa, za), sq_rest<18>(d.y, xb, zb), racc);
  }
  // two-qubit gates under lane masks; without one xb and zb are zero (spare)
  const T mc = mask(d.y, kDecCnot), mz = mask(d.y, kDecCz);
  const T flip = bop3<LUT_SELECT>(mz, bop3<LUT_AND_XOR_BC>(xb, za, zb), bop3<LUT_AND_XNOR>(zb, xb, za));
  racc = bop3<LUT_AND_XOR>(flip, xa, racc);
  za = bop3<LUT_AND_XOR>(zb, mc, bop3<LUT_AND_XOR>(xb, mz, za));
  xb = bop3<LUT_AND_XOR>(xa, mc, xb);
  zb = bop3<LUT_AND_XOR>(xa, mz, zb);
  if (flags & (1u << kStepSwap)) {   // seldom; a SWAP adds no sign
    const T ms = mask(d.y, kDecSwap), sx = (xa ^ xb) & ms, sz = (za ^ zb) & ms;
    racc = bop3<LUT_AND_XOR>(flip & ms, xa, racc);
    xa ^= sx;
    xb ^= sx;
    za ^= sz;
    zb ^= sz;
  }
  put_col(pb, xb, zb);
  put_col(pa, xa, za);
}

// All layers of a decoded stream on one row group, as fused_body does, in
// rounds of up to one step of 64 ops per wave (a layer takes one or more).
// sched[r]: the steps of round r, | kRoundEnds where the layer ends with it;
// 64 rounds' entries sit in a wave's lanes.  A wave loads its next kOpAhead
// rounds' ops ahead.  LDS: n columns, the spare ones, the sign word.
constexpr int kOpAhead = 4;
template <typename T>
__device__ __forceinline__ void decoded_body(uint64_t *X, uint64_t *Z, uint64_t *P, uint32_t n, uint32_t Wp,
                                             const uint2 *__restrict__ dec, const uint32_t *__restrict__ sched,
                                             uint32_t rounds, uint32_t unit) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool alone = nthr == 64;   // (one wave's LDS accesses are in order)
  const size_t cs = size_t(Wp) * 8 / sizeof(T);
  const T *XT = reinterpret_cast<const T *>(X);
  const T *ZT = reinterpret_cast<const T *>(Z);
  constexpr uint32_t kCol = sizeof(XZ<T>);
  T *sign = lds_at<T>((n + kSpareCols) * kCol);
  for (uint32_t j = tid; j < n; j += nthr) {
    XZ<T> *c = lds_at<XZ<T>>(j * kCol);
    copy_word(c->x, XT[j * cs + unit]);
    copy_word(c->z, ZT[j * cs + unit]);
  }
  if (tid < kSpareCols) *lds_at<XZ<T>>((n + tid) * kCol) = {};
  if (tid == 0) *sign = T{};
  const GlobalU32 *gsched = (const GlobalU32 *)sched;
  const GlobalU64 *gdec = (const GlobalU64 *)dec + size_t(wave) * 64;
  auto entries = [&](uint32_t r) -> uint32_t { return r + lane < rounds ? uint32_t(gsched[r + lane]) : 0u; };
  uint64_t ring[kOpAhead];
  uint32_t ctl[kOpAhead];
  uint32_t first = 0;   // step of the next round to load
  auto load = [&](int d, uint32_t e, uint32_t i) {
    const uint32_t c = uint32_t(__builtin_amdgcn_readlane(int(e), int(i))), cnt = c & (kRoundEnds - 1);
    ctl[d] = c;
    // (a wave past the round's steps loads from the stream's start: in range,
    // since the stream holds a round of every wave; see the launch)
    ring[d] = (gdec + size_t(wave < cnt ? first : 0u) * 64)[lane];
    first += cnt;
  };
  uint32_t e = entries(0);
#pragma unroll
  for (int d = 0; d < kOpAhead; ++d) load(d, e, uint32_t(d));
  __syncthreads();
  T racc{};
  for (uint32_t r0 = 0; r0 < rounds; r0 += 64) {
    e = entries(r0 + kOpAhead);
    asm volatile("" : "+v"(e));   // waited for here, and not with every turn of the loop below
    for (uint32_t q = 0; q < 64; q += kOpAhead) {
#pragma unroll
      for (int d = 0; d < kOpAhead; ++d) {
        const uint32_t c = ctl[d];
        if (wave < (c & (kRoundEnds - 1)))
          apply_decoded<T>(make_uint2(uint32_t(ring[d]), uint32_t(ring[d] >> 32)), racc);
        load(d, e, q + uint32_t(d));   // (after its use: a copy of it would wait for every load in flight)
        if ((c & kRoundEnds) && !alone) lds_barrier();
      }
      if (r0 + q + kOpAhead >= rounds) break;
    }
  }
  if (nonzero(racc)) lds_xor(sign, racc);
  __syncthreads();
  T *XW = reinterpret_cast<T *>(X);
  T *ZW = reinterpret_cast<T *>(Z);
  for (uint32_t j = tid; j < n; j += nthr) {
    const XZ<T> *c = lds_at<XZ<T>>(j * kCol);
    copy_word(XW[j * cs + unit], c->x);
    copy_word(ZW[j * cs + unit], c->z);
  }
  if (tid == 0) {
    const T r = *sign;
    if (nonzero(r)) reinterpret_cast<T *>(P)[unit] ^= r;   // this part of P is ours alone
  }
}

constexpr uint32_t kFusedMaxThreads = 1024;
__global__ void __launch_bounds__(kFusedMaxThreads) k_gates_decoded(TabDev t, const uint2 *__restrict__ dec,
                                                                   const uint32_t *__restrict__ sched, uint32_t rounds) {
  // consecutive row groups on one XCD (workgroups go round the 8 of them): the
  // groups of a 128-byte line of a column then share it in that XCD's L2
  const uint32_t per = gridDim.x / 8, more = gridDim.x % 8, xcd = blockIdx.x % 8;
  const uint32_t unit = xcd * per + min(xcd, more) + blockIdx.x / 8;
  decoded_body<uint32_t>(t.X, t.Z, t.P, t.n, t.Wp, dec, sched, rounds, unit);
}
template <typename T>
__global__ void __launch_bounds__(256) k_gates_many_decoded(const ManyDesc *__restrict__ descs) {
  const ManyDesc d = descs[blockIdx.y];
  constexpr uint32_t kBits = 8 * sizeof(T);
  if (blockIdx.x >= (2 * d.n + kBits - 1) / kBits) return;   // group past the tableau's 2n rows
  decoded_body<T>(d.X, d.Z, d.P, d.n, d.Wp, d.dec, d.sched, d.poffs[d.depth], blockIdx.x);
}

// One tableau, 32-row groups (twice as many workgroups as 64-row ones: a
// single tableau is latency-bound, not throughput-bound).  Launched with up
// to 1024 threads: 16 waves share a group's layer work, so that more LDS
// round trips are in flight per SIMD (n = 10,000, 20 layers: 30 % less time
// than with 256 threads).
__global__ void __launch_bounds__(kFusedMaxThreads) k_gates_fused(TabDev t, const uint64_t *__restrict__ ops,
                                                     const uint32_t *__restrict__ offs, uint32_t depth) {
  extern __shared__ uint64_t lds_u64[];
  __shared__ uint32_t s_r;
  uint32_t *sx = reinterpret_cast<uint32_t *>(lds_u64), *sz = sx + t.n;
  fused_body<uint32_t>(t.X, t.Z, t.P, t.n, t.Wp, ops, offs, depth, blockIdx.x, sx, sz, &s_r);
}

// Many tableaux in one launch: blockIdx.y picks the tableau, blockIdx.x its
// row group (groups past the tableau's 2n rows exit at once).
template <typename T>
__global__ void __launch_bounds__(256) k_gates_many(const ManyDesc *__restrict__ descs) {
  extern __shared__ uint64_t lds_u64[];
  __shared__ T s_r;
  const ManyDesc d = descs[blockIdx.y];
  constexpr uint32_t kBits = 8 * sizeof(T);
  if (blockIdx.x >= (2 * d.n + kBits - 1) / kBits) return;   // group past the tableau's 2n rows
  T *sx = reinterpret_cast<T *>(lds_u64), *sz = sx + d.n;
  fused_body<T>(d.X, d.Z, d.P, d.n, d.Wp, d.ops, d.offs, d.depth, blockIdx.x, sx, sz, &s_r);
}

// dst <- src with every sign column of dst set to src's column 0 (+ pending).
__global__ void __launch_bounds__(256) k_copy_tab(TabDev dst, TabDev src) {
  const size_t ncol = size_t(src.n) * src.Wp;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < ncol; i += stride) {
    dst.X[i] = src.X[i];
    dst.Z[i] = src.Z[i];
  }
  const size_t nr = size_t(dst.Wp) * dst.S;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < nr; i += stride) {
    const size_t w = i / dst.S;
    dst.R[i] = src.R[w * src.S] ^ src.P[w];
  }
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < dst.Wp; i += stride) dst.P[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *dst.abort_flag = 0;
}

// Words handed over in the kernel's arguments, stored to device memory (an
// upload that needs no staging buffer and no host-memory copy).
constexpr uint32_t kArgWords = 960;
struct ArgWords {
  uint32_t w[kArgWords];
};
__global__ void __launch_bounds__(256) k_store_words(uint32_t *dst, ArgWords a, uint32_t count) {
  for (uint32_t i = threadIdx.x; i < count; i += blockDim.x) dst[i] = a.w[i];
}

// Word words[q] of every column of X and Z, gathered for a host readout of a
// few rows: ox[q * n + j] = X[j * Wp + words[q]] (every words[q] < W).
__global__ void __launch_bounds__(256) k_gather_words(TabDev t, const uint32_t *__restrict__ words, uint32_t nw,
                                                      uint64_t *__restrict__ ox, uint64_t *__restrict__ oz) {
  const size_t total = size_t(nw) * t.n;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const size_t q = i / t.n, j = i % t.n;
    const size_t at = j * t.Wp + words[q];
    ox[i] = t.X[at];
    oz[i] = t.Z[at];
  }
}

// Outcomes of shots s0 .. s0 + rows and cnt measurements, transposed from the
// staging's [measurement][shot] into rows of `pitch` bytes (a multiple of 64)
// in host memory, and the random flags into `rnd`.  A block turns a tile of 64
// by 64 in LDS: reads and the writes over the host link are whole lines.
__global__ void __launch_bounds__(256) k_emit(TabDev t, uint32_t cnt, uint32_t s0, uint32_t rows,
                                              uint8_t *__restrict__ out, size_t pitch, uint8_t *__restrict__ rnd) {
  constexpr uint32_t kPad = 80;   // bytes of a tile row: 16-byte aligned, banks 20 apart
  __shared__ uint4 s_tile[64 * kPad / 16];
  uint8_t *tile = reinterpret_cast<uint8_t *>(s_tile);
  const uint32_t tid = threadIdx.x, i0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  const uint32_t iw = min(64u, cnt - i0);
  if (r0 < rows) {
    const uint32_t rw = min(64u, rows - r0);
    const uint8_t *src = t.out + size_t(i0) * t.S + s0 + r0;
    for (uint32_t j = tid; j < iw * rw; j += 256) {
      const uint32_t i = j / rw, r = j % rw;
      tile[r * kPad + i] = src[size_t(i) * t.S + r];
    }
    __syncthreads();
    const uint32_t r = tid / 4, part = tid % 4;
    if (r < rw && part * 16 < iw)   // (past cnt: whatever the tile holds, within the row's pitch)
      *reinterpret_cast<uint4 *>(out + size_t(r0 + r) * pitch + i0 + part * 16) = s_tile[(r * kPad) / 16 + part];
  }
  if (blockIdx.y == 0 && tid < iw) rnd[i0 + tid] = t.kind[i0 + tid];
}

// The same for short rows, written without gaps (fewer than 64 outcomes): a
// thread gathers 16 bytes, each read from a cached line of the staging.
__global__ void __launch_bounds__(256) k_emit_packed(TabDev t, uint32_t cnt, uint32_t s0, uint32_t rows,
                                                     uint8_t *__restrict__ out, uint8_t *__restrict__ rnd) {
  const uint32_t total = rows * cnt;   // (the caller's parts are of 16 MB at most)
  const uint32_t o = (blockIdx.x * 256 + threadIdx.x) * 16;
  if (o < total) {
    uint32_t s = o / cnt, i = o % cnt, v[4] = {};
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k) {
      if (o + k < total) v[k / 4] |= uint32_t(t.out[size_t(i) * t.S + s0 + s]) << (8 * (k % 4));
      if (++i == cnt) i = 0, ++s;
    }
    *reinterpret_cast<uint4 *>(out + o) = make_uint4(v[0], v[1], v[2], v[3]);
  }
  if (blockIdx.x == 0 && threadIdx.x < cnt) rnd[threadIdx.x] = t.kind[threadIdx.x];
}

// Outcomes of the last measurement pass (staging: out[i * S + s], kind[i])
// into a caller's record: rec[s * ld + col0 + i], random flags rnd[col0 + i].
__global__ void __launch_bounds__(256) k_record(TabDev t, uint32_t cnt, uint8_t *__restrict__ rec, size_t ld,
                                                size_t col0, uint8_t *__restrict__ rnd) {
  const size_t total = size_t(cnt) * t.S;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t j = size_t(blockIdx.x) * blockDim.x + threadIdx.x; j < total; j += stride) {
    const size_t s = j / cnt, i = j % cnt;
    rec[s * ld + col0 + i] = t.out[i * t.S + s];
  }
  if (rnd)
    for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < cnt; i += stride) rnd[col0 + i] = t.kind[i];
}

// Classically conditioned Paulis: op i = qubit (bits 0..23) | Pauli (bits
// 24..25: 1 X, 2 Y, 3 Z) | record column (bits 32..63).  In shot s, when
// rec[s * ld + column] is 1, every row that anticommutes with the Pauli
// flips sign: X flips rows with z_a = 1, Z rows with x_a = 1, Y rows with
// x_a ^ z_a = 1.  The ops only XOR into signs, so their order does not matter.
// A piece of work is 64 shots (one a lane) and a few row words.  With SPLIT a
// block takes a piece and its waves share out the ops, several loaded at a time
// (a thread a shot and word, op by op: 15 us a launch at n = 97, 256 shots, 20
// ops, a chain of loads; now 5.7); else every wave takes a piece of its own, of
// one row word.  That is for few ops, which do not fill a block's eight waves:
// 10^6 shots of n = 100, the whole call, 1 op 34 us (71 split), 5 54 (86), 10 80
// (95), 15 105 (108), 16 110 (107); 100 ops of 10^5 shots 84 (69).
constexpr uint32_t kCondWaves = 8, kCondOps = 4;
constexpr uint32_t kCondSplit = 16;
constexpr uint32_t cond_words(bool split) { return split ? 4 : 1; }
template <bool SPLIT>
__global__ void __launch_bounds__(64 * kCondWaves) k_cond_pauli(TabDev t, const uint64_t *__restrict__ ops, uint32_t k,
                                                                const uint8_t *__restrict__ rec, size_t ld) {
  constexpr uint32_t kWords = cond_words(SPLIT);
  __shared__ uint64_t s_flip[SPLIT ? kCondWaves : 1][kWords][64];
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t tiles = (t.S + 63) / 64, total = tiles * ((t.W + kWords - 1) / kWords);
  const uint32_t first = SPLIT ? blockIdx.x : blockIdx.x * kCondWaves + wave, step = SPLIT ? gridDim.x : gridDim.x * kCondWaves;
  for (uint32_t b = first; b < total; b += step) {
    const uint32_t s = (b % tiles) * 64 + lane, w0 = (b / tiles) * kWords;
    const uint8_t *row = rec + size_t(min(s, t.S - 1)) * ld;
    uint64_t flip[kWords] = {};
    auto take = [&](auto count, uint32_t i0) {   // ops i0 .. i0 + count - 1, past k none
      constexpr uint32_t N = decltype(count)::value;
      uint64_t op[N], x[N][kWords], z[N][kWords];
      uint32_t bit[N];
#pragma unroll
      for (uint32_t i = 0; i < N; ++i) {
        op[i] = ops[min(i0 + i, k - 1)];
        const uint32_t a = uint32_t(op[i] & kQubitMask);
        const bool on = i0 + i < k && a < t.n;
        bit[i] = on ? row[op[i] >> 32] & 1u : 0u;
#pragma unroll
        for (uint32_t w = 0; w < kWords; ++w) {
          const size_t at = size_t(on ? a : 0) * t.Wp + min(w0 + w, t.W - 1);
          x[i][w] = t.X[at];
          z[i][w] = t.Z[at];
        }
      }
#pragma unroll
      for (uint32_t i = 0; i < N; ++i) {
        const uint32_t p = uint32_t(op[i] >> 24) & 3u;
        const uint64_t on = 0ull - bit[i];
        // the Pauli's x part (X, Y) flips rows with z = 1, its z part (Y, Z) rows with x = 1
#pragma unroll
        for (uint32_t w = 0; w < kWords; ++w) flip[w] ^= ((p != 3u ? z[i][w] : 0ull) ^ (p != 1u ? x[i][w] : 0ull)) & on;
      }
    };
    using Four = std::integral_constant<uint32_t, kCondOps>;
    if constexpr (SPLIT) {
      for (uint32_t i0 = wave * kCondOps; i0 < k; i0 += kCondWaves * kCondOps) take(Four{}, i0);
    } else {
      uint32_t i0 = 0;
      for (; i0 + kCondOps <= k; i0 += kCondOps) take(Four{}, i0);
      for (; i0 < k; ++i0) take(std::integral_constant<uint32_t, 1>{}, i0);
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (uint32_t w = 0; w < kWords; ++w) s_flip[wave][w][lane] = flip[w];
      __syncthreads();
      if (wave < kWords && w0 + wave < t.W && s < t.S) {
        uint64_t f = 0;
#pragma unroll
        for (uint32_t v = 0; v < kCondWaves; ++v) f ^= s_flip[v][wave][lane];
        if (f) t.R[size_t(w0 + wave) * t.S + s] ^= f;
      }
      __syncthreads();
    } else if (s < t.S) {
#pragma unroll
      for (uint32_t w = 0; w < kWords; ++w)
        if (w0 + w < t.W && flip[w]) t.R[size_t(w0 + w) * t.S + s] ^= flip[w];
    }
  }
}

static inline uint32_t grid_for(size_t items, uint32_t block, uint32_t cap = 4096) {
  size_t g = (items + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return uint32_t(g);
}

hipError_t launch_init_zero(const TabDev &t, hipStream_t st) {
  const size_t items = size_t(t.n) * t.Wp;
  k_init_zero<<<grid_for(items, 256), 256, 0, st>>>(t);
  return hipGetLastError();
}

hipError_t launch_clear_state(const TabDev &t, hipStream_t st) {
  k_clear_state<<<1, 64, 0, st>>>(t);
  return hipGetLastError();
}

hipError_t launch_fold_pending(const TabDev &t, hipStream_t st) {
  k_fold_pending<<<grid_for(size_t(t.Wp) * t.S, 256), 256, 0, st>>>(t);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_clear_pending<<<grid_for(t.Wp, 256), 256, 0, st>>>(t);
  return hipGetLastError();
}

hipError_t launch_gate_layer(const TabDev &t, const uint64_t *ops, uint32_t nops, uint32_t w0, uint32_t w1,
                             hipStream_t st) {
  if (nops == 0) return hipSuccess;
  const uint32_t tiles = (w1 - w0 + 63) / 64;
  uint32_t per = 4 * kLayerOps;   // one turn of a block (two or four: the same or slower)
  while ((nops + per - 1) / per > 65535) per *= 2;
  dim3 grid(tiles, (nops + per - 1) / per);
  k_gate_layer<<<grid, 256, 0, st>>>(t, ops, nops, per, w0, w1);
  return hipGetLastError();
}

bool fused_gates_fit(uint32_t n) { return size_t(n) * 8 <= kFusedGateLds; }

hipError_t launch_gates_fused(const TabDev &t, const uint64_t *ops, const uint32_t *dev_offs,
                              uint32_t depth, hipStream_t st) {
  if (depth == 0) return hipSuccess;
  const size_t lds = size_t(t.n) * 8;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_gates_fused),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(kFusedGateLds));
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const uint32_t halves = (2 * t.n + 31) / 32;
  // (below n = 512 a layer has too few ops for 16 waves)
  const uint32_t threads = t.n >= 512 ? kFusedMaxThreads : 256;
  k_gates_fused<<<halves, threads, lds, st>>>(t, ops, dev_offs, depth);
  return hipGetLastError();
}

bool many_gates_fit(uint32_t max_n, uint32_t rows) { return 2 * size_t(max_n) * (rows / 8) <= kFusedGateLds; }

hipError_t launch_gates_many(const ManyDesc *dev_descs, uint32_t count, uint32_t max_n, uint32_t rows,
                             hipStream_t st) {
  if (count == 0) return hipSuccess;
  const int v = rows == 128 ? 2 : rows == 64 ? 1 : 0;
  const void *fn = v == 2 ? reinterpret_cast<const void *>(k_gates_many<U128>)
                 : v == 1 ? reinterpret_cast<const void *>(k_gates_many<uint64_t>)
                          : reinterpret_cast<const void *>(k_gates_many<uint32_t>);
  static bool attr_set[3] = {false, false, false};
  if (!attr_set[v]) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(kFusedGateLds));
    if (e != hipSuccess) return e;
    attr_set[v] = true;
  }
  const size_t lds = 2 * size_t(max_n) * (rows / 8);
  const dim3 grid((2 * max_n + rows - 1) / rows, count);
  if (v == 2)
    k_gates_many<U128><<<grid, 256, lds, st>>>(dev_descs);
  else if (v == 1)
    k_gates_many<uint64_t><<<grid, 256, lds, st>>>(dev_descs);
  else
    k_gates_many<uint32_t><<<grid, 256, lds, st>>>(dev_descs);
  return hipGetLastError();
}

// (decoded addresses count from 0: no LDS of the kernel's own)
static hipError_t allow_gate_lds(const void *fn, size_t more) {
  hipFuncAttributes a;
  hipError_t e = hipFuncGetAttributes(&a, fn);
  if (e != hipSuccess) return e;
  if (a.sharedSizeBytes != 0) return hipErrorInvalidConfiguration;
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(kFusedGateLds + more));
}

constexpr size_t kMoreLds = kSpareCols * 8 + 8, kMoreLdsMany = kSpareCols * 32 + 16;
bool decoded_gates_ready() {
  static std::atomic<bool> ready{false};   // (only success is kept: another call may ask again)
  if (ready) return true;
  const void *const many[3] = {reinterpret_cast<const void *>(k_gates_many_decoded<uint32_t>),
                               reinterpret_cast<const void *>(k_gates_many_decoded<uint64_t>),
                               reinterpret_cast<const void *>(k_gates_many_decoded<U128>)};
  bool ok = allow_gate_lds(reinterpret_cast<const void *>(k_gates_decoded), kMoreLds) == hipSuccess;
  for (const void *fn : many) ok = ok && allow_gate_lds(fn, kMoreLdsMany) == hipSuccess;
  if (!ok) (void)hipGetLastError();
  ready = ok;
  return ok;
}

// Workgroups of four waves for `depth` layers.
static uint32_t decode_grid(uint32_t depth, uint32_t most) { return depth / 4 + 1 < most ? depth / 4 + 1 : most; }

hipError_t launch_gates_decoded(const TabDev &t, const uint64_t *ops, const uint32_t *dev_offs,
                                const uint32_t *dev_poffs, const uint32_t *dev_sched, uint32_t depth, uint32_t rounds,
                                uint32_t max_steps, uint32_t waves, uint2 *dec, uint2 *dec_base, hipStream_t st) {
  if (rounds == 0) return hipSuccess;
  const uint32_t gx = decode_grid(depth, 4096), gz = std::min((max_steps + 3) / 4, 1024u);
  k_decode_ops<<<dim3(gx, 1, gz), 256, 0, st>>>(ops, dev_offs, dev_poffs, depth, t.n, dec);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_gates_decoded<<<(2 * t.n + 31) / 32, 64 * waves, size_t(t.n) * 8 + kMoreLds, st>>>(t, dec_base, dev_sched, rounds);
  return hipGetLastError();
}

hipError_t launch_gates_many_decoded(const ManyDesc *dev_descs, uint32_t count, uint32_t max_n, uint32_t rows,
                                     uint32_t max_depth, uint32_t max_steps, uint32_t waves, hipStream_t st) {
  if (count == 0 || max_depth == 0 || max_steps == 0) return hipSuccess;
  const int v = rows == 128 ? 2 : rows == 64 ? 1 : 0;
  const uint32_t gx = decode_grid(max_depth, 256), gz = std::min((max_steps + 3) / 4, 1024u);
  k_plan_many<<<count, 1024, 0, st>>>(dev_descs, waves);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_decode_many<<<dim3(gx, count, gz), 256, 0, st>>>(dev_descs, rows / 4);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = 2 * size_t(max_n + kSpareCols) * (rows / 8) + 16;
  const dim3 grid((2 * max_n + rows - 1) / rows, count);
  if (v == 2)
    k_gates_many_decoded<U128><<<grid, 64 * waves, lds, st>>>(dev_descs);
  else if (v == 1)
    k_gates_many_decoded<uint64_t><<<grid, 64 * waves, lds, st>>>(dev_descs);
  else
    k_gates_many_decoded<uint32_t><<<grid, 64 * waves, lds, st>>>(dev_descs);
  return hipGetLastError();
}

hipError_t launch_emit(const TabDev &t, uint32_t cnt, uint32_t s0, uint32_t rows, bool packed, uint8_t *out,
                       size_t pitch, uint8_t *rnd, hipStream_t st) {
  if (cnt == 0) return hipSuccess;
  if (packed) {
    const size_t groups = (size_t(rows) * cnt + 15) / 16;
    k_emit_packed<<<uint32_t(std::max<size_t>(1, (groups + 255) / 256)), 256, 0, st>>>(t, cnt, s0, rows, out, rnd);
    return hipGetLastError();
  }
  k_emit<<<dim3((cnt + 63) / 64, rows ? (rows + 63) / 64 : 1), 256, 0, st>>>(t, cnt, s0, rows, out, pitch, rnd);
  return hipGetLastError();
}

hipError_t launch_record(const TabDev &t, uint32_t cnt, uint8_t *rec, size_t ld, size_t col0, uint8_t *rnd,
                         hipStream_t st) {
  if (cnt == 0) return hipSuccess;
  k_record<<<grid_for(size_t(cnt) * t.S, 256), 256, 0, st>>>(t, cnt, rec, ld, col0, rnd);
  return hipGetLastError();
}

hipError_t launch_cond_pauli(const TabDev &t, const uint64_t *ops, uint32_t k, const uint8_t *rec, size_t ld,
                             hipStream_t st) {
  if (k == 0) return hipSuccess;
  const bool split = k >= kCondSplit;
  const size_t pieces = size_t((t.S + 63) / 64) * ((t.W + cond_words(split) - 1) / cond_words(split));
  const size_t blocks = split ? pieces : (pieces + kCondWaves - 1) / kCondWaves;
  (split ? k_cond_pauli<true> : k_cond_pauli<false>)<<<uint32_t(std::min<size_t>(blocks, 4096)), 64 * kCondWaves, 0, st>>>(
      t, ops, k, rec, ld);
  return hipGetLastError();
}

hipError_t launch_gather_words(const TabDev &t, const uint32_t *words, uint32_t nw, uint64_t *ox, uint64_t *oz,
                               hipStream_t st) {
  if (nw == 0) return hipSuccess;
  k_gather_words<<<grid_for(size_t(nw) * t.n, 256), 256, 0, st>>>(t, words, nw, ox, oz);
  return hipGetLastError();
}

hipError_t launch_copy_tab(const TabDev &dst, const TabDev &src, hipStream_t st) {
  const size_t items = size_t(src.n) * src.Wp;
  k_copy_tab<<<grid_for(items, 256), 256, 0, st>>>(dst, src);
  return hipGetLastError();
}

hipError_t launch_store_words(uint32_t *dst, const uint32_t *host, uint32_t count, hipStream_t st) {
  for (uint32_t at = 0; at < count; at += kArgWords) {
    ArgWords a;
    const uint32_t c = count - at < kArgWords ? count - at : kArgWords;
    memcpy(a.w, host + at, size_t(c) * 4);
    k_store_words<<<1, 256, 0, st>>>(dst + at, a, c);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace cliff
