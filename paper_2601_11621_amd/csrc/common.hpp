// Shared definitions of the gfx950 Catalan library: modular arithmetic for the
// three 32-bit NTT primes, descriptor structs, launch constants.
//
// Every multiplication of the reconstruction phase (Sec. 3.2, Alg. 2 of
// arXiv 2601.11621) is an exact product of little-endian uint32 limb vectors.
// Large products go through the FP64 transforms (fntt.hip), or on request (see
// cat_lazy_primes_set) through a cyclic convolution modulo three primes
//   p0 = 3*2^30+1, p1 = 13*2^28+1, p2 = 29*2^27+1   (all in (2^31, 2^32),
// 2-adicity >= 27, product ~2^95.1), one 32-bit limb per coefficient, and are
// recombined with Garner's CRT.  Exactness: a coefficient of a la x lb limb
// product is < min(la,lb) * 2^64 <= 2^90 for operands up to 2^26 limbs, below
// p0*p1*p2; the transform length N = 2^k <= 2^27 needs 2-adicity >= k.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define CAT_NPRIMES 3
#define CAT_MAX_LOGN 27
#define CAT_MAX_GROUPS 32       // e_p <= log2(2n) < 32
#define CAT_LDS_LOGT 12         // row length of the LDS-resident transforms
#define CAT_CRT_E 3             // limbs per thread in the CRT/carry kernel (>= 3)
#define CAT_CRT_THREADS 256
#define CAT_CRT_BLOCK (CAT_CRT_E * CAT_CRT_THREADS)

// ----------------------------------------------------------------------------
// Per-prime constants (host computes, device reads from __constant__).
// Montgomery radix R = 2^32.  A "twiddle pair" (w, wq) holds w = W*R mod p
// (Montgomery form of W) and wq = w * p^-1 mod 2^32; mul_tw(a, w, wq) = a*W
// mod p for every 32-bit a.
// ----------------------------------------------------------------------------
struct PrimeC {
  uint32_t p;
  uint32_t pinv;          // p^-1 mod 2^32
  uint32_t w16[8], w16q[8];    // omega_16^i (forward), Montgomery pairs
  uint32_t iw16[8], iw16q[8];  // omega_16^-i (inverse)
};

struct CrtC {
  // Garner: x0 = r0; x1 = (r1 - x0) * c01 mod p1; x2 = (r2 - x0) * c012 - x1 * c12 mod p2
  uint32_t c01, c01q;       // p0^-1 mod p1 (Montgomery pair for p1)
  uint32_t c12, c12q;       // p1^-1 mod p2 (Montgomery pair for p2)
  uint32_t c012, c012q;     // (p0*p1)^-1 mod p2 (Montgomery pair for p2)
  uint32_t p0, p1;
};

// ----------------------------------------------------------------------------
// Modular arithmetic, p odd, 2^31 < p < 2^32.  Inputs of add/sub reduced.
// ----------------------------------------------------------------------------
__device__ __forceinline__ uint32_t sub_mod(uint32_t a, uint32_t b, uint32_t p) {
  uint32_t d;
  const bool borrow = __builtin_usub_overflow(a, b, &d);   // one v_sub_co_u32
  return borrow ? d + p : d;
}
__device__ __forceinline__ uint32_t add_mod(uint32_t a, uint32_t b, uint32_t p) {
  return sub_mod(a, p - b, p);   // p - b in (0, p]
}

// Montgomery multiplication with a precomputed companion (Montgomery 1985,
// with the quotient digit precomputed as in Shoup's method): returns a*w/R
// mod p in [0,p) for any 32-bit a and w < p.
__device__ __forceinline__ uint32_t mul_tw(uint32_t a, uint32_t w, uint32_t wq, uint32_t p) {
  const uint32_t m = a * wq;
  const uint32_t hi = __umulhi(a, w);
  const uint32_t mh = __umulhi(m, p);
  return sub_mod(hi, mh, p);   // hi, mh < p
}
// General Montgomery product a*b/R mod p, a,b < p.
__device__ __forceinline__ uint32_t mont_mul(uint32_t a, uint32_t b, uint32_t p, uint32_t pinv) {
  uint32_t lo = a * b;
  uint32_t hi = __umulhi(a, b);
  const uint32_t m = lo * pinv;
  const uint32_t mh = __umulhi(m, p);
  return sub_mod(hi, mh, p);   // hi, mh < p
}
// limb (any 32-bit value) reduced mod p: 2^32 < 2p, so one subtraction suffices
__device__ __forceinline__ uint32_t reduce_limb(uint32_t x, uint32_t p) { return x >= p ? x - p : x; }

// ----------------------------------------------------------------------------
// The second prime set: q0 = 105*2^23+1, q1 = 107*2^23+1, q2 = 119*2^23+1, all
// below 2^30 (product ~2^89.35, 2-adicity 23).  A coefficient of a product
// with min(la, lb) <= 2^22 limbs is below 2^22 (2^32-1)^2 < 2^86, so
// transforms of up to 2^23 points can use it.  With 4q < 2^32, residues may
// stay unreduced between butterflies (Harvey 2014, "Faster arithmetic for
// number-theoretic transforms"): forward passes keep values in [0, 2q),
// inverse passes in [0, 4q), and only the outputs that leave the transform
// are reduced to [0, q).  Twiddles from tables are Shoup pairs (w in normal
// form, w' = floor(w 2^32 / q)); twiddles computed on the fly stay Montgomery
// pairs as in the first set.
// ----------------------------------------------------------------------------
#define CAT_LAZY_MAX_LOGN 23

// x < 2m -> x mod m (one subtraction, m = q or 2q)
__device__ __forceinline__ uint32_t red2(uint32_t x, uint32_t m) {
  uint32_t d;
  return __builtin_usub_overflow(x, m, &d) ? x : d;
}
// a*w mod q in [0, 2q) for every 32-bit a (Shoup): w < q, ws = floor(w 2^32 / q)
__device__ __forceinline__ uint32_t shoup(uint32_t a, uint32_t w, uint32_t ws, uint32_t q) {
  return a * w - __umulhi(a, ws) * q;
}
// a*w/2^32 mod q in (0, 2q) for every 32-bit a, w < q Montgomery form,
// wq = w * q^-1 mod 2^32: hi(a w) - hi(m q) lies in (-q, q)
__device__ __forceinline__ uint32_t mont_lazy(uint32_t a, uint32_t w, uint32_t wq, uint32_t q) {
  return __umulhi(a, w) - __umulhi(a * wq, q) + q;
}
// x*y/2^32 mod q in (0, 2q) for x, y < 2q (x y < 4q^2, so hi(x y) < q)
__device__ __forceinline__ uint32_t mont_mul_lazy(uint32_t x, uint32_t y, uint32_t q, uint32_t qinv) {
  const uint32_t lo = x * y;
  return __umulhi(x, y) - __umulhi(lo * qinv, q) + q;
}
// limb (any 32-bit value, < 8q) into [0, 2q)
__device__ __forceinline__ uint32_t limb_lazy(uint32_t x, uint32_t q) { return red2(red2(x, 4 * q), 2 * q); }
// [0, 4q) -> [0, q)
__device__ __forceinline__ uint32_t red4(uint32_t x, uint32_t q) { return red2(red2(x, 2 * q), q); }

// ----------------------------------------------------------------------------
// Descriptors of a batch of products c = a * b.
// Explicit: a table in device memory.  Tree: computed from the level of a
// forest of balanced product trees (one tree per exponent group): node i of
// group g at level j covers leaves [i*2^j, min((i+1)*2^j, K_g)) and has exactly
// that many limbs; its parent's output sits at the left child's offset.
// ----------------------------------------------------------------------------
struct MulDesc {
  uint64_t a_off, b_off, c_off, r_off;  // r_off: position in the residue arrays
  uint32_t la, lb;
};

struct TreeLevel {
  uint32_t ngroups;
  uint32_t j;                           // input node size 2^j limbs
  uint64_t base[CAT_MAX_GROUPS];        // arena offset of group g
  uint64_t K[CAT_MAX_GROUPS];           // leaves (limbs) of group g
  uint64_t mpref[CAT_MAX_GROUPS + 1];   // prefix count of products per group
  uint64_t rbase[CAT_MAX_GROUPS];       // residue position of group g, in limbs or in 64-bit digits:
  uint32_t rshift;                      // product i's residues at rbase + (i 2^(j+1) >> rshift)
};

#define CAT_INLINE_DESC 16

// A level of decimal joins (even lengths, 64-bit digits): product i < sq reads a
// at a0 + i sa (la limbs; la_last for product `last`) and writes residues at
// digit i (la + lb) / 2; the second operand, lb limbs at b0, is the same for
// all.  Product sq is b squared.
struct UniDesc {
  uint64_t a0, sa, b0;
  uint32_t la, lb, la_last, last, sq;
};

struct DescView {
  const MulDesc* table;  // device table (large explicit batches), or
  uint32_t ninl;         // > 0: explicit descriptors carried in the kernel arguments, or
  uint32_t uni;          // > 0: a level of decimal joins, or
  MulDesc inl[CAT_INLINE_DESC];
  UniDesc u;
  TreeLevel tree;        // tree mode
  __host__ __device__ __forceinline__ MulDesc get(uint64_t i) const {
    if (table) return table[i];
    if (ninl) return inl[i];
    if (uni) {
      MulDesc d;
      d.a_off = i == u.sq ? u.b0 : u.a0 + i * u.sa;
      d.b_off = u.b0;
      d.c_off = 0;             // the segments say where the digits go
      d.r_off = i * (((uint64_t)u.la + u.lb) / 2);
      d.la = i == u.sq ? u.lb : i == u.last ? u.la_last : u.la;
      d.lb = u.lb;
      return d;
    }
    uint32_t g = 0;
    while (g + 1 < tree.ngroups && i >= tree.mpref[g + 1]) g++;
    uint64_t il = i - tree.mpref[g];
    uint64_t sz = 1ull << tree.j;
    MulDesc d;
    d.a_off = tree.base[g] + 2 * il * sz;
    d.b_off = d.a_off + sz;
    d.c_off = d.a_off;
    d.r_off = tree.rbase[g] + ((2 * il * sz) >> tree.rshift);
    d.la = (uint32_t)sz;
    uint64_t rem = tree.K[g] - (2 * il + 1) * sz;
    d.lb = (uint32_t)(rem < sz ? rem : sz);
    return d;
  }
  // slot i of a tile over the products first .. end: those past the end have empty
  // operands, at the first one's place (a masked load still reads a limb there)
  __host__ __device__ __forceinline__ MulDesc slot(uint64_t i, uint64_t first, uint64_t end) const {
    MulDesc d = get(i < end ? i : first);
    if (i >= end) d.la = d.lb = 0;
    return d;
  }
  // where the residues of the segment of product i start (a group of a tree
  // level is one segment, any other product its own)
  __device__ __forceinline__ uint64_t seg_base(uint64_t i, const MulDesc& d) const {
    if (table || ninl || uni) return d.r_off;
    uint32_t g = 0;
    while (g + 1 < tree.ngroups && i >= tree.mpref[g + 1]) g++;
    return tree.rbase[g];
  }
};

// CRT/carry segments: out[out_pos + k] for k < len from residues at res_pos + k
// (decimal joins also add the limbs add[add_pos + k] for k < add_len).
struct CrtSeg {
  uint64_t out_pos, res_pos, len;
  uint64_t add_pos, add_len;
};

// ------------------------------------------------------------ radix 10^18
#define DEC_B 1000000000000000000ull
#define DEC_D 16000000000000000000ull       // 16 B: the normalised divisor
#define DEC_V ((uint64_t)(~(unsigned __int128)0 / DEC_D - ((unsigned __int128)1 << 64)))
// floor((r 2^64 + w) / D) and its remainder, for r < D: two-by-one division
// with a precomputed reciprocal (Moller and Granlund, "Improved division by
// invariant integers", IEEE TC 2011, Algorithm 4)
__device__ __forceinline__ uint64_t div_d(uint64_t r, uint64_t w, uint64_t* rem) {
  const unsigned __int128 q = (unsigned __int128)DEC_V * r + (((unsigned __int128)(r + 1) << 64) | w);
  uint64_t q1 = (uint64_t)(q >> 64);
  const uint64_t q0 = (uint64_t)q;
  uint64_t rr = w - q1 * DEC_D;
  if (rr > q0) {
    q1--;
    rr += DEC_D;
  }
  if (rr >= DEC_D) {
    q1++;
    rr -= DEC_D;
  }
  *rem = rr;
  return q1;
}

// Bits of the device error word
#define CAT_DEVERR_CARRY_OUT 1u     // a product overflowed its la+lb limbs
#define CAT_DEVERR_NEG_EXP 2u       // negative exponent (C(n) not integral)
#define CAT_DEVERR_BOUNDS 4u        // a prime count exceeded its buffer
#define CAT_DEVERR_SCAN 8u          // a carry look-back gave up waiting (never expected)
#define CAT_DEVERR_RANGE 16u        // an exponent reached 2^32

// Ranges copied unchanged from one arena to the other (the last node of a
// group with an odd node count is carried up a level).  Kernels that take a
// CopyList run extra workgroups for it: workgroup cb (counted from the first
// copy workgroup) copies chunk cb of TAIL_CHUNK words, ranges in order.
#define TAIL_CHUNK 4096u
struct CopyList {
  uint32_t n;
  uint64_t off[CAT_MAX_GROUPS];
  uint64_t len[CAT_MAX_GROUPS];
};
inline uint32_t tail_blocks(const CopyList& cl) {
  uint64_t b = 0;
  for (uint32_t r = 0; r < cl.n; r++) b += (cl.len[r] + TAIL_CHUNK - 1) / TAIL_CHUNK;
  return (uint32_t)b;
}
__device__ __forceinline__ void copy_tail_block(const CopyList& cl, const uint32_t* __restrict__ in,
                                                uint32_t* __restrict__ out, uint32_t cb) {
  for (uint32_t r = 0; r < cl.n; r++) {
    const uint64_t nb = (cl.len[r] + TAIL_CHUNK - 1) / TAIL_CHUNK;
    if (cb < nb) {
      const uint64_t k0 = (uint64_t)cb * TAIL_CHUNK, k1 = min(k0 + (uint64_t)TAIL_CHUNK, cl.len[r]);
      for (uint64_t k = k0 + threadIdx.x; k < k1; k += blockDim.x) out[cl.off[r] + k] = in[cl.off[r] + k];
      return;
    }
    cb -= (uint32_t)nb;
  }
}

// ----------------------------------------------------------------------------
// Helpers of the transform and carry kernels.
// ----------------------------------------------------------------------------
// Word 3 of the gfx9 buffer descriptor: 32-bit data format, which untyped
// accesses use for nothing but the range check against the buffer's size.
#define CAT_BUF_DW3 0x00020000

// bit reversal of an r-bit index, compile-time
__host__ __device__ constexpr int brev_c(int x, int r) {
  int y = 0;
  for (int i = 0; i < r; i++) y |= ((x >> i) & 1) << (r - 1 - i);
  return y;
}

__host__ __device__ constexpr uint32_t lds_pad(uint32_t i) { return i + (i >> 4); }

// Word arrays read and written through raw buffer resources with byte
// offsets in one VGPR: loads past the array's end return 0 and stores there
// are dropped (the range check of an unswizzled buffer), which the column
// kernels use for the zero padding of their operands and the end of a product.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t words_rsrc(const uint32_t* p, uint64_t words) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)(uint32_t)(words * 4u), CAT_BUF_DW3);
}
__device__ __forceinline__ uint32_t buf_ld(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, (int)byte_off, 0, 0);
}
__device__ __forceinline__ void buf_st(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)byte_off, 0, 0);
}

// radix of the pass at sub-problem size 2^logS
__host__ __device__ constexpr int pass_logr(int logS) { return (logS % 4) ? (logS % 4) : 4; }

// Synchronisation between two radix-16 passes.  Both have total/16 groups,
// and the 2^logSmall elements of a sub-problem of the smaller size are written
// and read by the same 2^logSmall consecutive groups, i.e. consecutive
// threads; in a plain vector (logC = 0) with 2^logSmall <= 64 those sit in one
// wave, which orders its own LDS traffic, so no workgroup barrier is needed.
// (Next to a pass of smaller radix the group counts differ: full barrier.)
__device__ __forceinline__ void pass_sync(int logSmall, uint32_t logC) {
  if (logC == 0 && logSmall <= 6) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// frequency held at output position q of the pass-structured transform of size 2^logS
__device__ __forceinline__ uint32_t out_freq(uint32_t q, int logS) {
  uint32_t f = 0, mult = 1;
  while (logS > 0) {
    const int r = pass_logr(logS);
    const int rest = logS - r;
    const uint32_t k1 = q >> rest;
    f += k1 * mult;
    mult <<= r;
    q &= (1u << rest) - 1;
    logS = rest;
  }
  return f;
}

// Workgroups are dealt round-robin to the 8 XCDs (each with its own L2) in
// the order of their linear index.  Neighbouring column tiles share cache
// lines (a tile row is C words), so block b of a grid of G is renumbered to
// put consecutive tiles on one XCD: XCD x gets the tiles
// [x ceil(G/8), ...) in order (a bijection of [0, G) for any G).
#define CAT_XCDS 8
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t G) {
  const uint32_t q = G / CAT_XCDS, r = G % CAT_XCDS;
  const uint32_t x = b % CAT_XCDS, k = b / CAT_XCDS;
  return x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

// Wave-level: carry into each lane for (g, p) with wave carry-in `cin`;
// returns lane's carry in, and the wave carry out in *cout.
__device__ __forceinline__ uint32_t wave_carry(bool g, bool pr, uint32_t cin, uint32_t* cout, bool* allprop) {
  const uint64_t gm = __ballot(g), pm = __ballot(pr);
  const uint64_t a = gm, b = gm | pm;
  const uint64_t s1 = a + b;
  const uint64_t c1 = s1 < a;
  const uint64_t s2 = s1 + cin;
  const uint64_t c2 = s2 < s1;
  *cout = (uint32_t)(c1 | c2);
  *allprop = (pm == ~0ull);
  const uint64_t cm = s2 ^ pm;   // carry into each bit position
  return (uint32_t)((cm >> (threadIdx.x & 63)) & 1ull);
}

// Segments of a CRT launch: device tables (many segments) or up to
// CAT_INLINE_SEG segments carried in the kernel arguments.
#define CAT_INLINE_SEG 32
struct SegView {
  const CrtSeg* segs;        // nullptr => inline tables
  const uint32_t* pref;      // pref[s] = first block of segment s (nseg+1 entries)
  const uint32_t* b2s;       // with segs: the segment of every block (one load, no search)
  uint32_t nseg;
  uint32_t ubl;              // > 0: uniform segments of ubl blocks each (below)
  CrtSeg iseg[CAT_INLINE_SEG];
  uint32_t ipref[CAT_INLINE_SEG + 1];
  // uniform: segment s is iseg[0] with out_pos, add_pos and res_pos advanced
  // by s * ustep[0 .. 2]; segment ulast is ulast_len long, segment usq goes to
  // usq_pos and adds nothing
  uint64_t ustep[3];
  uint64_t ulast_len, usq_pos;
  uint32_t ulast, usq;
  __device__ __forceinline__ CrtSeg uniform(uint32_t q) const {
    CrtSeg sg = iseg[0];
    sg.out_pos += q * ustep[0];
    sg.add_pos += q * ustep[1];
    sg.res_pos += q * ustep[2];
    if (q == ulast) sg.len = ulast_len;
    if (q == usq) {
      sg.out_pos = usq_pos;
      sg.add_pos = sg.add_len = 0;
    }
    return sg;
  }
  __device__ __forceinline__ void find(uint32_t b, CrtSeg* sg, uint32_t* first, uint32_t* end,
                                       uint32_t* segi = nullptr) const {
    if (ubl) {
      const uint32_t q = b / ubl;
      *sg = uniform(q);
      *first = q * ubl;
      *end = *first + ubl;
      if (segi) *segi = q;
      return;
    }
    const uint32_t* pr = segs ? pref : ipref;
    uint32_t lo = 0, hi = nseg;   // pr[lo] <= b < pr[lo+1]
    if (segs && b2s) {
      lo = b2s[b];
    } else {
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (pr[mid] <= b) lo = mid; else hi = mid;
      }
    }
    *sg = segs ? segs[lo] : iseg[lo];
    *first = pr[lo];
    *end = pr[lo + 1];
    if (segi) *segi = lo;
  }
};
