// Exact big-integer products for the reconstruction phase (Sec. 3.2, Alg. 2):
// cyclic convolution of 64-bit digits modulo three primes near 2^50 (or 2^51)
// by number-theoretic transforms whose modular arithmetic runs on the FP64 FMA
// units.
//
// Why FP64.  The transforms are bound by vector issue.  A modular product of
// two 50-bit residues costs six FP64 instructions (below) and a modular sum
// one; the 32-bit integer form costs four and about three, on residues that
// hold 30 bits.  Measured on registers (radix-16 DFT with its 15 twiddles):
// 1.26e11 per second in FP64, 1.50e11 in 30-bit integers, but each FP64
// transform carries 64-bit digits, so a product needs half as many points and
// one butterfly level less.
//
// Numbers.  A residue is a signed integer held exactly in a double, any
// representative with |x| < 2^53.  The product is the FMA form of van der Hoeven,
// Lecerf and Quintin ("Modular SIMD arithmetic in Mathemagix", ACM TOMS 2016),
// with the quotient rounded to nearest and the last correction left out: with h = fl(a w), l = a w - h (exact by
// FMA) and q = rint(fl(h / p)), the value (h - q p) + l is exactly a w - q p:
// h - q p is an integer below 2^53, so its FMA does not round, and neither
// does the last sum.  q is within 1/2 + e of a w / p, where e collects the
// roundings of the quotient (each 2^-53 |a w / p|), so the result is below
// (1/2 + e) p; sums and differences are plain additions.
//
// Ranges, in units of p, with |w| <= p/2 (table entries are balanced):
//  * a product by a constant with its own quotient (mulc: two roundings) is
//    at most 1/2 + a/8 for a < 8 and p near 2^50 (set 0), 1/2 + a/4 for a < 4
//    and p near 2^51 (set 1);
//  * a product with the quotient taken from h (mulm: three roundings) is at
//    most 1/2 + 3a/16 (set 0), 1/2 + 3a/8 (set 1);
//  * red() gives 1/2 (plus 2^-40).
// A DFT multiplies the second input of every butterfly (by a constant, or
// reduces it where the constant is 1 after the first stage), so a value grows
// as x -> x + 1/2 + x/8 per stage: four stages take inputs of A to at most
// 2.85 A + 1.70 (set 0).  Pass twiddles bring that back to 1/2 + 3/16 of it,
// and outputs without a twiddle are reduced, so A stays at or below 1.76 and
// every value below 6.8 < 8 = 2^53 / p.  Set 1 (limit 4) reduces all 16 inputs
// of a DFT first: 2, 3.5/2, ... at most 3.87.
//
// Exactness of the product: a coefficient is at most min(la, lb) (2^64 - 1)^2
// with the lengths in digits.  Set 0 (three primes above 2^50) covers operands
// of up to 2^22 digits, that is transforms of up to 2^23 points; set 1 (above
// 2^51) up to 2^25 digits, transforms of up to 2^26.
//
// Transform structure: passes of radix 16 or 8 (the first of radix 2^(log2 S
// mod 4), or mod 3) on registers, one thread holding as many values, with LDS
// between the passes.  A transform of up to 2^14 points runs in one workgroup
// (k_flds); longer ones are cut in rows of 2^11 or 2^12 points and column DFTs
// of 2^4 .. 2^10 points (Bailey 1990).  Both operands of a product pass through
// the same LDS buffer, the first one's outputs waiting in registers, so a
// transform of T points needs 8 T bytes of LDS.
#include "fntt.hpp"

#include <vector>

#pragma clang fp contract(off)

namespace {

struct FPrime {
  double p, pinv;
  double w[8], wp[8];     // omega_16^i and omega_16^i / p
  double iw[8], iwp[8];   // inverse roots
};
__constant__ FPrime c_fp[2][CAT_NPRIMES];

// Constants of the recombination, every constant with its quotient c / p:
// x0 = k00 r0 mod p0, x1 = k11 r1 + k10 x0 mod p1, x2 = k22 r2 + k20 x0 + k21
// x1 mod p2 (the transform's scale 2^-logD is in k00, k11, k22).
struct FCrt {
  double p[3], pinv[3];
  double k00, k00q, k10, k10q, k11, k11q, k20, k20q, k21, k21q, k22, k22q;
  uint64_t pi[2];         // p0, p1
};

#define FTWS_ENTRIES 32766u    // pass tables of sizes 2^1 .. 2^14, back to back
#define FTW2_BITS 13u          // two-level table: omega_{2^26}^y = hi[y >> 13] lo[y mod 2^13]
#define FTW2 (1u << FTW2_BITS)
struct FTables {
  const double* tws3;          // the same for passes of radix 8
  const double* itws3;
  const double* tws;           // [prime][FTWS_ENTRIES]: [2^s - 2 + (k << logSR) + j] = omega_S^(j k)
  const double* itws;
  const double* lo;            // [prime][FTW2]
  const double* hi;
  const double* ilo;
  const double* ihi;
};
FTables g_ft[2];

// ------------------------------------------------------------------ arithmetic
__device__ __forceinline__ double red(double a, double p, double pinv) {
  return __builtin_fma(-__builtin_rint(a * pinv), p, a);
}
// a w mod p for a constant w with wp = w / p
__device__ __forceinline__ double mulc(double a, double w, double wp, double p) {
  const double h = a * w;
  const double q = __builtin_rint(a * wp);
  const double l = __builtin_fma(a, w, -h);
  return __builtin_fma(-q, p, h) + l;
}
__device__ __forceinline__ double mulm(double a, double w, double p, double pinv) {
  const double h = a * w;
  const double q = __builtin_rint(h * pinv);
  const double l = __builtin_fma(a, w, -h);
  return __builtin_fma(-q, p, h) + l;
}

// Radix-R DFT on registers, natural input, output y[k] in v[brev(k)].  Stage t
// has 2^t blocks; block b takes (x, y) to x + w y, x - w y with w =
// omega_16^brev3(b).  ZHI: the upper half of the input is zero (a zero-padded
// operand, entries at most 1/2): the first stage copies, and the sums of
// reduced inputs need no reduction (at most 4 after four stages, set 0).
template <int LOGR, int PS, bool ZHI>
__device__ __forceinline__ void fdft(double* v, const FPrime& c) {
  constexpr int R = 1 << LOGR;
  const double p = c.p, pinv = c.pinv;
  if constexpr (PS == 1 && !ZHI) {
#pragma unroll
    for (int i = 0; i < R; i++) v[i] = red(v[i], p, pinv);
  }
#pragma unroll
  for (int t = 0; t < LOGR; t++) {
    const int h = R >> (t + 1);
#pragma unroll
    for (int b = 0; b < (1 << t); b++) {
#pragma unroll
      for (int i = 0; i < h; i++) {
        double& x = v[2 * b * h + i];
        double& y = v[2 * b * h + i + h];
        if (t == 0 && ZHI) {
          y = x;
          continue;
        }
        double z;
        if (b != 0) z = mulc(y, c.w[brev_c(b, 3)], c.wp[brev_c(b, 3)], p);
        else if (t == 0 || (ZHI && PS == 0)) z = y;
        else z = red(y, p, pinv);
        y = x - z;
        x = x + z;
      }
    }
  }
}

// Inverse: input y[k] in v[brev(k)], output R x[j] in v[j].
template <int LOGR, int PS>
__device__ __forceinline__ void fidft(double* v, const FPrime& c) {
  constexpr int R = 1 << LOGR;
  const double p = c.p, pinv = c.pinv;
  if constexpr (PS == 1) {
#pragma unroll
    for (int i = 0; i < R; i++) v[i] = red(v[i], p, pinv);
  }
#pragma unroll
  for (int t = 0; t < LOGR; t++) {
    const int h = 1 << t;
#pragma unroll
    for (int s = 0; s < R; s += 2 * h) {
#pragma unroll
      for (int i = 0; i < h; i++) {
        double& x = v[s + i];
        double& y = v[s + i + h];
        double z;
        if (i != 0) z = mulc(y, c.iw[i * (8 >> t)], c.iwp[i * (8 >> t)], p);
        else z = t == 0 ? y : red(y, p, pinv);
        y = x - z;
        x = x + z;
      }
    }
  }
}

// Pass twiddles omega_S^(j k) (S = R << logSR) of the R values y[k] in
// v[brev(k)], read through a buffer resource: the uniform part k << logSR is
// the scalar offset.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ftw_rsrc(const double* tw, uint32_t entries) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)tw, (short)0, (int)(entries * 8u), CAT_BUF_DW3);
}
__device__ __forceinline__ double buf_ldd(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  const auto u = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0);
  return __hiloint2double((int)u[1], (int)u[0]);
}
__device__ __forceinline__ void buf_std(__amdgpu_buffer_rsrc_t r, uint32_t voff, double x) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  u32x2 u;
  u[0] = (uint32_t)__double2loint(x);
  u[1] = (uint32_t)__double2hiint(x);
  __builtin_amdgcn_raw_buffer_store_b64(u, r, (int)voff, 0, 0);
}
template <int LOGR, int LE>
__device__ __forceinline__ void ptw(double* v, const double* tws, int logSR, uint32_t j, const FPrime& c) {
  constexpr int R = 1 << LOGR;
  const __amdgpu_buffer_rsrc_t rs = ftw_rsrc(tws + ((1u << (logSR + LOGR)) - 2u), (uint32_t)R << logSR);
  v[0] = red(v[0], c.p, c.pinv);
#pragma unroll
  for (int k = 1; k < R; k++) {
    const int r = brev_c(k, LOGR);
    v[r] = mulm(v[r], buf_ldd(rs, j * 8u, ((uint32_t)k << logSR) * 8u), c.p, c.pinv);
  }
}

// A 64-bit digit (lo, hi) as a residue: hi 2^32 reduced, plus lo (below
// p/2 + 2^32).
__device__ __forceinline__ double digit(uint32_t lo, uint32_t hi, double p, double pinv) {
  return red((double)hi * 4294967296.0, p, pinv) + (double)lo;
}

// ------------------------------------------------------ passes in a workgroup
// A thread holds E = 2^LE values (LE = 3 or 4).  LDS element e of a tile of C =
// 2^logC columns (1: a plain vector) sits at (e + e/E) C + column.  Every
// radix-E pass after the first has one group per thread: thread t = (h, c), h
// = t / C; its group in sub-problems of S = E SR elements is j = h mod SR of
// sub-problem h / SR.
template <int LE>
__device__ __forceinline__ constexpr uint32_t fpad(uint32_t i) { return i + (i >> LE); }
// radix (log2) of the pass at sub-problem size 2^logS
template <int LE>
__host__ __device__ constexpr int fpass(int logS) { return (logS % LE) ? (logS % LE) : LE; }

template <int LE, int LOGSR, int PS>
__device__ __forceinline__ void mid_fwd(double* lds, uint32_t logC, const double* tws, const FPrime& c, uint32_t tid) {
  constexpr uint32_t SR = 1u << LOGSR, E = 1u << LE;
  const uint32_t h = tid >> logC, j = h & (SR - 1);
  const uint32_t b = (fpad<LE>(((h >> LOGSR) << (LOGSR + LE)) + j) << logC) + (tid & ((1u << logC) - 1));
  const uint32_t st = (SR + SR / E) << logC;
  double v[E];
#pragma unroll
  for (int k = 0; k < (int)E; k++) v[k] = lds[b + k * st];
  fdft<LE, PS, false>(v, c);
  ptw<LE, LE>(v, tws, LOGSR, j, c);
#pragma unroll
  for (int k = 0; k < (int)E; k++) lds[b + k * st] = v[brev_c(k, LE)];
}
template <int LE, int LOGSR, int PS>
__device__ __forceinline__ void mid_inv(double* lds, uint32_t logC, const double* itws, const FPrime& c, uint32_t tid) {
  constexpr uint32_t SR = 1u << LOGSR, E = 1u << LE;
  const uint32_t h = tid >> logC, j = h & (SR - 1);
  const uint32_t b = (fpad<LE>(((h >> LOGSR) << (LOGSR + LE)) + j) << logC) + (tid & ((1u << logC) - 1));
  const uint32_t st = (SR + SR / E) << logC;
  double v[E];
#pragma unroll
  for (int k = 0; k < (int)E; k++) v[brev_c(k, LE)] = lds[b + k * st];
  ptw<LE, LE>(v, itws, LOGSR, j, c);
  fidft<LE, PS>(v, c);
#pragma unroll
  for (int k = 0; k < (int)E; k++) lds[b + k * st] = v[k];
}
// Passes below the first one, which left sub-problems of 2^LOGSUB points
// (LOGSUB a multiple of LE): radix-E passes through LDS until sub-problems of
// E are left, which each thread then takes into registers.
template <int LE, int LOGSUB, int PS>
__device__ __forceinline__ void rest_fwd(double* lds, uint32_t logC, const double* tws, const FPrime& c, uint32_t tid) {
  if constexpr (LOGSUB > LE) {
    mid_fwd<LE, LOGSUB - LE, PS>(lds, logC, tws, c, tid);
    pass_sync(LOGSUB - LE, logC);
    rest_fwd<LE, LOGSUB - LE, PS>(lds, logC, tws, c, tid);
  }
}
// the inverse of rest_fwd, each pass followed by its synchronisation except
// the last, which the caller does
template <int LE, int LOGSUB, int LOGTOP, int PS>
__device__ __forceinline__ void rest_inv(double* lds, uint32_t logC, const double* itws, const FPrime& c, uint32_t tid) {
  if constexpr (LOGSUB <= LOGTOP) {
    mid_inv<LE, LOGSUB - LE, PS>(lds, logC, itws, c, tid);
    if constexpr (LOGSUB < LOGTOP) pass_sync(LOGSUB, logC);
    rest_inv<LE, LOGSUB + LE, LOGTOP, PS>(lds, logC, itws, c, tid);
  }
}

// First forward pass (radix 2^LR) of a tile whose elements i < E of a thread
// are the groups d + D k, D = E / R: group d holds x[d + D k], k < R, and is
// group j of its sub-problem (element positions j + SR k).
template <int LE, int LR, int LOGSR, int PS, bool ZHI>
__device__ __forceinline__ void first_fwd(double* lds, const double* x, uint32_t NT, uint32_t logC, const double* tws,
                                          const FPrime& c, uint32_t tid) {
  constexpr int R = 1 << LR, D = (1 << LE) / R;
  constexpr uint32_t SR = 1u << LOGSR;
#pragma unroll
  for (int d = 0; d < D; d++) {
    const uint32_t g = tid + NT * d, h = g >> logC, j = h & (SR - 1);
    double v[R];
#pragma unroll
    for (int k = 0; k < R; k++) v[k] = (ZHI && k >= R / 2) ? 0.0 : x[d + D * k];
    fdft<LR, PS, ZHI>(v, c);
    ptw<LR, LE>(v, tws, LOGSR, j, c);
    const uint32_t b = (fpad<LE>(((h >> LOGSR) << (LOGSR + LR)) + j) << logC) + (g & ((1u << logC) - 1));
#pragma unroll
    for (int k = 0; k < R; k++) lds[b + k * ((SR + (SR >> LE)) << logC)] = v[brev_c(k, LR)];
  }
}
// Last inverse pass into x[d + D k].
template <int LE, int LR, int LOGSR, int PS>
__device__ __forceinline__ void last_inv(const double* lds, double* x, uint32_t NT, uint32_t logC, const double* itws,
                                         const FPrime& c, uint32_t tid) {
  constexpr int R = 1 << LR, D = (1 << LE) / R;
  constexpr uint32_t SR = 1u << LOGSR;
#pragma unroll
  for (int d = 0; d < D; d++) {
    const uint32_t g = tid + NT * d, h = g >> logC, j = h & (SR - 1);
    const uint32_t b = (fpad<LE>(((h >> LOGSR) << (LOGSR + LR)) + j) << logC) + (g & ((1u << logC) - 1));
    double v[R];
#pragma unroll
    for (int k = 0; k < R; k++) v[brev_c(k, LR)] = lds[b + k * ((SR + (SR >> LE)) << logC)];
    ptw<LR, LE>(v, itws, LOGSR, j, c);
    fidft<LR, PS>(v, c);
#pragma unroll
    for (int k = 0; k < R; k++) x[d + D * k] = v[k];
  }
}
// The synchronisation next to the pass of radix 2^LR over sub-problems of
// 2^LOGSR: wave-local only when that pass too has one group per thread.
template <int LE, int LR, int LOGSR>
__device__ __forceinline__ void edge_sync() {
  if constexpr (LR == LE) pass_sync(LOGSR, 0);
  else __syncthreads();
}
// the E consecutive slots of a thread
template <int LE>
__device__ __forceinline__ void slots_load(const double* lds, double* v, uint32_t tid, uint32_t logC) {
  const uint32_t b = (fpad<LE>((tid >> logC) << LE) << logC) + (tid & ((1u << logC) - 1));
#pragma unroll
  for (int k = 0; k < (1 << LE); k++) v[k] = lds[b + (k << logC)];
}
template <int LE>
__device__ __forceinline__ void slots_store(double* lds, const double* v, uint32_t tid, uint32_t logC) {
  const uint32_t b = (fpad<LE>((tid >> logC) << LE) << logC) + (tid & ((1u << logC) - 1));
#pragma unroll
  for (int k = 0; k < (1 << LE); k++) lds[b + (k << logC)] = v[k];
}
// the passes of one operand of a plain vector, from the values x of its first
// pass to the outputs of the last one in v
template <int LE, int LOGN, int PS, bool ZHI>
__device__ __forceinline__ void vec_fwd(double* lds, const double* x, double* v, uint32_t NT, const double* tws,
                                        const FPrime& c, uint32_t tid) {
  constexpr int LR = fpass<LE>(LOGN), LOGSR = LOGN - LR;
  first_fwd<LE, LR, LOGSR, PS, ZHI>(lds, x, NT, 0, tws, c, tid);
  edge_sync<LE, LR, LOGSR>();
  rest_fwd<LE, LOGSR, PS>(lds, 0, tws, c, tid);
  slots_load<LE>(lds, v, tid, 0);
}
// a (outputs of the last but one pass of the first operand), b (of the second)
// -> their product's inverse transform, in the order of the first pass
template <int LE, int LOGN, int PS>
__device__ __forceinline__ void vec_mul_inv(double* lds, double* a, double* b, uint32_t NT, const double* itws,
                                            const FPrime& c, uint32_t tid) {
  constexpr int LR = fpass<LE>(LOGN), LOGSR = LOGN - LR;
  fdft<LE, PS, false>(a, c);
  fdft<LE, PS, false>(b, c);
#pragma unroll
  for (int k = 0; k < (1 << LE); k++) a[k] = mulm(red(a[k], c.p, c.pinv), b[k], c.p, c.pinv);
  fidft<LE, PS>(a, c);
  slots_store<LE>(lds, a, tid, 0);
  if constexpr (LOGSR > LE) {
    pass_sync(LE, 0);
    rest_inv<LE, 2 * LE, LOGSR, PS>(lds, 0, itws, c, tid);
  }
  edge_sync<LE, LR, LOGSR>();
  last_inv<LE, LR, LOGSR, PS>(lds, a, NT, 0, itws, c, tid);
}

// Twiddles theta^(e0 + step i), i = 0 .. 15, times the 16 values of one or two
// arrays.  theta = omega_S^f; e0 f and step f as exponents of omega_{2^26}.
template <int PS>
struct Geo {
  double w[4], r4;
  double p, pinv;
  __device__ __forceinline__ static double tw2(const double* lo, const double* hi, uint32_t y, double p, double pinv) {
    return fix(mulm(lo[y & (FTW2 - 1)], hi[y >> FTW2_BITS], p, pinv), p, pinv);
  }
  // set 0: |w| <= 0.68 throughout; set 1 reduces every power
  __device__ __forceinline__ static double fix(double x, double p, double pinv) {
    if constexpr (PS == 1) return red(x, p, pinv);
    else return x;
  }
  __device__ __forceinline__ Geo(const double* lo, const double* hi, uint32_t y0, uint32_t ystep, double p_,
                                 double pinv_)
      : p(p_), pinv(pinv_) {
    const uint32_t mask = (1u << FNTT_MAX_LOGD) - 1;
    const double r1 = tw2(lo, hi, ystep & mask, p, pinv);
    w[0] = tw2(lo, hi, y0 & mask, p, pinv);
    const double r2 = fix(mulm(r1, r1, p, pinv), p, pinv);
    r4 = fix(mulm(r2, r2, p, pinv), p, pinv);
    w[1] = fix(mulm(w[0], r1, p, pinv), p, pinv);
    w[2] = fix(mulm(w[0], r2, p, pinv), p, pinv);
    w[3] = fix(mulm(w[1], r2, p, pinv), p, pinv);
  }
  __device__ __forceinline__ void step() {
#pragma unroll
    for (int i = 0; i < 4; i++) w[i] = fix(mulm(w[i], r4, p, pinv), p, pinv);
  }
};

// limbs of an operand: the digit at position pos (zero past the end)
__device__ __forceinline__ uint2 limb2(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off) {
  return make_uint2(buf_ld(rs, byte_off), buf_ld(rs, byte_off + 4u));
}

// ---------------------------------------------------------------------------
// Whole products in one workgroup, transforms of 2^LOGD digits.  A tile holds
// 2^LOGT slots (2^12 at least, 2^(LOGT - LOGD) products); grid: 3 x tiles,
// renumbered so that each XCD takes a contiguous run of (tile, prime) pairs
// and the three primes of a tile read the operands once from HBM.  ZHI: no
// operand of the batch is longer than N/2 digits.
constexpr int flds_tile(int logD) { return logD < 12 ? 12 : logD; }
// Values per thread: 8 (radix-8 passes, at most 64 registers, room for eight waves
// per SIMD) up to 2^12 digits and at 2^13 (66 registers: seven waves, of which a
// workgroup of 1,024 threads fills four, so one stays on a CU); 16 at 2^14, where a
// workgroup has 1,024 threads too.
// Against 16 everywhere (four waves): C(10^5) 0.238 -> 0.230 ms, C(10^7) 0.619
// -> 0.600, the 4,096-product batch 2.24 -> 2.18.  The rows of the four-step
// path, which are bound by vector issue and HBM and not by latency, lose 3 %
// with 8 (their twiddle loads and LDS passes weigh more): they keep 16.
constexpr int flds_le(int logD) { return logD <= 13 ? 3 : 4; }
template <int LOGD, bool ZHI>
__global__ void __launch_bounds__((1 << flds_tile(LOGD)) >> flds_le(LOGD))
    __attribute__((amdgpu_waves_per_eu(flds_le(LOGD) == 3 ? 6 : 4)))
k_flds(DescView dv, uint64_t m0_, uint64_t nmul, const uint32_t* __restrict__ ain, const uint32_t* __restrict__ bin,
       double* __restrict__ res, uint64_t stride, FTables tb) {
  constexpr int LOGT = flds_tile(LOGD), LE = flds_le(LOGD), LR = fpass<LE>(LOGD), LOGSR = LOGD - LR;
  constexpr uint32_t T = 1u << LOGT, NT = T >> LE, N = 1u << LOGD, PER = T / N, SR = 1u << LOGSR;
  constexpr int R = 1 << LR, E = 1 << LE, D = E / R;
  __shared__ double lds[fpad<LE>(T)];
  __shared__ MulDesc ds[PER];
  const uint32_t tid = threadIdx.x;
  const uint32_t wid = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t prime = wid % CAT_NPRIMES;
  const FPrime& c = c_fp[0][prime];
  const uint64_t m0 = (uint64_t)(wid / CAT_NPRIMES) * PER;
  const uint32_t cnt = (uint32_t)min((uint64_t)PER, nmul - m0);
  for (uint32_t i = tid; i < PER; i += NT) ds[i] = dv.slot(m0_ + m0 + i, m0_ + m0, m0_ + m0 + cnt);
  __syncthreads();
  const double* tws = (LE == 3 ? tb.tws3 : tb.tws) + (size_t)prime * FTWS_ENTRIES;
  const double* itws = (LE == 3 ? tb.itws3 : tb.itws) + (size_t)prime * FTWS_ENTRIES;
  double a[E], b[E];
  // thread t holds the elements t + NT i = group d of the first pass at k
  // (i = d + D k): position j + SR k of product blk
  constexpr int RK = ZHI ? R / 2 : R, NR = ZHI ? E / 2 : E;
  uint2 ra[NR], rb[NR];
#pragma unroll
  for (int d = 0; d < D; d++) {
    const uint32_t g = tid + NT * d, j = g & (SR - 1);
    const MulDesc& m = ds[g >> LOGSR];
    const uint32_t la = m.la, lb = m.lb;
    const uint32_t *sa = ain + m.a_off, *sb = bin + m.b_off;
#pragma unroll
    for (int k = 0; k < RK; k++) {
      // clamped addresses and masks: every load is issued at once
      const uint32_t q = 2 * (j + SR * k);
      const uint32_t x0 = sa[q < la ? q : 0], x1 = sa[q + 1 < la ? q + 1 : 0];
      const uint32_t y0 = sb[q < lb ? q : 0], y1 = sb[q + 1 < lb ? q + 1 : 0];
      ra[d + D * k] = make_uint2(q < la ? x0 : 0u, q + 1 < la ? x1 : 0u);
      rb[d + D * k] = make_uint2(q < lb ? y0 : 0u, q + 1 < lb ? y1 : 0u);
    }
  }
#pragma unroll
  for (int i = 0; i < NR; i++) a[i] = digit(ra[i].x, ra[i].y, c.p, c.pinv);
  vec_fwd<LE, LOGD, 0, ZHI>(lds, a, a, NT, tws, c, tid);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NR; i++) b[i] = digit(rb[i].x, rb[i].y, c.p, c.pinv);
  vec_fwd<LE, LOGD, 0, ZHI>(lds, b, b, NT, tws, c, tid);
  vec_mul_inv<LE, LOGD, 0>(lds, a, b, NT, itws, c, tid);
  double* out = res + (size_t)prime * stride;
#pragma unroll
  for (int d = 0; d < D; d++) {
    const uint32_t g = tid + NT * d, j = g & (SR - 1);
    const MulDesc& m = ds[g >> LOGSR];
    const uint32_t L = (m.la + m.lb + 1) / 2;
    double* o = out + m.r_off;
#pragma unroll
    for (int k = 0; k < R; k++) {
      const uint32_t pos = j + SR * k;
      if (pos < L) o[pos] = a[d + D * k];
    }
    if (j == 0 && L > N) o[N] = 0.0;   // la + lb = 2 N + 1: no coefficient there
  }
}

// ---------------------------------------------------------------------------
// Four-step: F[((m*3 + prime)*2 + op) * 2^logD + position], doubles.
struct FGeom {
  int logD, logS, logC;
  // tile bx of the pass over sub-problems of 2^logS with column length 2^logL
  __device__ __forceinline__ void locate(int logL, uint64_t bx, uint64_t* m, uint32_t* base, uint32_t* j0) const {
    const int lt = logS - logL - logC;                    // tiles per sub-problem (log2)
    const int lp = logD - logS + lt;                      // tiles per product
    *m = bx >> lp;
    const uint32_t r = (uint32_t)(bx & ((1ull << lp) - 1));
    *base = (r >> lt) << logS;
    *j0 = (r & ((1u << lt) - 1)) << logC;
  }
};

// Column DFT of 2^LOGL points over tiles of 2^LOGT values (C = 2^logC
// neighbouring columns), one thread per 16 values.  FIRST: the operands'
// digits come from limbs; otherwise from F, times the twiddles of the pass
// before (sub-problems 2^prevS, column length 2^prevL).  The results go to F,
// reduced; the twiddles of this pass are applied by the next one.
// Bound by HBM: 8 B written per digit slot, prime and operand (and 4 to 8
// read), about 70 FP64 instructions.
template <int LOGL, int PS, bool FIRST>
__global__ void __launch_bounds__(LOGL <= 8 ? 256 : 512)
k_fcol_fwd(DescView dv, FGeom fg, uint64_t m0_, int prevS, int prevL, const uint32_t* __restrict__ ain,
           const uint32_t* __restrict__ bin, double* __restrict__ F, FTables tb) {
  constexpr int LOGT = LOGL <= 8 ? 12 : 13, LR = pass_logr(LOGL), LOGSR = LOGL - LR;
  constexpr uint32_t T = 1u << LOGT, NT = T / 16;
  constexpr uint32_t logC = LOGT - LOGL;
  constexpr uint32_t C = 1u << logC, RI = NT >> logC;     // rows per step of i
  __shared__ double lds[LOGL > 4 ? ((1u << LOGL) + (1u << LOGL) / 16) * C : 1];
  const uint32_t tid = threadIdx.x;
  const uint32_t wid = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t prime = wid % CAT_NPRIMES, op = blockIdx.z;
  const FPrime& c = c_fp[PS][prime];
  uint64_t m;
  uint32_t base, j0;
  fg.locate(LOGL, wid / CAT_NPRIMES, &m, &base, &j0);
  if (op && m && dv.uni) return;     // one second operand for the whole batch
  const int logSig = fg.logS - LOGL;
  const uint64_t N = 1ull << fg.logD;
  double* f = F + ((m * 3 + prime) * 2 + op) * N;
  const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc((void*)f, (short)0, (int)(uint32_t)(N * 8), CAT_BUF_DW3);
  const uint32_t pos0 = base + ((tid >> logC) << logSig) + j0 + (tid & (C - 1));   // element i: + (RI i) << logSig
  const double* tws = tb.tws + (size_t)prime * FTWS_ENTRIES;
  double x[16];
  bool zhi = false;
  if constexpr (FIRST) {
    const MulDesc d = dv.get(m0_ + m);
    const uint32_t len = op ? d.lb : d.la;
    zhi = len <= N;                                       // at most N/2 digits
    const __amdgpu_buffer_rsrc_t rs = words_rsrc(op ? bin + d.b_off : ain + d.a_off, len);
    uint2 r[16];
    if (zhi) {
#pragma unroll
      for (int i = 0; i < 8; i++) r[i] = limb2(rs, (pos0 + ((RI * i) << logSig)) * 8u);
#pragma unroll
      for (int i = 0; i < 8; i++) x[i] = digit(r[i].x, r[i].y, c.p, c.pinv);
    } else {
#pragma unroll
      for (int i = 0; i < 16; i++) r[i] = limb2(rs, (pos0 + ((RI * i) << logSig)) * 8u);
#pragma unroll
      for (int i = 0; i < 16; i++) x[i] = digit(r[i].x, r[i].y, c.p, c.pinv);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; i++) x[i] = buf_ldd(rf, (pos0 + ((RI * i) << logSig)) * 8u, 0);
    const uint32_t fr = out_freq((base >> fg.logS) & ((1u << prevL) - 1), prevL) << (FNTT_MAX_LOGD - prevS);
    Geo<PS> gw(tb.lo + (size_t)prime * FTW2, tb.hi + (size_t)prime * FTW2, (pos0 - base) * fr, (RI << logSig) * fr,
               c.p, c.pinv);
#pragma unroll
    for (int i = 0; i < 16; i++) {
      x[i] = mulm(x[i], gw.w[i & 3], c.p, c.pinv);
      if ((i & 3) == 3 && i < 15) gw.step();
    }
  }
  double v[16];
  if constexpr (LOGL == 4) {
    if (FIRST && zhi) {
#pragma unroll
      for (int i = 8; i < 16; i++) x[i] = 0.0;
      fdft<4, PS, FIRST>(x, c);
    } else {
      fdft<4, PS, false>(x, c);
    }
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = x[k];
  } else {
    if (FIRST && zhi) first_fwd<4, LR, LOGSR, PS, FIRST>(lds, x, NT, logC, tws, c, tid);
    else first_fwd<4, LR, LOGSR, PS, false>(lds, x, NT, logC, tws, c, tid);
    __syncthreads();
    rest_fwd<4, LOGSR, PS>(lds, logC, tws, c, tid);
    slots_load<4>(lds, v, tid, logC);
    fdft<4, PS, false>(v, c);
  }
  const uint32_t q0 = base + ((16 * (tid >> logC)) << logSig) + j0 + (tid & (C - 1));
#pragma unroll
  for (int k = 0; k < 16; k++)
    buf_std(rf, (q0 + ((uint32_t)k << logSig)) * 8u, red(v[brev_c(k, 4)], c.p, c.pinv));
}

// Inverse column DFT.  FIRST (the outermost pass): the residues of positions
// below la + lb limbs; otherwise back to F, times the inverse twiddles of the
// pass before.
template <int LOGL, int PS, bool FIRST>
__global__ void __launch_bounds__(LOGL <= 8 ? 256 : 512)
k_fcol_inv(DescView dv, FGeom fg, uint64_t m0_, int prevS, int prevL, double* __restrict__ F,
           double* __restrict__ res, uint64_t stride, FTables tb) {
  constexpr int LOGT = LOGL <= 8 ? 12 : 13, LR = pass_logr(LOGL), LOGSR = LOGL - LR;
  constexpr uint32_t T = 1u << LOGT, NT = T / 16;
  constexpr uint32_t logC = LOGT - LOGL;
  constexpr uint32_t C = 1u << logC, RI = NT >> logC;
  __shared__ double lds[LOGL > 4 ? ((1u << LOGL) + (1u << LOGL) / 16) * C : 1];
  const uint32_t tid = threadIdx.x;
  const uint32_t prime = blockIdx.y;
  const FPrime& c = c_fp[PS][prime];
  uint64_t m;
  uint32_t base, j0;
  fg.locate(LOGL, xcd_remap(blockIdx.x, gridDim.x), &m, &base, &j0);
  const int logSig = fg.logS - LOGL;
  const uint64_t N = 1ull << fg.logD;
  double* f = F + ((m * 3 + prime) * 2 + 0) * N;
  const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc((void*)f, (short)0, (int)(uint32_t)(N * 8), CAT_BUF_DW3);
  const uint32_t pos0 = base + ((tid >> logC) << logSig) + j0 + (tid & (C - 1));
  const double* itws = tb.itws + (size_t)prime * FTWS_ENTRIES;
  double x[16];
  {
    const uint32_t q0 = base + ((16 * (tid >> logC)) << logSig) + j0 + (tid & (C - 1));
#pragma unroll
    for (int k = 0; k < 16; k++) x[brev_c(k, 4)] = buf_ldd(rf, (q0 + ((uint32_t)k << logSig)) * 8u, 0);
  }
  fidft<4, PS>(x, c);
  if constexpr (LOGL > 4) {
    slots_store<4>(lds, x, tid, logC);
    __syncthreads();
    if constexpr (LOGSR > 4) {
      rest_inv<4, 8, LOGSR, PS>(lds, logC, itws, c, tid);
      __syncthreads();
    }
    last_inv<4, LR, LOGSR, PS>(lds, x, NT, logC, itws, c, tid);
  }
  if constexpr (FIRST) {
    const MulDesc d = dv.get(m0_ + m);
    const uint64_t L = ((uint64_t)d.la + d.lb + 1) / 2;
    double* out = res + (size_t)prime * stride + d.r_off;
    // positions at or past L fall outside the buffer's range: not written
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)out, (short)0, (int)(uint32_t)(L * 8), CAT_BUF_DW3);
#pragma unroll
    for (int i = 0; i < 16; i++) buf_std(rs, (pos0 + ((RI * i) << logSig)) * 8u, x[i]);
    if (L > N && base == 0 && j0 == 0 && tid == 0) out[N] = 0.0;
  } else {
    const uint32_t fr = out_freq((base >> fg.logS) & ((1u << prevL) - 1), prevL) << (FNTT_MAX_LOGD - prevS);
    Geo<PS> gw(tb.ilo + (size_t)prime * FTW2, tb.ihi + (size_t)prime * FTW2, (pos0 - base) * fr, (RI << logSig) * fr,
               c.p, c.pinv);
#pragma unroll
    for (int i = 0; i < 16; i++) {
      x[i] = mulm(red(x[i], c.p, c.pinv), gw.w[i & 3], c.p, c.pinv);
      if ((i & 3) == 3 && i < 15) gw.step();
      buf_std(rf, (pos0 + ((RI * i) << logSig)) * 8u, x[i]);
    }
  }
}

// Rows of 2^LOGD points of both operands: the column pass's twiddles, both
// forward transforms, the pointwise product, the inverse transform and the
// inverse twiddles.  Grid: rows of the batch x primes.  Bound by vector issue
// and by HBM at once: 24 B per digit slot and prime, about 260 FP64
// instructions.  126 registers for rows of 2^12; rows of 2^11 spill two.
template <int LOGM, int PS>
__global__ void __launch_bounds__((1 << LOGM) / 16) __attribute__((amdgpu_waves_per_eu(4)))
k_frow(int logD, int logS, int logL, int bshared, double* __restrict__ F, FTables tb) {
  constexpr int LE = 4, E = 1 << LE;
  constexpr uint32_t M = 1u << LOGM, NT = M >> LE;
  __shared__ double lds[fpad<LE>(M)];
  const uint32_t tid = threadIdx.x, prime = blockIdx.y;
  const FPrime& c = c_fp[PS][prime];
  const int logQ = logD - LOGM;
  const uint64_t N = 1ull << logD;
  const uint64_t m = blockIdx.x >> logQ;
  const uint32_t q = blockIdx.x & ((1u << logQ) - 1);
  double* fa = F + ((m * 3 + prime) * 2 + 0) * N + ((uint64_t)q << LOGM);
  // a common second operand: product 0's
  const double* fb = F + (((bshared ? 0 : m) * 3 + prime) * 2 + 1) * N + ((uint64_t)q << LOGM);
  const double* tws = tb.tws + (size_t)prime * FTWS_ENTRIES;
  const double* itws = tb.itws + (size_t)prime * FTWS_ENTRIES;
  double a[E], b[E];
#pragma unroll
  for (int i = 0; i < E; i++) {
    a[i] = fa[tid + NT * i];
    b[i] = fb[tid + NT * i];
  }
  // position j of row q takes omega_S^(j f), f the frequency of q
  const uint32_t fr = out_freq(q & ((1u << logL) - 1), logL) << (FNTT_MAX_LOGD - logS);
  {
    Geo<PS> gw(tb.lo + (size_t)prime * FTW2, tb.hi + (size_t)prime * FTW2, tid * fr, NT * fr, c.p, c.pinv);
#pragma unroll
    for (int i = 0; i < E; i++) {
      a[i] = mulm(a[i], gw.w[i & 3], c.p, c.pinv);
      b[i] = mulm(b[i], gw.w[i & 3], c.p, c.pinv);
      if ((i & 3) == 3 && i < E - 1) gw.step();
    }
  }
  vec_fwd<LE, LOGM, PS, false>(lds, a, a, NT, tws, c, tid);
  __syncthreads();
  vec_fwd<LE, LOGM, PS, false>(lds, b, b, NT, tws, c, tid);
  vec_mul_inv<LE, LOGM, PS>(lds, a, b, NT, itws, c, tid);
  {
    Geo<PS> gw(tb.ilo + (size_t)prime * FTW2, tb.ihi + (size_t)prime * FTW2, tid * fr, NT * fr, c.p, c.pinv);
#pragma unroll
    for (int i = 0; i < E; i++) {
      fa[tid + NT * i] = mulm(red(a[i], c.p, c.pinv), gw.w[i & 3], c.p, c.pinv);
      if ((i & 3) == 3 && i < E - 1) gw.step();
    }
  }
}

// ---------------------------------------------------------------------------
// Recombination and carries.  V = x0 + p0 (x1 + p1 x2) < 2^153 by Garner's
// method, as v0 + v1 2^64 + v2 2^128.
__device__ __forceinline__ double canon(double x, double p, double pinv) {
  x = red(x, p, pinv);
  return x + (x < 0.0 ? p : 0.0);
}
// an integer 0 <= x < 2^52
__device__ __forceinline__ uint64_t to_u52(double x) {
  return (uint64_t)__double_as_longlong(x + 4503599627370496.0) & 0xFFFFFFFFFFFFFull;
}
// from x0, x1 and the third residue
__device__ __forceinline__ void fcrt_join(double x0, double x1, double r2, const FCrt& k, uint64_t& v0, uint64_t& v1,
                                          uint32_t& v2) {
  const double x2 = canon(mulc(r2, k.k22, k.k22q, k.p[2]) + (mulc(x0, k.k20, k.k20q, k.p[2]) +
                                                             mulc(x1, k.k21, k.k21q, k.p[2])),
                          k.p[2], k.pinv[2]);
  const unsigned __int128 t = (unsigned __int128)k.pi[1] * to_u52(x2) + to_u52(x1);
  const unsigned __int128 m1 = (unsigned __int128)k.pi[0] * (uint64_t)t + to_u52(x0);
  const unsigned __int128 m2 = (unsigned __int128)k.pi[0] * (uint64_t)(t >> 64) + (uint64_t)(m1 >> 64);
  v0 = (uint64_t)m1;
  v1 = (uint64_t)m2;
  v2 = (uint32_t)(m2 >> 64);
}
__device__ __forceinline__ void fcrt_value(double r0, double r1, double r2, const FCrt& k, uint64_t& v0, uint64_t& v1,
                                           uint32_t& v2) {
  const double x0 = canon(mulc(r0, k.k00, k.k00q, k.p[0]), k.p[0], k.pinv[0]);
  const double x1 = canon(mulc(r1, k.k11, k.k11q, k.p[1]) + mulc(x0, k.k10, k.k10q, k.p[1]), k.p[1], k.pinv[1]);
  fcrt_join(x0, x1, r2, k, v0, v1, v2);
}
// The column value in the radix of the carries, v0 + v1 R + v2 R^2: R = 2^64, or
// with DEC R = 10^18 (decimal joins; digits below R) after `add` is added.  There
// V < 2^25 R^2 + R, so both quotients that are below 2^31 come from FP64 (off by
// one at most, and seen from the remainder) and one division by the reciprocal is
// left: with d = 16 R, (u2, u1, u0) = 16 V, u1's remainder mod d tells an
// overestimate (just below 2^64) from an underestimate (just above d).
__device__ __forceinline__ void dec_split(uint64_t add, uint64_t& v0, uint64_t& v1, uint32_t& v2) {
  v0 += add;
  const uint32_t c = v0 < add;
  v1 += c;
  v2 += (v1 < c);
  const uint32_t u2 = (v2 << 4) | (uint32_t)(v1 >> 60);
  const uint64_t u1 = (v1 << 4) | (v0 >> 60), u0 = v0 << 4;
  uint32_t q1 = (uint32_t)(((double)u2 * 0x1p64 + (double)u1) * (1.0 / (double)DEC_D));
  uint64_t r = u1 - q1 * DEC_D;
  if (r >= DEC_D) {
    const bool under = r - DEC_D < (1ull << 60);
    q1 = under ? q1 + 1 : q1 - 1;
    r = under ? r - DEC_D : r + DEC_D;
  }
  const uint64_t q0 = div_d(r, u0, &r);
  v0 = r >> 4;
  v2 = (uint32_t)(((double)q1 * 0x1p64 + (double)q0) * (1.0 / (double)DEC_B));
  v1 = q0 - v2 * DEC_B;
  if ((int64_t)v1 < 0) {
    v2--;
    v1 += DEC_B;
  } else if (v1 >= DEC_B) {
    v2++;
    v1 -= DEC_B;
  }
}
template <bool DEC>
__device__ __forceinline__ void fcol_value(double r0, double r1, double r2, const FCrt& k, uint64_t add, uint64_t& v0,
                                           uint64_t& v1, uint32_t& v2) {
  fcrt_value(r0, r1, r2, k, v0, v1, v2);
  if constexpr (DEC) dec_split(add, v0, v1, v2);
}
// s = a + b + c as s mod R and the carry h = s / R
template <bool DEC>
__device__ __forceinline__ uint64_t fcol_sum(uint64_t a, uint64_t b, uint64_t c, uint32_t* h) {
  const uint64_t t = a + b, s = t + c;
  if constexpr (DEC) {
    *h = (s >= DEC_B) + (s >= 2 * DEC_B);
    return s - *h * DEC_B;
  } else {
    *h = (t < a) + (s < c);
    return s;
  }
}
// u = lo + carries of the column before (at most 2): does it generate a carry,
// does it pass one on?
template <bool DEC>
__device__ __forceinline__ bool fcol_gen(uint64_t u, uint64_t lo) {
  return DEC ? u >= DEC_B : u < lo;
}
template <bool DEC>
__device__ __forceinline__ bool fcol_prop(uint64_t u) {
  return u == (DEC ? DEC_B - 1 : ~0ull);
}
// the digit u + c and its carry
template <bool DEC>
__device__ __forceinline__ uint64_t fcol_digit(uint64_t u, bool gk, uint32_t* c) {
  uint64_t y = u + *c;
  if constexpr (DEC) {
    *c = y >= DEC_B;
    if (*c) y -= DEC_B;
  } else {
    *c = (y < u || gk) ? 1u : 0u;
  }
  return y;
}
// digit k of the addend (limbs at `add`, add_len of them)
__device__ __forceinline__ uint64_t add_digit(const uint32_t* __restrict__ add, uint64_t add_len, uint64_t k) {
  const uint64_t q = 2 * k < add_len ? 2 * k : 0;
  const uint64_t x = ((uint64_t)add[q + 1] << 32) | add[q];
  return 2 * k < add_len ? x : 0;
}

// Positions kb + E tid .. of a block, as in k_crt: digit k is v0(k) + v1(k-1)
// + v2(k-2) plus carries; with s_k that sum, x_k = s_k mod 2^64, y_k = s_k >>
// 64 and u_k = x_k + y_{k-1}, the carries left are binary.  The first wave
// recomputes the CTX positions below the block for the left context; unless
// every u of them propagates they also decide the carry into the block
// (*spec: 0 or 1, else 2).
#define FCRT_CTX 16
template <bool DEC>
__device__ __forceinline__ void fcrt_local(uint64_t len, const double* __restrict__ r0, const double* __restrict__ r1,
                                           const double* __restrict__ r2, const uint32_t* __restrict__ add,
                                           uint64_t add_len, const FCrt& kc, uint64_t kb, uint4* xv, uint32_t* tmp,
                                           uint64_t* ul, bool* gk, bool* Gt, bool* Pt, uint32_t* spec) {
  static_assert(FCRT_E >= 3, "a thread's last column must lie inside the thread");
  const uint32_t tid = threadIdx.x;
  const uint64_t k0 = kb + (uint64_t)tid * FCRT_E;
  const bool lctx = tid < FCRT_CTX && kb + tid >= FCRT_CTX;
  double x0[FCRT_E], x1[FCRT_E], x2[FCRT_E], y0 = 0.0, y1 = 0.0, y2 = 0.0;
  if (kb + FCRT_BLOCK <= len) {
    // read once: non-temporal
#pragma unroll
    for (int i = 0; i < FCRT_E; i++) {
      x0[i] = __builtin_nontemporal_load(r0 + k0 + i);
      x1[i] = __builtin_nontemporal_load(r1 + k0 + i);
      x2[i] = __builtin_nontemporal_load(r2 + k0 + i);
    }
  } else {
#pragma unroll
    for (int i = 0; i < FCRT_E; i++) {
      const bool in = k0 + i < len;
      const uint64_t kk = in ? k0 + i : 0;
      x0[i] = in ? r0[kk] : 0.0;
      x1[i] = in ? r1[kk] : 0.0;
      x2[i] = in ? r2[kk] : 0.0;
    }
  }
  if (lctx) {
    y0 = r0[kb + tid - FCRT_CTX];
    y1 = r1[kb + tid - FCRT_CTX];
    y2 = r2[kb + tid - FCRT_CTX];
  }
  uint64_t ad[FCRT_E] = {}, yd = 0;
  if constexpr (DEC) {
#pragma unroll
    for (int i = 0; i < FCRT_E; i++) ad[i] = add_digit(add, add_len, k0 + i);
    if (lctx) yd = add_digit(add, add_len, kb + tid - FCRT_CTX);
  }
  uint64_t a0[FCRT_E], a1[FCRT_E], lo[FCRT_E];
  uint32_t a2[FCRT_E], h[FCRT_E];
#pragma unroll
  for (int i = 0; i < FCRT_E; i++) fcol_value<DEC>(x0[i], x1[i], x2[i], kc, ad[i], a0[i], a1[i], a2[i]);
#pragma unroll
  for (int i = 2; i < FCRT_E; i++) lo[i] = fcol_sum<DEC>(a0[i], a1[i - 1], a2[i - 2], &h[i]);
  uint4 bctx = make_uint4(0, 0, 0, 0);
  uint32_t sp = 2;
  if (tid < 64) {
    uint64_t c0, c1;
    uint32_t c2;
    fcol_value<DEC>(y0, y1, y2, kc, yd, c0, c1, c2);
    const uint64_t b1 = __shfl_up((unsigned long long)c1, 1, 64);
    const uint32_t b2 = __shfl_up(c2, 1, 64), d2 = __shfl_up(c2, 2, 64);
    uint32_t hh;
    const uint64_t cl = fcol_sum<DEC>(c0, b1, d2, &hh);          // column kb - CTX + tid (lanes >= 2)
    const uint32_t hq = __shfl_up(hh, 1, 64);
    const uint64_t cu = cl + hq;                            // u of it (lanes >= 3)
    const bool g = fcol_gen<DEC>(cu, cl);
    const bool valid = tid >= 3 && tid < FCRT_CTX;
    const uint64_t gm = __ballot(valid && g);
    const uint64_t dm = gm | __ballot(valid && !g && !fcol_prop<DEC>(cu));
    if (dm) sp = (uint32_t)((gm >> (63 - __builtin_clzll(dm))) & 1ull);
    bctx = make_uint4((uint32_t)c1, (uint32_t)(c1 >> 32), c2 | (hh << 30), b2);
  }
  __syncthreads();   // xv may still be read by a previous call
  // v2 < 2^26: the column's carry h <= 2 rides in the two bits above it
  xv[tid + 1] = make_uint4((uint32_t)a1[FCRT_E - 1], (uint32_t)(a1[FCRT_E - 1] >> 32),
                           a2[FCRT_E - 1] | (h[FCRT_E - 1] << 30), a2[FCRT_E - 2]);
  if (tid == FCRT_CTX - 1) xv[0] = bctx;
  if (tid == 0) *spec = sp;
  __syncthreads();
  const uint4 z = xv[tid];
  const uint32_t zv2 = z.z & 0x3FFFFFFFu;
  lo[0] = fcol_sum<DEC>(a0[0], ((uint64_t)z.y << 32) | z.x, z.w, &h[0]);
  lo[1] = fcol_sum<DEC>(a0[1], a1[0], zv2, &h[1]);
  bool G = false, P = true;
  uint32_t hp = z.z >> 30;
#pragma unroll
  for (int i = 0; i < FCRT_E; i++) {
    ul[i] = lo[i] + hp;
    gk[i] = fcol_gen<DEC>(ul[i], lo[i]);
    hp = h[i];
    const bool pr = fcol_prop<DEC>(ul[i]);
    G = gk[i] || (pr && G);
    P = P && pr;
  }
  *Gt = G;
  *Pt = P;
  uint32_t cout;
  bool ap;
  wave_carry(G, P, 0, &cout, &ap);
  if ((tid & 63) == 0) tmp[tid >> 6] = cout | (ap ? 2u : 0u);
  __syncthreads();
}
__device__ __forceinline__ uint32_t fcrt_pair(const uint32_t* tmp) {
  uint32_t bG = 0, bP = 1;
  for (uint32_t w = 0; w < FCRT_THREADS / 64; w++) {
    const uint32_t x = tmp[w];
    bG = (x & 1u) | ((x >> 1) & bG);
    bP = bP & (x >> 1);
  }
  return bG | (bP << 1);
}

// The outermost inverse column pass of all three primes with the recombination:
// the residues stay in registers, and digits leave instead of them.  A wave's
// lanes hold runs of CR = min(C, 64) neighbouring digits (C columns of a tile);
// the carries inside a run are resolved here (shuffles and ballots), and what
// leaves it at the top, below 2^96, goes to two words per run: 8 + 16 / CR B
// written per digit and read again by the carry kernel instead of 24.
// Bound by HBM: 24 B read per digit.  About 200 registers (the first two primes'
// values, the loads of the next one), so two waves per SIMD; with three, which
// spill, it is 3 % slower at C(2,050,572,903).  There: the carry kernel 0.44 -> 0.24
// ms a level, this pass as long as k_fcol_inv; 69.1 -> 67.6 ms in all.
template <int LOGL, int PS, bool DEC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_fcol_crt(DescView dv, SegView sv, FGeom fg, FCrt kc, const double* __restrict__ F, double* __restrict__ res,
           uint64_t stride, const uint32_t* __restrict__ add, FTables tb) {
  constexpr int LOGT = 12, LR = pass_logr(LOGL), LOGSR = LOGL - LR;
  constexpr uint32_t T = 1u << LOGT, NT = T / 16;
  constexpr uint32_t logC = LOGT - LOGL, logCR = logC < 6 ? logC : 6;
  constexpr uint32_t C = 1u << logC, RI = NT >> logC, CR = 1u << logCR;
  __shared__ double lds[LOGL > 4 ? ((1u << LOGL) + (1u << LOGL) / 16) * C : 1];
  const uint32_t tid = threadIdx.x, lane = tid & (CR - 1);
  uint64_t m;
  uint32_t base, j0;
  fg.locate(LOGL, xcd_remap(blockIdx.x, gridDim.x), &m, &base, &j0);
  const int logSig = fg.logS - LOGL;
  const uint64_t N = 1ull << fg.logD;
  const uint32_t q0 = base + ((16 * (tid >> logC)) << logSig) + j0 + (tid & (C - 1));
  auto load = [&](int prime, double* y) {
    const double* f = F + (m * 3 + prime) * 2 * N;
    const __amdgpu_buffer_rsrc_t rf =
        __builtin_amdgcn_make_buffer_rsrc((void*)f, (short)0, (int)(uint32_t)(N * 8), CAT_BUF_DW3);
#pragma unroll
    for (int k = 0; k < 16; k++) y[k] = buf_ldd(rf, (q0 + ((uint32_t)k << logSig)) * 8u, 0);
  };
  double x[16], nx[16], y0[16], y1[16];
  load(0, nx);
  for (int prime = 0; prime < CAT_NPRIMES; prime++) {
    const FPrime& c = c_fp[PS][prime];
    const double* itws = tb.itws + (size_t)prime * FTWS_ENTRIES;
#pragma unroll
    for (int k = 0; k < 16; k++) x[brev_c(k, 4)] = nx[k];
    if (prime + 1 < CAT_NPRIMES) load(prime + 1, nx);   // in flight during this prime's passes
    fidft<4, PS>(x, c);
    if constexpr (LOGL > 4) {
      if (prime) __syncthreads();
      slots_store<4>(lds, x, tid, logC);
      __syncthreads();
      if constexpr (LOGSR > 4) {
        rest_inv<4, 8, LOGSR, PS>(lds, logC, itws, c, tid);
        __syncthreads();
      }
      last_inv<4, LR, LOGSR, PS>(lds, x, NT, logC, itws, c, tid);
    }
    if (prime == 0) {
#pragma unroll
      for (int i = 0; i < 16; i++) y0[i] = canon(mulc(x[i], kc.k00, kc.k00q, kc.p[0]), kc.p[0], kc.pinv[0]);
    } else if (prime == 1) {
#pragma unroll
      for (int i = 0; i < 16; i++)
        y1[i] = canon(mulc(x[i], kc.k11, kc.k11q, kc.p[1]) + mulc(y0[i], kc.k10, kc.k10q, kc.p[1]), kc.p[1], kc.pinv[1]);
    }
  }
  const MulDesc d = dv.get(m);
  const uint64_t L = ((uint64_t)d.la + d.lb + 1) / 2;
  uint64_t* out = (uint64_t*)res + d.r_off;
  const uint64_t sb = dv.seg_base(m, d);
  uint64_t* ev = (uint64_t*)(res + stride) + sb;
  const uint32_t run0 = (uint32_t)((d.r_off - sb) >> logCR);
  const uint32_t pos0 = base + ((tid >> logC) << logSig) + j0 + (tid & (C - 1));   // element i: + (RI i) << logSig
  const uint32_t* ad = nullptr;
  uint64_t add_len = 0;
  if constexpr (DEC) {
    const CrtSeg sg = sv.uniform((uint32_t)m);
    ad = add + sg.add_pos;
    add_len = sg.add_len;
  }
  constexpr uint64_t TOP = CR == 64 ? 1ull << 63 : ((~0ull / ((1ull << CR) - 1)) << (CR - 1));
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const uint32_t k = pos0 + ((RI * i) << logSig);
    uint64_t v0, v1;
    uint32_t v2;
    fcrt_join(y0[i], y1[i], x[i], kc, v0, v1, v2);
    if constexpr (DEC) dec_split(add_digit(ad, add_len, k), v0, v1, v2);
    uint64_t t1 = __shfl_up((unsigned long long)v1, 1, 64);
    const uint32_t b2 = __shfl_up(v2, 1, 64);
    uint32_t t2 = __shfl_up(v2, 2, 64), h;
    if (lane < 1) t1 = 0;
    if (lane < 2) t2 = 0;
    const uint64_t lo = fcol_sum<DEC>(v0, t1, t2, &h);
    const uint32_t hp = __shfl_up(h, 1, 64);
    const uint64_t u = lo + (lane ? hp : 0);
    const bool gk = fcol_gen<DEC>(u, lo), pr = fcol_prop<DEC>(u);
    const uint64_t gm = __ballot(gk) & ~TOP, bm = (__ballot(pr) & ~TOP) | gm;
    const uint64_t cm = (gm + bm) ^ gm ^ bm;            // carry into each lane
    uint32_t cy = (uint32_t)((cm >> (tid & 63)) & 1ull);
    const uint64_t dg = fcol_digit<DEC>(u, gk, &cy);
    if (k < L) out[k] = dg;
    if (lane == CR - 1 && k + 1 <= L) {
      // v1 of this digit, v2 of the one below and the carries; v2 above them
      uint32_t eh;
      const uint64_t e0 = fcol_sum<DEC>(v1, b2, (uint64_t)h + cy, &eh);
      const uint64_t at = 2 * (uint64_t)(run0 + ((k + 1) >> logCR));
      ev[at] = e0;
      ev[at + 1] = (uint64_t)v2 + eh;
    }
  }
  if (L > N && base == 0 && j0 == 0 && tid == 0) out[N] = 0;
}

// The digits and run carries of k_fcol_crt, in the role of fcrt_local: u = digit
// + what its run's neighbour left, and binary carries.
template <bool DEC>
__device__ __forceinline__ void fpart_local(uint64_t len, const uint64_t* __restrict__ dg,
                                            const uint64_t* __restrict__ ev, uint32_t logCR, uint64_t kb,
                                            uint32_t* tmp, uint64_t* ul, bool* gk, bool* Gt, bool* Pt, uint32_t* spec) {
  const uint32_t tid = threadIdx.x, CR = 1u << logCR;
  const uint64_t k0 = kb + (uint64_t)tid * FCRT_E;
  auto extra = [&](uint64_t k) -> uint64_t {
    const uint32_t r = (uint32_t)k & (CR - 1);
    return r < 2 && k >= CR && k < len ? ev[2 * (k >> logCR) + r] : 0;
  };
  uint64_t lo[FCRT_E], e[FCRT_E], cl = 0, ce = 0;
#pragma unroll
  for (int i = 0; i < FCRT_E; i++) {
    const uint64_t k = k0 + i;
    lo[i] = k < len ? dg[k] : 0;
    e[i] = extra(k);
  }
  const bool lctx = tid < FCRT_CTX && kb >= FCRT_CTX;
  if (lctx) {
    cl = dg[kb + tid - FCRT_CTX];
    ce = extra(kb + tid - FCRT_CTX);
  }
  if (tid < 64) {
    const uint64_t cu = cl + ce;
    const bool g = fcol_gen<DEC>(cu, cl);
    const uint64_t gm = __ballot(lctx && g);
    const uint64_t dm = gm | __ballot(lctx && !g && !fcol_prop<DEC>(cu));
    if (tid == 0) *spec = dm ? (uint32_t)((gm >> (63 - __builtin_clzll(dm))) & 1ull) : 2u;
  }
  bool G = false, P = true;
#pragma unroll
  for (int i = 0; i < FCRT_E; i++) {
    ul[i] = lo[i] + e[i];
    gk[i] = fcol_gen<DEC>(ul[i], lo[i]);
    const bool pr = fcol_prop<DEC>(ul[i]);
    G = gk[i] || (pr && G);
    P = P && pr;
  }
  *Gt = G;
  *Pt = P;
  uint32_t cout;
  bool ap;
  wave_carry(G, P, 0, &cout, &ap);
  if ((tid & 63) == 0) tmp[tid >> 6] = cout | (ap ? 2u : 0u);
  __syncthreads();
}

struct FWords {
  uint32_t w[2 * FCRT_E];
};

// Block b < nblk covers FCRT_BLOCK digits of one segment (out_pos and len in
// limbs, res_pos in digits); blocks from nblk on copy tail ranges.  The carry
// into a block and the look-back are those of k_crt.  Bound by HBM: 24 B read
// and 8 B written per digit.
// DEC: radix-10^18 digits, plus the segments' addends (limbs relative to `add`).
// PART: the digits and run carries of k_fcol_crt (runs of 2^logCR; the addends are in).
template <bool DEC, bool PART>
__global__ void __launch_bounds__(FCRT_THREADS)
k_fcrt(SegView sv, FCrt kc, uint32_t logCR, const double* __restrict__ res, uint64_t stride, const uint32_t* __restrict__ add,
       uint32_t* __restrict__ out, uint32_t nblk, uint32_t* __restrict__ flags, uint32_t epoch, uint32_t polls, CopyList tails,
       const uint32_t* __restrict__ tin, uint32_t* __restrict__ tout, uint32_t* __restrict__ err) {
  __shared__ uint32_t tmp[FCRT_THREADS / 64], tmp2[FCRT_THREADS / 64];
  __shared__ uint4 xv[FCRT_THREADS + 1];
  __shared__ uint32_t s_state, s_pair, s_spec, s_spec2;
  const uint32_t b = blockIdx.x, tid = threadIdx.x;
  if (b >= nblk) {
    copy_tail_block(tails, tin, tout, b - nblk);
    return;
  }
  CrtSeg sg;
  uint32_t first, end;
  sv.find(b, &sg, &first, &end);
  const uint64_t len = (sg.len + 1) / 2;
  const double* r0 = res + sg.res_pos;
  const double* r1 = r0 + stride;
  const double* r2 = r1 + stride;
  const uint64_t kb = (uint64_t)(b - first) * FCRT_BLOCK;
  const uint32_t* ad = nullptr;
  if constexpr (DEC) {
    if (kb >= len) return;     // a shorter last segment: its end is before these blocks
    end = first + (uint32_t)((len + FCRT_BLOCK - 1) / FCRT_BLOCK);
    ad = add + sg.add_pos;
  }
  uint64_t ul[FCRT_E];
  bool gk[FCRT_E], G, P;
  const uint64_t *dg = (const uint64_t*)r0, *ev = (const uint64_t*)r1;
  if constexpr (PART) fpart_local<DEC>(len, dg, ev, logCR, kb, tmp, ul, gk, &G, &P, &s_spec);
  else fcrt_local<DEC>(len, r0, r1, r2, ad, sg.add_len, kc, kb, xv, tmp, ul, gk, &G, &P, &s_spec);
  const uint32_t own = fcrt_pair(tmp);
  if (tid == 0)
    __hip_atomic_store(flags + b, (epoch << 3) | (own << 1) | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t cin = 0, k = b;
  bool done = (b == first);
  if (!done && s_spec < 2u) {
    cin = s_spec;
    done = true;
  }
  while (!done) {
    k--;
    if (tid == 0) {
      uint32_t f = 0;
      for (uint32_t i = 0; i < polls; i++) {
        f = __hip_atomic_load(flags + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((f & 1u) && (f >> 3) == epoch) break;
        f = 0;
        __builtin_amdgcn_s_sleep(2);
      }
      s_state = f ? 1u : 2u;
      s_pair = (f >> 1) & 3u;
    }
    __syncthreads();
    const uint32_t state = s_state;
    uint32_t pair = s_pair;
    __syncthreads();
    if (state == 2u) {
      // not published yet: recompute block k's pair from its residues
      uint64_t ul2[FCRT_E];
      bool gk2[FCRT_E], G2, P2;
      const uint64_t kb2 = (uint64_t)(k - first) * FCRT_BLOCK;
      if constexpr (PART) fpart_local<DEC>(len, dg, ev, logCR, kb2, tmp2, ul2, gk2, &G2, &P2, &s_spec2);
      else fcrt_local<DEC>(len, r0, r1, r2, ad, sg.add_len, kc, kb2, xv, tmp2, ul2, gk2, &G2, &P2, &s_spec2);
      pair = fcrt_pair(tmp2);
    }
    if (pair & 1u) { cin = 1; done = true; }           // block k generates a carry
    else if (!(pair & 2u)) done = true;                 // block k absorbs any carry-in
    else if (k == first) done = true;                   // all-propagate back to the start
  }
  if (tid == 0 && b + 1 == end && ((own & 1u) | ((own >> 1) & cin))) atomicOr(err, CAT_DEVERR_CARRY_OUT);
  if constexpr (PART) {   // what the last run left above the segment
    const uint64_t q = len >> logCR;
    if (tid == 0 && b + 1 == end && (len & ((1ull << logCR) - 1)) == 0 && q && (ev[2 * q] | ev[2 * q + 1]))
      atomicOr(err, CAT_DEVERR_CARRY_OUT);
  }
  uint32_t wc = cin;
  for (uint32_t w = 0; w < (tid >> 6); w++) {
    const uint32_t x = tmp[w];
    wc = (x & 1u) | ((x >> 1) & wc);
  }
  uint32_t cout;
  bool ap;
  uint32_t c = wave_carry(G, P, wc, &cout, &ap);
  uint32_t* o = out + sg.out_pos;
  const uint64_t w0 = 2 * (kb + (uint64_t)tid * FCRT_E);
  FWords r;
#pragma unroll
  for (int i = 0; i < FCRT_E; i++) {
    const uint64_t y = fcol_digit<DEC>(ul[i], gk[i], &c);
    r.w[2 * i] = (uint32_t)y;
    r.w[2 * i + 1] = (uint32_t)(y >> 32);
  }
  if (2 * (kb + FCRT_BLOCK) <= sg.len) {
    *(FWords*)(o + w0) = r;
  } else {
    bool over = false;
#pragma unroll
    for (int i = 0; i < 2 * FCRT_E; i++) {
      if (w0 + i < sg.len) o[w0 + i] = r.w[i];
      else over = over || r.w[i] != 0;
    }
    if (over) atomicOr(err, CAT_DEVERR_CARRY_OUT);     // a limb past la + lb
  }
}

// ---------------------------------------------------------------------------
// Products of up to 2^11 digits with the three primes and the carries in one
// workgroup: T / 8 threads of 8 values per prime, then T / 4 threads of 4 digits
// recombine and carry, so that the residues never leave LDS and a tree level is
// one launch.  The tile is one product, or 2^9 slots of shorter ones: the
// smallest that gives every prime whole waves, because a level of few products
// is bound by how much of it one CU has to issue (tiles of 2^11 slots held three
// waves per SIMD on one CU while the others stood idle).
// Every product has la + lb <= 2 N limbs, so nothing is carried out of its N
// slots and one scan over the tile serves all its products.
#define FF_MAX_LOGD FNTT_FUSED_MAX_LOGD
constexpr int ff_tile(int logD) { return logD < 9 ? 9 : logD; }
constexpr int ff_threads(int logD) { return CAT_NPRIMES << (ff_tile(logD) - 3); }
#define FF_E 4
// DEC: the carries in radix 10^18, with the addends and lengths of the segments sg.
template <int LOGD, bool ZHI, int LOGT = ff_tile(LOGD), bool DEC = false>
__device__ __forceinline__ void ffused_tile(double* lds, MulDesc* ds, CrtSeg* sg, uint4* xw, uint32_t* tmp,
                                            const uint32_t* __restrict__ ain, const uint32_t* __restrict__ bin,
                                            uint32_t* __restrict__ out, const FTables& tb, const FCrt& kc,
                                            uint32_t* __restrict__ err) {
  constexpr int LE = 3, LR = fpass<LE>(LOGD), LOGSR = LOGD - LR;
  constexpr uint32_t T = 1u << LOGT, NT = T >> LE, N = 1u << LOGD, SR = 1u << LOGSR, TP = fpad<LE>(T);
  constexpr int R = 1 << LR, E = 1 << LE, D = E / R;
  const uint32_t prime = __builtin_amdgcn_readfirstlane(threadIdx.x / NT), tid = threadIdx.x % NT;
  const FPrime& c = c_fp[0][prime];
  double* l = lds + prime * TP;
  const double* tws = tb.tws3 + (size_t)prime * FTWS_ENTRIES;
  const double* itws = tb.itws3 + (size_t)prime * FTWS_ENTRIES;
  double a[E], b[E];
  constexpr int RK = ZHI ? R / 2 : R, NR = ZHI ? E / 2 : E;
  uint2 ra[NR], rb[NR];
#pragma unroll
  for (int d = 0; d < D; d++) {
    const uint32_t g = tid + NT * d, j = g & (SR - 1);
    const MulDesc& m = ds[g >> LOGSR];
    const uint32_t la = m.la, lb = m.lb;
    const uint32_t *sa = ain + m.a_off, *sb = bin + m.b_off;
#pragma unroll
    for (int k = 0; k < RK; k++) {
      const uint32_t q = 2 * (j + SR * k);
      const uint32_t x0 = sa[q < la ? q : 0], x1 = sa[q + 1 < la ? q + 1 : 0];
      const uint32_t y0 = sb[q < lb ? q : 0], y1 = sb[q + 1 < lb ? q + 1 : 0];
      ra[d + D * k] = make_uint2(q < la ? x0 : 0u, q + 1 < la ? x1 : 0u);
      rb[d + D * k] = make_uint2(q < lb ? y0 : 0u, q + 1 < lb ? y1 : 0u);
    }
  }
#pragma unroll
  for (int i = 0; i < NR; i++) a[i] = digit(ra[i].x, ra[i].y, c.p, c.pinv);
  vec_fwd<LE, LOGD, 0, ZHI>(l, a, a, NT, tws, c, tid);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NR; i++) b[i] = digit(rb[i].x, rb[i].y, c.p, c.pinv);
  vec_fwd<LE, LOGD, 0, ZHI>(l, b, b, NT, tws, c, tid);
  vec_mul_inv<LE, LOGD, 0>(l, a, b, NT, itws, c, tid);
  // the residues in order, in the slots that this thread read last
#pragma unroll
  for (int d = 0; d < D; d++) {
    const uint32_t g = tid + NT * d, j = g & (SR - 1);
    const uint32_t s = fpad<LE>(((g >> LOGSR) << LOGD) + j);
#pragma unroll
    for (int k = 0; k < R; k++) l[s + k * (SR + (SR >> LE))] = a[d + D * k];
  }
  __syncthreads();
  // recombination and carries: thread t < T / 4 has the slots 4 t .. 4 t + 3
  const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const bool on = t < T / FF_E;
  const uint32_t k0 = (FF_E * t) & (N - 1);
  uint64_t a0[FF_E], a1[FF_E], lo[FF_E], ul[FF_E];
  uint32_t a2[FF_E], h[FF_E];
  bool gk[FF_E], G = false, P = false;
  if (on) {
    const uint32_t s = fpad<LE>(FF_E * t);
#pragma unroll
    for (int i = 0; i < FF_E; i++) {
      uint64_t ad = 0;
      if constexpr (DEC) {
        const CrtSeg& q = sg[(FF_E * t) >> LOGD];
        ad = add_digit(ain + q.add_pos, q.add_len, k0 + i);
      }
      fcol_value<DEC>(lds[s + i], lds[TP + s + i], lds[2 * TP + s + i], kc, ad, a0[i], a1[i], a2[i]);
    }
#pragma unroll
    for (int i = 2; i < FF_E; i++) lo[i] = fcol_sum<DEC>(a0[i], a1[i - 1], a2[i - 2], &h[i]);
    // the left neighbour's last two columns (none at a product's start)
    const uint32_t p0 = (uint32_t)a1[FF_E - 1], p1 = (uint32_t)(a1[FF_E - 1] >> 32),
                   p2 = a2[FF_E - 1] | (h[FF_E - 1] << 30), p3 = a2[FF_E - 2];
    uint4 z = make_uint4(__shfl_up(p0, 1, 64), __shfl_up(p1, 1, 64), __shfl_up(p2, 1, 64), __shfl_up(p3, 1, 64));
    if (lane == 63) xw[wave] = make_uint4(p0, p1, p2, p3);
    ul[0] = ((uint64_t)z.y << 32) | z.x;   // kept across the barrier
    ul[1] = ((uint64_t)z.w << 32) | z.z;
  }
  __syncthreads();
  if (on) {
    uint4 z = make_uint4((uint32_t)ul[0], (uint32_t)(ul[0] >> 32), (uint32_t)ul[1], (uint32_t)(ul[1] >> 32));
    if (lane == 0 && wave > 0) z = xw[wave - 1];
    if (k0 == 0) z = make_uint4(0, 0, 0, 0);
    lo[0] = fcol_sum<DEC>(a0[0], ((uint64_t)z.y << 32) | z.x, z.w, &h[0]);
    lo[1] = fcol_sum<DEC>(a0[1], a1[0], z.z & 0x3FFFFFFFu, &h[1]);
    P = true;
    uint32_t hp = z.z >> 30;
#pragma unroll
    for (int i = 0; i < FF_E; i++) {
      ul[i] = lo[i] + hp;
      gk[i] = fcol_gen<DEC>(ul[i], lo[i]);
      hp = h[i];
      const bool pr = fcol_prop<DEC>(ul[i]);
      G = gk[i] || (pr && G);
      P = P && pr;
    }
    uint32_t cout;
    bool ap;
    wave_carry(G, P, 0, &cout, &ap);
    if (lane == 0) tmp[wave] = cout | (ap ? 2u : 0u);
  }
  __syncthreads();
  if (!on) return;
  uint32_t wc = 0;
  for (uint32_t w = 0; w < wave; w++) {
    const uint32_t x = tmp[w];
    wc = (x & 1u) | ((x >> 1) & wc);
  }
  uint32_t cout;
  bool ap;
  uint32_t cy = wave_carry(G, P, wc, &cout, &ap);
  const MulDesc& m = ds[(FF_E * t) >> LOGD];
  uint32_t L = m.la + m.lb;
  uint64_t cpos = m.c_off;
  if constexpr (DEC) {
    const CrtSeg& q = sg[(FF_E * t) >> LOGD];
    L = (uint32_t)q.len;
    cpos = q.out_pos;
  }
  const uint32_t w0 = 2 * k0;
  struct W8 {
    uint32_t w[2 * FF_E];
  } r;
#pragma unroll
  for (int i = 0; i < FF_E; i++) {
    const uint64_t y = fcol_digit<DEC>(ul[i], gk[i], &cy);
    r.w[2 * i] = (uint32_t)y;
    r.w[2 * i + 1] = (uint32_t)(y >> 32);
  }
  uint32_t* o = out + cpos + w0;
  if (w0 + 2 * FF_E <= L) {
    *(W8*)o = r;
  } else {
    bool over = false;
#pragma unroll
    for (int i = 0; i < 2 * FF_E; i++) {
      if (w0 + i < L) o[i] = r.w[i];
      else over = over || r.w[i] != 0;
    }
    if (over) atomicOr(err, CAT_DEVERR_CARRY_OUT);
  }
}

// One bucket of products of `dv`; workgroups from `tiles`
// on copy tail ranges.
template <int LOGD, bool ZHI>
__global__ void __launch_bounds__(ff_threads(LOGD)) __attribute__((amdgpu_waves_per_eu(6)))
k_ffused(DescView dv, uint64_t m0, uint64_t nmul, uint32_t tiles, const uint32_t* __restrict__ ain,
         const uint32_t* __restrict__ bin, uint32_t* __restrict__ out, FTables tb, FCrt kc, CopyList tails,
         const uint32_t* __restrict__ tin, uint32_t* __restrict__ tout, uint32_t* __restrict__ err) {
  constexpr uint32_t PER = 1u << (ff_tile(LOGD) - LOGD);
  __shared__ double lds[CAT_NPRIMES * fpad<3>(1u << ff_tile(LOGD))];
  __shared__ MulDesc ds[PER];
  __shared__ uint4 xw[8];
  __shared__ uint32_t tmp[8];
  if (blockIdx.x >= tiles) {
    copy_tail_block(tails, tin, tout, blockIdx.x - tiles);
    return;
  }
  const uint64_t i0 = (uint64_t)blockIdx.x * PER;
  if (threadIdx.x < PER) ds[threadIdx.x] = dv.slot(m0 + i0 + threadIdx.x, m0 + i0, m0 + nmul);
  __syncthreads();
  ffused_tile<LOGD, ZHI>(lds, ds, nullptr, xw, tmp, ain, bin, out, tb, kc, err);
}

// A level of decimal joins (operands of at most N/2 digits): product i has the
// segment i of sv, addends relative to `ain`.
template <int LOGD>
__global__ void __launch_bounds__(ff_threads(LOGD)) __attribute__((amdgpu_waves_per_eu(6)))
k_ffused10(DescView dv, SegView sv, uint64_t nmul, uint32_t tiles, const uint32_t* __restrict__ ain,
           const uint32_t* __restrict__ bin, uint32_t* __restrict__ out, FTables tb, FCrt kc, CopyList tails,
           const uint32_t* __restrict__ tin, uint32_t* __restrict__ tout, uint32_t* __restrict__ err) {
  constexpr uint32_t PER = 1u << (ff_tile(LOGD) - LOGD);
  __shared__ double lds[CAT_NPRIMES * fpad<3>(1u << ff_tile(LOGD))];
  __shared__ MulDesc ds[PER];
  __shared__ CrtSeg sg[PER];
  __shared__ uint4 xw[8];
  __shared__ uint32_t tmp[8];
  if (blockIdx.x >= tiles) {
    copy_tail_block(tails, tin, tout, blockIdx.x - tiles);
    return;
  }
  const uint64_t i0 = (uint64_t)blockIdx.x * PER;
  if (threadIdx.x < PER) {
    CrtSeg q{};
    if (i0 + threadIdx.x < nmul) q = sv.uniform((uint32_t)i0 + threadIdx.x);
    ds[threadIdx.x] = dv.slot(i0 + threadIdx.x, i0, nmul);
    sg[threadIdx.x] = q;
  }
  __syncthreads();
  ffused_tile<LOGD, true, ff_tile(LOGD), true>(lds, ds, sg, xw, tmp, ain, bin, out, tb, kc, err);
}

// Several short buckets of a generic batch in one launch: workgroup b takes the
// products tiles[b].x .. of `desc`, all of one bucket (tiles[b].y: log2 of the
// transform in limbs, products << 8), in a tile of 2^11 slots.  Against a launch
// per bucket: the 4,096-product batch 2.203 -> 2.164 ms.
__constant__ FCrt c_fcrt[FF_MAX_LOGD + 1];
__global__ void __launch_bounds__(ff_threads(FF_MAX_LOGD)) __attribute__((amdgpu_waves_per_eu(6)))
k_ffused_mix(const MulDesc* __restrict__ desc, const uint2* __restrict__ tiles, const uint32_t* __restrict__ ain,
             const uint32_t* __restrict__ bin, uint32_t* __restrict__ out, FTables tb, uint32_t* __restrict__ err) {
  __shared__ double lds[CAT_NPRIMES * fpad<3>(1u << FF_MAX_LOGD)];
  __shared__ MulDesc ds[1u << (FF_MAX_LOGD - FNTT_LDS_MIN_LOGD)];
  __shared__ uint4 xw[8];
  __shared__ uint32_t tmp[8];
  const uint2 tl = tiles[blockIdx.x];
  const int logD = (int)(tl.y & 255u) - 1;
  const uint32_t cnt = tl.y >> 8;
  if (threadIdx.x < (1u << (FF_MAX_LOGD - logD))) {
    MulDesc d = desc[tl.x + (threadIdx.x < cnt ? threadIdx.x : 0)];
    if (threadIdx.x >= cnt) d.la = d.lb = 0;   // as DescView::slot
    ds[threadIdx.x] = d;
  }
  __syncthreads();
#define T(X)                                                                                   \
  case X:                                                                                      \
    ffused_tile<X, false, FF_MAX_LOGD>(lds, ds, nullptr, xw, tmp, ain, bin, out, tb, c_fcrt[X], err);   \
    break
  switch (logD) {
    T(5); T(6); T(7); T(8); T(9); T(10); T(11);
    default: break;
  }
#undef T
}

// ------------------------------------------------------------------ host side
static const uint64_t kPF[2][CAT_NPRIMES] = {{1125900443713537ull, 1125905745313793ull, 1125906550620161ull},
                                             {2251800350556161ull, 2251801155862529ull, 2251803907325953ull}};
static const uint64_t kGF[2][CAT_NPRIMES] = {{5, 3, 6}, {6, 3, 5}};   // primitive roots

uint64_t mulmod64(uint64_t a, uint64_t b, uint64_t p) { return (uint64_t)((unsigned __int128)a * b % p); }
uint64_t powmod64(uint64_t b, uint64_t e, uint64_t p) {
  uint64_t r = 1;
  for (; e; e >>= 1) {
    if (e & 1) r = mulmod64(r, b, p);
    b = mulmod64(b, b, p);
  }
  return r;
}
uint64_t invmod64(uint64_t a, uint64_t p) { return powmod64(a % p, p - 2, p); }
double balanced(uint64_t x, uint64_t p) { return x > p / 2 ? -(double)(p - x) : (double)x; }

void fill_powers(uint64_t w, uint64_t p, size_t n, double* out) {
  uint64_t x = 1;
  for (size_t i = 0; i < n; i++) {
    out[i] = balanced(x, p);
    x = mulmod64(x, w, p);
  }
}

FCrt g_crt[FNTT_MAX_LOGD + 1];

FCrt make_crt(int logD) {
  const uint64_t* P = kPF[fntt_set(logD)];
  FCrt k{};
  for (int i = 0; i < 3; i++) {
    k.p[i] = (double)P[i];
    k.pinv[i] = 1.0 / (double)P[i];
  }
  k.pi[0] = P[0];
  k.pi[1] = P[1];
  auto put = [&](uint64_t v, int i, double* c, double* q) {
    *c = balanced(v % P[i], P[i]);
    *q = *c / (double)P[i];
  };
  uint64_t s[3];
  for (int i = 0; i < 3; i++) s[i] = invmod64(1ull << logD, P[i]);
  const uint64_t c01 = invmod64(P[0] % P[1], P[1]);
  const uint64_t c12 = invmod64(P[1] % P[2], P[2]);
  const uint64_t c012 = mulmod64(invmod64(P[0] % P[2], P[2]), c12, P[2]);
  put(s[0], 0, &k.k00, &k.k00q);
  put(mulmod64(s[1], c01, P[1]), 1, &k.k11, &k.k11q);
  put(P[1] - c01, 1, &k.k10, &k.k10q);
  put(mulmod64(s[2], c012, P[2]), 2, &k.k22, &k.k22q);
  put(P[2] - c012, 2, &k.k20, &k.k20q);
  put(P[2] - c12, 2, &k.k21, &k.k21q);
  return k;
}

#define FCHK(x)                        \
  do {                                 \
    const hipError_t e_ = (x);         \
    if (e_ != hipSuccess) return e_;   \
  } while (0)

hipError_t upload(const std::vector<double>& h, const double** d) {
  void* q = nullptr;
  FCHK(hipMalloc(&q, h.size() * sizeof(double)));
  FCHK(hipMemcpy(q, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice));
  *d = (const double*)q;
  return hipSuccess;
}

}  // namespace

hipError_t fntt_init() {
  FPrime fp[2][CAT_NPRIMES];
  for (int s = 0; s < 2; s++) {
    std::vector<double> tws[2], tws3[2], lo[2], hi[2];
    for (int d = 0; d < 2; d++) {
      tws3[d].assign((size_t)CAT_NPRIMES * FTWS_ENTRIES, 1.0);
      tws[d].assign((size_t)CAT_NPRIMES * FTWS_ENTRIES, 1.0);
      lo[d].resize((size_t)CAT_NPRIMES * FTW2);
      hi[d].resize((size_t)CAT_NPRIMES * FTW2);
    }
    for (int i = 0; i < CAT_NPRIMES; i++) {
      const uint64_t p = kPF[s][i];
      const uint64_t w = powmod64(kGF[s][i], (p - 1) >> FNTT_MAX_LOGD, p);
      if (powmod64(w, 1ull << (FNTT_MAX_LOGD - 1), p) != p - 1) return hipErrorUnknown;
      FPrime& c = fp[s][i];
      c.p = (double)p;
      c.pinv = 1.0 / (double)p;
      for (int d = 0; d < 2; d++) {
        const uint64_t r = d ? invmod64(w, p) : w;
        double* cw = d ? c.iw : c.w;
        double* cq = d ? c.iwp : c.wp;
        fill_powers(powmod64(r, 1ull << (FNTT_MAX_LOGD - 4), p), p, 8, cw);
        for (int k = 0; k < 8; k++) cq[k] = cw[k] / c.p;
        // pass tables: omega_S^(j k) over j < S / R, k < R, R the pass's radix
        std::vector<double> pw(1u << 14);
        for (int ls = 1; ls <= 14; ls++) {
          const uint32_t S = 1u << ls;
          fill_powers(powmod64(r, 1ull << (FNTT_MAX_LOGD - ls), p), p, S, pw.data());
          for (int le = 3; le <= 4; le++) {
            const int lr = le == 3 ? fpass<3>(ls) : fpass<4>(ls), lsr = ls - lr;
            double* t = &(le == 3 ? tws3 : tws)[d][(size_t)i * FTWS_ENTRIES + S - 2];
            for (uint32_t k = 0; k < (1u << lr); k++)
              for (uint32_t j = 0; j < (1u << lsr); j++) t[(k << lsr) + j] = pw[(uint64_t)j * k % S];
          }
        }
        fill_powers(r, p, FTW2, &lo[d][(size_t)i * FTW2]);
        fill_powers(powmod64(r, FTW2, p), p, FTW2, &hi[d][(size_t)i * FTW2]);
      }
    }
    FTables& t = g_ft[s];
    FCHK(upload(tws3[0], &t.tws3));
    FCHK(upload(tws3[1], &t.itws3));
    FCHK(upload(tws[0], &t.tws));
    FCHK(upload(tws[1], &t.itws));
    FCHK(upload(lo[0], &t.lo));
    FCHK(upload(lo[1], &t.ilo));
    FCHK(upload(hi[0], &t.hi));
    FCHK(upload(hi[1], &t.ihi));
  }
  for (int l = 0; l <= FNTT_MAX_LOGD; l++) g_crt[l] = make_crt(l);
  FCHK(hipMemcpyToSymbol(HIP_SYMBOL(c_fcrt), g_crt, sizeof(FCrt) * (FF_MAX_LOGD + 1)));
  return hipMemcpyToSymbol(HIP_SYMBOL(c_fp), fp, sizeof(fp));
}

hipError_t fntt_lds(const FBatch& b, hipStream_t st) {
  const int lt = b.logD < 12 ? 12 : b.logD;
  const uint64_t per = 1ull << (lt - b.logD);
  const uint64_t tiles = (b.cnt + per - 1) / per;
  const dim3 grid((uint32_t)(tiles * CAT_NPRIMES)), block((1u << lt) >> flds_le(b.logD));
#define L(X)                                                                                                  \
  case X:                                                                                                     \
    if (b.half)                                                                                               \
      hipLaunchKernelGGL((k_flds<X, true>), grid, block, 0, st, b.dv, b.m0, b.cnt, b.ain, b.bin, b.res,       \
                         b.stride, g_ft[0]);                                                                  \
    else                                                                                                      \
      hipLaunchKernelGGL((k_flds<X, false>), grid, block, 0, st, b.dv, b.m0, b.cnt, b.ain, b.bin, b.res,      \
                         b.stride, g_ft[0]);                                                                  \
    break
  switch (b.logD) {
    L(5); L(6); L(7); L(8); L(9); L(10); L(11); L(12); L(13); L(14);
    default: return hipErrorInvalidValue;
  }
#undef L
  return hipGetLastError();
}

bool fntt_fused_fits(int logD) { return logD >= FNTT_LDS_MIN_LOGD && logD <= FF_MAX_LOGD; }
hipError_t fntt_fused(const FBatch& b, uint32_t* out, const CopyList& tails, const uint32_t* tin, uint32_t* tout,
                      uint32_t* err, hipStream_t st) {
  const uint64_t per = 1ull << (ff_tile(b.logD) - b.logD);
  const uint32_t tiles = (uint32_t)((b.cnt + per - 1) / per);
  const dim3 grid(tiles + tail_blocks(tails)), block(ff_threads(b.logD));
#define L(X)                                                                                                  \
  case X:                                                                                                     \
    if (b.half)                                                                                               \
      hipLaunchKernelGGL((k_ffused<X, true>), grid, block, 0, st, b.dv, b.m0, b.cnt, tiles, b.ain, b.bin,     \
                         out, g_ft[0], g_crt[X], tails, tin, tout, err);                                      \
    else                                                                                                      \
      hipLaunchKernelGGL((k_ffused<X, false>), grid, block, 0, st, b.dv, b.m0, b.cnt, tiles, b.ain, b.bin,    \
                         out, g_ft[0], g_crt[X], tails, tin, tout, err);                                      \
    break
  switch (b.logD) {
    L(5); L(6); L(7); L(8); L(9); L(10); L(11);
    default: return hipErrorInvalidValue;
  }
#undef L
  return hipGetLastError();
}

hipError_t fntt_fused10(const FBatch& b, const SegView& sv, uint32_t* out, const CopyList& tails, const uint32_t* tin,
                        uint32_t* tout, uint32_t* err, hipStream_t st) {
  const uint64_t per = 1ull << (ff_tile(b.logD) - b.logD);
  const uint32_t tiles = (uint32_t)((b.cnt + per - 1) / per);
  const dim3 grid(tiles + tail_blocks(tails)), block(ff_threads(b.logD));
#define L(X)                                                                                                    \
  case X:                                                                                                       \
    hipLaunchKernelGGL((k_ffused10<X>), grid, block, 0, st, b.dv, sv, b.cnt, tiles, b.ain, b.bin, out, g_ft[0], \
                       g_crt[X], tails, tin, tout, err);                                                        \
    break
  switch (b.logD) {
    L(5); L(6); L(7); L(8); L(9); L(10); L(11);
    default: return hipErrorInvalidValue;
  }
#undef L
  return hipGetLastError();
}

hipError_t fntt_fused_mix(const MulDesc* desc, const uint2* tiles, uint32_t ntiles, const uint32_t* ain,
                          const uint32_t* bin, uint32_t* out, uint32_t* err, hipStream_t st) {
  hipLaunchKernelGGL(k_ffused_mix, dim3(ntiles), dim3(ff_threads(FF_MAX_LOGD)), 0, st, desc, tiles, ain, bin, out,
                     g_ft[0], err);
  return hipGetLastError();
}

// The launches below instantiate what fp_passes asks for.
template <int LOGL, int PS>
static hipError_t col_fwd_launch(const FBatch& b, int logS, bool first, int prevS, int prevL, hipStream_t st) {
  constexpr int LOGT = LOGL <= 8 ? 12 : 13;
  const FGeom fg{b.logD, logS, LOGT - LOGL};
  const dim3 grid((uint32_t)((b.cnt << (b.logD - LOGT)) * CAT_NPRIMES), 1, 2), block((1u << LOGT) / 16);
  if constexpr (fcol_used(PS, LOGL, true)) {
    if (first) {
      hipLaunchKernelGGL((k_fcol_fwd<LOGL, PS, true>), grid, block, 0, st, b.dv, fg, b.m0, prevS, prevL, b.ain, b.bin,
                         b.F, g_ft[PS]);
      return hipGetLastError();
    }
  }
  if constexpr (fcol_used(PS, LOGL, false)) {
    if (!first) {
      hipLaunchKernelGGL((k_fcol_fwd<LOGL, PS, false>), grid, block, 0, st, b.dv, fg, b.m0, prevS, prevL, b.ain, b.bin,
                         b.F, g_ft[PS]);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}
template <int LOGL, int PS>
static hipError_t col_inv_launch(const FBatch& b, int logS, bool first, int prevS, int prevL, hipStream_t st) {
  constexpr int LOGT = LOGL <= 8 ? 12 : 13;
  const FGeom fg{b.logD, logS, LOGT - LOGL};
  const dim3 grid((uint32_t)(b.cnt << (b.logD - LOGT)), CAT_NPRIMES), block((1u << LOGT) / 16);
  if constexpr (fcol_residues_used(PS, LOGL)) {
    if (first) {
      hipLaunchKernelGGL((k_fcol_inv<LOGL, PS, true>), grid, block, 0, st, b.dv, fg, b.m0, prevS, prevL, b.F, b.res,
                         b.stride, g_ft[PS]);
      return hipGetLastError();
    }
  }
  if constexpr (fcol_used(PS, LOGL, false)) {
    if (!first) {
      hipLaunchKernelGGL((k_fcol_inv<LOGL, PS, false>), grid, block, 0, st, b.dv, fg, b.m0, prevS, prevL, b.F, b.res,
                         b.stride, g_ft[PS]);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}
#define COL_SWITCH(FN)                                                                                          \
  switch (logL) {                                                                                               \
    COL_CASE(FN, 4);                                                                                            \
    COL_CASE(FN, 5);                                                                                            \
    COL_CASE(FN, 6);                                                                                            \
    COL_CASE(FN, 7);                                                                                            \
    COL_CASE(FN, 8);                                                                                            \
    COL_CASE(FN, 9);                                                                                            \
    COL_CASE(FN, 10);                                                                                           \
    default: return hipErrorInvalidValue;                                                                       \
  }
#define COL_CASE(FN, X)                                                                                         \
  case X:                                                                                                       \
    return fntt_set(b.logD) == 0 ? FN<X, 0>(b, logS, first, prevS, prevL, st)                                   \
                                 : FN<X, 1>(b, logS, first, prevS, prevL, st)

hipError_t fntt_col_fwd(const FBatch& b, int logS, int logL, bool first, int prevS, int prevL, hipStream_t st) {
  COL_SWITCH(col_fwd_launch);
}
hipError_t fntt_col_inv(const FBatch& b, int logS, int logL, bool first, int prevS, int prevL, hipStream_t st) {
  COL_SWITCH(col_inv_launch);
}

template <int LOGM, int PS>
static hipError_t row_launch(const FBatch& b, int logS, int logL, hipStream_t st) {
  if constexpr (frow_used(PS, LOGM)) {
    const dim3 grid((uint32_t)(b.cnt << (b.logD - LOGM)), CAT_NPRIMES), block((1u << LOGM) / 16);
    hipLaunchKernelGGL((k_frow<LOGM, PS>), grid, block, 0, st, b.logD, logS, logL, b.dv.uni, b.F, g_ft[PS]);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}
hipError_t fntt_row(const FBatch& b, int logM, int logS, int logL, hipStream_t st) {
  const bool set1 = fntt_set(b.logD) != 0;
  switch (logM) {
    case 11: return set1 ? row_launch<11, 1>(b, logS, logL, st) : row_launch<11, 0>(b, logS, logL, st);
    case 12: return set1 ? row_launch<12, 1>(b, logS, logL, st) : row_launch<12, 0>(b, logS, logL, st);
    default: return hipErrorInvalidValue;
  }
}

template <int LOGL, int PS>
static hipError_t col_crt_launch(const FBatch& b, int logS, const SegView& sv, const uint32_t* add, hipStream_t st) {
  if constexpr (fcol_used(PS, LOGL, true)) {
    constexpr int LOGT = 12;
    const FGeom fg{b.logD, logS, LOGT - LOGL};
    const dim3 grid((uint32_t)(b.cnt << (b.logD - LOGT))), block((1u << LOGT) / 16);
    if (add)
      hipLaunchKernelGGL((k_fcol_crt<LOGL, PS, true>), grid, block, 0, st, b.dv, sv, fg, g_crt[b.logD], b.F, b.res,
                         b.stride, add, g_ft[PS]);
    else
      hipLaunchKernelGGL((k_fcol_crt<LOGL, PS, false>), grid, block, 0, st, b.dv, sv, fg, g_crt[b.logD], b.F, b.res,
                         b.stride, add, g_ft[PS]);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}
hipError_t fntt_col_crt(const FBatch& b, int logL, const SegView& sv, const uint32_t* add, hipStream_t st) {
#define L(X)                                                                                                   \
  case X: return fntt_set(b.logD) == 0 ? col_crt_launch<X, 0>(b, b.logD, sv, add, st)                          \
                                       : col_crt_launch<X, 1>(b, b.logD, sv, add, st)
  switch (logL) {
    L(4); L(5); L(6); L(7);
    default: return hipErrorInvalidValue;
  }
#undef L
}

hipError_t fntt_crt(const SegView& sv, int logD, int logCR, const double* res, uint64_t stride, const uint32_t* add,
                    uint32_t* out, uint32_t nblk, uint32_t* flags, uint32_t epoch, uint32_t polls,
                    const CopyList& tails, const uint32_t* tin, uint32_t* tout, uint32_t* err, hipStream_t st) {
  const dim3 grid(nblk + tail_blocks(tails)), block(FCRT_THREADS);
#define L(D, P)                                                                                                       \
  hipLaunchKernelGGL((k_fcrt<D, P>), grid, block, 0, st, sv, g_crt[logD], (uint32_t)logCR, res, stride, add, out,     \
                     nblk, flags, epoch, polls, tails, tin, tout, err)
  if (add) {
    if (logCR) L(true, true);
    else L(true, false);
  } else {
    if (logCR) L(false, true);
    else L(false, false);
  }
#undef L
  return hipGetLastError();
}
