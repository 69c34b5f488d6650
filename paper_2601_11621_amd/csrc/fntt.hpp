// Host interface of the floating-point transform kernels (fntt.hip).
#pragma once
#include "common.hpp"

#include <algorithm>

#define FNTT_MAX_LOGD 26       // longest transform (64-bit digits): products of up to 2^27 limbs
#define FNTT_SMALL_MAX_LOGD 23 // longest transform of prime set 0 (primes just above 2^50)
#define FNTT_LDS_MIN_LOGD 5    // one-workgroup transforms
#define FNTT_LDS_MAX_LOGD 14
#define FNTT_FUSED_MAX_LOGD 11 // with recombination and carries in the same workgroup
#define FNTT_ROW_MAX 12        // four-step rows (2^11 and 2^12 digits)
#define FNTT_COL_MIN 4         // column DFTs
#define FNTT_COL_MAX 10
#define FCRT_E 3               // digits per thread of the carry kernel
#define FCRT_THREADS 256
#define FCRT_BLOCK (FCRT_E * FCRT_THREADS)

// prime set of a transform of 2^logD digits
constexpr int fntt_set(int logD) { return logD <= FNTT_SMALL_MAX_LOGD ? 0 : 1; }

// Four-step schedule.  Rows of 2^12 digits (2^11 under the shortest column DFT)
// and as few column passes as fit, at every size: with rows of 2^11 / 2^13 C(10^8)
// takes 2.51 / 2.78 ms instead of 2.41, 5 10^6 x 3 10^6 limbs 0.357 / 0.363
// instead of 0.300; 2^13 at any one size lost up to 3 %, 2^11 won nothing beyond
// noise.
struct FpPasses {
  int P = 0, logM = 0, logL[4] = {}, logS[4] = {};
};
constexpr FpPasses fp_passes(int logD) {
  FpPasses f;
  f.logM = std::min(FNTT_ROW_MAX, logD - FNTT_COL_MIN);
  const int rest = logD - f.logM;
  f.P = (rest + FNTT_COL_MAX - 1) / FNTT_COL_MAX;
  for (int k = 0, ls = logD; k < f.P; k++) {
    f.logL[k] = rest / f.P + (k < rest % f.P ? 1 : 0);
    f.logS[k] = ls;
    ls -= f.logL[k];
  }
  return f;
}
// Which kernels that schedule launches (fntt.hip instantiates no others): column
// passes of 2^logL as a transform's outermost pass or as a later one, rows of
// 2^logM, the outermost inverse pass with residues (not always replaced by
// fntt_col_crt).
#define FP_RUN_MIN_LOG 22      // fntt_col_crt: from 2^22 digits a batch
#define FNTT_RUN_MAX_LOGL 7    // and with columns of at most 2^7 (see fp_run_log)
constexpr bool fcol_used(int set, int logL, bool outer) {
  for (int d = FNTT_LDS_MAX_LOGD + 1; d <= FNTT_MAX_LOGD; d++) {
    const FpPasses f = fp_passes(d);
    for (int k = 0; k < f.P; k++)
      if (fntt_set(d) == set && (k == 0) == outer && f.logL[k] == logL) return true;
  }
  return false;
}
constexpr bool fcol_residues_used(int set, int logL) {
  for (int d = FNTT_LDS_MAX_LOGD + 1; d <= FNTT_MAX_LOGD; d++)
    if (fntt_set(d) == set && fp_passes(d).logL[0] == logL && (d < FP_RUN_MIN_LOG || logL > FNTT_RUN_MAX_LOGL))
      return true;
  return false;
}
constexpr bool frow_used(int set, int logM) {
  for (int d = FNTT_LDS_MAX_LOGD + 1; d <= FNTT_MAX_LOGD; d++)
    if (fntt_set(d) == set && fp_passes(d).logM == logM) return true;
  return false;
}

// Constants and twiddle tables (on the current device); once per process.
hipError_t fntt_init();

// One transform batch: products m0 .. m0 + cnt of `dv`, 2^logD digits each.
// Residues (unreduced, times 2^logD) go to res[prime * stride + r_off + k].
struct FBatch {
  DescView dv;
  uint64_t m0, cnt;
  int logD;
  bool half;             // no operand is longer than 2^(logD - 1) digits
  const uint32_t* ain;
  const uint32_t* bin;
  double* F;             // four-step scratch: 6 * cnt * 2^logD doubles
  double* res;
  uint64_t stride;       // doubles between the residues of two primes
};

hipError_t fntt_lds(const FBatch& b, hipStream_t st);
// Products with carries in one launch (la + lb <= 2^(logD + 1) limbs each; the
// limbs go to out + c_off), with tail copies; for the sizes that fit.
bool fntt_fused_fits(int logD);
hipError_t fntt_fused(const FBatch& b, uint32_t* out, const CopyList& tails, const uint32_t* tin, uint32_t* tout,
                      uint32_t* err, hipStream_t st);
// One level of decimal joins (uniform batch, segment i of sv for product i,
// addends relative to b.ain), for the same sizes.
hipError_t fntt_fused10(const FBatch& b, const SegView& sv, uint32_t* out, const CopyList& tails, const uint32_t* tin,
                        uint32_t* tout, uint32_t* err, hipStream_t st);
// The same for several buckets over device tables: tile b is the products
// tiles[b].x .. (tiles[b].y: logD + 1, products << 8; 2^11 slots at most).
hipError_t fntt_fused_mix(const MulDesc* desc, const uint2* tiles, uint32_t ntiles, const uint32_t* ain,
                          const uint32_t* bin, uint32_t* out, uint32_t* err, hipStream_t st);
// column pass over sub-problems of 2^logS digits, L = 2^logL of them along the
// column; outer (prevS, prevL): the pass before it, whose twiddles this pass
// applies (0: none).  first: the operands come from limbs, the results go to
// the residues.
hipError_t fntt_col_fwd(const FBatch& b, int logS, int logL, bool first, int prevS, int prevL, hipStream_t st);
hipError_t fntt_col_inv(const FBatch& b, int logS, int logL, bool first, int prevS, int prevL, hipStream_t st);
// rows of 2^logM digits under a column pass of sub-problems 2^logS, length 2^logL
hipError_t fntt_row(const FBatch& b, int logM, int logS, int logL, hipStream_t st);
// residues -> limbs with carries (blocks [0, nblk) of sv; res_pos in digits);
// with `add`, in radix 10^18 with the addends of the segments (relative to it)
// (logCR > 0: the digits and run carries of fntt_col_crt instead of residues)
hipError_t fntt_crt(const SegView& sv, int logD, int logCR, const double* res, uint64_t stride, const uint32_t* add,
                    uint32_t* out, uint32_t nblk, uint32_t* flags, uint32_t epoch, uint32_t polls,
                    const CopyList& tails, const uint32_t* tin, uint32_t* tout, uint32_t* err, hipStream_t st);
// The outermost inverse pass (2^logL) with the recombination: digits, and what
// carries out of each run of 2^fntt_run_log(logL) of them.  `add`: decimal joins.
hipError_t fntt_col_crt(const FBatch& b, int logL, const SegView& sv, const uint32_t* add, hipStream_t st);
inline int fntt_run_log(int logL) { return std::min(12 - logL, 6); }
