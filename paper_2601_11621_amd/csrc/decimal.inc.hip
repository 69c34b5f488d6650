// Radix conversion to decimal (the optional decimal text output of Sec. 3.2):
// device kernels.  The integer is converted bottom-up in radix B = 10^18, a
// digit in two limbs: leaves of 29 limbs become sixteen digits, and each level
// joins two neighbours as hi * 2^(928 * 2^j) + lo, where the power of two is
// itself held in radix B.  The products are the FP64 transforms of the library
// (64-bit digits, so radix-B digits go in as they are) with radix-B carries
// that also add lo.
//
// 29 limbs: 2^928 has 15.52 digits, so the 2^j 15.52 digits of an operand at
// level j fill 97 % of half a transform of 2^(j+5).  (Leaves of 16 limbs and
// radix 10^9 filled 53 %.)
#define DEC_LEAF_LIMBS 29
#define DEC_LEAF_DIGITS 16         // 2^928 < 10^288

// 64-bit words that hold what is left of a leaf after d digits (59 bits at
// least each)
__host__ __device__ constexpr int dec_words(int d) { return (32 * DEC_LEAF_LIMBS - 59 * d + 63) / 64; }
#define DEC_LEAF_WORDS 15
static_assert(dec_words(0) == DEC_LEAF_WORDS && dec_words(DEC_LEAF_DIGITS) <= 0, "leaf words");

// Leaves: limbs [29 i, 29 (i + 1)) of x (zero past L) as sixteen radix-B digits
// at out[32 i ..], least significant first (schoolbook division by 10^18 in
// 64-bit words: 123 two-by-one divisions).  Bound by vector issue.
__global__ void __launch_bounds__(64) k_dec_leaf(const uint32_t* __restrict__ x, uint64_t L, uint32_t* __restrict__ out,
                                                 uint64_t nleaves) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nleaves) return;
  uint64_t w[DEC_LEAF_WORDS];
#pragma unroll
  for (int k = 0; k < DEC_LEAF_WORDS; k++) {
    const uint64_t at = i * DEC_LEAF_LIMBS + 2 * k;
    const uint32_t lo = at < L ? x[at] : 0u;
    const uint32_t hi = 2 * k + 1 < DEC_LEAF_LIMBS && at + 1 < L ? x[at + 1] : 0u;
    w[k] = ((uint64_t)hi << 32) | lo;
  }
#pragma unroll
  for (int d = 0; d < DEC_LEAF_DIGITS; d++) {
    constexpr int W0 = DEC_LEAF_WORDS;
    const int W = dec_words(d) < W0 ? dec_words(d) : W0;
    // 16 x word by word, so that the divisor has its top bit set
    uint64_t r = w[W - 1] >> 60;
#pragma unroll
    for (int k = W - 1; k >= 0; k--) w[k] = div_d(r, (w[k] << 4) | (k ? w[k - 1] >> 60 : 0), &r);
    r >>= 4;
    out[i * 2 * DEC_LEAF_DIGITS + 2 * d] = (uint32_t)r;
    out[i * 2 * DEC_LEAF_DIGITS + 2 * d + 1] = (uint32_t)(r >> 32);
  }
}

// Text of the digits dig[0 ..], most significant first: eighteen characters a
// digit, the leading digit without its zeros.  top (device) is one past the
// highest nonzero limb (0 for x = 0).  The character count and the error word go to
// the pinned words pin[0], pin[1]; nothing is written when the count exceeds cap.
// Grid: one thread per digit that can exist.
__global__ void __launch_bounds__(256) k_dec_ascii(const uint32_t* __restrict__ dig,
                                                   const unsigned long long* __restrict__ top, uint64_t cap,
                                                   char* __restrict__ out, const uint32_t* __restrict__ err,
                                                   unsigned long long* __restrict__ pin) {
  const unsigned long long t = *top;
  const uint64_t ti = t ? (t - 1) / 2 : 0;
  const uint64_t vt = ((uint64_t)dig[2 * ti + 1] << 32) | dig[2 * ti];
  uint32_t width = 1;
  for (uint64_t q = vt; q >= 10u; q /= 10u) width++;
  const uint64_t n = width + 18 * ti;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    pin[0] = n;
    pin[1] = *err;
  }
  if (n > cap || i > ti) return;
  uint64_t v = ((uint64_t)dig[2 * i + 1] << 32) | dig[2 * i];
  if (i == ti) {
    for (int k = (int)width - 1; k >= 0; k--) {
      out[k] = (char)('0' + v % 10u);
      v /= 10u;
    }
    return;
  }
  char* o = out + width + 18 * (ti - 1 - i);
  uint32_t h[2] = {(uint32_t)(v / 1000000000u), (uint32_t)(v % 1000000000u)};
#pragma unroll
  for (int q = 0; q < 2; q++) {
#pragma unroll
    for (int k = 8; k >= 0; k--) {
      o[9 * q + k] = (char)('0' + h[q] % 10u);
      h[q] /= 10u;
    }
  }
}

// P_0 = 2^928, written by a kernel that takes it as an argument
struct DecWords {
  uint32_t w[2 * DEC_LEAF_DIGITS];
};
__global__ void k_dec_p0(DecWords p0, uint32_t* __restrict__ out) {
  if (threadIdx.x < 2 * DEC_LEAF_DIGITS) out[threadIdx.x] = p0.w[threadIdx.x];
}
