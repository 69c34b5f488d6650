// Small products of the reconstruction tree (Sec. 3.2, Alg. 2: the lower
// levels of BalancedProductTree(G_e)), plus utility kernels.
//
//  * k_base: one wave forms a node of 256 limbs from its consecutive primes,
//    eight limbs at a time by one lane, then five schoolbook levels in LDS.
//  * k_school: one wave per product of la, lb <= 128 limbs: column sums (a
//    lane holds up to four consecutive columns, a 64-bit sum and a carry
//    count each), then the ballot carry-lookahead.

// ---------------------------------------------------------------------------
// Schoolbook products, la, lb <= 128.  4 waves per block, one product each;
// blocks from ceil(nmul / 4) on copy the tail ranges.
#define SCHOOL_MAX 128
// ---------------------------------------------------------------------------
// Long times short (the shorter operand <= COLSUM_MAX_LB limbs): the exact
// column sums V(k) = sum_j a[k-j] b[j] (< 2^74) for k < la + lb, written as
// three words to the residue rows (v0, v1, v2 at r[k], r[stride + k],
// r[2 stride + k]); the raw mode of the CRT kernel then propagates the carries.
// Workgroup b covers the CRT block b (COLSUM_COLS = CAT_CRT_BLOCK columns of
// one product, found with the stage's segment map); it stages the window
// a[kb - lb, kb + COLSUM_COLS) and b in LDS, and each thread slides a window of
// COLSUM_E values of a down j.  Each column keeps a 64-bit sum and a count of
// its carries out of bit 64 (at most lb), one multiply-add and one add-carry
// per 32x32 product.
#define COLSUM_MAX_LB 1024
#define COLSUM_E CAT_CRT_E
#define COLSUM_T CAT_CRT_THREADS
#define COLSUM_COLS (COLSUM_E * COLSUM_T)
static_assert(COLSUM_COLS == CAT_CRT_BLOCK, "column-sum blocks are the CRT blocks");
__device__ __forceinline__ uint32_t uni32(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uni64(uint64_t x) {
  return ((uint64_t)uni32((uint32_t)(x >> 32)) << 32) | uni32((uint32_t)x);
}
// acc_e += w_e * bj (64-bit, carry out of bit 64 counted in top_e) for three
// columns: the carry of each multiply-add goes to a mask of its own and is
// added two instructions after it was written
__device__ __forceinline__ void colsum_mac3(uint64_t& a0, uint64_t& a1, uint64_t& a2, uint32_t& t0, uint32_t& t1,
                                            uint32_t& t2, uint32_t w0, uint32_t w1, uint32_t w2, uint32_t bj) {
  uint64_t c0, c1, c2;
  asm("v_mad_u64_u32 %0, %6, %9, %12, %0\n\t"
      "v_mad_u64_u32 %1, %7, %10, %12, %1\n\t"
      "v_mad_u64_u32 %2, %8, %11, %12, %2\n\t"
      "v_addc_co_u32_e64 %3, %6, 0, %3, %6\n\t"
      "v_addc_co_u32_e64 %4, %7, 0, %4, %7\n\t"
      "v_addc_co_u32_e64 %5, %8, 0, %5, %8"
      : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(t0), "+v"(t1), "+v"(t2), "=&s"(c0), "=&s"(c1), "=&s"(c2)
      : "v"(w0), "v"(w1), "v"(w2), "v"(bj));
}
static_assert(COLSUM_E == 3, "colsum_mac3 covers three columns");
// the same for one, two and four columns (one and two with wait states
// between a carry's write and its read)
__device__ __forceinline__ void colsum_mac1(uint64_t& a0, uint32_t& t0, uint32_t w0, uint32_t bj) {
  uint64_t c0;
  asm("v_mad_u64_u32 %0, %2, %3, %4, %0\n\t"
      "s_nop 1\n\t"
      "v_addc_co_u32_e64 %1, %2, 0, %1, %2"
      : "+v"(a0), "+v"(t0), "=&s"(c0)
      : "v"(w0), "v"(bj));
}
__device__ __forceinline__ void colsum_mac2(uint64_t& a0, uint64_t& a1, uint32_t& t0, uint32_t& t1, uint32_t w0,
                                            uint32_t w1, uint32_t bj) {
  uint64_t c0, c1;
  asm("v_mad_u64_u32 %0, %4, %6, %8, %0\n\t"
      "v_mad_u64_u32 %1, %5, %7, %8, %1\n\t"
      "s_nop 0\n\t"
      "v_addc_co_u32_e64 %2, %4, 0, %2, %4\n\t"
      "v_addc_co_u32_e64 %3, %5, 0, %3, %5"
      : "+v"(a0), "+v"(a1), "+v"(t0), "+v"(t1), "=&s"(c0), "=&s"(c1)
      : "v"(w0), "v"(w1), "v"(bj));
}
__device__ __forceinline__ void colsum_mac4(uint64_t& a0, uint64_t& a1, uint64_t& a2, uint64_t& a3, uint32_t& t0,
                                            uint32_t& t1, uint32_t& t2, uint32_t& t3, uint32_t w0, uint32_t w1,
                                            uint32_t w2, uint32_t w3, uint32_t bj) {
  uint64_t c0, c1, c2, c3;
  asm("v_mad_u64_u32 %0, %8, %12, %16, %0\n\t"
      "v_mad_u64_u32 %1, %9, %13, %16, %1\n\t"
      "v_mad_u64_u32 %2, %10, %14, %16, %2\n\t"
      "v_mad_u64_u32 %3, %11, %15, %16, %3\n\t"
      "v_addc_co_u32_e64 %4, %8, 0, %4, %8\n\t"
      "v_addc_co_u32_e64 %5, %9, 0, %5, %9\n\t"
      "v_addc_co_u32_e64 %6, %10, 0, %6, %10\n\t"
      "v_addc_co_u32_e64 %7, %11, 0, %7, %11"
      : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3), "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3), "=&s"(c0), "=&s"(c1),
        "=&s"(c2), "=&s"(c3)
      : "v"(w0), "v"(w1), "v"(w2), "v"(w3), "v"(bj));
}
template <int E>
__device__ __forceinline__ void mac_cols(uint64_t* acc, uint32_t* top, const uint32_t* w, uint32_t bj) {
  if constexpr (E == 1) colsum_mac1(acc[0], top[0], w[0], bj);
  if constexpr (E == 2) colsum_mac2(acc[0], acc[1], top[0], top[1], w[0], w[1], bj);
  if constexpr (E == 3) colsum_mac3(acc[0], acc[1], acc[2], top[0], top[1], top[2], w[0], w[1], w[2], bj);
  if constexpr (E == 4)
    colsum_mac4(acc[0], acc[1], acc[2], acc[3], top[0], top[1], top[2], top[3], w[0], w[1], w[2], w[3], bj);
}
__global__ void __launch_bounds__(COLSUM_T) k_colsum(DescView dv, SegView sv, const uint32_t* __restrict__ ain,
                                                const uint32_t* __restrict__ bin, uint32_t* __restrict__ res,
                                                uint64_t stride, uint32_t* __restrict__ err) {
  // lb rounded up to even (b padded with a zero limb); sw[t] = a[kb - lbe + t]
  __shared__ uint32_t sw[COLSUM_COLS + COLSUM_MAX_LB];
  __shared__ __align__(8) uint32_t sbv[COLSUM_MAX_LB];
  CrtSeg sg;
  uint32_t first, end, si;
  sv.find(blockIdx.x, &sg, &first, &end, &si);
  const MulDesc d = dv.get(uni32(si));
  // the longer operand slides, the shorter one is the kernel of the sums
  const uint32_t da = uni32(d.la), db = uni32(d.lb);
  const bool sw_ab = da < db;
  const uint32_t* a = sw_ab ? bin + uni64(d.b_off) : ain + uni64(d.a_off);
  const uint32_t* b = sw_ab ? ain + uni64(d.a_off) : bin + uni64(d.b_off);
  const uint32_t la = sw_ab ? db : da, lb = sw_ab ? da : db;
  const uint32_t tid = threadIdx.x;
  if (lb > COLSUM_MAX_LB) {
    if (tid == 0) atomicOr(err, CAT_DEVERR_BOUNDS);
    return;
  }
  const uint32_t L = la + lb;
  const uint32_t kb = (uni32(blockIdx.x) - uni32(first)) * COLSUM_COLS;
  const uint32_t lbe = (lb + 1) & ~1u;
  const uint32_t wn = COLSUM_COLS + lbe;
  for (uint32_t i = tid; i < wn; i += COLSUM_T) {
    const int64_t idx = (int64_t)kb - (int64_t)lbe + i;
    sw[i] = (idx >= 0 && idx < (int64_t)la) ? a[idx] : 0u;
  }
  for (uint32_t i = tid; i < lbe; i += COLSUM_T) sbv[i] = i < lb ? b[i] : 0u;
  __syncthreads();
  // column k = kb + COLSUM_E tid + e takes a[k - j] = sw[c0 + e - j]; the
  // reads for j + 1 and j + 2 at the last pair (down to sw[COLSUM_E tid])
  // stay in the window
  const uint32_t c0 = COLSUM_E * tid + lbe;
  uint32_t w[COLSUM_E];
#pragma unroll
  for (int e = 0; e < COLSUM_E; e++) w[e] = sw[c0 + e];
  uint64_t acc[COLSUM_E];
  uint32_t top[COLSUM_E];
#pragma unroll
  for (int e = 0; e < COLSUM_E; e++) {
    acc[e] = 0;
    top[e] = 0;
  }
  for (uint32_t j = 0; j < lbe; j += 2) {
    const uint2 bj = *(const uint2*)&sbv[j];
    const uint32_t wn1 = sw[c0 - j - 1], wn2 = sw[c0 - j - 2];
    colsum_mac3(acc[0], acc[1], acc[2], top[0], top[1], top[2], w[0], w[1], w[2], bj.x);
    // j + 1: every column moves one position down a
    colsum_mac3(acc[0], acc[1], acc[2], top[0], top[1], top[2], wn1, w[0], w[1], bj.y);
    w[2] = w[0];
    w[1] = wn1;
    w[0] = wn2;
  }
  uint32_t* r = res + sg.res_pos;
  const uint32_t k0 = kb + COLSUM_E * tid;
#pragma unroll
  for (int e = 0; e < COLSUM_E; e++) {
    if (k0 + e >= L) break;
    r[k0 + e] = (uint32_t)acc[e];
    r[stride + k0 + e] = (uint32_t)(acc[e] >> 32);
    r[2 * stride + k0 + e] = top[e];
  }
}

#define SCHOOL_WAVES 4
#define SCHOOL_WIN (3 * SCHOOL_MAX)
// Column sums of one product in one wave: lane owns the E consecutive columns
// k = E lane + e (64 E >= la + lb - 1) and runs over j < lbe (the shorter
// operand rounded up to even, padded with a zero limb): V(k) = sum_j
// a[k - j] b[j], with sa[t] = a[t - lbe] (zero outside [0, la)).  Each column
// keeps a 64-bit sum and its count of carries out of bit 64; the three words
// go to sv[.][k + 3].
template <int E>
__device__ __forceinline__ void school_cols(const uint32_t* sa, const uint32_t* sbv, uint32_t lbe, uint32_t lane,
                                            uint32_t (*sv)[2 * SCHOOL_MAX + 4]) {
  const uint32_t c0 = E * lane + lbe;
  uint32_t w[E];
#pragma unroll
  for (int e = 0; e < E; e++) w[e] = sa[c0 + e];
  uint64_t acc[E];
  uint32_t top[E];
#pragma unroll
  for (int e = 0; e < E; e++) {
    acc[e] = 0;
    top[e] = 0;
  }
  for (uint32_t j = 0; j < lbe; j += 2) {
    const uint2 bj = *(const uint2*)&sbv[j];
    const uint32_t wn1 = sa[c0 - j - 1], wn2 = sa[c0 - j - 2];
    mac_cols<E>(acc, top, w, bj.x);
    // j + 1: every column one position further down a
    uint32_t w1[E];
    w1[0] = wn1;
#pragma unroll
    for (int e = 1; e < E; e++) w1[e] = w[e - 1];
    mac_cols<E>(acc, top, w1, bj.y);
#pragma unroll
    for (int e = E - 1; e >= 2; e--) w[e] = w[e - 2];
    if constexpr (E >= 2) w[1] = wn1;
    w[0] = wn2;
  }
#pragma unroll
  for (int e = 0; e < E; e++) {
    const uint32_t k = E * lane + e;
    sv[0][k + 3] = (uint32_t)acc[e];
    sv[1][k + 3] = (uint32_t)(acc[e] >> 32);
    sv[2][k + 3] = top[e];
  }
  for (uint32_t k = 64 * E + lane; k < 2 * SCHOOL_MAX; k += 64) {
    sv[0][k + 3] = 0;
    sv[1][k + 3] = 0;
    sv[2][k + 3] = 0;
  }
}

// One product of da x db limbs (both at most SCHOOL_MAX) in one wave; sa, sb, sv
// are the wave's own LDS.
__device__ __forceinline__ void school_wave(const uint32_t* __restrict__ pa, uint32_t da,
                                            const uint32_t* __restrict__ pb, uint32_t db, uint32_t* __restrict__ out,
                                            uint32_t* sa, uint32_t* sb, uint32_t (*sv)[2 * SCHOOL_MAX + 4],
                                            uint32_t lane, uint32_t* __restrict__ err) {
  // the longer operand slides (la), the shorter one is summed over (lb)
  const bool swp = da < db;
  const uint32_t* a = swp ? pb : pa;
  const uint32_t* b = swp ? pa : pb;
  const uint32_t la = swp ? db : da, lb = swp ? da : db, L = la + lb;
  const uint32_t lbe = (lb + 1) & ~1u;
  {
    // every load of the lane in flight together: clamped addresses, masks
    uint32_t xa[SCHOOL_WIN / 64], xb[2];
#pragma unroll
    for (int i = 0; i < SCHOOL_WIN / 64; i++) {
      const uint32_t idx = lane + 64 * i - lbe;    // wraps when t < lbe
      xa[i] = idx < la ? a[idx] : 0u;
    }
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const uint32_t t = lane + 64 * i;
      xb[i] = t < lb ? b[t] : 0u;
    }
#pragma unroll
    for (int i = 0; i < SCHOOL_WIN / 64; i++) sa[lane + 64 * i] = xa[i];
#pragma unroll
    for (int i = 0; i < 2; i++) sb[lane + 64 * i] = xb[i];
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const uint32_t ncol = (L - 1 + 63) / 64;   // columns per lane; k < L - 1 carry the sums
  if (ncol <= 1)
    school_cols<1>(sa, sb, lbe, lane, sv);
  else if (ncol == 2)
    school_cols<2>(sa, sb, lbe, lane, sv);
  else if (ncol == 3)
    school_cols<3>(sa, sb, lbe, lane, sv);
  else
    school_cols<4>(sa, sb, lbe, lane, sv);
  if (lane < 3) { sv[0][lane] = 0; sv[1][lane] = 0; sv[2][lane] = 0; }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  // lane owns limbs 4*lane .. 4*lane+3 (position k stored at index k+3)
  constexpr int E = 4;
  const uint32_t k0 = lane * E;
  uint64_t u[E];
  uint32_t yprev = (uint32_t)(((uint64_t)sv[0][k0 + 2] + sv[1][k0 + 1] + sv[2][k0]) >> 32);
  bool G = false, P = true;
#pragma unroll
  for (int i = 0; i < E; i++) {
    const uint32_t k = k0 + i;
    uint64_t s = 0;
    if (k < L) s = (uint64_t)sv[0][k + 3] + sv[1][k + 2] + sv[2][k + 1];
    u[i] = (s & 0xFFFFFFFFull) + yprev;
    yprev = (uint32_t)(s >> 32);
    const bool g = u[i] >= (1ull << 32), pr = u[i] == 0xFFFFFFFFull;
    G = g || (pr && G);
    P = P && pr;
  }
  uint32_t cout;
  bool ap;
  uint32_t c = wave_carry(G, P, 0, &cout, &ap);
#pragma unroll
  for (int i = 0; i < E; i++) {
    const uint32_t k = k0 + i;
    const uint64_t t = u[i] + c;
    c = (uint32_t)(t >> 32);
    if (k < L) out[k] = (uint32_t)t;
  }
  if (lane == 0 && cout) atomicOr(err, CAT_DEVERR_CARRY_OUT);
}

__global__ void __launch_bounds__(64 * SCHOOL_WAVES)
k_school(DescView dv, uint64_t nmul, const uint32_t* __restrict__ ain, const uint32_t* __restrict__ bin,
         uint32_t* __restrict__ out, uint32_t* __restrict__ err, uint32_t prod_blocks, CopyList tails,
         const uint32_t* __restrict__ tin, uint32_t* __restrict__ tout) {
  __shared__ uint32_t sa[SCHOOL_WAVES][SCHOOL_WIN];
  __shared__ __align__(8) uint32_t sb[SCHOOL_WAVES][SCHOOL_MAX];
  __shared__ uint32_t sv[SCHOOL_WAVES][3][2 * SCHOOL_MAX + 4];
  if (blockIdx.x >= prod_blocks) {
    copy_tail_block(tails, tin, tout, blockIdx.x - prod_blocks);
    return;
  }
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint64_t mi = (uint64_t)blockIdx.x * SCHOOL_WAVES + w;
  if (mi >= nmul) return;   // whole wave leaves together; no block barrier below
  const MulDesc d = dv.get(uni64(mi));
  school_wave(ain + uni64(d.a_off), uni32(d.la), bin + uni64(d.b_off), uni32(d.lb), out + d.c_off, sa[w], sb[w], sv[w],
              lane, err);
}

// ---------------------------------------------------------------------------
// The bottom of the product trees: node i of a group, 256 limbs, is the product
// of the entries [i 32 s8, (i+1) 32 s8) of the group.  s8 entries below 2^B fit
// eight limbs when s8 B <= 256, so a node takes 32 floor(256 / B) entries and not
// 256: the tree over C(10^7)'s 25-bit primes has 0.69 M limbs in its slots, not
// 0.87 M, and C(10^5)'s half as many and one level less.
// One wave per node: lanes 0 .. 31 multiply s8 entries each (an accumulator of
// eight limbs), then five schoolbook levels (8 x 8 up to 128 x 128 limbs) with
// four columns per lane, in the wave's own LDS and without a barrier: operand a
// of product t at sa[3 h t + h ..), zeros on both sides, operand b at sb[h t ..).
// About 2,600 instructions per wave; before, a thread formed 64 limbs alone
// (2,016 dependent multiply-adds, 25 us in a level of any size) and two
// schoolbook launches followed (7 to 18 us together).  With one group of prime
// powers instead of a group per exponent (k_groups): C(10^3) 0.106 -> 0.064 ms,
// C(10^5) 0.212 -> 0.138, C(10^7) 0.581 -> 0.480, C(10^8) 2.83 -> 2.53.
#define BASE_J 8                 // nodes of 2^8 limbs
#define BASE_S8_MAX 24
#define BASE_WAVES 4
struct BaseLevel {
  uint32_t ngroups;
  uint32_t nodes;                          // of all groups
  uint64_t src[CAT_MAX_GROUPS];            // first entry of group g
  uint64_t dst[CAT_MAX_GROUPS];            // limb position of its first node
  uint64_t K[CAT_MAX_GROUPS];              // entries
  uint32_t s8[CAT_MAX_GROUPS];             // entries per eight limbs
  uint32_t mpref[CAT_MAX_GROUPS + 1];      // prefix count of nodes
};
__global__ void __launch_bounds__(64 * BASE_WAVES)
k_base(BaseLevel bl, const uint32_t* __restrict__ in, uint32_t* __restrict__ out) {
  __shared__ __align__(16) uint32_t sa_[BASE_WAVES][384];
  __shared__ __align__(16) uint32_t sb_[BASE_WAVES][128];
  __shared__ uint32_t st_[BASE_WAVES][32 * BASE_S8_MAX];
  const uint32_t w = uni32(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t node = uni32(blockIdx.x * BASE_WAVES + w);
  if (node >= bl.nodes) return;   // whole wave leaves together; no block barrier below
  uint32_t* sa = sa_[w];
  uint32_t* sb = sb_[w];
  uint32_t* st = st_[w];
  uint32_t g = 0;
  while (g + 1 < bl.ngroups && node >= bl.mpref[g + 1]) g++;
  const uint32_t il = node - bl.mpref[g], s8 = bl.s8[g];
  const uint64_t e0 = (uint64_t)il * 32 * s8, K = bl.K[g];
  const uint32_t cnt = (uint32_t)min((uint64_t)(32 * s8), K - e0);   // entries of this node
  {
    const uint32_t* src = in + bl.src[g] + e0;
    for (uint32_t i = lane; i < cnt; i += 64) st[i] = src[i];
  }
  auto wsync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  wsync();
  // eight limbs per lane (1 where the group has ended)
  if (lane < 32) {
    uint32_t acc[8] = {1, 0, 0, 0, 0, 0, 0, 0};
    const uint32_t i0 = lane * s8, i1 = min(i0 + s8, cnt);
    for (uint32_t i = i0; i < i1; i++) {
      const uint32_t q = st[i];
      uint32_t carry = 0;
#pragma unroll
      for (int l = 0; l < 8; l++) {
        const uint64_t t = (uint64_t)acc[l] * q + carry;
        acc[l] = (uint32_t)t;
        carry = (uint32_t)(t >> 32);
      }
    }
    // h = 8: piece 2 t is operand a of product t, piece 2 t + 1 operand b
    const uint32_t t = lane >> 1;
#pragma unroll
    for (int l = 0; l < 8; l++) {
      if (lane & 1) {
        sb[8 * t + l] = acc[l];
      } else {
        sa[24 * t + l] = 0;
        sa[24 * t + 8 + l] = acc[l];
        sa[24 * t + 16 + l] = 0;
      }
    }
  }
  wsync();
  uint32_t r[4];
  for (uint32_t lh = 3; lh <= 7; lh++) {
    const uint32_t h = 1u << lh;
    // columns k0 .. k0 + 3 of product t
    const uint32_t t = (4 * lane) >> (lh + 1), k0 = (4 * lane) & (2 * h - 1);
    const uint32_t* pa = sa + 3 * h * t + h + k0;
    const uint32_t* pb = sb + h * t;
    uint32_t wv[4], top[4] = {0, 0, 0, 0};
    uint64_t acc[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 4; e++) wv[e] = pa[e];
    const uint32_t* pw = pa;
#pragma unroll 2
    for (uint32_t j = 0; j < h; j += 4) {
      const uint4 b = *(const uint4*)&pb[j];
      const uint32_t n0 = pw[-1], n1 = pw[-2], n2 = pw[-3], n3 = pw[-4];
      pw -= 4;
      colsum_mac4(acc[0], acc[1], acc[2], acc[3], top[0], top[1], top[2], top[3], wv[0], wv[1], wv[2], wv[3], b.x);
      colsum_mac4(acc[0], acc[1], acc[2], acc[3], top[0], top[1], top[2], top[3], n0, wv[0], wv[1], wv[2], b.y);
      colsum_mac4(acc[0], acc[1], acc[2], acc[3], top[0], top[1], top[2], top[3], n1, n0, wv[0], wv[1], b.z);
      colsum_mac4(acc[0], acc[1], acc[2], acc[3], top[0], top[1], top[2], top[3], n2, n1, n0, wv[0], b.w);
      wv[0] = n3;
      wv[1] = n2;
      wv[2] = n1;
      wv[3] = n0;
    }
    // limb k: lo(V_k) + mid(V_(k-1)) + hi(V_(k-2)) and carries; a product's
    // columns take nothing from the lane of the product before it
    const bool first = k0 == 0;
    uint32_t m3 = __shfl_up((uint32_t)(acc[3] >> 32), 1, 64), t3 = __shfl_up(top[3], 1, 64),
             t2 = __shfl_up(top[2], 1, 64);
    if (first) m3 = t3 = t2 = 0;
    uint64_t s[4];
    s[0] = (uint64_t)(uint32_t)acc[0] + m3 + t2;
    s[1] = (uint64_t)(uint32_t)acc[1] + (uint32_t)(acc[0] >> 32) + t3;
    s[2] = (uint64_t)(uint32_t)acc[2] + (uint32_t)(acc[1] >> 32) + top[0];
    s[3] = (uint64_t)(uint32_t)acc[3] + (uint32_t)(acc[2] >> 32) + top[1];
    uint32_t y = __shfl_up((uint32_t)(s[3] >> 32), 1, 64);
    if (first) y = 0;
    uint64_t u[4];
    bool G = false, P = true;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      u[e] = (s[e] & 0xFFFFFFFFull) + y;
      y = (uint32_t)(s[e] >> 32);
      const bool gg = u[e] >= (1ull << 32), pp = u[e] == 0xFFFFFFFFull;
      G = gg || (pp && G);
      P = P && pp;
    }
    // (no product carries out of its 2 h limbs, so one scan serves them all)
    uint32_t cout;
    bool ap;
    uint32_t c = wave_carry(G, P, 0, &cout, &ap);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const uint64_t x = u[e] + c;
      c = (uint32_t)(x >> 32);
      r[e] = (uint32_t)x;
    }
    if (lh == 7) break;
    wsync();   // every lane has read this level's operands
    // product t of 2 h limbs: operand a (t even) or b of product t / 2
    const uint32_t h2 = 2 * h, t2i = t >> 1;
    if (t & 1) {
      *(uint4*)&sb[h2 * t2i + k0] = make_uint4(r[0], r[1], r[2], r[3]);
    } else {
      uint32_t* q = sa + 3 * h2 * t2i + k0;
      *(uint4*)q = make_uint4(0, 0, 0, 0);
      *(uint4*)(q + h2) = make_uint4(r[0], r[1], r[2], r[3]);
      *(uint4*)(q + 2 * h2) = make_uint4(0, 0, 0, 0);
    }
    wsync();
  }
  // the node's slot: 256 limbs; in the last one eight per started piece, and one
  // per entry at most
  const uint64_t left = min(K, 8 * ((K + s8 - 1) / s8)) - ((uint64_t)il << BASE_J);
  const uint32_t len = (uint32_t)min((uint64_t)256, left);
  uint32_t* o = out + bl.dst[g] + ((uint64_t)il << BASE_J) + 4 * lane;
  if (4 * lane + 4 <= len) {
    struct W4 {
      uint32_t w[4];
    } v = {{r[0], r[1], r[2], r[3]}};
    *(W4*)o = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (4 * lane + e < len) o[e] = r[e];
  }
}

// A chain of schoolbook steps in one workgroup, each step's products (one wave
// each) reading the results of earlier steps: the powers P_e and their product
// R, whose steps hold a few short products.  As launches of their own they cost
// 3 us each and 6 to 10 us more in a graph that has to carry the dependency from
// one node of the side branch to the next, and the main branch waits for R: at
// n = 10^5 the chain took 64 us of a 230 us call.  Positions are words from W;
// a and b carry the operand's length above bit 56.
#define CHAIN_WAVES 16
#define CHAIN_STEPS 32
#define CHAIN_PRODS 128
struct ChainProd {
  uint64_t a, b, c;
};
struct Chain {
  uint32_t nstep;
  uint32_t fill_len;        // words cleared at fill_pos
  uint64_t fill_pos;
  uint16_t pref[CHAIN_STEPS + 1];
  ChainProd p[CHAIN_PRODS];
};
__global__ void __launch_bounds__(64 * CHAIN_WAVES)
k_school_chain(Chain ch, uint32_t* W, uint32_t* __restrict__ err) {
  __shared__ uint32_t sa[CHAIN_WAVES][SCHOOL_WIN];
  __shared__ __align__(8) uint32_t sb[CHAIN_WAVES][SCHOOL_MAX];
  __shared__ uint32_t sv[CHAIN_WAVES][3][2 * SCHOOL_MAX + 4];
  const uint32_t w = uni32(threadIdx.x >> 6), lane = threadIdx.x & 63;
  for (uint32_t k = threadIdx.x; k < ch.fill_len; k += blockDim.x) W[ch.fill_pos + k] = 0;
  for (uint32_t s = 0; s < ch.nstep; s++) {
    for (uint32_t i = ch.pref[s] + w; i < ch.pref[s + 1]; i += CHAIN_WAVES) {
      const ChainProd q = ch.p[i];
      const uint64_t m = (1ull << 56) - 1;
      school_wave(W + uni64(q.a & m), uni32((uint32_t)(q.a >> 56)), W + uni64(q.b & m), uni32((uint32_t)(q.b >> 56)),
                  W + uni64(q.c), sa[w], sb[w], sv[w], lane, err);
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    // the step's limbs are in memory for every wave before the next one reads
    __threadfence_block();
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Copy of up to CAT_MAX_GROUPS ranges (the odd nodes carried up a level).
__global__ void k_copy_ranges(CopyList cl, const uint32_t* __restrict__ in, uint32_t* __restrict__ out) {
  const uint32_t r = blockIdx.y;
  if (r >= cl.n) return;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < cl.len[r];
       k += (uint64_t)gridDim.x * blockDim.x)
    out[cl.off[r] + k] = in[cl.off[r] + k];
}

// Copies of up to CAT_MAX_GROUPS ranges from one array to another, each to
// an offset of its own (the primes of the requests of a batch, compacted).
struct MoveList {
  uint32_t n;
  uint64_t src[CAT_MAX_GROUPS], dst[CAT_MAX_GROUPS], len[CAT_MAX_GROUPS];
};
__global__ void k_move_ranges(MoveList ml, const uint32_t* __restrict__ in, uint32_t* __restrict__ out) {
  const uint32_t r = blockIdx.y;
  if (r >= ml.n) return;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < ml.len[r];
       k += (uint64_t)gridDim.x * blockDim.x)
    out[ml.dst[r] + k] = in[ml.src[r] + k];
}

__global__ void k_fill(uint32_t* __restrict__ p, uint64_t n, uint32_t v) {
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (uint64_t)gridDim.x * blockDim.x)
    p[k] = v;
}

// Highest index with a nonzero limb, +1 (0 if all zero) -> *top; limbs below
// ncopy are also copied to dst (the caller's output), and with `tail` the last
// block copies those from there to the length, at most `tail`, so that nothing is
// written behind the result (one result only, with `pub`).  One result per grid.y;
// each block reduces in LDS and issues one atomicMax.  With `pub`, the last block
// of the launch (a counter at *done, zero before) copies pub_words words from
// there to pinned host memory: the lengths and the error word reach the host with
// the launch itself, where a copy of its own took another 12 us.
#define TOP_UNROLL 8
struct TopReq {
  const uint32_t* x;
  uint64_t n;
  unsigned long long* top;
  uint32_t* dst;
  uint64_t ncopy, tail;
};
template <int NR>
struct TopBatch {
  TopReq r[NR];
};
template <int NR>
__global__ void __launch_bounds__(256)
k_top_nonzero(TopBatch<NR> tb, uint32_t* done, const uint32_t* pub, uint32_t* pub_dst, uint32_t pub_words) {
  __shared__ unsigned long long part[4];
  __shared__ uint32_t s_last;
  const TopReq& q = tb.r[NR == 1 ? 0 : blockIdx.y];
  const uint32_t* __restrict__ x = q.x;
  uint32_t* __restrict__ dst = q.dst;
  const uint64_t n = q.n, ncopy = q.ncopy;
  unsigned long long best = 0;
  // TOP_UNROLL loads in flight per thread: one at a time, 16 and more rounds of
  // memory latency were the kernel's time (C(10^8) 2.43 -> 2.36 ms)
  const uint64_t T = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k0 < n; k0 += TOP_UNROLL * T) {
    uint32_t v[TOP_UNROLL];
#pragma unroll
    for (int i = 0; i < TOP_UNROLL; i++) v[i] = x[k0 + i * T < n ? k0 + i * T : k0];
#pragma unroll
    for (int i = 0; i < TOP_UNROLL; i++) {
      const uint64_t k = k0 + i * T;
      if (k < n && v[i]) best = k + 1;
      if (k < n && k < ncopy) dst[k] = v[i];
    }
  }
  for (int d = 32; d >= 1; d >>= 1) {
    unsigned long long o = __shfl_xor(best, d, 64);
    best = o > best ? o : best;
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); w++) best = part[w] > best ? part[w] : best;
    if (best) atomicMax(q.top, best);
    if (pub) {
      __threadfence();
      s_last = atomicAdd(done, 1u) + 1 == gridDim.x * gridDim.y;
    }
  }
  if (!pub) return;
  __syncthreads();
  if (s_last) {
    __threadfence();
    for (uint32_t k = threadIdx.x; k < pub_words; k += blockDim.x)
      pub_dst[k] = __hip_atomic_load(pub + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (NR == 1) {
      const unsigned long long len = __hip_atomic_load(q.top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint64_t end = min((uint64_t)len, q.tail);
      for (uint64_t k = ncopy + threadIdx.x; k < end; k += blockDim.x) dst[k] = x[k];
    }
  }
}

// Limb k of floor(x / 2^s) for x[0..lx) (zero past the top).
__device__ __forceinline__ uint32_t shifted_limb(const uint32_t* __restrict__ x, uint64_t lx, uint64_t s, uint64_t k) {
  const uint64_t w = k + (s >> 5);
  const uint32_t r = (uint32_t)(s & 31);
  const uint32_t lo = w < lx ? x[w] : 0u;
  if (r == 0) return lo;
  const uint32_t hi = w + 1 < lx ? x[w + 1] : 0u;
  return (lo >> r) | (hi << (32 - r));
}

// 1 + the highest index where X = floor(x / 2^s) and Y = y differ (0 if X = Y),
// limbs past the ends being zero -> *top (atomicMax; zero it before).  n: the
// limbs to scan (at least the longer of X and Y).
__global__ void __launch_bounds__(256) k_diff_top(const uint32_t* __restrict__ x, uint64_t lx, uint64_t s,
                                                  const uint32_t* __restrict__ y, uint64_t ly, uint64_t n,
                                                  unsigned long long* top) {
  __shared__ unsigned long long part[4];
  unsigned long long best = 0;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t a = shifted_limb(x, lx, s, k), b = k < ly ? y[k] : 0u;
    if (a != b) best = k + 1;
  }
  for (int d = 32; d >= 1; d >>= 1) {
    unsigned long long o = __shfl_xor(best, d, 64);
    best = o > best ? o : best;
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); w++) best = part[w] > best ? part[w] : best;
    if (best) atomicMax(top, best);
  }
}

// Fingerprints of a limb vector: x mod (2^32 - 5), x mod (2^32 + 1), x mod
// (2^32 - 1).  Workgroup b reduces the 4096 limbs [4096 b, 4096 b + 4096):
// thread t holds the RES_C limbs at 4096 b + 256 i + t (coalesced loads) and
// the block's partial is sum_k x_k (2^32)^(k - 4096 b) mod q; the library
// combines the partials with the weights (2^32)^(4096 b) on the host.  With
// 2^32 = 5, -1 and 1 modulo the three moduli, the weight of limb 256 i + t
// is 5^(256 i + t), (-1)^t and 1: a Horner pass over i with the constant
// 5^256 (two folds of 2^32 = 5 per step) for the first, plain 64-bit sums
// for the others.
#define RES_T 256
#define RES_C 16
#define RES_BLOCK (RES_T * RES_C)
#define RES_Q0 4294967291ull   // 2^32 - 5
#define RES_Q1 4294967297ull   // 2^32 + 1
#define RES_Q2 4294967295ull   // 2^32 - 1
// y mod (2^32 - 5) for any 64-bit y: fold 2^32 = 5 twice, then one subtraction
__device__ __forceinline__ uint32_t mod_q0(uint64_t y) {
  const uint64_t r = (y >> 32) * 5ull + (y & 0xFFFFFFFFull);   // < 6 * 2^32
  const uint64_t r2 = (r >> 32) * 5ull + (r & 0xFFFFFFFFull);  // < 2^32 + 30
  return (uint32_t)(r2 >= RES_Q0 ? r2 - RES_Q0 : r2);
}
__global__ void __launch_bounds__(RES_T) k_residues(const uint32_t* __restrict__ x, uint64_t n, uint32_t w256,
                                                    uint64_t* __restrict__ part) {
  __shared__ uint64_t red[3][RES_T / 64];
  const uint32_t t = threadIdx.x;
  const uint64_t base = (uint64_t)blockIdx.x * RES_BLOCK;
  uint32_t v[RES_C];
#pragma unroll
  for (int i = 0; i < RES_C; i++) {
    const uint64_t k = base + (uint64_t)i * RES_T + t;
    v[i] = k < n ? x[k] : 0u;
  }
  uint32_t h = 0;
  uint64_t s = 0;
#pragma unroll
  for (int i = RES_C - 1; i >= 0; i--) {
    h = mod_q0((uint64_t)h * w256 + v[i]);
    s += v[i];
  }
  // lane weight 5^t mod q0 by square-and-multiply over the bits of t < 256
  uint32_t w = 1, b5 = 5;
  for (uint32_t e = t; e; e >>= 1) {
    if (e & 1) w = mod_q0((uint64_t)w * b5);
    b5 = mod_q0((uint64_t)b5 * b5);
  }
  uint64_t a0 = mod_q0((uint64_t)h * w);      // < 2^32: 256 of them sum below 2^40
  uint64_t ap = (t & 1) ? 0 : s, am = (t & 1) ? s : 0;   // s < 2^36
  for (int d = 32; d >= 1; d >>= 1) {
    a0 += __shfl_xor(a0, d, 64);
    ap += __shfl_xor(ap, d, 64);
    am += __shfl_xor(am, d, 64);
  }
  if ((t & 63) == 0) {
    red[0][t >> 6] = a0;
    red[1][t >> 6] = ap;
    red[2][t >> 6] = am;
  }
  __syncthreads();
  if (t == 0) {
    uint64_t s0 = 0, sp = 0, sm = 0;
    for (int k = 0; k < RES_T / 64; k++) {
      s0 += red[0][k];
      sp += red[1][k];
      sm += red[2][k];
    }
    part[3 * (uint64_t)blockIdx.x + 0] = s0 % RES_Q0;
    part[3 * (uint64_t)blockIdx.x + 1] = (sp % RES_Q1 + RES_Q1 - sm % RES_Q1) % RES_Q1;
    part[3 * (uint64_t)blockIdx.x + 2] = (sp + sm) % RES_Q2;
  }
}

// ---------------------------------------------------------------------------
// Twiddle tables.  roots[prime][s] = omega_{2^s} in Montgomery form, for
// each prime set (the second set has roots up to 2^CAT_LAZY_MAX_LOGN).
struct RootsC {
  uint32_t r[CAT_NPRIMES][CAT_MAX_LOGN + 1];     // forward, Montgomery form
  uint32_t ir[CAT_NPRIMES][CAT_MAX_LOGN + 1];    // inverse
  uint32_t one[CAT_NPRIMES];                     // R mod p
};
__constant__ RootsC c_roots;
__constant__ RootsC c_roots1;
template <int AS>
__device__ __forceinline__ const RootsC& rootsc() {
  if constexpr (AS == 0) return c_roots;
  else return c_roots1;
}

__device__ __forceinline__ uint32_t mont_pow(uint32_t b, uint64_t e, uint32_t one, uint32_t p, uint32_t pinv) {
  uint32_t r = one;
  while (e) {
    if (e & 1) r = mont_mul(r, b, p, pinv);
    b = mont_mul(b, b, p, pinv);
    e >>= 1;
  }
  return r;
}
__device__ __forceinline__ uint2 tw_pair(uint32_t w, uint32_t pinv) { return make_uint2(w, w * pinv); }
// Shoup pair of the value whose Montgomery form is w: (W, floor(W 2^32 / p))
__device__ __forceinline__ uint2 shoup_pair(uint32_t w, uint32_t p, uint32_t pinv) {
  const uint32_t W = mont_mul(w, 1u, p, pinv);
  return make_uint2(W, (uint32_t)(((uint64_t)W << 32) / p));
}

// Pass tables: for s = 1..14, S = 2^s, radix R = 2^pass_logr(s), entry
// (k1, j2) at tws_off(s) + (k1 << (s - r)) + j2 = omega_S^{+-j2*k1}:
// Montgomery pairs (set 0) or Shoup pairs (set 1).
template <int AS>
__global__ void k_build_tws(uint2* __restrict__ tws, uint2* __restrict__ itws) {
  const uint32_t prime = blockIdx.y;
  const PrimeC& pc = primec<AS>(prime);
  const RootsC& rc = rootsc<AS>();
  const uint32_t p = pc.p, pinv = pc.pinv;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < TWS_ENTRIES; i += gridDim.x * blockDim.x) {
    int s = 1;
    while (tws_off(s + 1) <= i) s++;
    const uint32_t li = i - tws_off(s);
    const int r = pass_logr(s);
    const uint32_t k1 = li >> (s - r), j2 = li & ((1u << (s - r)) - 1);
    const uint64_t e = (uint64_t)j2 * k1;
    const uint32_t w = mont_pow(rc.r[prime][s], e, rc.one[prime], p, pinv);
    const uint32_t iw = mont_pow(rc.ir[prime][s], e, rc.one[prime], p, pinv);
    tws[(size_t)prime * TWS_ENTRIES + i] = AS == 0 ? tw_pair(w, pinv) : shoup_pair(w, p, pinv);
    itws[(size_t)prime * TWS_ENTRIES + i] = AS == 0 ? tw_pair(iw, pinv) : shoup_pair(iw, p, pinv);
  }
}

// Two-level tables of omega = omega_{2^tw_logn}: lo[i] = omega^i (i < 2^14,
// Montgomery pairs), hi[i] = omega^{i*2^14} (i < 2^(tw_logn - 14), Montgomery
// form); and the inverse.
template <int AS>
__global__ void k_build_tw2(uint2* __restrict__ lo, uint32_t* __restrict__ hi, uint2* __restrict__ ilo,
                            uint32_t* __restrict__ ihi) {
  const uint32_t prime = blockIdx.y;
  const PrimeC& pc = primec<AS>(prime);
  const RootsC& rc = rootsc<AS>();
  const uint32_t p = pc.p, pinv = pc.pinv;
  const uint32_t one = rc.one[prime];
  const uint32_t r = rc.r[prime][tw_logn<AS>()], ir = rc.ir[prime][tw_logn<AS>()];
  const uint32_t nhi = 1u << (tw_logn<AS>() - TW2_LO_BITS);
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < TW2_LO; i += gridDim.x * blockDim.x) {
    lo[(size_t)prime * TW2_LO + i] = tw_pair(mont_pow(r, i, one, p, pinv), pinv);
    ilo[(size_t)prime * TW2_LO + i] = tw_pair(mont_pow(ir, i, one, p, pinv), pinv);
    if (i < nhi) {
      hi[(size_t)prime * TW2_HI + i] = mont_pow(r, (uint64_t)i << TW2_LO_BITS, one, p, pinv);
      ihi[(size_t)prime * TW2_HI + i] = mont_pow(ir, (uint64_t)i << TW2_LO_BITS, one, p, pinv);
    }
  }
}
