// Radix conversion to decimal text (the optional decimal output of Sec. 3.2):
// plan and C ABI.
//
// x (L limbs) is cut into n_0 = ceil(L/29) leaves of 29 limbs, each turned into
// sixteen radix-10^18 digits (two limbs a digit; lengths below are limbs).
// Level j holds n_j nodes; node i is the value of limbs [i 29 2^j, (i+1) 29 2^j)
// and has len_j limbs, the last one last_j (as many digits as its bits need).
// Two neighbours join as hi * P_j + lo with P_j = 2^(928 2^j), len_j limbs as
// well; a last node without a partner is carried up.  The products of a level
// are one uniform batch with one second operand, and the squaring that makes
// P_{j+1} is one more product of the same batch: a level is one launch up to 2^11
// digits, and no second stream is needed.  A product too long for one transform
// (the top one, beyond 29 2^22 limbs) is cut along hi into pieces:
// T_0 = hi_0 P + lo, T_k = hi_k P + T_{k-1} / B^m above the copied T_{k-1} mod B^m.

struct DecLevel {
  uint64_t nodes = 0, len = 0, last = 0;   // n_j, len_j, last_j
  uint64_t pw = 0;                         // P_j
};

struct DecPlan {
  uint64_t L = 0;
  std::vector<DecLevel> lv;      // levels 0 .. h (level h: one node)
  std::vector<std::vector<Stage>> join;   // stages of level j -> j+1
  uint64_t x[2] = {0, 0};        // uint32 offsets
  size_t off_res = 0, off_F = 0, off_ctl = 0, ctl_words = 0, total = 0;   // bytes
  uint64_t res_len = 0;
  uint64_t products = 0, product_digits = 0;
};

// limbs (even) for a value of at most 2^k in radix 10^18 (exact, or one digit
// more when k log10(2) is within 1e-6 below a multiple of 18)
uint64_t dec_limbs(uint64_t k) { return 2 * ((uint64_t)((long double)k * 0.30102999566398119521L / 18.0L + 1e-6L) + 1); }

// np joins with second operand u.b0, and its square if sq_len
bool dec_stage(Stage* s, uint64_t np, UniDesc u, const CrtSeg& seg, uint64_t step_out, uint64_t step_add,
               uint64_t last_len, uint64_t sq_pos, bool sq) {
  const uint64_t len = (uint64_t)u.la + u.lb;
  int k = ceil_log2(len / 2);            // digits of the longest product
  // the one-workgroup kernels take operands of half a transform
  if (k <= FNTT_LDS_MAX_LOGD) k = std::max(k, ceil_log2(std::max(u.la, u.lb) / 2) + 1);
  if (k > FNTT_MAX_LOGD) return false;
  s->fp = true;
  s->logN = std::max(k, FNTT_LDS_MIN_LOGD) + 1;
  s->nmul = np + (sq ? 1 : 0);
  s->limbs = s->nmul * len;
  u.last = (uint32_t)(np - 1);
  u.sq = sq ? (uint32_t)np : ~0u;
  s->dv = DescView{};
  s->dv.uni = 1;
  s->dv.u = u;
  s->sv = SegView{};
  s->sv.ubl = crt_blocks(true, seg.len);
  s->sv.nseg = (uint32_t)s->nmul;
  s->sv.iseg[0] = seg;
  s->sv.ustep[0] = step_out;
  s->sv.ustep[1] = step_add;
  s->sv.ustep[2] = len / 2;
  s->sv.ulast = u.last;
  s->sv.ulast_len = last_len;
  s->sv.usq = u.sq;
  s->sv.usq_pos = sq_pos;
  s->nseg = (uint32_t)s->nmul;
  const uint64_t nb = s->nmul * s->sv.ubl;
  s->nblk = (uint32_t)nb;
  return nb < (1ull << 31);
}

cat_status make_dec_plan(uint64_t L, DecPlan* D) {
  DecPlan& P = *D;
  P = DecPlan{};
  P.L = L;
  if (L > (1ull << CAT_MAX_LOGN)) return CAT_ERANGE;
  uint64_t o = 0, xsize = 0;
  auto take = [&](uint64_t words) {
    const uint64_t r = o;
    o = align_up(o + words, 64);
    return r;
  };
  // levels
  DecLevel c;
  c.nodes = std::max<uint64_t>(1, (L + DEC_LEAF_LIMBS - 1) / DEC_LEAF_LIMBS);
  for (uint64_t span = DEC_LEAF_LIMBS;; span *= 2) {
    c.len = dec_limbs(32 * span);
    const uint64_t rest = L > (c.nodes - 1) * span ? L - (c.nodes - 1) * span : 0;
    // (the leaf kernel writes all digits of every leaf)
    c.last = span == DEC_LEAF_LIMBS ? c.len : std::min(c.len, dec_limbs(32 * rest));
    c.pw = c.nodes > 1 ? take(c.len) : 0;
    xsize = std::max(xsize, c.nodes * c.len);
    P.lv.push_back(c);
    if (c.nodes == 1) break;
    c.nodes = (c.nodes + 1) / 2;
  }
  P.x[0] = take(xsize);
  P.x[1] = take(xsize);
  // joins
  uint64_t F_words = 0, nblk_max = 0;
  for (size_t j = 0; j + 1 < P.lv.size(); j++) {
    const DecLevel& a = P.lv[j];
    const DecLevel& b = P.lv[j + 1];
    const uint64_t xin = P.x[j & 1], xout = P.x[(j + 1) & 1];
    const uint64_t np = a.nodes / 2;
    const bool odd = a.nodes & 1, sq = j + 2 < P.lv.size();
    std::vector<Stage> v;
    UniDesc u{xin + a.len, 2 * a.len, a.pw, (uint32_t)a.len, (uint32_t)a.len, (uint32_t)(odd ? a.len : a.last)};
    if (np == 1) u.la = u.la_last;
    Stage s;
    const CrtSeg seg{xout, 0, b.len, xin, a.len};
    if (dec_stage(&s, np, u, seg, b.len, 2 * a.len, odd ? b.len : b.last, b.pw, sq)) {
      if (odd) {
        s.tails.n = 1;
        s.tails.len[0] = a.last;
        s.tail_in_base = xin + (a.nodes - 1) * a.len;
        s.tail_out_base = xout + np * b.len;
      }
      v.push_back(s);
    } else {
      // one product only, cut along hi
      if (np != 1 || odd || sq) return CAT_ERANGE;
      const uint64_t m = (2ull << FNTT_MAX_LOGD) - a.len;
      uint64_t add_pos = xin, add_len = a.len, tmp[2] = {0, 0};
      for (uint64_t h0 = 0, i = 0; h0 < a.last; h0 += m, i++) {
        const bool end = h0 + m >= a.last;
        const uint64_t la = end ? a.last - h0 : m, ol = end ? b.last - h0 : la + a.len;
        if (!end && i < 2) tmp[i] = take(m + a.len);
        const uint64_t dst = end ? xout + h0 : tmp[i & 1];
        UniDesc ui{xin + a.len + h0, 0, a.pw, (uint32_t)la, (uint32_t)a.len, (uint32_t)la};
        Stage si;
        if (ol > la + a.len ||
            !dec_stage(&si, 1, ui, CrtSeg{dst, 0, ol, add_pos, add_len}, 0, 0, ol, 0, false))
          return CAT_ERANGE;
        if (i) {   // T_{i-1} mod B^m is final
          si.tails.n = 1;
          si.tails.len[0] = m;
          si.tail_in_base = add_pos - m;
          si.tail_out_base = xout + h0 - m;
        }
        v.push_back(si);
        add_pos = dst + m;
        add_len = a.len;
      }
    }
    for (const Stage& t : v) {
      P.res_len = std::max(P.res_len, t.limbs / 2);
      if (t.logN - 1 > FNTT_LDS_MAX_LOGD) F_words = std::max<uint64_t>(F_words, t.nmul * 12ull << (t.logN - 1));
      nblk_max = std::max<uint64_t>(nblk_max, t.nblk);
      P.products += t.nmul;
      P.product_digits += t.limbs;
    }
    P.join.push_back(v);
  }
  size_t off = o * 4;
  auto takeb = [&](size_t bytes) {
    const size_t r = off;
    off = align_up(off + bytes, 256);
    return r;
  };
  P.off_res = takeb(3 * (P.res_len + 64) * 8);
  P.off_F = takeb(F_words * 4);
  // control block: error word, -, top (8 bytes), look-back flags
  P.ctl_words = 4 + nblk_max + 1;
  P.off_ctl = takeb(P.ctl_words * 4);
  P.total = off;
  return CAT_OK;
}

// P_0 = 2^(32 DEC_LEAF_LIMBS) in radix 10^18, least significant digit first
DecWords dec_p0() {
  uint32_t w[DEC_LEAF_LIMBS + 1] = {0};   // as 32-bit limbs, by long division
  w[DEC_LEAF_LIMBS] = 1;
  DecWords d;
  for (int k = 0; k < DEC_LEAF_DIGITS; k++) {
    unsigned __int128 r = 0;
    for (int i = DEC_LEAF_LIMBS; i >= 0; i--) {
      const unsigned __int128 cur = (r << 32) | w[i];
      w[i] = (uint32_t)(cur / DEC_B);
      r = cur % DEC_B;
    }
    d.w[2 * k] = (uint32_t)r;
    d.w[2 * k + 1] = (uint32_t)(r >> 32);
  }
  return d;
}

cat_status launch_join(Exec& X, const Stage& s) {
  const uint32_t* tin = X.W + s.tail_in_base;
  uint32_t* tout = X.W + s.tail_out_base;
  if (fntt_fused_fits(s.logN - 1)) {
    const FBatch b = fp_batch(X, s, s.dv, s.nmul);
    KTime kt("k_ffused10", X.st, bfly(9.0 * b.cnt, b.logD));
    HIPCHK(fntt_fused10(b, s.sv, X.W, s.tails, tin, tout, X.err, X.st));
    X.launches++;
    return CAT_OK;
  }
  STCHK(launch_fp(X, s, s.dv, s.nmul, X.W));
  KTime kt("k_fcrt10", X.st, (double)s.nblk * FCRT_BLOCK);
  X.crt_epoch++;
  HIPCHK(fntt_crt(s.sv, s.logN - 1, fp_run_log(s, s.nmul), (const double*)X.res, X.res_stride / 2, X.W, X.W, s.nblk,
                  X.flags, X.crt_epoch, crt_polls(s.nblk), s.tails, tin, tout, X.err, X.st));
  X.launches++;
  return CAT_OK;
}

extern "C" {

cat_status decimal_sizes(size_t n_limbs, size_t* max_chars, size_t* work_bytes) {
  if (!max_chars || !work_bytes) return CAT_EINVAL;
  DecPlan P;
  STCHK(make_dec_plan(n_limbs, &P));
  // decimal digits of a number below 2^(32 L)
  *max_chars = (size_t)((long double)n_limbs * 32.0L * 0.30102999566398119521L) + 2;
  *work_bytes = P.total;
  return CAT_OK;
}

// The whole conversion is queued directly (clear the control block, P_0, the
// leaves, the joins, the top digit, the text): its launches, at most 100, queue
// faster than they run.
cat_status bigint_to_decimal(const uint32_t* d_x, size_t n_limbs, char* d_out, size_t cap, size_t* n_chars,
                             void* d_work, size_t work_bytes, void* stream) {
  if (!n_chars || !d_work || (n_limbs && !d_x)) return CAT_EINVAL;
  std::lock_guard<std::recursive_mutex> lk(g.mu);
  STCHK(init_locked(-1));
  STCHK(set_device());
  DecPlan P;
  STCHK(make_dec_plan(n_limbs, &P));
  if (work_bytes < P.total) return CAT_ENOMEM;
  hipStream_t st = (hipStream_t)stream;
  char* wb = (char*)d_work;
  Exec X;
  X.W = (uint32_t*)wb;
  X.res = (uint32_t*)(wb + P.off_res);
  X.res_stride = 2 * (P.res_len + 64);
  X.F = (uint32_t*)(wb + P.off_F);
  X.err = (uint32_t*)(wb + P.off_ctl);
  X.flags = X.err + 4;
  X.st = st;
  unsigned long long* top = (unsigned long long*)(X.err + 2);
  const size_t h = P.lv.size() - 1;
  hipLaunchKernelGGL(k_fill, dim3((uint32_t)std::min<uint64_t>((P.ctl_words + 255) / 256, 1024)), dim3(256), 0, st,
                     X.err, (uint64_t)P.ctl_words, 0u);
  LAUNCHCHK();
  if (h > 0) {
    static const DecWords p0 = dec_p0();
    hipLaunchKernelGGL(k_dec_p0, dim3(1), dim3(64), 0, st, p0, X.W + P.lv[0].pw);
    LAUNCHCHK();
  }
  const uint64_t n0 = P.lv[0].nodes;
  {
    KTime kt("k_dec_leaf", st, (double)n0);
    hipLaunchKernelGGL(k_dec_leaf, dim3((uint32_t)((n0 + 63) / 64)), dim3(64), 0, st, d_x, (uint64_t)n_limbs,
                       X.W + P.x[0], n0);
  }
  LAUNCHCHK();
  for (size_t j = 0; j < h; j++)
    for (const Stage& s : P.join[j]) STCHK(launch_join(X, s));
  const uint32_t* dig = X.W + P.x[h & 1];
  const uint64_t nw = P.lv[h].last;
  STCHK(launch_top(st, dig, nw, top, nullptr, 0));
  {
    KTime kt("k_dec_ascii", st, (double)nw / 2);
    hipLaunchKernelGGL(k_dec_ascii, dim3((uint32_t)((nw / 2 + 255) / 256)), dim3(256), 0, st, dig,
                       (const unsigned long long*)top, d_out ? (uint64_t)cap : (uint64_t)0, d_out, X.err,
                       (unsigned long long*)g.pin);
  }
  LAUNCHCHK();
  // (the last launch left the count and the error word in pinned memory)
  HIPCHK(hipStreamSynchronize(st));
  uint64_t pin[2];
  memcpy(pin, g.pin, sizeof(pin));
  cat_stats stats{};
  stats.products = P.products;
  stats.product_limbs = P.product_digits;
  stats.levels = (uint32_t)h;
  g.stats = stats;
  if (pin[1]) return CAT_EINTERNAL;
  *n_chars = (size_t)pin[0];
  if (!d_out || cap < pin[0]) return CAT_ERANGE;
  return CAT_OK;
}

}  // extern "C"
