// prompt seeding: the dense [m x L] causal rows on the matrix cores, merge, decision.
// Part of one translation unit: included by corm_kernels.hip, in this order, after <hip/hip_runtime.h> and corm.h.
#ifndef CORM_PREFILL_HPP
#define CORM_PREFILL_HPP

namespace {

// ---------------------------------------------------------------- prompt seeding (dense, matrix cores)
//
// The prompt's last m queries (steps tau_j = t - m + 1 + j) against all its keys: the causal rows of
// Eq. 2, thresholded (Def. 3.1) into last_hit and stored in the ring exactly where m decode steps would
// have put them.  [m x L] logits per head are a dense contraction, so q.K^T runs on the MFMA units; the
// elementwise tail (exp, rounding, compare) and the ring store bound the rest.
//
// Two passes over the same products:
//   pass 1   query-major, workgroup = up to 16 tiles of 16 queries, loops over the keys of its segment: per query the sum of
//            exp relative to a reference -> partials [head, key segment, query]
//   merge    per query: reference and 1/sum over the segments, and what pass 2 compares with
//   pass 2   key-major, workgroup = 256 (128) keys of a unit, loops over all query tiles; p = exp2(s - reference) / sum,
//            stored to the ring row of the query's step at the key's position, and per key the latest step whose
//            stored score reaches the threshold
// In pass 2 the workgroup keeps its keys in registers as the A operand (lane l: row l%16 of a 16-key tile, the
// 16 bytes 64*c + 16*(l/16) .. of each 64-byte chunk c of the row); a tile of 16 queries is the B
// operand in the same layout, read from LDS, where the workgroup stages the queries in double-buffered
// blocks.  D: lane l holds query l%16 and rows 4*(l/16) .. +3 of each key tile.
//
// Query tiles are walked in the order (16 queries, head of the group): tile tt = (queries 16*(tt/G) .., head
// tt%G).  The step of a lane's query never falls from one tile to the next, so one register per key holds its
// latest hit over all heads.  A launch with few units deals the tiles of a key block to several workgroups
// (segments); their last_hit then meet in an atomic max.

constexpr int PREFILL_XCDS = 8;   // accelerator dies of the device

// Groups of 16 queries of a call: pass 2 keeps latest hits as 1 + such a number in 16 bits, and forms offsets into the queries of up to four
// heads, of 512 bytes each, in 32; the clear launch has a grid row for each.
constexpr int SEED_MAX_TILES = 65535;
static_assert(SEED_MAX_TILES <= 0xffff, "latest hits: two keys to a word");
static_assert(4ull * SEED_MAX_TILES * 16 * 512 <= 0xffffffffull, "offsets into a block's queries (a descriptor's length is below a half of it)");

struct PrefillArgs {
  const void* q_tail;   // [B, Hq, m, d]
  const void* K;
  const int32_t* lens;
  const int32_t* pos;
  int32_t* last_hit;
  const int32_t* t;
  void* ring;
  float2* part;    // [B*Hq, nkb, w]  (reference, sum) per key segment (nks <= nkb of them)
  float4* stats;   // [B*Hq, w]       per query: see prefill_query_stats
  int32_t* status;
  int32_t Hq, Hkv, Lcap, Tcap, w, m, nkb, ring_bf16;
  int32_t units;                   // B * Hkv
  int32_t nqb, nks, kseg;          // pass 1: query blocks of a unit, key segments of a unit, keys per segment
  int32_t nseg, seg_blocks;        // pass 2: workgroups that share the query blocks of a key block, blocks each
  int32_t ring_bits, ring_words;   // boolean message: one bit per (row, position), words per row
  float thr_scale, scale_log2;
};

template <typename DT> struct PrefillMma;
template <> struct PrefillMma<BF16> {
  __device__ static __forceinline__ f32x4_t mma(const uint4& a, const uint4& b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                   0, 0, 0);
  }
};
template <> struct PrefillMma<F32> {
  // four k-steps of v_mfma_f32_16x16x4_f32: lane group l/16 supplies element 4*(l/16) + e of the chunk in step e
  __device__ static __forceinline__ f32x4_t mma(const uint4& a, const uint4& b, f32x4_t c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
};

typedef float f32x2_t __attribute__((ext_vector_type(2)));

// two fp32 -> two bf16 (round to nearest even) in one word, first value in the low half
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// the score of a raw logit: the one formula every ring type starts from
__device__ __forceinline__ float prefill_score(float d, float scale_log2, float ms, float inv) {
  return fast_exp2(fmaf(d, scale_log2, -ms)) * fabsf(inv);   // (its sign: see prefill_query_stats)
}

typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bit_select(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }

// Two 16-bit integers in a word: all ones in the half where x > limit.  (In assembly: as a
// comparison of vectors the compiler takes it apart into two compares and two selects.)
__device__ __forceinline__ uint32_t above16x2(uint32_t x, uint32_t limit) {
  uint32_t m;
  asm("v_pk_sub_i16 %0, %1, %2 clamp\n\tv_pk_ashrrev_i16 %0, 15, %0 op_sel_hi:[0,1]" : "=&v"(m) : "v"(limit), "v"(x));
  return m;
}

// the least of near, |a| and |b| (those that are numbers)
__device__ __forceinline__ float least_abs(float near, float a, float b) {
  asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(near) : "v"(a), "v"(b));
  return near;
}

// (x << 1) | the sign of t, in one instruction that touches no scalar register: a compare would put its result there,
// and every reader of it waits
__device__ __forceinline__ uint32_t shift_in_sign(uint32_t x, float t) {
  return __builtin_amdgcn_alignbit(x, __float_as_uint(t), 31);
}

// What the ring holds: which form of Def. 3.1 pass 2 evaluates (an instance each).
enum { SEED_BF16 = 0, SEED_F32 = 1, SEED_BITS = 2 };

// Per query, for pass 2: x = reference, y = 1/sum (z, the sum of exp2(logit - reference)) and, so that pass 2 neither unpacks what it stores nor forms scores
// that it does not store,
//   score rings   z = the smallest fp32 score whose stored value reaches thr.  bf16: rounding to nearest even is
//                 monotone, so "stored >= thr" is "score >= z" with z the midpoint below the smallest bf16 >= thr
//                 (or the next fp32, where that midpoint rounds down).  fp32: z = thr.  bf16, w: that smallest bf16 minus one
//                 (as an integer: for scores that are numbers the order is the same) in both halves of a word, for whole blocks.
//                 A row with a logit that is not finite (its reference or sum is not a finite number either), in which scores may
//                 be no numbers, has the sign of y set: no block with such a row is a fast one, and general blocks decide by z.
//   boolean ring  raw logits above z + w are important, those below z - w are not, and only those between
//                 need the score itself.  The band is the threshold in the logit domain -+ a bound on every
//                 rounding between a logit and its score (products, fma, exp2, 1/sum, the logarithms and z -+ w here: together
//                 below 2e-6 of the terms), so the decisions are bit for bit those of the score.
//                 A query without such a band has w = infinity and is decided by the score
//                 throughout: thresholds 0 or near the ends of the fp32 range, and rows with a logit that is not finite.
// The reference is near the row's maximum, so that no term of the sum overflows and those that make it up do not vanish: at most
// 1/2 above it, and at most log2(STATS_JUMP times the key tiles looked at together) below, in log2 units; it is the maximum where the
// reference could not follow the logits.
__device__ __forceinline__ float4 prefill_query_stats(const PrefillArgs& a, float ms, float z, float thr) {
  float4 s = make_float4(ms, z > 0.f ? 1.0f / z : 0.f, thr, 0.f);
  if (a.ring_bits) {
    const float lt = log2f(thr), lz = log2f(z);
    const float at = ms + lt + lz, pad = 1e-5f + 2e-6f * (fabsf(ms) + fabsf(lt) + fabsf(lz));
    s.z = at / a.scale_log2;
    s.w = 1.0001f * (pad / a.scale_log2);
    if (!(lt + lz > -100.f) || !(fabsf(s.z) < 1e30f) || !(s.w < 1e30f)) s = make_float4(s.x, s.y, 0.f, __builtin_inff());
  } else if (a.ring_bf16) {
    const uint32_t up = (__float_as_uint(thr) + 0xffffu) >> 16;   // the smallest bf16 >= thr (thr >= 0)
    s.z = up ? __uint_as_float(((up - 1u) << 16) + 0x8000u + (up & 1u)) : 0.f;
    s.w = __uint_as_float(((up - 1u) & 0xffffu) * 0x10001u);
    if (!(fabsf(ms) < __builtin_inff()) || !(z < __builtin_inff())) s.y = -s.y;
  }
  return s;
}

template <int ROWB>
struct PrefillGeom {
  static constexpr int NCH = ROWB / 64;            // 64-byte chunks of a row
  static constexpr int T = NCH <= 4 ? 4 : 2;       // 16-key tiles per wave
  static constexpr int WKEYS = T * 16;             // keys per wave
  static constexpr int KB = WAVES * WKEYS;         // keys per workgroup
  static constexpr int QBLK = ROWB <= 256 ? 64 : 32;   // queries staged in LDS at a time
  static constexpr int QT = QBLK / 16;             // query tiles of a block
  static constexpr int QROW = ROWB + 16;           // LDS row pitch (padded against bank conflicts)
  static constexpr int QLOADS = QBLK * ROWB / (WG * 16);   // 16-byte loads per thread and block
  static_assert(QBLK * ROWB % (WG * 16) == 0 && QBLK <= WG, "a block is loaded in whole passes of the workgroup");
};

// ---------------------------------------------------------------- pass 1: the sum of exp per query
//
// Query-major, the other way round than pass 2: a wave keeps QW tiles of 16 queries in registers (B operand) and all keys of
// its segment pass by through LDS (A operand, double-buffered blocks).  A lane then holds four keys of ONE query per tile,
// so its sum stays in a register: nothing crosses lanes inside the loop, and every 256 keys the register is added to a word
// of LDS.  The elementwise tail is little more than fma, exp2, add per pair: the reference of a sum (a power of two,
// each lane its own) is not the running maximum but follows it: where a tile's four terms add up to more than STATS_JUMP, the
// reference is moved to their maximum and they are formed again, which is rare after the first block.  So, as with the maximum,
// the terms that make up a sum come from small differences.  A workgroup with a lane whose reference could not be set, or whose
// sum is not finite, does the loop again, first for the maxima and then for the sums against them.
// Bound by the products, at the rate the card's power leaves (with the tail dropped 480 us for 512 heads x 1024 queries x 4096 keys:
// 1.0 PFLOP/s; a large library product 1.15), and by what of the tail does not fit beside them.  Inside whole calls, key-major with
// a maximum per tile, as before, and now, traced in turn: 600 to 616 us, 588 to 596 (bf16), 512 x 1024 x 8192 1170, 1041; the merge
// 23 -> 6 and 40 -> 7 us, since a row has a partial per segment and no longer one per 256 keys.  (578 and 1025 us with one register for
// the sum of a row and lanes that are not asked for themselves: wrong sums for logits of 10^6, low bits lost on long rows.)
// Tried, as kernels alone in a row of runs, where key-major takes 768 and this one took 697: against the fixed reference 0 640, but its
// terms carry the rounding of whole logits (fp32 ring 8.3e-7 from 64 bits, 5.6e-7 as it is); a whole block done again in
// place of a tile 729; 32 x 32 tiles at two waves per SIMD 686 and 702, 128 queries per wave 709 to 764 (all against the reference 0).

constexpr float STATS_JUMP = 16.f;

// Blocks of keys (the first is one for itself) whose sums are added up by themselves before they join the sum of all: with one register
// from the first key to the last, a few large terms at a prompt's start swallow the low bits of the thousands of tiles after them.
// Error of the row sum on the CPU (rms), in this order | one register | partials of 256 keys against their maximum (as pass 1 was when it
// went key-major), the first 16 keys 2^24 above the others: 8192 keys 1.0e-7 | 3.6e-6 | 1.6e-7, 32768 keys 1.8e-7 | 1.4e-5 | 3.1e-7; without
// such keys, 32768: 0.9e-7 | 3.3e-7 | 1.6e-7.
constexpr int STATS_FOLD = 4;

// QW query tiles per wave.  bf16: as many as the registers of three waves per SIMD hold, so that a key tile read from LDS serves as
// many products as it can; one where the launch is short of workgroups (stats_segments).  fp32: one, its products take long
// enough for any LDS traffic.
template <typename DT>
constexpr int stats_qw() { return std::is_same<DT, F32>::value ? 1 : 4; }

template <int ROWB, int QW>
struct StatsGeom {
  static constexpr int NCH = ROWB / 64;
  static constexpr int KBLK = ROWB <= 256 ? 64 : 32;   // keys staged in LDS at a time
  static constexpr int KT = KBLK / 16;
  static constexpr int NT = QW >= KT ? 1 : KT / QW;    // key tiles worked on together: independent chains of products
  static constexpr int KROW = ROWB + 16;           // LDS row pitch (padded against bank conflicts)
  static constexpr int KLOADS = KBLK * ROWB / (WG * 16);
  static_assert(KBLK * ROWB % (WG * 16) == 0 && KBLK <= 64, "a block is loaded in whole passes of the workgroup");
};

template <typename DT, int D, int QW>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(3, 3))) void corm_prefill_stats_kernel(
    const PrefillArgs a) {
  constexpr int ROWB = D * DT::ESZ;
  using Geo = StatsGeom<ROWB, QW>;
  constexpr int NCH = Geo::NCH, KBLK = Geo::KBLK, KT = Geo::KT, KROW = Geo::KROW, KLOADS = Geo::KLOADS;
  constexpr int NT = Geo::NT;
  constexpr int NEVER = 0x7fffffff;   // position of a slot that holds no key: visible to no query

  // workgroup id % 8 names the XCD; the workgroups of a unit (its query blocks first, they read the same keys) follow one
  // another on it
  const int per_xcd = (a.units + PREFILL_XCDS - 1) / PREFILL_XCDS;
  const int li = (int)(blockIdx.x / PREFILL_XCDS);
  const int qblk = li % a.nqb, lk = li / a.nqb;
  const int ks = lk % a.nks;
  const int unit = (int)(blockIdx.x % PREFILL_XCDS) * per_xcd + lk / a.nks;
  if (lk / a.nks >= per_xcd || unit >= a.units) return;
  const int b = unit / a.Hkv, hkv = unit - b * a.Hkv;
  const int G = a.Hq / a.Hkv;
  const int lgG = 31 - __clz(G);   // G is a power of two
  int L = a.lens[unit];
  L = L < 0 ? 0 : (L > a.Lcap ? a.Lcap : L);
  const int key_beg = ks * a.kseg, key_end = min(key_beg + a.kseg, L);
  if (key_beg >= L) return;
  const int tcur = a.t[b];
  const int tau0 = tcur - a.m + 1;   // step of tail query 0
  if (tau0 < 1 || tcur > a.Tcap) return;   // (pass 2 reports it)
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // (uniform: what hangs on it
  // takes scalar registers; in vector registers it had them spilled, and a reload in the loop waits for the keys in flight)
  const int n = lane & 15, lg = lane >> 4;

  __shared__ __attribute__((aligned(16))) char sh_k[2][KBLK * KROW];
  __shared__ __attribute__((aligned(16))) int32_t sh_pos[2][KBLK];

  const int ntt = ((a.m + 15) / 16) << lgG;                    // query tiles of the group
  const int wtt = (qblk * WAVES + wv) * QW;                    // this wave's first
  const int tt_end = min((qblk + 1) * WAVES * QW, ntt);        // end of the workgroup's
  const int nqt = min(max(ntt - wtt, 0), QW);                  // tiles of this wave
  // the last position the workgroup sees, the last and the first query of the wave: positions they see
  const int wg_last = tau0 + min(((tt_end - 1) >> lgG) * 16 + 15, a.m - 1) - 1;
  const int vis_last = tau0 + min(((wtt + nqt - 1) >> lgG) * 16 + 15, a.m - 1) - 1;
  const int vis_first = tau0 + (wtt >> lgG) * 16 - 1;

  uint4 qb[QW][NCH];
#pragma unroll
  for (int qt = 0; qt < QW; ++qt) {
    const int tt = min(wtt + qt, ntt - 1), j = (tt >> lgG) * 16 + n;
    const char* q = reinterpret_cast<const char*>(a.q_tail) +
                    ((size_t)(b * a.Hq + hkv * G + (tt & (G - 1))) * a.m + min(j, a.m - 1)) * ROWB;
#pragma unroll
    for (int c = 0; c < NCH; ++c) qb[qt][c] = *reinterpret_cast<const uint4*>(q + c * 64 + 16 * lg);
  }

  const __amdgpu_buffer_rsrc_t rk = make_rsrc(
      reinterpret_cast<const char*>(a.K) + (size_t)unit * a.Lcap * ROWB, (uint32_t)key_end * ROWB);
  const __amdgpu_buffer_rsrc_t rp = make_rsrc(a.pos + (size_t)unit * a.Lcap, (uint32_t)key_end * 4);
  u32x4_t kr[KLOADS];
  int pr;
  auto fetch = [&](int key0) __attribute__((always_inline)) {   // (past the end: zeros, no traffic)
#pragma unroll
    for (int i = 0; i < KLOADS; ++i)
      kr[i] = __builtin_amdgcn_raw_buffer_load_b128(rk, (int)((uint32_t)key0 * ROWB + (uint32_t)(i * WG + tid) * 16), 0, 0);
    pr = __builtin_amdgcn_raw_buffer_load_b32(rp, (key0 + tid % KBLK) * 4, 0, 0);
  };
  auto stage = [&](int buf, int key0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KLOADS; ++i) {
      const int o = (i * WG + tid) * 16;   // row o / ROWB, column o % ROWB
      *reinterpret_cast<u32x4_t*>(&sh_k[buf][(o / ROWB) * KROW + (o % ROWB)]) = kr[i];
    }
    const bool held = key0 + tid % KBLK < key_end && pr >= 0 && pr < a.Tcap;
    sh_pos[buf][tid % KBLK] = held ? pr : NEVER;
  };
  auto mma_tile = [&](int cur, int kt, f32x4_t (&d)[QW]) __attribute__((always_inline)) {
    uint4 ka[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      ka[c] = *reinterpret_cast<const uint4*>(&sh_k[cur][(kt * 16 + n) * KROW + c * 64 + 16 * lg]);
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) d[qt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int qt = 0; qt < QW; ++qt) d[qt] = PrefillMma<DT>::mma(ka[c], qb[qt][c], d[qt]);
  };

  // of this lane's keys of a query: reference of the sum, maximum (raw logits), sum of up to STATS_FOLD blocks; in LDS (the
  // registers are full) the sum of the blocks before them and its reference, a thread's own words
  float ms[QW], mx[QW], z[QW];
  __shared__ __attribute__((aligned(16))) float sh_z[WG][QW], sh_zref[WG][QW];
  uint32_t any = 0u;             // bit qt: the query saw a key; bit 16 + qt: its reference is set
#pragma unroll
  for (int qt = 0; qt < QW; ++qt) {
    ms[qt] = 0.f;
    mx[qt] = neg_inf();
  }
  float unset = 2.f * STATS_JUMP * NT;   // (0 from the first block on) the wave's references are to be set
  // Moves a reference to the maximum m of a tile's raw logits, if it is higher or the first.  A first one that is lower than the 0 it
  // replaces comes too late for keys seen before (their terms may have vanished): the sum is not a number from then on.
  auto follow = [&](int qt, float m) __attribute__((always_inline)) {
    const float to = rintf(m * a.scale_log2);
    if (fabsf(to) < 1e6f && (to > ms[qt] || !((any >> (16 + qt)) & 1u))) {
      z[qt] = to >= ms[qt] || !((any >> qt) & 1u) ? ldexpf(z[qt], (int)(ms[qt] - to)) : __builtin_nanf("");
      ms[qt] = to;
      any |= 0x10000u << qt;
    }
  };
  enum { FOLLOW, MAXIMA, FIXED };   // the reference follows the sum; the maxima instead; the sum against the maxima
  auto fold = [&](int mode) __attribute__((always_inline)) {
    int th = tid;
    asm volatile("" : "+v"(th));   // (its addresses are formed here, not kept in registers through the loop)
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) {
      float before = sh_z[th][qt];
      if (mode == FOLLOW) {   // (the reference rose, or was set before anything was summed)
        before = ldexpf(before, (int)(sh_zref[th][qt] - ms[qt]));
        sh_zref[th][qt] = ms[qt];
      }
      sh_z[th][qt] = before + z[qt];
      z[qt] = 0.f;
    }
  };
  auto walk = [&](int mode) __attribute__((always_inline)) {
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) {
      z[qt] = 0.f;
      sh_z[tid][qt] = 0.f;
      sh_zref[tid][qt] = ms[qt];
    }
    fetch(key_beg);
    stage(0, key_beg);
    int cur = 0;
    for (int key0 = key_beg; key0 < key_end; key0 += KBLK, cur ^= 1) {
      __syncthreads();   // the block is staged; nobody reads the other buffer any more
      const int first = sh_pos[cur][0];
      if (first > wg_last && first != NEVER) break;   // (uniform) positions ascend: nothing more to be seen
      fetch(key0 + KBLK);
      const int p = sh_pos[cur][lane % KBLK];
      if (__all(p <= vis_first) && nqt == QW && mode != MAXIMA) {
        // (uniform over the wave) every query sees every key: straight-line code, the next tile's products under this tile's tail
        f32x4_t dn[NT][QW];
#pragma unroll
        for (int x = 0; x < NT; ++x) mma_tile(cur, x, dn[x]);
#pragma unroll
        for (int kt = 0; kt < KT; kt += NT) {
          f32x4_t d[NT][QW];
#pragma unroll
          for (int x = 0; x < NT; ++x)
#pragma unroll
            for (int qt = 0; qt < QW; ++qt) d[x][qt] = dn[x][qt];
#pragma unroll
          for (int x = 0; x < NT; ++x)
            if (kt + NT < KT) mma_tile(cur, kt + NT + x, dn[x]);
          float sum[QW], big = kt ? 0.f : unset;
          auto terms = [&](int x, int qt) __attribute__((always_inline)) {
            float e[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) e[r] = fast_exp2(fmaf(d[x][qt][r], a.scale_log2, -ms[qt]));
            return (e[0] + e[1]) + (e[2] + e[3]);
          };
#pragma unroll
          for (int qt = 0; qt < QW; ++qt) {
            sum[qt] = 0.f;
#pragma unroll
            for (int x = 0; x < NT; ++x) sum[qt] += terms(x, qt);
            big = fmaxf(big, sum[qt]);
          }
          if (__builtin_expect(__any(big > STATS_JUMP * NT) && mode == FOLLOW, 0)) {
#pragma unroll
            for (int qt = 0; qt < QW; ++qt) {
              asm volatile("" : "+v"(ms[qt]));   // (nothing of this is to be done ahead of the branch)
              float m = neg_inf();
#pragma unroll
              for (int x = 0; x < NT; ++x)
#pragma unroll
                for (int r = 0; r < 4; ++r) m = fmaxf(m, d[x][qt][r]);
              follow(qt, m);
              sum[qt] = 0.f;
#pragma unroll
              for (int x = 0; x < NT; ++x) sum[qt] += terms(x, qt);
            }
          }
#pragma unroll
          for (int qt = 0; qt < QW; ++qt) z[qt] += sum[qt];
          any |= (1u << QW) - 1u;
        }
        unset = 0.f;
      } else if (__any(p <= vis_last) && nqt > 0) {
        unset = 0.f;
        int vis[QW], nl = lane;   // this lane's query of the tile sees positions <= vis
        asm volatile("" : "+v"(nl));   // (formed here, not kept in registers through the other blocks)
#pragma unroll
        for (int qt = 0; qt < QW; ++qt) {
          const int j = ((wtt + qt) >> lgG) * 16 + (nl & 15);
          vis[qt] = wtt + qt < ntt && j < a.m ? tau0 + j - 1 : -1;
        }
#pragma unroll 1
        for (int kt = 0; kt < KT; ++kt) {
          f32x4_t d[QW];
          mma_tile(cur, kt, d);
          const int4 kp = *reinterpret_cast<const int4*>(&sh_pos[cur][kt * 16 + 4 * lg]);
#pragma unroll
          for (int qt = 0; qt < QW; ++qt) {
            const bool s[4] = {kp.x <= vis[qt], kp.y <= vis[qt], kp.z <= vis[qt], kp.w <= vis[qt]};
            float m = neg_inf();
#pragma unroll
            for (int r = 0; r < 4; ++r) m = fmaxf(m, s[r] ? d[qt][r] : neg_inf());
            if (mode == MAXIMA) {
              mx[qt] = fmaxf(mx[qt], m);
            } else {
              if (mode == FOLLOW) follow(qt, m);
              float e[4];
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                e[r] = fast_exp2(fmaf(d[qt][r], a.scale_log2, -ms[qt]));
                e[r] = s[r] ? e[r] : 0.f;
              }
              z[qt] += (e[0] + e[1]) + (e[2] + e[3]);
            }
            any |= (s[0] || s[1] || s[2] || s[3]) ? 1u << qt : 0u;
          }
        }
      }
      if (mode != MAXIMA && (key0 - key_beg) / KBLK % STATS_FOLD == 0) fold(mode);   // (uniform)
      stage(cur ^ 1, key0 + KBLK);
    }
    fold(mode);
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) z[qt] = sh_z[tid][qt];
    __syncthreads();
  };

  walk(FOLLOW);
  // A lane whose reference was set in time holds a sum of at least 2^-1/2, its largest term.  Any other that saw a key summed
  // against the reference 0, which a sum below 1/2 does not fit (terms may have vanished), or set one too late: asked per lane,
  // since the other lane groups of the query hide it.
  bool out_of_range = false;
#pragma unroll
  for (int qt = 0; qt < QW; ++qt) {   // the four lane groups of a query, each with a reference of its own
    out_of_range |= ((any >> qt) & 1u) && !(z[qt] >= 0.5f && z[qt] < __builtin_inff());
    const float m = z[qt] > 0.f ? ms[qt] : neg_inf();
    ms[qt] = rows_allreduce_max(m);
    z[qt] = rows_allreduce_sum(z[qt] > 0.f ? ldexpf(z[qt], (int)(m - ms[qt])) : z[qt]);
    if (ms[qt] == neg_inf()) ms[qt] = 0.f;
  }
  if (__syncthreads_or(out_of_range)) {   // (rare)
    walk(MAXIMA);
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) {
      mx[qt] = rows_allreduce_max(mx[qt]);
      ms[qt] = mx[qt] == neg_inf() ? 0.f : mx[qt] * a.scale_log2;
    }
    walk(FIXED);
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) {
      z[qt] = rows_allreduce_sum(z[qt]);
      if (mx[qt] == neg_inf()) ms[qt] = neg_inf();
    }
  }
  any = rows_allreduce_or(any);
#pragma unroll
  for (int qt = 0; qt < QW; ++qt) {
    const int tt = wtt + qt, j = (tt >> lgG) * 16 + n;
    if (lg == 0 && tt < ntt && j < a.m)
      a.part[((size_t)(b * a.Hq + hkv * G + (tt & (G - 1))) * a.nkb + ks) * a.w + j] =
          make_float2((any >> qt) & 1u ? ms[qt] : neg_inf(), z[qt]);
  }
}

// ---------------------------------------------------------------- pass 2: scores, ring rows, last hits

// FAR: a head's ring reaches beyond the 32-bit offsets of a buffer descriptor (pass 2).
template <typename DT, int D, int MODE, bool FAR>
__device__ __forceinline__ void prefill_scores(const PrefillArgs& a) {
  constexpr int ROWB = D * DT::ESZ;
  using Geo = PrefillGeom<ROWB>;
  constexpr int NCH = Geo::NCH, T = Geo::T, KB = Geo::KB, WKEYS = Geo::WKEYS, QT = Geo::QT;
  constexpr int QBLK = Geo::QBLK, QROW = Geo::QROW, QLOADS = Geo::QLOADS;
  constexpr int NEVER = 0x7fffffff;   // position of a slot that holds no key: visible to no query
  // Which key of the wave sits in row 4*lg + r of key tile tl: where a lane's 4*T values leave as bf16 or as bits,
  // 4*T consecutive keys (they pack into whole words of the lane); fp32 scores leave per key tile, 64
  // consecutive bytes per query.
  constexpr bool RUN = MODE != SEED_F32;

  // One-dimensional grid of 8 * ceil(units / 8) * nkb * nseg workgroups.  Workgroups are dealt round-robin to the 8
  // XCDs, so id % 8 names the XCD; each XCD takes a contiguous range of units and runs the key blocks of a unit
  // one after the other: they all read the same tail queries, which then stay in that XCD's L2.  (As many workgroups as the chip
  // holds, which take the blocks from a queue per XCD and then from the others': the whole call 1 % shorter, not kept.)
  const int per_xcd = (a.units + PREFILL_XCDS - 1) / PREFILL_XCDS;
  const int li = (int)(blockIdx.x / PREFILL_XCDS);
  const int seg = li % a.nseg, lk = li / a.nseg;
  const int unit = (int)(blockIdx.x % PREFILL_XCDS) * per_xcd + lk / a.nkb;
  const int kb = lk % a.nkb;
  if (lk / a.nkb >= per_xcd || unit >= a.units) return;
  const int b = unit / a.Hkv, hkv = unit - b * a.Hkv;
  const int G = a.Hq / a.Hkv;
  const int lgG = 31 - __clz(G);   // G is a power of two
  int L = a.lens[unit];
  L = L < 0 ? 0 : (L > a.Lcap ? a.Lcap : L);
  const int key_blk = kb * KB;
  if (key_blk >= L) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = lane & 15, lg = lane >> 4;
  const int tcur = a.t[b];
  const int tau0 = tcur - a.m + 1;   // step of tail query 0
  if (tau0 < 1 || tcur > a.Tcap) {
    if (tid == 0 && a.status) atomicOr(a.status, CORM_DEV_BAD_STEP);
    return;
  }
  const int s0 = (tau0 - 1) % a.w;   // ring slot of tail query 0

  constexpr int STB = 4;   // (one behind is still read from when the next is staged)
  __shared__ __attribute__((aligned(16))) char sh_q[2][QBLK * QROW];     // query blocks, double buffered
  __shared__ __attribute__((aligned(16))) float4 sh_st[STB][QBLK];   // prefill_query_stats per query
  __shared__ __attribute__((aligned(16))) int32_t sh_pos[KB];            // positions of the workgroup's keys

  // Pass 2, bf16 ring: a wave's tile of stored scores is turned through LDS so that every query's consecutive
  // positions leave as one piece of its ring row (16 bytes per lane).  Rows are padded by 16 bytes.
  // (Stored straight from the lanes that hold them, a lane's 16 bytes in pieces of 64: the whole call 3 to 6 % longer.)
  constexpr int TROW = WKEYS + 8;
  constexpr bool TURN = MODE == SEED_BF16;
  __shared__ __attribute__((aligned(16))) uint16_t sh_t[TURN ? WAVES : 1][TURN ? 16 : 1][TURN ? TROW : 1];

  const char* Kb = reinterpret_cast<const char*>(a.K) + (size_t)unit * a.Lcap * ROWB;
  const int32_t* posb = a.pos + (size_t)unit * a.Lcap;
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(Kb, (uint32_t)L * ROWB);
  const int wkey0 = key_blk + wv * WKEYS;   // first key of this wave

  uint4 ka[T][NCH];
#pragma unroll
  for (int tl = 0; tl < T; ++tl) {
    const int row = wkey0 + (RUN ? (n >> 2) * (4 * T) + tl * 4 + (n & 3) : tl * 16 + n);
#pragma unroll
    for (int c = 0; c < NCH; ++c) ka[tl][c] = buffer_load16(rk, (uint32_t)row * ROWB + (uint32_t)(c * 64 + 16 * lg));
  }
  int my_pos = NEVER;   // of key wkey0 + lane
  if (lane < WKEYS && wkey0 + lane < L) {
    my_pos = posb[wkey0 + lane];
    if (my_pos < 0 || my_pos >= a.Tcap) {
      if (a.status) atomicOr(a.status, CORM_DEV_BAD_STEP);
      my_pos = NEVER;
    }
  }
  if (lane < WKEYS) sh_pos[wv * WKEYS + lane] = my_pos;
  // every slot of the wave holds a key; its positions are consecutive; the first and the last of them
  const bool wave_whole = __all(lane >= WKEYS || my_pos != NEVER);
  const int pos_w0 = __builtin_amdgcn_readfirstlane(my_pos), pos_wlast = __builtin_amdgcn_readlane(my_pos, WKEYS - 1);
  const bool wave_run = wave_whole && __all(lane >= WKEYS || my_pos == pos_w0 + lane);
  // Pass 2 stores whole pieces of a row where the wave's keys are consecutive and every piece is aligned (rows of
  // the ring then start at multiples of a piece as well).
  const bool rows_ok = a.ring == nullptr ||
                       (wave_run && (MODE == SEED_BF16  ? ((pos_w0 | a.Tcap) & 7) == 0
                                     : MODE == SEED_F32 ? ((pos_w0 | a.Tcap) & 3) == 0
                                                        : WKEYS % 32 == 0 && (pos_w0 & 31) == 0));
  const int pos_wmax = wave_whole ? pos_wlast : NEVER;
  // Positions ascend with the slot, so queries before the one that sees the block's first key see none of it.
  const int pfirst = posb[key_blk];
  const int jt_first = max(pfirst - tau0 + 1, 0) / 16;

  const int jt_wave = pos_w0 == NEVER ? jt_first : max(pos_w0 - tau0 + 1, 0) / 16;   // the same of the wave's first key

  const int ntt = ((a.m + 15) / 16) << lgG;                    // query tiles of the group
  const int blk_end = min((seg + 1) * a.seg_blocks, (ntt + QT - 1) / QT);
  const int blk_vis = min((jt_first << lgG) / QT, blk_end);    // first block with a query that sees a key
  const int blk_seg = seg * a.seg_blocks;                      // first block of this workgroup
  const int blk_beg = max(blk_seg, blk_vis);
  const char* qg = reinterpret_cast<const char*>(a.q_tail) + (size_t)(b * a.Hq + hkv * G) * a.m * ROWB;
  const float4* stats = a.stats + (size_t)(b * a.Hq + hkv * G) * a.w;

  // Queries reach the waves through LDS, QBLK at a time: the block after the current one is in flight
  // (registers) while the current one is worked on, so the loop never waits on a load it has just
  // issued.  Two LDS buffers, one barrier per block.  Loads and stores share one in-order counter: the registers
  // go to LDS where the number of ring stores issued behind the loads is known to the compiler.
  u32x4_t qr[QLOADS];
  float4 str = make_float4(0.f, 0.f, 0.f, 0.f);
  // A block's tiles start at a multiple of QT: tile x of the block is head h0 + x % G, 16 queries jt0 + x / G (G <= QT) or, for
  // larger groups, head h0 + x.  What hangs on x alone is formed here, so that a block costs few scalar instructions.
  constexpr int RPP = WG * 16 / ROWB;   // rows per pass of the workgroup
  const int half = RPP == 32 ? __builtin_amdgcn_readfirstlane(tid >> 7) : 0;
  uint32_t q_off[QLOADS], q_row[QLOADS];   // bytes from the block's first query, and of queries of its head before it
#pragma unroll
  for (int i = 0; i < QLOADS; ++i) {
    const int x = i * RPP / 16 + half;
    q_row[i] = (uint32_t)(x >> lgG) * 16u * ROWB;
    q_off[i] = (uint32_t)(x & (G - 1)) * (uint32_t)a.m * ROWB + q_row[i];
  }
  const int st_x = (tid % QBLK) / 16;   // (every wave the same QBLK queries: no branch, whose join would cost the exact wait count)
  const float4* stats_lane = stats + (size_t)(st_x & (G - 1)) * a.w + (st_x >> lgG) * 16 + (tid & 15);
  auto fetch = [&](int blk, u32x4_t (&qr)[QLOADS], float4& str) __attribute__((always_inline)) {
    const int h0 = (blk * QT) & (G - 1), j0 = ((blk * QT) >> lgG) * 16;
    const char* q0 = qg + ((size_t)h0 * a.m + j0) * ROWB;
    const uint32_t left = (uint32_t)(a.m - j0) * ROWB;
#pragma unroll
    for (int i = 0; i < QLOADS; ++i) {
      // (uniform over the wave) a descriptor that ends with the head's last query: zeros past it, which are masked
      const __amdgpu_buffer_rsrc_t rq = make_rsrc(q0 + q_off[i], (uint32_t)max((int)(left - q_row[i]), 0));
      qr[i] = __builtin_amdgcn_raw_buffer_load_b128(rq, (i * RPP * ROWB + tid * 16) % (16 * ROWB), 0, 0);
    }
    str = stats_lane[(size_t)h0 * a.w + j0];   // (past the last query: up to 63 more, which the workspace holds)
  };
  auto read_tile = [&](int cur, int ti, uint4 (&qb)[NCH]) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      qb[c] = *reinterpret_cast<const uint4*>(&sh_q[cur][(ti * 16 + n) * QROW + c * 64 + 16 * lg]);
  };
  auto mma = [&](const uint4 (&qb)[NCH], f32x4_t (&d)[T]) __attribute__((always_inline)) {
#pragma unroll
    for (int tl = 0; tl < T; ++tl) d[tl] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int tl = 0; tl < T; ++tl) d[tl] = PrefillMma<DT>::mma(ka[tl][c], qb[c], d[tl]);
  };
  auto mma_tile = [&](int cur, int ti, f32x4_t (&d)[T]) __attribute__((always_inline)) {
    uint4 qb[NCH];
    read_tile(cur, ti, qb);
    mma(qb, d);
  };
  // Fast blocks store through a buffer descriptor with 32-bit offsets: of one head's ring, or (FAR; as an instance of its
  // own, since the few scalar instructions per tile cost the others 1 to 3 %) of the rows of a tile's 16 queries, which lie
  // in a row unless the ring wraps among them.  Without a ring its length is 0, which drops the stores (no branch
  // around them); so are those at DEAD_OFFSET, as long as the descriptor ends in front of it.
  const uint64_t row_bytes64 = MODE == SEED_BITS ? (uint64_t)a.ring_words * 4 : (uint64_t)a.Tcap * (MODE == SEED_BF16 ? 2 : 4);
  const uint64_t head_bytes = a.w * row_bytes64;
  const uint32_t row_bytes = (uint32_t)row_bytes64;
  // ring slot of query j; row of the ring that query j of head g is recorded in
  auto slot_of = [&](int j) __attribute__((always_inline)) -> uint32_t {
    const int slot = s0 + j;
    return (uint32_t)(slot >= a.w ? slot - a.w : slot);
  };
  const uint64_t ring0 = reinterpret_cast<uint64_t>(a.ring) + (uint64_t)(b * a.Hq + hkv * G) * head_bytes;   // of the group's first head
  const uint32_t ring_len = a.ring ? (FAR ? 16 * row_bytes : (uint32_t)head_bytes) : 0u;
  auto ring_row = [&](int g, int j) __attribute__((always_inline)) -> size_t {
    return (size_t)(b * a.Hq + hkv * G + g) * a.w + slot_of(j);
  };

  // The latest hit of every key of the lane, over the queries n of every tile: fp32 ring, the step; else 1 + the number of the 16
  // queries (0: none), two keys to a word, in the order of the lane's keys.
  constexpr bool PACKED = MODE != SEED_F32;
  int hm[PACKED ? 1 : T][4];
  uint32_t hm2[PACKED ? 2 * T : 1];
#pragma unroll
  for (int tl = 0; tl < (PACKED ? 1 : T); ++tl)
#pragma unroll
    for (int r = 0; r < 4; ++r) hm[tl][r] = 0;
#pragma unroll
  for (int i = 0; i < (PACKED ? 2 * T : 1); ++i) hm2[i] = 0u;
  auto hit_at = [&](int i, int jt) __attribute__((always_inline)) {   // key i of the lane, 16 queries jt
    hm2[PACKED ? i >> 1 : 0] = i & 1 ? (hm2[PACKED ? i >> 1 : 0] & 0xffffu) | ((uint32_t)(jt + 1) << 16)
                                     : (hm2[PACKED ? i >> 1 : 0] & 0xffff0000u) | (uint32_t)(jt + 1);
  };
  auto raise = [&](int i, uint32_t at0, uint32_t at1) __attribute__((always_inline)) {   // word i, to at least these
    uint32_t& h = hm2[PACKED ? i : 0];
    h = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, h), __builtin_bit_cast(u16x2_t, at0 | (at1 << 16))));
  };
  // Boolean ring: fast blocks collect the latest hits of up to 32 tiles in bit slices: bit i of `seen` says that one found key i
  // important, bit i of slice k is bit k of the latest such tile's number in the run.  A block adds its tiles together, 10
  // instructions for four tiles of the lane's 16 keys (a history per key: 64).  After 32 tiles, or where their run ends, they join the above.
  constexpr bool HIST = MODE == SEED_BITS;
  constexpr int SLICES = 5;
  uint32_t seen_run = 0u, slice[SLICES] = {};
  int run_n = 0, run_tt = 0;   // tiles in the run, its first
  auto settle = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4 * T; i += 2) {
      uint32_t at[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        int k = 0;
#pragma unroll
        for (int b = 0; b < SLICES; ++b) k |= (int)((slice[b] >> (i + x)) & 1u) << b;
        at[x] = (seen_run >> (i + x)) & 1u ? (uint32_t)((run_tt + k) >> lgG) + 1u : 0u;
      }
      raise(i >> 1, at[0], at[1]);   // (a general block after the run may have found a later one)
    }
    seen_run = 0u;
    run_n = 0;
  };

  auto stage = [&](int blk, const u32x4_t (&qr)[QLOADS], const float4& str) __attribute__((always_inline)) {
    const int buf = blk & 1;
#pragma unroll
    for (int i = 0; i < QLOADS; ++i) {
      const int o = (i * WG + tid) * 16;   // row o / ROWB, column o % ROWB
      *reinterpret_cast<u32x4_t*>(&sh_q[buf][(o / ROWB) * QROW + (o % ROWB)]) = qr[i];
    }
    sh_st[blk % STB][tid % QBLK] = str;
  };
  if (blk_beg < blk_end) {
    fetch(blk_beg, qr, str);
    stage(blk_beg, qr, str);
    __syncthreads();
  }
  // Fast blocks (uniform over the wave): every query of the block exists and sees every key of the wave, and whole pieces can be
  // stored: straight-line code, the next tile's MFMAs under this tile's tail.  They follow one another; with FAR, but for a block
  // whose rows go on at the ring's start, and with a bf16 ring, but for a block with a marked row (prefill_query_stats).
  // (Asked once the block is staged.)
  const int fast_beg = !rows_ok || pos_wmax == NEVER || (FAR && 16 * row_bytes64 > DEAD_OFFSET)
                           ? blk_end
                           : ((((max(pos_wmax - tau0 + 1, 0) + 15) / 16) << lgG) + QT - 1) / QT;
  const int fast_end = min(blk_end, ((a.m / 16) << lgG) / QT);
  auto is_fast = [&](int blk) __attribute__((always_inline)) {
    const int tt0 = blk * QT;
    return blk >= fast_beg && blk < fast_end &&
           (!FAR || slot_of((tt0 >> lgG) * 16) <= slot_of(((tt0 + QT - 1) >> lgG) * 16 + 15)) &&
           (!TURN || !__any(__float_as_int(sh_st[blk % STB][lane % QBLK].y) < 0));
  };
  uint64_t x_ring[QT];    // of tile x of a block, see fetch: bytes of ring from the block's first head (FAR: and row)
  uint32_t x_row[QT];
#pragma unroll
  for (int x = 0; x < QT; ++x) {
    x_row[x] = (uint32_t)(x >> lgG) * 16u * row_bytes;
    x_ring[x] = (uint64_t)(x & (G - 1)) * head_bytes + (FAR ? (uint64_t)(x >> lgG) * 16u * row_bytes64 : 0);
  }
  // A pipeline over the tiles, across blocks: under the tail of a tile run the next one's products (dn), whose queries were
  // read under the tail before (qn).  So the next block is staged, and the barrier passed, in front of the last but one tile.
  auto fast_block = [&](int blk, f32x4_t (&dn)[T], uint4 (&qn)[NCH]) __attribute__((always_inline)) {
    const int cur = blk & 1, tt0 = blk * QT, jt0 = tt0 >> lgG;
    const uint32_t slot0 = slot_of(jt0 * 16);
    const uint64_t ring_blk = ring0 + (uint64_t)(tt0 & (G - 1)) * head_bytes + (FAR ? slot0 * row_bytes64 : 0);
    // Ring offsets of tile x: the lane's row of the 16 and the column in it are in `lane_off`.  (One head's ring: where the rows
    // reach beyond its end, they go on at its start.  Unsigned: the lower of the two is the one inside.)
    const uint32_t first_blk = slot0 * row_bytes;
    auto tile_off = [&](int x, uint32_t lane_off) __attribute__((always_inline)) -> uint32_t {
      if (FAR) return lane_off;
      const uint32_t first = first_blk + x_row[x];
      return min(lane_off + first, lane_off + (first - (uint32_t)head_bytes));
    };
    uint32_t hits[QT];   // boolean ring: bit i, the tile's query found key i of the lane important
#pragma unroll
    for (int ti = 0; ti < QT; ++ti) {
      f32x4_t d[T];
#pragma unroll
      for (int tl = 0; tl < T; ++tl) d[tl] = dn[tl];
      const int jt = jt0 + (ti >> lgG);
      const float4 st = sh_st[blk % STB][ti * 16 + n];
      if (ti == QT - 2) {
        stage(blk + 1, qr, str);
        __syncthreads();
      }
      if (ti + 1 < QT || blk + 1 < fast_end) mma(qn, dn);   // (uniform)
      if (ti + 2 < QT) read_tile(cur, ti + 2, qn);
      else read_tile(cur ^ 1, ti + 2 - QT, qn);
      const __amdgpu_buffer_rsrc_t rr = make_rsrc(reinterpret_cast<const char*>(ring_blk + x_ring[ti]), ring_len);
      if (MODE == SEED_BITS) {
        uint32_t hbits = 0u;
        float near = __builtin_inff();
#pragma unroll
        for (int i = 4 * T - 1; i >= 0; i -= 2) {   // key i of the lane's run: row i % 4 of key tile i / 4
          const float x1 = st.z - d[i >> 2][i & 3], x0 = st.z - d[(i - 1) >> 2][(i - 1) & 3];
          hbits = shift_in_sign(shift_in_sign(hbits, x1), x0);
          near = least_abs(near, x1, x0);
        }
        if (__any(near <= st.w)) {   // (uniform, rare) what lies in the band is decided by the score
          const float thr = importance_threshold(a.thr_scale, tau0 + jt * 16 + n);
          hbits = 0u;
#pragma unroll 1
          for (int tl = 0; tl < T; ++tl) {
            const f32x4_t x = tl == 0 ? d[0] : tl == 1 ? d[1] : tl == 2 ? d[T > 2 ? 2 : 0] : d[T > 2 ? 3 : 0];
#pragma unroll
            for (int r = 0; r < 4; ++r)
              hbits |= (prefill_score(x[r], a.scale_log2, st.x, st.y) >= thr ? 1u : 0u) << (4 * tl + r);
          }
        }
        hits[ti] = hbits;
        // the wave owns whole words of every query's row: plain stores
        if (T == 4) {   // 16 keys per lane: two lane groups to a word
          const auto sw = __builtin_amdgcn_permlane16_swap(hbits, hbits, false, false);
          const uint32_t at = tile_off(ti, n * row_bytes + (uint32_t)(pos_w0 >> 5) * 4 + (lg >> 1) * 4);
          __builtin_amdgcn_raw_buffer_store_b32(sw[0] | (sw[1] << 16), rr, (lg & 1) ? DEAD_OFFSET : at, 0, 0);
        } else {        // 8 keys per lane: four lane groups to a word
          const uint32_t w = rows_allreduce_or(hbits << (8 * lg));
          const uint32_t at = tile_off(ti, n * row_bytes + (uint32_t)(pos_w0 >> 5) * 4);
          __builtin_amdgcn_raw_buffer_store_b32(w, rr, lg ? DEAD_OFFSET : at, 0, 0);
        }
      } else {
        float pv[T][4];
#pragma unroll
        for (int tl = 0; tl < T; ++tl)
#pragma unroll
          for (int r = 0; r < 4; ++r) pv[tl][r] = prefill_score(d[tl][r], a.scale_log2, st.x, st.y);
        if (MODE == SEED_F32) {
          const int tau = tau0 + jt * 16 + n;
#pragma unroll
          for (int tl = 0; tl < T; ++tl)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              hm[PACKED ? 0 : tl][r] = pv[tl][r] >= st.z ? tau : hm[PACKED ? 0 : tl][r];
              // (said to be read here: left alone, the compiler keeps the compares of all tiles of the block in
              // scalar registers, spills those, and selects at the end)
              asm volatile("" : "+v"(hm[PACKED ? 0 : tl][r]));
            }
          const uint32_t at = tile_off(ti, n * row_bytes + (uint32_t)(pos_w0 + 4 * lg) * 4);
#pragma unroll
          for (int tl = 0; tl < T; ++tl) {
            const u32x4_t v = {__float_as_uint(pv[tl][0]), __float_as_uint(pv[tl][1]), __float_as_uint(pv[tl][2]),
                               __float_as_uint(pv[tl][3])};
            __builtin_amdgcn_raw_buffer_store_b128(v, rr, at + tl * 64, 0, 0);
          }
        } else {
          constexpr int PIECES = WKEYS / 8;        // 16-byte pieces of a query's row
          constexpr int RPS = 64 / PIECES;         // rows per store of the wave
          uint32_t pk[2 * T];
#pragma unroll
          for (int i = 0; i < 2 * T; ++i) {
            pk[i] = pack_bf16x2(pv[i >> 1][2 * (i & 1)], pv[i >> 1][2 * (i & 1) + 1]);
            hm2[PACKED ? i : 0] = bit_select(above16x2(pk[i], __float_as_uint(st.w)), (uint32_t)(jt + 1) * 0x10001u,
                                             hm2[PACKED ? i : 0]);
          }
#pragma unroll
          for (int h = 0; h < T / 2; ++h)
            *reinterpret_cast<uint4*>(&sh_t[wv][n][lg * (4 * T) + h * 8]) =
                make_uint4(pk[4 * h], pk[4 * h + 1], pk[4 * h + 2], pk[4 * h + 3]);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS is in order within a wave
#pragma unroll
          for (int h = 0; h < 16 / RPS; ++h) {
            const int qi = h * RPS + lane / PIECES, ch = lane % PIECES;
            const u32x4_t v = *reinterpret_cast<const u32x4_t*>(&sh_t[wv][qi][ch * 8]);
            __builtin_amdgcn_raw_buffer_store_b128(v, rr, tile_off(ti, qi * row_bytes + (uint32_t)(pos_w0 + ch * 8) * 2), 0, 2);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
      }
    }
    if (HIST) {
      if (run_n + QT > 32 || (run_n && run_tt + run_n != tt0)) settle();
      if (!run_n) run_tt = tt0;
      constexpr int LOW = QT == 4 ? 2 : 1;
      static_assert(QT == 2 || QT == 4, "the latest hit of a block's tiles");
      uint32_t low[2], any = hits[0] | hits[1];
      low[0] = QT == 4 ? hits[QT - 1] | (hits[1] & ~hits[QT - 2]) : hits[1];
      low[1] = QT == 4 ? hits[QT - 2] | hits[QT - 1] : 0u;
      if (QT == 4) any |= low[1];
#pragma unroll
      for (int b = 0; b < SLICES; ++b)
        slice[b] = bit_select(any, b < LOW ? low[b & 1] : (run_n >> b) & 1 ? ~0u : 0u, slice[b]);
      seen_run |= any;
      run_n += QT;
    }
  };
  // the general block: queries that see a part of the keys, units with holes, the ends of tails and units
  auto general_block = [&](int blk, int tt0) __attribute__((always_inline)) {
#pragma unroll 1
    for (int ti = 0; ti < QT; ++ti) {
      const int tt = tt0 + ti, jt = tt >> lgG, g = tt & (G - 1);
      if (tt >= ntt || jt < jt_wave || wkey0 >= L) continue;   // (uniform) past the end / no key to be seen
      f32x4_t d[T];
      mma_tile(blk & 1, ti, d);
      const int j = jt * 16 + n;                 // this lane's query
      const int tau = tau0 + j;
      const int vis = j < a.m ? tau - 1 : -1;    // the query sees positions <= vis
      int kp[T][4];                              // positions of this lane's keys
      uint32_t seen = 0u;
#pragma unroll
      for (int tl = 0; tl < T; ++tl) {
        const int4 v = *reinterpret_cast<const int4*>(
            &sh_pos[wv * WKEYS + (RUN ? lg * (4 * T) + tl * 4 : tl * 16 + 4 * lg)]);
        kp[tl][0] = v.x; kp[tl][1] = v.y; kp[tl][2] = v.z; kp[tl][3] = v.w;
#pragma unroll
        for (int r = 0; r < 4; ++r) seen |= (kp[tl][r] <= vis ? 1u : 0u) << (4 * tl + r);
      }
      const float4 st = sh_st[blk % STB][ti * 16 + n];
      const float thr = MODE == SEED_BITS ? importance_threshold(a.thr_scale, tau) : st.z;
      float pv[T][4];
      uint32_t hbits = 0u;
#pragma unroll
      for (int tl = 0; tl < T; ++tl)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool s = (seen >> (4 * tl + r)) & 1u;
          const float e = prefill_score(d[tl][r], a.scale_log2, st.x, st.y);
          pv[tl][r] = s ? e : 0.f;
          const bool hit = s && e >= thr;
          if (PACKED) {
            if (hit) hit_at(4 * tl + r, jt);
          } else {
            hm[PACKED ? 0 : tl][r] = hit ? tau : hm[PACKED ? 0 : tl][r];
          }
          hbits |= (hit ? 1u : 0u) << (4 * tl + r);
        }
      if (!a.ring) continue;   // summary-only state: nothing is recorded but last_hit
      const size_t row = ring_row(g, min(j, a.m - 1));   // (no lane stores for a query past the last)
      if (MODE == SEED_BITS) {
        uint32_t* roww = reinterpret_cast<uint32_t*>(a.ring) + row * a.ring_words;
        if (rows_ok) {        // (uniform) whole words
          if (T == 4) {
            const auto sw = __builtin_amdgcn_permlane16_swap(hbits, hbits, false, false);
            if (!(lg & 1) && j < a.m) roww[(pos_w0 >> 5) + (lg >> 1)] = sw[0] | (sw[1] << 16);
          } else {
            const uint32_t w = rows_allreduce_or(hbits << (8 * lg));
            if (lg == 0 && j < a.m) roww[pos_w0 >> 5] = w;
          }
        } else {              // rows were cleared by the launch before: set single bits
#pragma unroll
          for (int tl = 0; tl < T; ++tl)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if ((hbits >> (4 * tl + r)) & 1u) atomicOr(&roww[kp[tl][r] >> 5], 1u << (kp[tl][r] & 31));
        }
      } else {
#pragma unroll
        for (int tl = 0; tl < T; ++tl) {
          // four consecutive positions, all seen, whole and aligned: one store
          const bool quad = ((seen >> (4 * tl)) & 15u) == 15u && kp[tl][1] == kp[tl][0] + 1 &&
                            kp[tl][2] == kp[tl][0] + 2 && kp[tl][3] == kp[tl][0] + 3 &&
                            ((row * a.Tcap + (size_t)kp[tl][0]) & 3) == 0;
          if (MODE == SEED_BF16) {
            uint16_t* dst = reinterpret_cast<uint16_t*>(a.ring) + row * a.Tcap;
            const uint32_t p0 = pack_bf16x2(pv[tl][0], pv[tl][1]), p1 = pack_bf16x2(pv[tl][2], pv[tl][3]);
            if (quad) {
              *reinterpret_cast<uint2*>(dst + kp[tl][0]) = make_uint2(p0, p1);
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if ((seen >> (4 * tl + r)) & 1u)
                  dst[kp[tl][r]] = (uint16_t)((r & 2 ? p1 : p0) >> (16 * (r & 1)));
            }
          } else {
            float* dst = reinterpret_cast<float*>(a.ring) + row * a.Tcap;
            if (quad) {
              *reinterpret_cast<float4*>(dst + kp[tl][0]) = make_float4(pv[tl][0], pv[tl][1], pv[tl][2], pv[tl][3]);
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if ((seen >> (4 * tl + r)) & 1u) dst[kp[tl][r]] = pv[tl][r];
            }
          }
        }
      }
    }
  };
  // Every wave passes the barrier of every block, whichever of the two loops it is in: behind it the next block is staged, and
  // nobody reads this one any more.  (Loops of their own: where the two kinds of block share one, the compiler takes a block's loads
  // for unfinished on some way round it and waits for everything, the ring stores of the block before included, at its top.)
  for (int blk = blk_beg; blk < blk_end;) {
    for (; blk < blk_end && !is_fast(blk); ++blk) {
      fetch(min(blk + 1, blk_end - 1), qr, str);
      general_block(blk, blk * QT);
      stage(blk + 1, qr, str);
      __syncthreads();
    }
    if (blk >= blk_end) break;
    f32x4_t dn[T];
    uint4 qn[NCH];
    mma_tile(blk & 1, 0, dn);
    read_tile(blk & 1, 1, qn);
    for (; blk < blk_end && is_fast(blk); ++blk) {
      fetch(min(blk + 1, blk_end - 1), qr, str);
      fast_block(blk, dn, qn);
    }
  }

  if (HIST) settle();
  // the latest hit of every key over the 16 queries of a tile, one key per lane (through LDS: a lane's 4*T keys
  // read and written one after the other cost as many memory latencies)
  __syncthreads();   // sh_pos of this wave is free
#pragma unroll
  for (int tl = 0; tl < T; ++tl) {
    int last[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = (int)((hm2[PACKED ? 2 * tl + (r >> 1) : 0] >> (16 * (r & 1))) & 0xffffu);
      int v = PACKED ? (k ? tau0 + (k - 1) * 16 + n : 0) : hm[PACKED ? 0 : tl][r];
      v = max(v, __shfl_xor(v, 1));
      v = max(v, __shfl_xor(v, 2));
      v = max(v, __shfl_xor(v, 4));
      last[r] = max(v, __shfl_xor(v, 8));
    }
    if (n == 0)
      *reinterpret_cast<int4*>(&sh_pos[wv * WKEYS + (RUN ? lg * (4 * T) + tl * 4 : tl * 16 + 4 * lg)]) =
          make_int4(last[0], last[1], last[2], last[3]);
  }
  __syncthreads();
  const int key = wkey0 + lane;
  if (lane < WKEYS && key < L) {
    int32_t* lh = a.last_hit + (size_t)unit * a.Lcap + key;
    const int v = sh_pos[wv * WKEYS + lane];
    if (v > *lh) {
      if (a.nseg == 1) *lh = v;
      else atomicMax(lh, v);
    }
  }
}

// Pass 2 on 256-byte rows takes the registers of two waves per SIMD (held to three it spills: 1.27 -> 1.76 ms); fp32 rows of
// 512 bytes, two key tiles per wave, fit three.  Per tile of 16 queries x 64 keys, 16 MFMAs: bf16 scores 74 other vector instructions
// (102 with both kinds of block in one loop), bits 46 (111), and 29 or 25 scalar ones (36 and 26).  One loop | two, us, this kernel traced and the whole
// call: 512 heads x 1024 queries x 4096 keys, bf16 ring 1264 | 1177 and 1858 | 1776 (calls in a row by themselves 1877 | 1792, without a ring 1453 | 1341);
// 512 x 1024 x 8192 with the boolean ring 1628 | 1173 and 2677 | 2234.  Calls of 18 to 45 us, of a block or a few per wave, take 0 to 1 us longer.  What still
// bounds it: with bf16 scores the 3.76 GB of ring, which 450 us of the 640 to 750 they take alone do not hide behind the rest; else products, scalar and
// vector issue of two waves that share a SIMD (products and LDS reads alone: 10.8 ns an MFMA on every SIMD, as it is 19).
template <typename DT, int D, int MODE, bool FAR>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2, 3))) void corm_prefill_scores_kernel(
    const PrefillArgs a) {
  prefill_scores<DT, D, MODE, FAR>(a);
}

// boolean message: zero the words of the rows of steps tau_0 .. tau_{m-1} that pass 2 may set single bits in
// (positions < tau); workgroup = 16 rows of one head.  Words that pass 2 stores whole are left to it: slot and position
// agree over the 64 slots that hold the word and its neighbour (positions ascend, so the first and the last tell), all
// of them have a column, and every query whose step lies behind the word's first position sees a key there.  A prompt without holes leaves
// next to nothing to clear: 512 heads x 1024 rows x 8192 positions 132 -> 37 us.
__global__ __launch_bounds__(256) void corm_prefill_clear_bits_kernel(const PrefillArgs a) {
  const int head = blockIdx.x;   // (heads in x: B * Hq may exceed the 65535 rows a grid has in y)
  const int b = head / a.Hq;
  const int tcur = a.t[b];
  const int tau0 = tcur - a.m + 1;
  if (tau0 < 1 || tcur > a.Tcap) return;
  const int unit = b * a.Hkv + (head - b * a.Hq) / (a.Hq / a.Hkv);
  int L = a.lens[unit];
  L = L < 0 ? 0 : (L > a.Lcap ? a.Lcap : L);
  const int32_t* posb = a.pos + (size_t)unit * a.Lcap;
  const int s0 = (tau0 - 1) % a.w;
  const int j0 = blockIdx.y * 16, j1 = min(j0 + 16, a.m);
  const int nw_max = min((tau0 + j1 - 1 + 31) >> 5, a.ring_words);
  for (int i = threadIdx.x; i < nw_max; i += 256) {
    const int k0 = (i >> 1) * 64;
    if (k0 + 64 <= min(L, a.Tcap) && posb[k0] == k0 && posb[k0 + 63] == k0 + 63) continue;
    for (int j = j0; j < j1; ++j) {
      int slot = s0 + j;
      if (slot >= a.w) slot -= a.w;
      if (i < (tau0 + j + 31) >> 5)
        reinterpret_cast<uint32_t*>(a.ring)[((size_t)head * a.w + slot) * a.ring_words + i] = 0u;
    }
  }
}

// per query: reference (the largest of them) and 1/sum over the key segments of its unit
__global__ __launch_bounds__(256) void corm_prefill_merge_kernel(const PrefillArgs a) {
  const int head = blockIdx.x;   // (heads in x: B * Hq may exceed the 65535 rows a grid has in y)
  const int j = blockIdx.y * 256 + threadIdx.x;
  if (j >= a.m) return;
  const int unit = (head / a.Hq) * a.Hkv + (head % a.Hq) / (a.Hq / a.Hkv);
  int L = a.lens[unit];
  L = L < 0 ? 0 : (L > a.Lcap ? a.Lcap : L);
  const int nblk = (L + a.kseg - 1) / a.kseg;
  const float2* part = a.part + (size_t)head * a.nkb * a.w + j;
  float mx = neg_inf();
  for (int k = 0; k < nblk; ++k) mx = fmaxf(mx, part[(size_t)k * a.w].x);
  const float ms = mx == neg_inf() ? 0.f : mx;
  float z = 0.f;
  for (int k = 0; k < nblk; ++k) {
    const float2 pk = part[(size_t)k * a.w];
    z = fmaf(pk.y, exp2f(pk.x - ms), z);
  }
  const int tau = a.t[head / a.Hq] - a.m + 1 + j;
  a.stats[(size_t)head * a.w + j] =
      prefill_query_stats(a, ms, z, importance_threshold(a.thr_scale, tau >= 1 ? tau : 1));
}

// Def. 4.1 + recent r from last_hit for whole units (no append): wave ballots and survivors per chunk
// for the compaction, optionally one byte per slot; writes t_first.
__global__ __launch_bounds__(WG) void corm_decide_kernel(const int32_t* lens, const int32_t* last_hit, const int32_t* t,
                                                         int32_t* t_first, unsigned long long* keepbits,
                                                         int32_t* counts, int2* unit_state, uint8_t* keep, int Hkv,
                                                         int Lcap, int nsplit, int kb_stride, int w, int r, int m) {
  __shared__ int sh_cnt[WAVES];
  const int split = blockIdx.x, unit = blockIdx.y;
  const int b = unit / Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int tcur = t[b];
  if (split == 0 && unit % Hkv == 0 && tid == 0) t_first[b] = tcur - m + 1;
  int L = lens[unit];
  L = L < 0 ? 0 : (L > Lcap ? Lcap : L);
  if (split == 0 && tid == 0) unit_state[unit] = make_int2(L, SUM_COUNTS);
  const int cbeg = split * CHUNK;
  if (cbeg >= L) return;
  const int cend = min(cbeg + CHUNK, L);
  const bool full = m >= w;
  const int32_t* lhb = last_hit + (size_t)unit * Lcap;
  unsigned long long* bitsb = keepbits + (size_t)unit * kb_stride;
  int kept = 0;
  for (int i0 = cbeg; i0 < cbeg + CHUNK; i0 += WG) {
    const int i = i0 + tid;
    bool k = false;
    if (i < cend) {
      k = !full || lhb[i] > tcur - w || i >= L - r;
      if (keep) keep[(size_t)unit * Lcap + i] = k ? 1 : 0;
    }
    const unsigned long long bal = __ballot(k);
    if (lane == 0 && i0 + wv * 64 < cend) bitsb[(i0 >> 6) + wv] = bal;
    kept += __popcll(bal);
  }
  if (lane == 0) sh_cnt[wv] = kept;
  __syncthreads();
  if (tid == 0) {
    int tot = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) tot += sh_cnt[i];
    counts[(size_t)unit * nsplit + split] = tot;
  }
}

}  // namespace

#endif  // CORM_PREFILL_HPP
