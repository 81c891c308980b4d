// split path, second launch: merge of the partials, record and decide.
// Part of one translation unit: included by corm_kernels.hip, in this order, after <hip/hip_runtime.h> and corm.h.
#ifndef CORM_RECORD_HPP
#define CORM_RECORD_HPP

namespace {

// ---------------------------------------------------------------- record (+ keep flags)

// RECORD_CHUNKS: 512-slot chunks per workgroup (more keys per workgroup amortize its fixed chain of
// dependent loads; fewer keep the chip full when the launch has few units).  NT: threads.  A workgroup of one chunk has a thread per key: such
// launches leave the chip mostly idle, and a thread's G scores per key run one after the other (9 units x 600 of 1600 slots, eight heads, 256
// threads 9.4 us, 512 6.4; 16 units x 2600, two heads 5.1, 4.4; 32 units x 4200, one head: equal).
constexpr int OUT_WAVE_PARTS = 16;   // up to here one wave folds the partial rows of an item alone
constexpr int OUT_BATCH = 8;         // of them in flight together

// Global max and sum of Eq. 2 of a head, by one wave, from its split partials; the first 64 stay in registers between the
// max and the sum.  (The same bits in every lane.)
__device__ __forceinline__ float2 head_stats(const float* part0, int pstride, int nparts) {
  const int lane = threadIdx.x & 63;
  float2 first = make_float2(neg_inf(), 0.f);
  if (lane < nparts) first = *reinterpret_cast<const float2*>(part0 + (size_t)lane * pstride);
  float mx = first.x;
  for (int s = lane + 64; s < nparts; s += 64) mx = fmaxf(mx, part0[(size_t)s * pstride]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  const float ms = mx == neg_inf() ? 0.f : mx;
  float zt = first.y * exp2f(first.x - ms);
  for (int s = lane + 64; s < nparts; s += 64) {
    const float* ps = part0 + (size_t)s * pstride;
    zt = fmaf(ps[1], exp2f(ps[0] - ms), zt);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) zt += __shfl_xor(zt, off);
  return make_float2(ms, zt);
}

// out (Eq. 1) of a unit, by the n_out workgroups that share it; stats(g, part0, nparts): global max and sum of a head.
// (head, block of 64 columns) items are dealt to them; lane = column, so every split's
// partial row is read as one contiguous 256-byte piece and the loads of all splits are independent (no cross-lane
// reduction, one memory latency per item).  Few splits: an item belongs to one wave,
// the rows in whole batches (a remainder loop is a chain of latencies: 16 units of up to 15 splits 5.7 us, in batches 4.7, as by
// the other way).  Many splits: to one workgroup, whose waves take the splits round-robin and meet in LDS.
template <int G, int NT, typename Stats>
__device__ __forceinline__ void record_out(const Params& p, int unit, int L, int nparts, int D, int wg, int n_out,
                                           const Stats& stats) {
  __shared__ float sh_out[WAVES][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int b = unit / p.Hkv, hq0 = (unit - b * p.Hkv) * G;
  const int pstride = D + 2, cblocks = D / 64;
  const float* part_u = p.partials + (size_t)(b * p.Hq + hq0) * p.npart * pstride;
  float* out_u = p.out + (size_t)(b * p.Hq + hq0) * D;
  if (nparts <= OUT_WAVE_PARTS) {
    for (int item = wg * (NT / 64) + wv; item < G * cblocks; item += n_out * (NT / 64)) {
      const int g = item / cblocks, c = (item - g * cblocks) * 64 + lane;
      const float* part0 = part_u + (size_t)g * p.npart * pstride;
      const float2 st = stats(g, part0, nparts);
      float at = 0.f;
      for (int s0 = 0; s0 < nparts; s0 += OUT_BATCH) {
        float m[OUT_BATCH], v[OUT_BATCH];
#pragma unroll
        for (int u = 0; u < OUT_BATCH; ++u) {
          const float* ps = part0 + (size_t)min(s0 + u, nparts - 1) * pstride;
          m[u] = ps[0];
          v[u] = ps[2 + c];
        }
#pragma unroll
        for (int u = 0; u < OUT_BATCH; ++u) at = fmaf(s0 + u < nparts ? v[u] : 0.f, exp2f(m[u] - st.x), at);
      }
      out_u[(size_t)g * D + c] = L > 0 ? at / st.y : 0.f;
    }
    return;
  }
  for (int item = wg; item < G * cblocks; item += n_out) {   // (uniform over the workgroup)
    const int g = item / cblocks, c = (item - g * cblocks) * 64 + lane;
    const float* part0 = part_u + (size_t)g * p.npart * pstride;
    const float2 st = stats(g, part0, nparts);
    if (wv < WAVES) {   // (four of them, whatever the workgroup: the order of the sums)
      float at = 0.f;
#pragma unroll 4
      for (int s = wv; s < nparts; s += WAVES) {
        const float* ps = part0 + (size_t)s * pstride;
        at = fmaf(ps[2 + c], exp2f(ps[0] - st.x), at);
      }
      sh_out[wv][lane] = at;
    }
    __syncthreads();
    if (wv == 0) {
      float tot = 0.f;
#pragma unroll
      for (int i = 0; i < WAVES; ++i) tot += sh_out[i][lane];
      out_u[(size_t)g * D + c] = L > 0 ? tot / st.y : 0.f;
    }
    __syncthreads();
  }
}

// A column of the grid is a unit, a row the same workgroup of every unit: first those that record, then (APART) n_out that do out alone.  So what
// has work comes in front of what the units leave empty and spreads over the dies, whatever the rows.  (Unit by unit, with out in front, the
// record workgroups of all units met on a few dies where a unit's workgroups were a multiple of 8, and on a full chip they waited
// for those that did out: eight heads, 193 units x 1520 of 1600 slots 19.2 us, 64 x 12000 of 32768 51.5, before out had workgroups of its own 12.4 and 37.2.
// Whole steps, us, unit by unit | row by row: 250 units x 1900 of 2048 slots, eight heads, 74.8 | 68.3; 120 x 460 of 3072 34.9 | 29.1, one head
// 16.1 | 15.9; 200 x 2457 of 16384, four heads, 182 | 155; 30 x 16000 of 16384 57.3 | 59.2, where the dies that attended to the chunks record them unit by unit.)
// Not APART: the workgroups that record share out, in front of the record, which lengthens their chain of latencies (this launch, us, so with two keys a
// thread | apart, with the threads of the host's rule: 32 units x 4200 keys 5.2 | 4.0, 16 x 2600 of two heads 5.8 | 4.1, 9 x 600 of eight 10.5 | 6.3, 128 x 33000 24.6 | 24.1).
template <int G, int RECORD_CHUNKS, int NT, bool APART>
__global__ __launch_bounds__(NT) void corm_record_kernel(const Params p, const int D, const int n_out) {
  constexpr int RECORD_ROWS = RECORD_CHUNKS * CHUNK;  // keys per workgroup
  constexpr int KPT = RECORD_ROWS / NT;  // keys per thread
  constexpr int KPC = CHUNK / NT;        // of which per chunk
  constexpr int NW = NT / 64;
  static_assert(CHUNK % NT == 0 && NT >= 64 * WAVES, "whole keys per thread and chunk; the waves of record_out");
  const int PSTRIDE = D + 2;
  const int unit = blockIdx.x;
  const UnitLen ul = unit_len(p, unit);
  const int L = ul.L;
  const int nparts = (L + p.part_keys - 1) / p.part_keys;           // attend partials that hold keys
  const int rsplit = blockIdx.y;   // this workgroup covers chunks [rsplit*RECORD_CHUNKS, +RECORD_CHUNKS)
  const int nrec = (p.nsplit + RECORD_CHUNKS - 1) / RECORD_CHUNKS;
  if (APART && rsplit >= nrec) {
    record_out<G, NT>(p, unit, L, nparts, D, rsplit - nrec, n_out,
                      [&](int, const float* part0, int nparts) { return head_stats(part0, PSTRIDE, nparts); });
    return;
  }
  const int tid = threadIdx.x;
  if (rsplit == 0 && tid == 0 && ul.flags && p.status) atomicOr(p.status, ul.flags);
  const int nlive = (L + CHUNK - 1) / CHUNK;                        // chunks that hold keys
  const int nwg = max((L + RECORD_ROWS - 1) / RECORD_ROWS, APART ? 0 : 1);   // record workgroups that have work
  if (rsplit >= nwg) return;

  const int b = unit / p.Hkv;
  const int hkv = unit - b * p.Hkv;
  const int hq0 = hkv * G;
  const int lane = tid & 63, wv = tid >> 6;
  const int rbeg = rsplit * RECORD_ROWS;
  const int rend = min(rbeg + RECORD_ROWS, L);

  __shared__ float sh_M[G], sh_Z[G];
  __shared__ int sh_cnt[RECORD_CHUNKS][NW];

  // this thread's keys: issue their loads first, they are consumed after the merge below
  const int32_t* posb = p.pos + (size_t)unit * p.Lcap;
  int32_t* lhb = p.last_hit + (size_t)unit * p.Lcap;
  const float* logit_u = p.logits + (size_t)(b * p.Hq + hq0) * p.Lcap;
  unsigned long long* bitsb = p.keepbits + (size_t)unit * p.kb_stride;
  unsigned long long* liveb = p.lazy ? p.live + (size_t)unit * p.kb_stride : nullptr;
  int my_pos[KPT], my_lh[KPT];
  bool my_live[KPT];   // lazy mode: the slot holds a key that was not evicted earlier
  float lg[KPT][G];
#pragma unroll
  for (int k = 0; k < KPT; ++k) {
    const int i = min(rbeg + k * NT + tid, max(rend - 1, 0));   // clamped: a live slot (or 0 in an empty unit)
    my_pos[k] = posb[i];
    my_lh[k] = lhb[i];
    my_live[k] = p.lazy ? ((liveb[i >> 6] >> (i & 63)) & 1ull) != 0 : true;
#pragma unroll
    for (int g = 0; g < G; ++g) lg[k][g] = logit_u[(size_t)g * p.Lcap + i];
  }
  const int tcur = p.t[b];
  const int tfirst = p.do_evict ? p.t_first[b] : tcur;

  for (int g = wv; g < G; g += NW) {   // (wave g handles head g, g + NW, ...)
    const float2 st = head_stats(p.partials + (size_t)(b * p.Hq + hq0 + g) * p.npart * PSTRIDE, PSTRIDE, nparts);
    if (lane == 0) {
      sh_M[g] = st.x;
      sh_Z[g] = st.y;
    }
  }
  __syncthreads();

  if (!APART) {
    record_out<G, NT>(p, unit, L, nparts, D, rsplit, nwg, [&](int g, const float*, int) { return make_float2(sh_M[g], sh_Z[g]); });
    if (L == 0) return;   // an empty unit: nothing to record
  }

  // record (Def. 3.1) and decide (Def. 4.1 + recent r) for the keys of this workgroup
  const bool step_ok = tcur >= 1 && tcur <= p.Tcap;
  if (!step_ok && rsplit == 0 && tid == 0 && p.status) atomicOr(p.status, CORM_DEV_BAD_STEP);
  const int slot = step_ok ? (tcur - 1) % p.w : 0;
  const float thr = importance_threshold(p.thr_scale, step_ok ? tcur : 1);
  const bool full = p.do_evict && step_ok && (tcur - tfirst + 1 >= p.w);
  uint8_t* keepb = p.keep ? p.keep + (size_t)unit * p.Lcap : nullptr;

  int kept[RECORD_CHUNKS];
#pragma unroll
  for (int c = 0; c < RECORD_CHUNKS; ++c) kept[c] = 0;
#pragma unroll
  for (int k = 0; k < KPT; ++k) {
    const int i = rbeg + k * NT + tid;
    const bool live = i < rend && my_live[k];
    bool keep = false;
    if (p.ring_bits) {   // (uniform) boolean message: compare the fp32 score, set bits wave by wave
      const bool pos_ok = live && my_pos[k] >= 0 && my_pos[k] < p.Tcap;
      if (live && !pos_ok && p.status) atomicOr(p.status, CORM_DEV_BAD_STEP);
      bool hit = false;
      const BitRun run = bit_run(my_pos[k], pos_ok);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float sc = live ? exp2f(lg[k][g] - sh_M[g]) / sh_Z[g] : 0.f;
        const bool hg = live && sc >= thr;
        hit |= hg;
        if (p.ring && step_ok)
          record_bits(reinterpret_cast<uint32_t*>(p.ring) + ((size_t)(b * p.Hq + hq0 + g) * p.w + slot) * p.ring_words,
                      p.ring_words, run, my_pos[k], hg && pos_ok);
      }
      if (live) {
        int lh = my_lh[k];
        if (hit && step_ok) {
          lh = tcur;
          lhb[i] = tcur;
        }
        const bool recent = p.lazy ? (my_pos[k] >= tcur - p.r) : (i >= L - p.r);
        keep = !full || (lh > tcur - p.w) || recent;
      }
    } else if (live) {
      const bool pos_ok = my_pos[k] >= 0 && my_pos[k] < p.Tcap;
      if (!pos_ok && p.status) atomicOr(p.status, CORM_DEV_BAD_STEP);
      bool hit = false;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float sc = exp2f(lg[k][g] - sh_M[g]) / sh_Z[g];
        float stored;
        const size_t ri = ((size_t)(b * p.Hq + hq0 + g) * p.w + slot) * p.Tcap + (size_t)my_pos[k];
        if (p.ring_bf16) {
          const uint16_t hb = f32_to_bf16_rne(sc);
          stored = __uint_as_float((uint32_t)hb << 16);
          if (step_ok && pos_ok && p.ring) reinterpret_cast<uint16_t*>(p.ring)[ri] = hb;
        } else {
          stored = sc;
          if (step_ok && pos_ok && p.ring) reinterpret_cast<float*>(p.ring)[ri] = sc;
        }
        hit |= (stored >= thr);
      }
      int lh = my_lh[k];
      if (hit && step_ok) {
        lh = tcur;
        lhb[i] = tcur;
      }
      // the r newest keys: the last r slots, or (lazy mode, where dead slots lie between) by position
      const bool recent = p.lazy ? (my_pos[k] >= tcur - p.r) : (i >= L - p.r);
      keep = !full || (lh > tcur - p.w) || recent;
    }
    if (p.do_evict && keepb && i < rend) keepb[i] = keep ? 1 : 0;
    const unsigned long long bal = __ballot(keep);
    if (p.do_evict && lane == 0 && rbeg + k * NT + wv * 64 < rend) {
      bitsb[((rbeg + k * NT) >> 6) + wv] = bal;
      if (p.lazy) liveb[((rbeg + k * NT) >> 6) + wv] = bal;
    }
    kept[k / KPC] += __popcll(bal);
  }
  if (p.do_evict) {
    if (lane == 0) {
#pragma unroll
      for (int c = 0; c < RECORD_CHUNKS; ++c) sh_cnt[c][wv] = kept[c];
    }
    __syncthreads();
    if (tid < RECORD_CHUNKS && rsplit * RECORD_CHUNKS + tid < nlive) {
      int tot = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) tot += sh_cnt[tid][i];
      const int chunk = rsplit * RECORD_CHUNKS + tid;
      p.counts[(size_t)unit * p.nsplit + chunk] = tot;
      // (a plain store: whoever lost a key stores the same)
      if (tot != min(CHUNK, L - chunk * CHUNK)) p.unit_state[unit].y = SUM_COUNTS;
    }
  }
}

}  // namespace

#endif  // CORM_RECORD_HPP
