// a whole decode step of small units in one launch: append, attend, record, decide and compact by one workgroup per unit.
// Part of one translation unit: included by corm_kernels.hip, in this order, after <hip/hip_runtime.h> and corm.h.
#ifndef CORM_SMALL_HPP
#define CORM_SMALL_HPP

namespace {

// ---------------------------------------------------------------- small units: one launch
//
// A few units of a few hundred slots leave nothing to share out: what a step costs is its launches and, in each, a chain of
// memory latencies (lengths, then rows or partials, then masks, then rows again).  Here a workgroup does the whole step of
// a unit: the logits stay in LDS as in the unit kernel, the new row is attended to from k_new and v_new directly (nothing is
// written to be read back), pos and last_hit are read once and stored once, at the slot the key ends in, and the
// survivors' list never leaves LDS.  Bound by that chain, and with hundreds of rows by what one workgroup streams: 4 units of 52 keys
// that evict at every step (fp32, d 64) 4.1 + 4.8 + 2.1 us in three launches, 6.9 in one with the inputs in the caches; with new
// inputs at every step 4.4 + 5.2 + 5.0 and 11.0 (a step of the program 13.8 -> 11.4).  small_step says where that pays.

constexpr int SMALL_WG = 512;
constexpr int SMALL_WAVES = SMALL_WG / 64;
constexpr int SMALL_TILES = 2;                           // slots per thread
constexpr int SMALL_MAX_SLOTS = SMALL_TILES * SMALL_WG;

// LDS for logits: whole stage pairs, and the stage of the new row behind the last slot
template <typename DT, int D, int G>
constexpr int small_stage_rows() { return SMALL_WAVES * (64 / (D * DT::ESZ / 16)) * (G == 1 ? UNROLL : UNROLL / 2); }

template <typename DT, int D, int G>
__global__ __launch_bounds__(SMALL_WG) void corm_small_kernel(const Params p, const int lstride) {
  using A = Attend<DT, D, G, SMALL_WAVES, (G == 1 ? UNROLL : UNROLL / 2)>;
  constexpr int EPL = A::EPL, ROWB = A::ROWB, LPR = A::LPR, RPL = A::RPL;
  static_assert(A::STAGE_ROWS == small_stage_rows<DT, D, G>(), "the host sizes the LDS by it");

  extern __shared__ float sh_logit[];   // [G][lstride] raw logits of the unit (log2 domain)
  __shared__ float sh_m[G][SMALL_WAVES];
  __shared__ float sh_z[G][SMALL_WAVES];
  __shared__ float sh_acc[G][SMALL_WAVES][D];
  __shared__ float sh_M[G], sh_Z[G];
  __shared__ unsigned long long sh_keep[SMALL_TILES * SMALL_WAVES];   // ballots, 64 slots each
  __shared__ uint16_t sh_src[SMALL_MAX_SLOTS];                        // old slots of the survivors

  const int unit = blockIdx.x;
  const int b = unit / p.Hkv, hkv = unit - b * p.Hkv, hq0 = hkv * G;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int sub = lane / LPR, cl = lane % LPR;
  const int lane_row = wv * RPL + sub;

  // everything that does not hang on the unit's length is requested with it
  const int lens_value = p.lens[unit], tcur = p.t[b], tfirst = p.t_first[b];
  uint4 qreg[G];
#pragma unroll
  for (int g = 0; g < G; ++g)
    qreg[g] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(p.q) +
                                              ((size_t)(b * p.Hq + hq0 + g) * ROWB + (size_t)cl * 16));
  const char* knew = reinterpret_cast<const char*>(p.k_new) + (size_t)unit * ROWB;
  const char* vnew = reinterpret_cast<const char*>(p.v_new) + (size_t)unit * ROWB;
  typename A::Stage sn;   // row 0 of the workgroup: the new one; the others are out of range
  A::template load<false>(sn, make_rsrc(knew, ROWB), make_rsrc(vnew, ROWB), (uint32_t)lane_row * ROWB + (uint32_t)cl * 16,
                          nullptr, 0);

  const UnitLen ul = unit_len_of(p, __builtin_amdgcn_readfirstlane(lens_value));
  const int L0 = ul.L0, L = ul.L;
  if (tid == 0 && ul.flags && p.status) atomicOr(p.status, ul.flags);
  char* Kb = reinterpret_cast<char*>(p.K) + (size_t)unit * p.Lcap * ROWB;
  char* Vb = reinterpret_cast<char*>(p.V) + (size_t)unit * p.Lcap * ROWB;
  int32_t* posb = p.pos + (size_t)unit * p.Lcap;
  int32_t* lhb = p.last_hit + (size_t)unit * p.Lcap;

  const __amdgpu_buffer_rsrc_t rk = make_rsrc(Kb, (uint32_t)L0 * ROWB);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(Vb, (uint32_t)L0 * ROWB);
  uint32_t off = (uint32_t)lane_row * ROWB + (uint32_t)cl * 16;
  constexpr uint32_t STAGE_BYTES = (uint32_t)A::STAGE_ROWS * ROWB;
  typename A::Stage s0, s1;
  A::template load<false>(s0, rk, rv, off, nullptr, 0);
  int my_pos[SMALL_TILES], my_lh[SMALL_TILES];   // of the slots tid, tid + SMALL_WG
  const __amdgpu_buffer_rsrc_t rp = make_rsrc(posb, (uint32_t)L0 * 4), rl = make_rsrc(lhb, (uint32_t)L0 * 4);
#pragma unroll
  for (int k = 0; k < SMALL_TILES; ++k) {
    const int i = k * SMALL_WG + tid;
    my_pos[k] = __builtin_amdgcn_raw_buffer_load_b32(rp, i * 4, 0, 0);
    my_lh[k] = __builtin_amdgcn_raw_buffer_load_b32(rl, i * 4, 0, 0);
  }
  clear_bit_rows(p, b, hq0, G, SMALL_WG);   // (ordered before the record phase by the barriers of the merge)

  float m_run[G], z_run[G], acc[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m_run[g] = neg_inf();
    z_run[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
  }
  for (int it = 0; it < L0; it += 2 * A::STAGE_ROWS) {
    A::template load<false>(s1, rk, rv, off + STAGE_BYTES, nullptr, 0);
    A::compute(s0, it + lane_row, it + lane_row, L0, cl, qreg, p.scale_log2, sh_logit, lstride, m_run, z_run, acc);
    off += 2 * STAGE_BYTES;
    A::template load<false>(s0, rk, rv, off, nullptr, 0);
    A::compute(s1, it + A::STAGE_ROWS + lane_row, it + A::STAGE_ROWS + lane_row, L0, cl, qreg, p.scale_log2, sh_logit,
               lstride, m_run, z_run, acc);
  }
  __syncthreads();   // (the logits of the rows behind L0 that the last stages covered are in place)
  if (ul.appended && wv == 0) {
    A::compute(sn, L0 + lane_row, L0 + lane_row, L, cl, qreg, p.scale_log2, sh_logit, lstride, m_run, z_run, acc);
    if (sub == 0) {
      *reinterpret_cast<uint4*>(Kb + (size_t)L0 * ROWB + (size_t)cl * 16) = sn.k[0];
      *reinterpret_cast<uint4*>(Vb + (size_t)L0 * ROWB + (size_t)cl * 16) = sn.v[0];
    }
  }

  // merge the row groups of each wave (scaled once, to the wave's maximum), then the waves
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float mw = m_run[g];
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) mw = fmaxf(mw, __shfl_xor(mw, o));
    const float a = fast_exp2(m_run[g] - (mw == neg_inf() ? 0.f : mw));
    m_run[g] = mw;
    z_run[g] *= a;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] *= a;
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
      z_run[g] += __shfl_xor(z_run[g], o);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] += __shfl_xor(acc[g][e], o);
    }
    if (sub == 0) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) sh_acc[g][wv][cl * EPL + e] = acc[g][e];
      if (cl == 0) {
        sh_m[g][wv] = m_run[g];
        sh_z[g][wv] = z_run[g];
      }
    }
  }
  __syncthreads();

  // out (Eq. 1) and the unit's max / sum (Eq. 2)
  for (int idx = tid; idx < G * D; idx += SMALL_WG) {
    const int g = idx / D, c = idx - g * D;
    float mx = neg_inf();
#pragma unroll
    for (int i = 0; i < SMALL_WAVES; ++i) mx = fmaxf(mx, sh_m[g][i]);
    float zt = 0.f, at = 0.f;
#pragma unroll
    for (int i = 0; i < SMALL_WAVES; ++i) {
      const float a = fast_exp2(sh_m[g][i] - mx);
      zt = fmaf(sh_z[g][i], a, zt);
      at = fmaf(sh_acc[g][i][c], a, at);
    }
    p.out[(size_t)(b * p.Hq + hq0 + g) * D + c] = at / zt;
    if (c == 0) {
      sh_M[g] = mx;
      sh_Z[g] = zt;
    }
  }
  __syncthreads();

  // record (Def. 3.1) and decide (Def. 4.1 + recent r)
  const bool step_ok = tcur >= 1 && tcur <= p.Tcap;
  if (!step_ok && tid == 0 && p.status) atomicOr(p.status, CORM_DEV_BAD_STEP);
  const int slot = step_ok ? (tcur - 1) % p.w : 0;
  const float thr = importance_threshold(p.thr_scale, step_ok ? tcur : 1);
  const bool full = step_ok && (tcur - tfirst + 1 >= p.w);
  uint8_t* keepb = p.keep ? p.keep + (size_t)unit * p.Lcap : nullptr;
  bool kept[SMALL_TILES], changed[SMALL_TILES];   // changed: what the slot holds is not what is stored there
#pragma unroll
  for (int k = 0; k < SMALL_TILES; ++k) {
    const int i = k * SMALL_WG + tid;
    const bool live = i < L;
    changed[k] = ul.appended && i == L0;
    if (changed[k]) {
      my_pos[k] = tcur - 1;
      my_lh[k] = 0;
    }
    const bool pos_ok = live && my_pos[k] >= 0 && my_pos[k] < p.Tcap;
    if (live && !pos_ok && p.status) atomicOr(p.status, CORM_DEV_BAD_STEP);
    bool hit = false;
    const BitRun run = bit_run(my_pos[k], pos_ok);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float sc = live ? exp2f(sh_logit[g * lstride + i] - sh_M[g]) / sh_Z[g] : 0.f;
      float stored = sc;
      const size_t row = (size_t)(b * p.Hq + hq0 + g) * p.w + slot;
      if (p.ring_bf16) {
        const uint16_t hb = f32_to_bf16_rne(sc);
        stored = __uint_as_float((uint32_t)hb << 16);
        if (step_ok && pos_ok && p.ring) reinterpret_cast<uint16_t*>(p.ring)[row * p.Tcap + (size_t)my_pos[k]] = hb;
      } else if (!p.ring_bits) {
        if (step_ok && pos_ok && p.ring) reinterpret_cast<float*>(p.ring)[row * p.Tcap + (size_t)my_pos[k]] = sc;
      }
      const bool hg = live && stored >= thr;
      hit |= hg;
      if (p.ring_bits && p.ring && step_ok)   // (uniform)
        record_bits(reinterpret_cast<uint32_t*>(p.ring) + row * p.ring_words, p.ring_words, run, my_pos[k], hg && pos_ok);
    }
    if (hit && step_ok) {
      my_lh[k] = tcur;
      changed[k] = true;
    }
    kept[k] = live && (!full || (my_lh[k] > tcur - p.w) || (i >= L - p.r));
    if (keepb && live) keepb[i] = kept[k] ? 1 : 0;
    const unsigned long long bal = __ballot(kept[k]);
    if (lane == 0) sh_keep[k * SMALL_WAVES + wv] = bal;
  }
  __syncthreads();

  // survivors: rank of this thread's keys, the list of old slots; pos and last_hit go where they end
  int T = 0, fixed = L;   // survivors; survivors in front of the first hole
  int before[SMALL_TILES];
#pragma unroll
  for (int w = 0; w < SMALL_TILES * SMALL_WAVES; ++w) {
    const unsigned long long word = sh_keep[w];
    if (w % SMALL_WAVES == wv) before[w / SMALL_WAVES] = T;
    T += __popcll(word);
    if (~word != 0ull) fixed = min(fixed, w * 64 + __ffsll((long long)~word) - 1);
  }
  int32_t* idxb = p.kept_idx ? p.kept_idx + (size_t)unit * p.Lcap : nullptr;
#pragma unroll
  for (int k = 0; k < SMALL_TILES; ++k) {
    const int i = k * SMALL_WG + tid;
    const int rank = before[k] + __popcll(sh_keep[k * SMALL_WAVES + wv] & ((1ull << lane) - 1ull));
    int at = -1;   // a survivor's slot is its rank; a slot behind the last survivor keeps its own
    if (kept[k]) {
      sh_src[rank] = (uint16_t)i;
      if (idxb) idxb[rank] = i;
      if (rank != i || changed[k]) at = rank;
    }
    if (at >= 0) {
      posb[at] = my_pos[k];
      lhb[at] = my_lh[k];
    }
    if (changed[k] && i >= T) {
      posb[i] = my_pos[k];
      lhb[i] = my_lh[k];
    }
  }
  if (tid == 0) p.lens[unit] = T;
  if (T == L) return;   // (uniform) nothing went
  __syncthreads();      // the list, and the new row in its slot

  // ascending batches: sources lie behind every destination of the batches before; a batch is stored when all of its
  // loads, of every wave, are in
  constexpr int RPP = SMALL_WG / LPR;   // rows per pass
  constexpr int NP = 4;                 // passes in flight together
  const int mrow = tid / LPR;
  const size_t col = (size_t)(tid % LPR) * 16;
  const int n = T - fixed;
  for (int j0 = 0; j0 < n; j0 += RPP * NP) {
    u32x4_t kr[NP], vr[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {   // (clamped: every load reads a valid row)
      const size_t o = (size_t)sh_src[fixed + min(j0 + u * RPP + mrow, n - 1)] * ROWB + col;
      kr[u] = *reinterpret_cast<const u32x4_t*>(Kb + o);
      vr[u] = *reinterpret_cast<const u32x4_t*>(Vb + o);
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) asm volatile("" ::"v"(kr[u]), "v"(vr[u]));
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int j = j0 + u * RPP + mrow;
      if (j < n) {
        const size_t o = (size_t)(fixed + j) * ROWB + col;
        *reinterpret_cast<u32x4_t*>(Kb + o) = kr[u];
        *reinterpret_cast<u32x4_t*>(Vb + o) = vr[u];
      }
    }
  }
}

}  // namespace

#endif  // CORM_SMALL_HPP
