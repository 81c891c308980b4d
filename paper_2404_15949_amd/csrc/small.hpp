// a whole decode step of small units in one launch: append, attend, record, decide and compact by one workgroup per unit.
// Part of one translation unit: included by corm_kernels.hip, in this order, after <hip/hip_runtime.h> and corm.h.
#ifndef CORM_SMALL_HPP
#define CORM_SMALL_HPP

namespace {

// ---------------------------------------------------------------- small units: one launch
//
// A few units of a few hundred slots leave nothing to share out: what a step costs is its launches and, in each, a chain of
// memory latencies (lengths, then rows or partials, then masks, then rows again).  Here a workgroup does the whole step of
// a unit: logits and partials stay in LDS, the new row is attended to from k_new and v_new directly (nothing is
// written to be read back), pos and last_hit are read once and stored once, at the slot the key ends in, and the
// survivors' list never leaves LDS.  Bound by that chain, and with hundreds of rows by what one workgroup streams: small_step says
// where that pays.
//
// The bits are those of the split launches, which the calls that do a part of a step keep to (corm_decode_attend, the two
// phases, the deferred step): the same parts of p.part_keys keys, each walked by four waves in the order of
// corm_attend_kernel and merged as there (two groups of four waves take the parts in turn), the partials folded as in
// corm_record_kernel.

constexpr int SMALL_WG = 512;
constexpr int SMALL_WAVES = SMALL_WG / 64;
constexpr int SMALL_GROUPS = SMALL_WAVES / WAVES;        // groups of waves that walk a part each
constexpr int SMALL_TILES = 2;                           // slots per thread
constexpr int SMALL_MAX_SLOTS = SMALL_TILES * SMALL_WG;
constexpr int SMALL_MAX_PARTS = SMALL_MAX_SLOTS / (CHUNK / MAX_PARTS_PER_CHUNK);

// (max, sum, products) of one column over the four waves of a part, as corm_attend_kernel merges them
struct SmallPart {
  float m, z, at;
};
__device__ __forceinline__ SmallPart small_part(const float* m, const float* z, const float* acc, int stride) {
  SmallPart r = {neg_inf(), 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < WAVES; ++i) r.m = fmaxf(r.m, m[i]);
  const float ms = r.m == neg_inf() ? 0.f : r.m;
#pragma unroll
  for (int i = 0; i < WAVES; ++i) {
    const float a = fast_exp2(m[i] - ms);
    r.z = fmaf(z[i], a, r.z);
    r.at = fmaf(acc[i * stride], a, r.at);
  }
  return r;
}

// floats of dynamic LDS: logits [G][lstride], partials of the waves: max and sum [parts][G][WAVES], products [parts][G][WAVES][D]
inline size_t small_lds_floats(int G, int D, int lstride, int parts) {
  return (size_t)G * lstride + (size_t)parts * G * WAVES * (D + 2);
}

template <typename DT, int D, int G>
__global__ __launch_bounds__(SMALL_WG) void corm_small_kernel(const Params p, const int lstride, const int max_parts) {
  using A = Attend<DT, D, G, WAVES>;
  constexpr int EPL = A::EPL, ROWB = A::ROWB, LPR = A::LPR, RPL = A::RPL;

  extern __shared__ float sh_dyn[];     // see small_lds_floats
  float* sh_logit = sh_dyn;             // raw logits of the unit (log2 domain)
  float* sh_m = sh_logit + G * lstride;
  float* sh_z = sh_m + max_parts * G * WAVES;
  float* sh_acc = sh_z + max_parts * G * WAVES;
  __shared__ float sh_M[G], sh_Z[G];
  __shared__ unsigned long long sh_keep[SMALL_TILES * SMALL_WAVES];   // ballots, 64 slots each
  __shared__ uint16_t sh_src[SMALL_MAX_SLOTS];                        // old slots of the survivors

  const int unit = blockIdx.x;
  const int b = unit / p.Hkv, hkv = unit - b * p.Hkv, hq0 = hkv * G;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wv / WAVES, gwv = wv % WAVES;
  const int sub = lane / LPR, cl = lane % LPR;
  const int lane_row = gwv * RPL + sub;   // this lane's row inside a load of its group

  // everything that does not hang on the unit's length is requested with it
  const int lens_value = p.lens[unit], tcur = p.t[b], tfirst = p.t_first[b];
  uint4 qreg[G];
#pragma unroll
  for (int g = 0; g < G; ++g)
    qreg[g] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(p.q) +
                                              ((size_t)(b * p.Hq + hq0 + g) * ROWB + (size_t)cl * 16));
  const uint4 knew = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(p.k_new) + (size_t)unit * ROWB + (size_t)cl * 16);
  const uint4 vnew = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(p.v_new) + (size_t)unit * ROWB + (size_t)cl * 16);

  const UnitLen ul = unit_len_of(p, __builtin_amdgcn_readfirstlane(lens_value));
  const int L0 = ul.L0, L = ul.L;   // (L >= 1: there is room in an empty unit)
  if (tid == 0 && ul.flags && p.status) atomicOr(p.status, ul.flags);
  char* Kb = reinterpret_cast<char*>(p.K) + (size_t)unit * p.Lcap * ROWB;
  char* Vb = reinterpret_cast<char*>(p.V) + (size_t)unit * p.Lcap * ROWB;
  int32_t* posb = p.pos + (size_t)unit * p.Lcap;
  int32_t* lhb = p.last_hit + (size_t)unit * p.Lcap;

  // The stages of a group: those of its parts (grp, grp + SMALL_GROUPS, ...) one after the other, the next one's loads always in
  // flight.  The descriptors end at row L0; the new row is put in its place where a stage holds it.
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(Kb, (uint32_t)L0 * ROWB);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(Vb, (uint32_t)L0 * ROWB);
  const int spp = p.part_keys / A::STAGE_ROWS, lg_spp = 31 - __clz(spp);   // stages per part: a power of two
  auto stage_part = [&](int n) __attribute__((always_inline)) { return grp + (n >> lg_spp) * SMALL_GROUPS; };
  auto stage_row = [&](int n) __attribute__((always_inline)) {   // first row of the group's stage n
    return stage_part(n) * p.part_keys + (n & (spp - 1)) * A::STAGE_ROWS;
  };
  auto fetch = [&](typename A::Stage& st, int row) __attribute__((always_inline)) {
    A::template load<false>(st, rk, rv, (uint32_t)(row + lane_row) * ROWB + (uint32_t)cl * 16, nullptr, 0);
  };
  typename A::Stage s0, s1;
  fetch(s0, stage_row(0));
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
  auto begin_part = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      m_run[g] = neg_inf();
      z_run[g] = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
    }
  };
  auto work = [&](typename A::Stage& st, int n) __attribute__((always_inline)) {
    const int row = stage_row(n);
    if (row >= L) return;   // (uniform over the wave)
    if (ul.appended && L0 >= row && L0 < row + A::STAGE_ROWS) {   // (uniform) the append
#pragma unroll
      for (int j = 0; j < A::U; ++j)
        if (row + lane_row + j * A::LOAD_ROWS == L0) {
          st.k[j] = knew;
          st.v[j] = vnew;
          *reinterpret_cast<uint4*>(Kb + (size_t)L0 * ROWB + (size_t)cl * 16) = knew;
          *reinterpret_cast<uint4*>(Vb + (size_t)L0 * ROWB + (size_t)cl * 16) = vnew;
        }
    }
    A::compute(st, row + lane_row, row + lane_row, L, cl, qreg, p.scale_log2, sh_logit, lstride, m_run, z_run, acc);
    if (stage_part(n + 1) != stage_part(n) || stage_row(n + 1) >= L) {   // (uniform) the last of its part with a key
      const int part = stage_part(n);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        A::merge_rows(m_run[g], z_run[g], acc[g]);
        const int at = (part * G + g) * WAVES + gwv;
        if (sub == 0) {
#pragma unroll
          for (int e = 0; e < EPL; ++e) sh_acc[at * D + cl * EPL + e] = acc[g][e];
          if (cl == 0) {
            sh_m[at] = m_run[g];
            sh_z[at] = z_run[g];
          }
        }
      }
      begin_part();
    }
  };
  begin_part();
  for (int n = 0; stage_row(n) < L; n += 2) {
    fetch(s1, stage_row(n + 1));
    work(s0, n);
    fetch(s0, stage_row(n + 2));
    work(s1, n + 1);
  }
  __syncthreads();

  // out (Eq. 1) and the unit's max / sum (Eq. 2)
  const int nparts = (L + p.part_keys - 1) / p.part_keys;
  for (int idx = tid; idx < G * D; idx += SMALL_WG) {
    const int g = idx / D, c = idx - g * D;
    SmallPart part[SMALL_MAX_PARTS];
    float mx = neg_inf();
#pragma unroll
    for (int s = 0; s < SMALL_MAX_PARTS; ++s) {
      part[s] = SmallPart{neg_inf(), 0.f, 0.f};
      if (s < nparts) {   // (uniform)
        const int at = (s * G + g) * WAVES;
        part[s] = small_part(sh_m + at, sh_z + at, sh_acc + at * D + c, D);
      }
      mx = fmaxf(mx, part[s].m);
    }
    const float ms = mx == neg_inf() ? 0.f : mx;
    float zs[SMALL_MAX_PARTS], at = 0.f;
#pragma unroll
    for (int s = 0; s < SMALL_MAX_PARTS; ++s) {
      const float a = exp2f(part[s].m - ms);
      zs[s] = part[s].z * a;
      asm volatile("" : "+v"(zs[s]));   // (rounded: not fused with the sums below)
      at = fmaf(part[s].at, a, at);
    }
    // (the order of a wave that adds up a partial per lane)
#pragma unroll
    for (int o = SMALL_MAX_PARTS / 2; o > 0; o >>= 1)
#pragma unroll
      for (int s = 0; s < o; ++s) zs[s] += zs[s + o];
    p.out[(size_t)(b * p.Hq + hq0 + g) * D + c] = at / zs[0];
    if (c == 0) {
      sh_M[g] = ms;
      sh_Z[g] = zs[0];
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
