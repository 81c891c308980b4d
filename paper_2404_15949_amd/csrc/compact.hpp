// stable in-place compaction: column slabs in one launch, or chunks in two (local and boundary).
// Part of one translation unit: included by corm_kernels.hip, in this order, after <hip/hip_runtime.h> and corm.h.
#ifndef CORM_COMPACT_HPP
#define CORM_COMPACT_HPP

namespace {

// ---------------------------------------------------------------- stable in-place compaction
//
// Survivor number rho of a unit (in slot order) must end in slot rho.  No cross-workgroup synchronization inside a
// launch; the unit's length is handed over through the workspace by the launch before (lens is written here).
//
// Many units, or short ones (compact_by_slabs), one launch: a workgroup owns a slab of columns of K or V over the whole
// unit (one more the metadata), so nobody else reads or writes what it moves: it walks the survivors behind the first
// hole in ascending batches (every destination <= its source; all loads of a batch complete before any of its
// stores).
//
// Few long units, two launches, where slabs would be a few long serial walks:
//   local     grid (splits, units).  R_c = survivors before chunk c (from the per-split counts).
//             The workgroup of chunk c = slots [a_c, a_c + CHUNK) moves its survivors with rho >= a_c
//             to slot rho -- inside its own chunk, so it reads and writes only its own slots -- in
//             ascending batches.  Its first survivors, those with rho < a_c ("boundary rows", at most
//             as many as slots were freed before the chunk), belong in earlier chunks, whose owners
//             may not have read those slots yet: they go to the chunk's staging area instead.
//   boundary  grid (splits, units).  Workgroup c copies its staged rows to slots
//             [R_c, min(a_c, R_{c+1})): slots no local workgroup writes, and whose old contents were
//             consumed in the previous launch.  Workgroup 0 writes lens, the live count and, in lazy
//             mode, the reset live masks.
//
// Policy (lazy mode): a unit is compacted only when its dead slots reach dead_num/dead_den of its
// slots (or its slots are about to run out); otherwise the launches leave it alone, its dead rows
// stay in place and the attend kernels skip them by their live masks.  Exact mode: dead_num = 0.

// The local launch runs one thread per slot of a chunk: a chunk is scanned in one step and its rows are requested
// 64 to 256 at a time (four passes of the workgroup), so a unit that lost a single key (the common case of a
// dense cache) costs a few memory latencies.
constexpr int CWG = CHUNK;
constexpr int CWAVES = CWG / 64;

struct CompactShared {
  int32_t wave_count[CWAVES];
  int32_t first_hole;   // first slot of the chunk (relative) that does not survive
  int32_t src_of[CWG];
};

struct CompactArgs {
  char* K;
  char* V;
  int32_t* pos;
  int32_t* last_hit;
  int32_t* lens;
  const uint8_t* keep;           // caller's byte mask (corm_compact only)
  unsigned long long* keepbits;  // [units, kb_stride] wave ballots (workspace)
  unsigned long long* live;      // lazy mode: the caller's live masks, reset where a unit is compacted
  int32_t* kept_idx;             // optional
  const int32_t* counts;         // [units, nsplit]
  int2* unit_state;              // [units] (slots, survivors or SUM_COUNTS) of the unit in this step, by the launch before
  int32_t* nlive;                // optional [units]: live keys after the step
  char* stage_k;                 // [units, nsplit, CHUNK, ROWB]
  char* stage_v;
  int32_t* stage_meta;           // [units, nsplit, CHUNK, 2] (pos, last_hit)
  int32_t units, nsplit, Lcap, kb_stride;
  int32_t lazy, dead_num, dead_den;
};

__device__ __forceinline__ bool compact_now(const CompactArgs& a, int L, int T) {
  return compact_policy(a.lazy, a.dead_num, a.dead_den, a.Lcap, L, T);
}

// Moves the n_rows survivors listed in src_of (ascending) to consecutive destinations starting at
// survivor number rho0: slot rho if rho >= own_begin, else staging row (rho - stage_rho0).  Every destination
// is <= its source; all loads of a batch complete before any of its stores.
template <int ROWB>
__device__ __forceinline__ void move_rows(char* Kb, char* Vb, char* sk, char* sv, const int32_t* src_of, int n_rows,
                                          int rho0, int own_begin, int stage_rho0) {
  constexpr int LPR = ROWB / 16;
  constexpr int RPP = CWG / LPR;  // rows per pass of the workgroup
  // Four passes in flight together, in named registers (an indexed array would be demoted to scratch).  Eight
  // (94 registers, two workgroups per compute unit) moved a full launch 2 % faster and made the launches that
  // find nothing to do slower: the workgroups that only look at their unit's word then come in more rounds.
  constexpr int NP = 4;
  const int tid = threadIdx.x;
  const int sub = tid / LPR;
  const size_t col = (size_t)(tid % LPR) * 16;
  const int last = n_rows - 1;
  for (int base = 0; base < n_rows; base += RPP * NP) {
    // clamped row numbers: every load reads a valid row, stores are predicated
#define CORM_LOAD_ROW(U)                                                                          \
    const size_t o##U = (size_t)src_of[min(base + sub + (U) * RPP, last)] * ROWB + col;            \
    const uint4 k##U = *reinterpret_cast<const uint4*>(Kb + o##U);                                \
    const uint4 v##U = *reinterpret_cast<const uint4*>(Vb + o##U);
    CORM_LOAD_ROW(0) CORM_LOAD_ROW(1) CORM_LOAD_ROW(2) CORM_LOAD_ROW(3)
#undef CORM_LOAD_ROW
    wait_vm_loads();
    __syncthreads();
#define CORM_STORE_ROW(U)                                                      \
    {                                                                            \
      const int j = base + sub + (U) * RPP;                                      \
      if (j < n_rows) {                                                          \
        const int rho = rho0 + j;                                                \
        if (rho >= own_begin) {                                                  \
          const size_t d = (size_t)rho * ROWB + col;                             \
          *reinterpret_cast<uint4*>(Kb + d) = k##U;                              \
          *reinterpret_cast<uint4*>(Vb + d) = v##U;                              \
        } else {                                                                 \
          const size_t d = (size_t)(rho - stage_rho0) * ROWB + col;              \
          *reinterpret_cast<uint4*>(sk + d) = k##U;                              \
          *reinterpret_cast<uint4*>(sv + d) = v##U;                              \
        }                                                                        \
      }                                                                          \
    }
    CORM_STORE_ROW(0) CORM_STORE_ROW(1) CORM_STORE_ROW(2) CORM_STORE_ROW(3)
#undef CORM_STORE_ROW
  }
  static_assert(NP == 4, "four named passes");
}

// The scan of a chunk.  keep: this thread's flag (0 for slots >= L).  Returns this thread's rank among the
// chunk's survivors and their number (via *kept).
__device__ __forceinline__ int chunk_scan(bool keep, CompactShared& sh, int* kept) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const unsigned long long bal = __ballot(keep);
  const int rank = __popcll(bal & ((1ull << lane) - 1ull));
  if (lane == 0) sh.wave_count[wv] = __popcll(bal);
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int i = 0; i < CWAVES; ++i) {
    const int c = sh.wave_count[i];
    if (i < wv) before += c;
    total += c;
  }
  *kept = total;
  return before + rank;
}

// survivors before chunk `split` (R) and of the whole unit (T), by one wave-wide pass over the counts
__device__ __forceinline__ void unit_counts(const int32_t* cnt, int nlive, int split, int* R, int* T) {
  int r = 0, t = 0;
  for (int s = (threadIdx.x & 63); s < nlive; s += 64) {
    const int c = min(max(cnt[s], 0), CHUNK);   // (whatever the workspace holds, rows stay inside the unit)
    if (s < split) r += c;
    t += c;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    r += __shfl_xor(r, off);
    t += __shfl_xor(t, off);
  }
  *R = r;
  *T = t;
}

// What the launch before left in a unit's state: its slots, and its survivors or, where several workgroups counted and a
// key went, SUM_COUNTS.  (Adding up in the record launch, by atomics on one word of the unit, cost that launch 0.6 to
// 1.5 us.)  A unit that lost nothing is known by this one load: the chunk launches, which have a workgroup per 512
// slots, leave then (128 units x 33000 slots with nothing to move, local launch: 5.1 us, 7.0 with the counts read as well).
// Slots are held to [0, Lcap] and survivors to [0, slots] whatever the workspace holds (corm_step_evict may be called on
// one that no corm_step_attend filled): nothing outside the unit is touched.
__device__ __forceinline__ int unit_slots(const CompactArgs& a, int2 state) { return min(max(state.x, 0), a.Lcap); }

// The slab launch: slots L and survivors T.  The counts are requested with the state and cost no further latency.
__device__ __forceinline__ void unit_totals(const CompactArgs& a, int unit, int* L, int* T) {
  const int lane = threadIdx.x & 63;
  const int32_t* cnt = a.counts + (size_t)unit * a.nsplit;   // (at most 32: SLAB_MAX_SLOTS / CHUNK)
  const int2 state = a.unit_state[unit];
  const int c = lane < a.nsplit ? cnt[lane] : 0;
  *L = unit_slots(a, state);
  int total = state.y;
  if (total == SUM_COUNTS) {   // (uniform)
    total = lane * CHUNK < *L ? min(max(c, 0), CHUNK) : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off);
  }
  *T = min(max(total, 0), *L);
}

// a caller's byte mask (corm_compact) -> wave ballots and survivors per split
__global__ __launch_bounds__(WG) void corm_count_kernel(const CompactArgs a, int32_t* counts) {
  __shared__ int sh_cnt[WAVES];
  const int split = blockIdx.x, unit = blockIdx.y;
  int L = a.lens[unit];
  L = L < 0 ? 0 : (L > a.Lcap ? a.Lcap : L);
  const int cbeg = split * CHUNK;
  if (split == 0 && threadIdx.x == 0) a.unit_state[unit] = make_int2(L, SUM_COUNTS);
  if (cbeg >= L) return;
  const int cend = min(cbeg + CHUNK, L);
  const uint8_t* keepb = a.keep + (size_t)unit * a.Lcap;
  unsigned long long* bitsb = a.keepbits + (size_t)unit * a.kb_stride;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int kept = 0;
  for (int i0 = cbeg; i0 < cbeg + CHUNK; i0 += WG) {
    const int i = i0 + threadIdx.x;
    const unsigned long long bal = __ballot(i < cend && keepb[i] != 0);
    if (lane == 0 && i0 + wv * 64 < cend) bitsb[(i0 >> 6) + wv] = bal;
    kept += __popcll(bal);
  }
  if (lane == 0) sh_cnt[wv] = kept;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) tot += sh_cnt[i];
    counts[(size_t)unit * a.nsplit + split] = tot;
  }
}

template <int ROWB>
__global__ __launch_bounds__(CWG) void corm_compact_local_kernel(const CompactArgs a) {
  __shared__ CompactShared sh_c;
  const int split = blockIdx.x, unit = blockIdx.y;
  const int tid = threadIdx.x;
  const int2 state = a.unit_state[unit];
  if (state.x == state.y && !a.kept_idx) return;   // nothing went
  const int L = unit_slots(a, state);
  const int nlive = (L + CHUNK - 1) / CHUNK;
  if (split >= nlive) return;
  const int32_t* cnt = a.counts + (size_t)unit * a.nsplit;
  int R, T;   // survivors before this chunk, survivors of the unit
  unit_counts(cnt, nlive, split, &R, &T);
  T = min(T, L);
  int32_t* idxb = a.kept_idx ? a.kept_idx + (size_t)unit * a.Lcap : nullptr;
  const int cbeg = split * CHUNK;
  const int cend = min(cbeg + CHUNK, L);
  const int i = cbeg + tid;   // this thread's slot
  if (!compact_now(a, L, T)) {   // nothing evicted, or (lazy mode) not enough dead slots yet
    if (idxb && T == L && i < cend) idxb[i] = i;
    return;
  }
  const int my_cnt = min(max(cnt[split], 0), CHUNK);
  if (R == cbeg && my_cnt == cend - cbeg) {   // no hole before or inside this chunk
    if (idxb && i < cend) idxb[i] = i;
    return;
  }
  char* Kb = a.K + (size_t)unit * a.Lcap * ROWB;
  char* Vb = a.V + (size_t)unit * a.Lcap * ROWB;
  int32_t* posb = a.pos + (size_t)unit * a.Lcap;
  int32_t* lhb = a.last_hit + (size_t)unit * a.Lcap;
  const unsigned long long* bitsb = a.keepbits + (size_t)unit * a.kb_stride;
  const size_t stage_row0 = ((size_t)unit * a.nsplit + split) * CHUNK;
  char* sk = a.stage_k + stage_row0 * ROWB;
  char* sv = a.stage_v + stage_row0 * ROWB;
  int32_t* sm = a.stage_meta + stage_row0 * 2;
  // a chunk whose count equals its size lost nothing: its flags are implied (and may be unwritten)
  const bool chunk_full = my_cnt == cend - cbeg;

  const bool kp = i < cend && (chunk_full || ((bitsb[i >> 6] >> (i & 63)) & 1ull) != 0);
  int my_pos = 0, my_lh = 0;
  if (kp) {
    my_pos = posb[i];
    my_lh = lhb[i];
  }
  if (tid == 0) sh_c.first_hole = CWG;
  wait_vm_loads();
  int kept;
  const int rank = chunk_scan(kp, sh_c, &kept);
  const int rho = R + rank;   // survivor number of this thread's key
  if (kp) {
    sh_c.src_of[rank] = i;
    if (idxb) idxb[rho] = i;
    if (rho >= cbeg) {
      if (rho != i) {
        posb[rho] = my_pos;
        lhb[rho] = my_lh;
      }
    } else {
      sm[(rho - R) * 2] = my_pos;
      sm[(rho - R) * 2 + 1] = my_lh;
    }
  } else if (i < cend) {
    atomicMin(&sh_c.first_hole, tid);
  }
  __syncthreads();
  // with no hole before the chunk, the survivors in front of its first hole already lie where they belong
  const int fixed = R == cbeg ? min(sh_c.first_hole, kept) : 0;
  move_rows<ROWB>(Kb, Vb, sk, sv, sh_c.src_of + fixed, kept - fixed, R + fixed, cbeg, R);
}

// by one workgroup of a unit: lens, the live count and, in lazy mode, the live masks of a unit that was compacted
__device__ __forceinline__ void unit_bookkeeping(const CompactArgs& a, int unit, int L, int T, bool compacted) {
  if (threadIdx.x == 0) {
    a.lens[unit] = compacted ? T : L;
    if (a.nlive) a.nlive[unit] = T;
  }
  if (a.lazy && compacted) {   // every slot below T is live again
    unsigned long long* liveb = a.live + (size_t)unit * a.kb_stride;
    for (int wd = threadIdx.x; wd < a.kb_stride; wd += blockDim.x) {
      const int lo = wd * 64;
      liveb[wd] = T >= lo + 64 ? ~0ull : (T > lo ? ((1ull << (T - lo)) - 1ull) : 0ull);
    }
  }
}

template <int ROWB>
__global__ __launch_bounds__(WG) void corm_compact_boundary_kernel(const CompactArgs a) {
  constexpr int LPR = ROWB / 16;
  const int split = blockIdx.x, unit = blockIdx.y;
  const int tid = threadIdx.x;
  const int2 state = a.unit_state[unit];
  if (state.x == state.y && split != 0) return;   // nothing went
  const int L = unit_slots(a, state);
  const int nlive = (L + CHUNK - 1) / CHUNK;
  if (split >= nlive && split != 0) return;
  const int32_t* cnt = a.counts + (size_t)unit * a.nsplit;
  int R, T;
  unit_counts(cnt, nlive, split, &R, &T);
  T = min(T, L);
  const bool compacted = compact_now(a, L, T);
  if (compacted && split > 0) {
    const int nb = min(split * CHUNK, R + min(max(cnt[split], 0), CHUNK)) - R;   // boundary rows of this chunk: survivors [R, R + nb)
    if (nb > 0) {
      char* Kb = a.K + (size_t)unit * a.Lcap * ROWB;
      char* Vb = a.V + (size_t)unit * a.Lcap * ROWB;
      int32_t* posb = a.pos + (size_t)unit * a.Lcap;
      int32_t* lhb = a.last_hit + (size_t)unit * a.Lcap;
      const size_t stage_row0 = ((size_t)unit * a.nsplit + split) * CHUNK;
      const size_t col = (size_t)(tid % LPR) * 16;
      for (int j = tid / LPR; j < nb; j += WG / LPR) {
        const size_t s = (stage_row0 + j) * ROWB + col;
        const size_t d = (size_t)(R + j) * ROWB + col;
        *reinterpret_cast<uint4*>(Kb + d) = *reinterpret_cast<const uint4*>(a.stage_k + s);
        *reinterpret_cast<uint4*>(Vb + d) = *reinterpret_cast<const uint4*>(a.stage_v + s);
      }
      for (int j = tid; j < nb; j += WG) {
        posb[R + j] = a.stage_meta[(stage_row0 + j) * 2];
        lhb[R + j] = a.stage_meta[(stage_row0 + j) * 2 + 1];
      }
    }
  }
  if (split == 0) unit_bookkeeping(a, unit, L, T, compacted);
}

// ---------------------------------------------------------------- one launch, a slab of columns per workgroup
//
// A slab is 128 bytes of a row, one cache line: 5 workgroups make a unit of 256-byte rows.  Bound by the bytes it has
// to move where many units evict (512 units of 1100 to 4300 keys, a hole each: 0.42 GB read and written in 82 us,
// 5.1 TB/s, what a plain copy reaches here; the two chunk launches 101 + 6 us), by what one compute unit loads and stores
// where few do (a batch of 512 pieces 1.5 us: 4000 rows 12 us and the list; compact_by_slabs says where chunks are the better
// choice), by the launch itself where none does (4.9 us for 512 units, 2.4 for 32; the chunks 4.9 + 4.8 and 2.2 + 2.4).
// Measured beside it on the 512 units: slabs of 64 bytes 102 us and 7.4 us for the launch that finds nothing, whole rows
// 89 us; 256 threads 89 us, 1024 threads 83 us but 7.2 us idle; four passes in flight 87 us.
constexpr int SLAB_WG = 512;
constexpr int SLAB_WAVES = SLAB_WG / 64;
constexpr int SLAB_MAX_SLOTS = 16384;          // a 64-slot word per thread and a 16-bit source slot per survivor in LDS
static_assert(SLAB_MAX_SLOTS <= SLAB_WG * 64 && SLAB_MAX_SLOTS <= 65536, "words of a unit, source slots");
constexpr int SLAB_XCDS = 8;                   // accelerator dies of the device
constexpr int slab_bytes(int rowb) { return rowb < 128 ? rowb : 128; }

template <int ROWB>
__global__ __launch_bounds__(SLAB_WG) void corm_compact_slab_kernel(const CompactArgs a) {
  constexpr int SLAB_BYTES = slab_bytes(ROWB);
  constexpr int SLABS = 2 * ROWB / SLAB_BYTES;   // of K, then of V; one more workgroup: metadata
  constexpr int LPR = SLAB_BYTES / 16;           // lanes per piece of a row
  constexpr int RPP = SLAB_WG / LPR;             // rows per pass of the workgroup
  constexpr int NP = 8;                          // passes in flight together, two such batches
  extern __shared__ uint16_t sh_src[];           // [Lcap] old slots of the survivors behind the first hole
  __shared__ int sh_wave[SLAB_WAVES], sh_first[SLAB_WAVES];
  __shared__ unsigned long long sh_word[SLAB_WG];
  __shared__ int sh_before[SLAB_WG];

  // XCD id % 8 takes the same contiguous range of units as the unit kernel
  const int per_xcd = (a.units + SLAB_XCDS - 1) / SLAB_XCDS;
  const int li = (int)(blockIdx.x / SLAB_XCDS);
  const int slab = li % (SLABS + 1);
  const int unit = (int)(blockIdx.x % SLAB_XCDS) * per_xcd + li / (SLABS + 1);
  if (li / (SLABS + 1) >= per_xcd || unit >= a.units) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int L, T;
  unit_totals(a, unit, &L, &T);
  const bool compacted = compact_now(a, L, T);
  int32_t* idxb = a.kept_idx ? a.kept_idx + (size_t)unit * a.Lcap : nullptr;
  if (slab == SLABS) unit_bookkeeping(a, unit, L, T, compacted);
  if (!compacted) {   // nothing evicted, or (lazy mode) not enough dead slots yet
    if (slab == SLABS && idxb && T == L)
      for (int i = tid; i < L; i += SLAB_WG) idxb[i] = i;
    return;
  }

  // survivors before every 64-slot word and the first hole: a word per thread, scanned over the workgroup
  const unsigned long long* bitsb = a.keepbits + (size_t)unit * a.kb_stride;
  const int nword = (L + 63) / 64;
  unsigned long long word = 0ull;
  int hole = 0x7fffffff;
  if (tid < nword) {
    word = bitsb[tid];
    const int valid = L - tid * 64;   // slots of this word that are in use
    if (valid < 64) word &= (1ull << valid) - 1ull;
    if (~word != 0ull) hole = tid * 64 + __ffsll((long long)~word) - 1;   // (>= L: no hole)
  }
  int before = __popcll(word);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int x = __shfl_up(before, off);
    if (lane >= off) before += x;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) hole = min(hole, __shfl_xor(hole, off));
  if (lane == 63) sh_wave[wv] = before;
  if (lane == 0) sh_first[wv] = hole;
  before -= __popcll(word);
  __syncthreads();
  int listed = 0;   // survivors by the masks: T, unless the workspace holds something else
#pragma unroll
  for (int i = 0; i < SLAB_WAVES; ++i) {
    if (i < wv) before += sh_wave[i];
    listed += sh_wave[i];
    hole = min(hole, sh_first[i]);
  }
  sh_word[tid] = word;
  sh_before[tid] = before;
  __syncthreads();
  const int fixed = min(hole, L);   // the survivors in front of the first hole lie where they belong
  // the list of old slots: a slot per lane, the words dealt to the waves
#pragma unroll 4
  for (int w = (fixed >> 6) + wv; w < nword; w += SLAB_WAVES) {
    const unsigned long long bw = sh_word[w];
    const int r = sh_before[w] + __popcll(bw & ((1ull << lane) - 1ull));
    if (((bw >> lane) & 1ull) && r >= fixed) sh_src[r - fixed] = (uint16_t)(w * 64 + lane);
  }
  __syncthreads();
  const int n = min(T, listed) - fixed;   // rows to move, to slots fixed, fixed + 1, ...

  if (slab == SLABS) {   // metadata: a slot per thread and step
    int32_t* posb = a.pos + (size_t)unit * a.Lcap;
    int32_t* lhb = a.last_hit + (size_t)unit * a.Lcap;
    if (idxb)
      for (int i = tid; i < fixed; i += SLAB_WG) idxb[i] = i;
    constexpr int MP = 4;   // in flight together
    for (int base = 0; base < n; base += SLAB_WG * MP) {
      int p[MP], h[MP], src[MP];
#pragma unroll
      for (int u = 0; u < MP; ++u) {
        src[u] = sh_src[min(base + u * SLAB_WG + tid, n - 1)];
        p[u] = posb[src[u]];
        h[u] = lhb[src[u]];
      }
      wait_vm_loads();
      __syncthreads();
#pragma unroll
      for (int u = 0; u < MP; ++u) {
        const int j = base + u * SLAB_WG + tid;
        if (j < n) {
          posb[fixed + j] = p[u];
          lhb[fixed + j] = h[u];
          if (idxb) idxb[fixed + j] = src[u];
        }
      }
    }
    return;
  }
  if (n <= 0) return;   // what went lay behind every survivor

  constexpr int HALF = SLABS / 2;
  char* base = (slab < HALF ? a.K : a.V) + (size_t)unit * a.Lcap * ROWB + (slab % HALF) * SLAB_BYTES + (tid % LPR) * 16;
  const int sub = tid / LPR;
  // Two batches of NP passes, the next one's loads issued before this one is stored (its sources lie behind every
  // destination of this batch).  A batch is stored once all of its loads, of every wave, are in.  (The stores are
  // predicated, so the compiler waits for both batches together.  Straight-line stores through a buffer descriptor, with
  // exact counts, measured 2 % faster on 512 units x 4096 rows and 0.5 to 0.8 us slower on units of 1000.)
  u32x4_t ra[NP], rb[NP];
  auto load = [&](int j0, u32x4_t (&r)[NP]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NP; ++u)   // (clamped: every load reads a valid row)
      r[u] = *reinterpret_cast<const u32x4_t*>(base + (size_t)sh_src[min(j0 + u * RPP + sub, n - 1)] * ROWB);
  };
  auto store = [&](int j0, const u32x4_t (&r)[NP]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NP; ++u) asm volatile("" ::"v"(r[u]));   // this wave's loads of the batch are in ...
    __syncthreads();                                             // ... and everybody's
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int j = j0 + u * RPP + sub;
      if (j < n) *reinterpret_cast<u32x4_t*>(base + (size_t)(fixed + j) * ROWB) = r[u];
    }
  };
  constexpr int BATCH = RPP * NP;
  load(0, ra);
  for (int j0 = 0; j0 < n; j0 += 2 * BATCH) {
    if (j0 + BATCH < n) load(j0 + BATCH, rb);
    store(j0, ra);
    if (j0 + BATCH >= n) break;
    if (j0 + 2 * BATCH < n) load(j0 + 2 * BATCH, ra);
    store(j0 + BATCH, rb);
  }
}

}  // namespace

#endif  // CORM_COMPACT_HPP
