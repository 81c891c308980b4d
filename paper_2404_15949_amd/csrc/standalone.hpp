// small standalone kernels: append, literal and summary masks, threshold, fill.
// Part of one translation unit: included by corm_kernels.hip, in this order, after <hip/hip_runtime.h> and corm.h.
#ifndef CORM_STANDALONE_HPP
#define CORM_STANDALONE_HPP

namespace {

// ---------------------------------------------------------------- standalone kernels

__global__ __launch_bounds__(64) void corm_append_kernel(char* K, char* V, int32_t* lens, int32_t* pos,
                                                         int32_t* last_hit, const char* k_new, const char* v_new,
                                                         const int32_t* t, int32_t* status, int Hkv, int Lcap,
                                                         int rowb) {
  const int unit = blockIdx.x;
  const int b = unit / Hkv;
  const int L0 = lens[unit];
  if (L0 < 0 || L0 >= Lcap) {
    if (threadIdx.x == 0 && status) atomicOr(status, L0 == Lcap ? CORM_DEV_UNIT_FULL : CORM_DEV_BAD_LENS);
    return;
  }
  const int lane = threadIdx.x;
  if (lane * 16 < rowb) {
    size_t dst = ((size_t)unit * Lcap + L0) * rowb + (size_t)lane * 16;
    size_t src = (size_t)unit * rowb + (size_t)lane * 16;
    *reinterpret_cast<uint4*>(K + dst) = *reinterpret_cast<const uint4*>(k_new + src);
    *reinterpret_cast<uint4*>(V + dst) = *reinterpret_cast<const uint4*>(v_new + src);
  }
  if (lane == 0) {
    pos[(size_t)unit * Lcap + L0] = t[b] - 1;
    last_hit[(size_t)unit * Lcap + L0] = 0;
    lens[unit] = L0 + 1;
  }
}

// The literal rule's look-up, in two halves so that many loads can be in flight: the word of a ring row that holds
// position pi, and whether it says "score >= thr" (bit ring: the recorded boolean itself).
template <int MODE>
__device__ __forceinline__ uint32_t ring_word(uint64_t row, int pi) {   // row: address in global memory
#define CORM_GLOBAL(T) reinterpret_cast<const __attribute__((address_space(1))) T*>(row)
  if (MODE == CORM_BIT) return CORM_GLOBAL(uint32_t)[pi >> 5];
  return MODE == CORM_BF16 ? (uint32_t)CORM_GLOBAL(uint16_t)[pi] : CORM_GLOBAL(uint32_t)[pi];
#undef CORM_GLOBAL
}
template <int MODE>
__device__ __forceinline__ bool ring_word_hit(uint32_t word, int pi, float thr) {
  if (MODE == CORM_BIT) return (word >> (pi & 31)) & 1u;
  return __uint_as_float(MODE == CORM_BF16 ? word << 16 : word) >= thr;
}

// Literal windowed OR over the ring (Def. 4.1 + recent r + group rule).
// Bound by the latency of the w * G reads per key and, where keys are rarely important, by the bytes of the window.  One
// workgroup takes 64 consecutive slots, one per lane, and its eight waves share the window's (row, head) pairs, newest
// row first, up to eight loads in flight each.  After every round the waves pool what they found and stop once all 64 keys
// are decided; the first round is short (16 pairs, then 64), since most keys are found important within a few rows.
// Measured against one thread per key that walked the window alone (a load, a division and a modulo per row, in series):
// 16 units of ~1460 keys, w 256, G 2: 197 -> 18 us; 512 units of 4096 keys, w 1024, G 1, nearly all kept: 1528 -> 407 us,
// 64 % evicted: 932 -> 322 us (bit ring 819 -> 129 us).
constexpr int MASK_WAVES = 8;

template <int MODE>
__global__ __launch_bounds__(MASK_WAVES * 64) void corm_evict_mask_kernel(const void* ring, const int32_t* lens,
                                                                          const int32_t* pos, const int32_t* t,
                                                                          const int32_t* t_first, uint8_t* keep, int Hq,
                                                                          int Hkv, int Lcap, int Tcap, int w, int r,
                                                                          float c) {
  __shared__ unsigned long long sh_hit;
  const int unit = blockIdx.y;
  const int b = unit / Hkv, hkv = unit - b * Hkv;
  const int G = Hq / Hkv;   // a power of two
  const int gshift = 31 - __clz(G);
  int L = lens[unit];
  L = L < 0 ? 0 : (L > Lcap ? Lcap : L);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x * 64 >= L) return;
  const int i = blockIdx.x * 64 + lane;
  const int tcur = t[b];
  const int tf = t_first[b];
  const bool full = tcur - tf + 1 >= w;
  const bool kept = !full || i >= L - r;   // decided without the ring
  const int pi = i < L ? pos[(size_t)unit * Lcap + i] : -1;
  const bool look = !kept && pi >= 0 && pi < Tcap;
  const int lo = max(max(tf, tcur - w + 1), 1);
  const long long pairs = tcur >= lo ? (long long)(tcur - lo + 1) << gshift : 0;
  const size_t row0 = (size_t)(b * Hq + hkv * G) * w;   // ring rows of the group's first head
  if (threadIdx.x == 0) sh_hit = 0ull;
  __syncthreads();

  const unsigned long long todo = __ballot(look);   // the same in every wave
  unsigned long long open = todo;
  bool hit = false;
  const int slot0 = pairs > 0 ? (tcur - 1) % w : 0;   // ring slot of the newest row
  const size_t rowb = MODE == CORM_BIT ? (size_t)((Tcap + 31) >> 5) * 4 : (size_t)Tcap * (MODE == CORM_BF16 ? 2 : 4);
  // Pair k: head k % G of step tcur - k / G.  What belongs to a pair and not to a key (the row's address, the IEEE quotient
  // of its threshold, the newest position its query saw) is formed by the lanes at once, one pair each.
  auto round = [&](auto batch, long long k0) {
    constexpr int N = decltype(batch)::value;
    const long long k = k0 + (lane & (N - 1));
    const int back = (int)(k >> gshift);   // (< w, like the window's rows, wherever the pair is looked up)
    const int slot = slot0 - back + (slot0 < back ? w : 0);
    const float thr = importance_threshold(c, max(tcur - back, 1));
    // (a key younger than the row did not exist at its step: minor there)
    const int seen = k < pairs ? tcur - back - 1 : -1;
    const uint64_t at = reinterpret_cast<uint64_t>(ring) + (row0 + (size_t)(k & (G - 1)) * w + (size_t)slot) * rowb;
    const bool mine = (open >> lane) & 1ull;
    uint32_t word[N];
    bool ok[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const uint64_t row = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(at >> 32), j) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)at, j);
      ok[j] = mine & (pi <= __builtin_amdgcn_readlane(seen, j));
      word[j] = 0u;
      if (ok[j]) word[j] = ring_word<MODE>(row, pi);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float thr_j = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(thr), j));
      hit |= ok[j] & ring_word_hit<MODE>(word[j], pi, thr_j);
    }
  };
  for (long long k0 = 0; k0 < pairs && open != 0ull;) {   // (uniform over the workgroup)
    if (k0 == 0) {
      round(std::integral_constant<int, 2>(), wv * 2);
      k0 += MASK_WAVES * 2;
    } else {
      round(std::integral_constant<int, 8>(), k0 + wv * 8);
      k0 += MASK_WAVES * 8;
    }
    const unsigned long long found = __ballot(hit);
    if (lane == 0 && found != 0ull) atomicOr(&sh_hit, found);
    __syncthreads();
    open = todo & ~sh_hit;
    __syncthreads();   // (every wave has read the pool before the next round adds to it)
  }
  if (wv == 0 && i < L) keep[(size_t)unit * Lcap + i] = (kept || ((sh_hit >> lane) & 1ull)) ? 1 : 0;
}

__global__ __launch_bounds__(WG) void corm_evict_mask_summary_kernel(const int32_t* last_hit, const int32_t* lens,
                                                                     const int32_t* t, const int32_t* t_first,
                                                                     uint8_t* keep, int Hkv, int Lcap, int w, int r) {
  const int unit = blockIdx.y;
  const int b = unit / Hkv;
  int L = lens[unit];
  L = L < 0 ? 0 : (L > Lcap ? Lcap : L);
  const int i = blockIdx.x * WG + threadIdx.x;
  if (i >= L) return;
  const int tcur = t[b];
  const bool full = tcur - t_first[b] + 1 >= w;
  const bool k = !full || last_hit[(size_t)unit * Lcap + i] > tcur - w || i >= L - r;
  keep[(size_t)unit * Lcap + i] = k ? 1 : 0;
}

// Diagnostic (Section 3, attention sparsity): per query head, the share of the unit's live keys whose
// recorded score of step t reaches c/t.  One workgroup per head.
__global__ __launch_bounds__(WG) void corm_row_density_kernel(const void* ring, int ring_mode, const int32_t* lens,
                                                              const int32_t* pos, const int32_t* t, float* density,
                                                              int Hq, int Hkv, int Lcap, int Tcap, int w, float c) {
  __shared__ int sh_cnt[WAVES];
  const int head = blockIdx.x;
  const int b = head / Hq, hq = head - b * Hq;
  const int unit = b * Hkv + hq / (Hq / Hkv);
  int L = lens[unit];
  L = L < 0 ? 0 : (L > Lcap ? Lcap : L);
  const int tcur = t[b];
  const bool step_ok = tcur >= 1 && tcur <= Tcap;
  const float thr = importance_threshold(c, step_ok ? tcur : 1);
  const size_t row = (size_t)head * w + (size_t)(step_ok ? (tcur - 1) % w : 0);
  int cnt = 0;
  for (int i0 = 0; i0 < L; i0 += WG) {
    const int i = i0 + (int)threadIdx.x;
    bool hit = false;
    if (i < L && step_ok) {
      const int pi = pos[(size_t)unit * Lcap + i];
      if (pi >= 0 && pi < Tcap && pi <= tcur - 1) {
        if (ring_mode == CORM_BIT) {
          hit = ((reinterpret_cast<const uint32_t*>(ring)[row * ((Tcap + 31) >> 5) + (size_t)(pi >> 5)] >> (pi & 31)) & 1u) != 0;
        } else {
          const size_t ri = row * Tcap + (size_t)pi;
          const float v = ring_mode == CORM_BF16
                              ? __uint_as_float((uint32_t) reinterpret_cast<const uint16_t*>(ring)[ri] << 16)
                              : reinterpret_cast<const float*>(ring)[ri];
          hit = v >= thr;
        }
      }
    }
    cnt += __popcll(__ballot(hit));
  }
  if ((threadIdx.x & 63) == 0) sh_cnt[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) tot += sh_cnt[i];
    density[head] = L > 0 ? (float)tot / (float)L : 0.f;
  }
}

__global__ void corm_threshold_kernel(float c, const int32_t* t, int n, float* thr) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) thr[i] = importance_threshold(c, t[i]);
}

__global__ void corm_fill_i32_kernel(int32_t* p, size_t n, int32_t v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace

#endif  // CORM_STANDALONE_HPP
