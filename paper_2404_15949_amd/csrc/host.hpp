// host side: workspace layout, validation, path selection and launches.
// Part of one translation unit: included by corm_kernels.hip, in this order, after <hip/hip_runtime.h> and corm.h.
#ifndef CORM_HOST_HPP
#define CORM_HOST_HPP

namespace {

// ---------------------------------------------------------------- host side

struct WorkspaceLayout {
  size_t counts_off, unit_state_off, keepbits_off, partials_off, logits_off, stage_meta_off, stage_k_off, stage_v_off;
  size_t seed_part_off, seed_stats_off, total;
  int nsplit, kb_stride;
  int seed_kb, seed_nkb;   // prompt seeding: keys per workgroup, key blocks per unit
};

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int row_bytes(const corm_desc* d) { return d->d * (d->kv_dtype == CORM_F32 ? 4 : 2); }

WorkspaceLayout workspace_layout(const corm_desc& d) {
  WorkspaceLayout w;
  w.nsplit = (d.Lcap + CHUNK - 1) / CHUNK;
  const size_t units = (size_t)d.B * d.Hkv, heads = (size_t)d.B * d.Hq;
  const size_t stage_rows = units * w.nsplit * CHUNK;   // every survivor of a chunk may be a boundary row
  w.counts_off = 0;
  w.kb_stride = (d.Lcap + 63) / 64;
  w.unit_state_off = align_up(units * w.nsplit * sizeof(int32_t), 256);
  w.keepbits_off = align_up(w.unit_state_off + units * sizeof(int2), 256);
  w.partials_off = align_up(w.keepbits_off + units * w.kb_stride * sizeof(unsigned long long), 256);
  w.logits_off = align_up(w.partials_off + heads * w.nsplit * MAX_PARTS_PER_CHUNK * (d.d + 2) * sizeof(float), 256);
  w.stage_meta_off = align_up(w.logits_off + heads * d.Lcap * sizeof(float), 256);   // (what lies in front of it is all that attend and record need)
  // (pass 2 of prompt seeding reads up to 63 queries past the last of a head: there is memory behind the last head's)
  w.seed_stats_off = align_up(w.stage_meta_off + stage_rows * 2 * sizeof(int32_t), 256);
  w.stage_k_off = align_up(w.seed_stats_off + heads * d.w * sizeof(float4), 256);
  w.stage_v_off = align_up(w.stage_k_off + stage_rows * row_bytes(&d), 256);
  w.seed_kb = row_bytes(&d) / 64 <= 4 ? PrefillGeom<256>::KB : PrefillGeom<512>::KB;
  w.seed_nkb = (d.Lcap + w.seed_kb - 1) / w.seed_kb;
  w.seed_part_off = align_up(w.stage_v_off + stage_rows * row_bytes(&d), 256);
  w.total = align_up(w.seed_part_off + heads * w.seed_nkb * d.w * sizeof(float2), 256);
  return w;
}

int validate_desc(const corm_desc* d) {
  if (!d) return CORM_EINVAL;
  if (d->B < 1 || d->Hq < 1 || d->Hkv < 1 || d->Lcap < 1 || d->Tcap < 1 || d->w < 1 || d->r < 1) return CORM_EINVAL;
  if (d->Hq % d->Hkv != 0) return CORM_EINVAL;
  if (!(d->thr_scale >= 0.f) || !std::isfinite(d->thr_scale)) return CORM_EINVAL;
  if (!(d->sm_scale >= 0.f) || !std::isfinite(d->sm_scale)) return CORM_EINVAL;
  if ((long long)d->B * d->Hkv > 2147483647LL / 2 || (long long)d->B * d->Hq > 2147483647LL / 2) return CORM_EINVAL;
  if (d->B * d->Hkv > 65535) return CORM_EUNSUPPORTED;  // grid.y limit
  if ((long long)d->Lcap * 512 >= (1LL << 31)) return CORM_EUNSUPPORTED;  // byte offsets inside a unit are 32-bit
  if (d->kv_dtype != CORM_F32 && d->kv_dtype != CORM_BF16) return CORM_EUNSUPPORTED;
  if (d->score_dtype != CORM_F32 && d->score_dtype != CORM_BF16 && d->score_dtype != CORM_BIT) return CORM_EUNSUPPORTED;
  if (d->d != 64 && d->d != 128) return CORM_EUNSUPPORTED;
  const int G = d->Hq / d->Hkv;
  if (G != 1 && G != 2 && G != 4 && G != 8) return CORM_EUNSUPPORTED;
  return CORM_OK;
}

bool misaligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }
bool misaligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) != 0; }

int launch_status() { return hipGetLastError() == hipSuccess ? CORM_OK : CORM_EHIP; }

// Per-call launch context: what corm_launch_opts asks for, plus the compute-unit count of the current
// device.  Nothing here outlives the call.
struct LaunchCtx {
  int path = 0;                               // 0 = choose by shape, 1 = split kernels (attend + record), 2 = fused
                                              // unit kernel, 3 = split kernels with q.K^T on the vector ALU even
                                              // where the MFMA kernel applies
  hipEvent_t ev0 = nullptr, ev1 = nullptr;    // recorded around the launch that streams K and V
  int cus = 256;
};

// Compute units of the current device, asked once per device (thread safe); 256 where no device answers.
constexpr int MAX_DEVICES = 64;
std::mutex g_device_mutex;
int g_device_cus[MAX_DEVICES] = {};

int device_cus() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return 256;
  std::lock_guard<std::mutex> lock(g_device_mutex);
  if (g_device_cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    g_device_cus[dev] = n;
  }
  return g_device_cus[dev];
}

int make_ctx(const corm_launch_opts* o, LaunchCtx* c) {
  *c = LaunchCtx();
  if (o) {
    if (o->path < 0 || o->path > 3) return CORM_EINVAL;
    if ((o->attend_start_event == nullptr) != (o->attend_stop_event == nullptr)) return CORM_EINVAL;
    c->path = o->path;
    c->ev0 = (hipEvent_t)o->attend_start_event;
    c->ev1 = (hipEvent_t)o->attend_stop_event;
  }
  c->cus = device_cus();
  return CORM_OK;
}

int check_workspace(const corm_desc* d, void* workspace, size_t workspace_bytes, WorkspaceLayout* wl) {
  *wl = workspace_layout(*d);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return CORM_EINVAL;
  if (workspace_bytes < wl->total) return CORM_ECAPACITY;
  return CORM_OK;
}

// fills the descriptor- and workspace-derived fields of p
void bind_params(const corm_desc* d, const WorkspaceLayout& wl, void* workspace, Params& p) {
  char* ws = reinterpret_cast<char*>(workspace);
  p.counts = reinterpret_cast<int32_t*>(ws + wl.counts_off);
  p.unit_state = reinterpret_cast<int2*>(ws + wl.unit_state_off);
  p.keepbits = reinterpret_cast<unsigned long long*>(ws + wl.keepbits_off);
  p.kb_stride = wl.kb_stride;
  p.partials = reinterpret_cast<float*>(ws + wl.partials_off);
  p.logits = reinterpret_cast<float*>(ws + wl.logits_off);
  p.B = d->B; p.Hq = d->Hq; p.Hkv = d->Hkv; p.Lcap = d->Lcap; p.Tcap = d->Tcap; p.w = d->w; p.r = d->r;
  p.nsplit = wl.nsplit;
  p.npart = wl.nsplit * MAX_PARTS_PER_CHUNK;
  p.part_keys = CHUNK;
  p.head_groups = 1;
  p.thr_scale = d->thr_scale;
  const float sm = d->sm_scale > 0.f ? d->sm_scale : 1.0f / sqrtf((float)d->d);
  p.scale_log2 = sm * LOG2E;
  p.ring_bf16 = d->score_dtype == CORM_BF16;
  p.ring_bits = d->score_dtype == CORM_BIT;
  p.ring_words = (d->Tcap + 31) / 32;
}

template <typename DT, int D, bool LAZY>
int launch_attend_g(const Params& p, int G, dim3 grid, hipStream_t s) {
  switch (G) {
    case 1: hipLaunchKernelGGL((corm_attend_kernel<DT, D, 1, LAZY>), grid, dim3(WG), 0, s, p); break;
    case 2: hipLaunchKernelGGL((corm_attend_kernel<DT, D, 2, LAZY>), grid, dim3(WG), 0, s, p); break;
    case 4: hipLaunchKernelGGL((corm_attend_kernel<DT, D, 4, LAZY>), grid, dim3(WG), 0, s, p); break;
    case 8: hipLaunchKernelGGL((corm_attend_kernel<DT, D, 8, LAZY>), grid, dim3(WG), 0, s, p); break;
    default: return CORM_EUNSUPPORTED;
  }
  return launch_status();
}

template <bool LAZY>
int launch_attend_gqa(const Params& p, int G, dim3 grid, hipStream_t s) {
  switch (G) {
    case 2: hipLaunchKernelGGL((corm_attend_gqa_kernel<2, LAZY>), grid, dim3(WG), 0, s, p); break;
    case 4: hipLaunchKernelGGL((corm_attend_gqa_kernel<4, LAZY>), grid, dim3(WG), 0, s, p); break;
    case 8: hipLaunchKernelGGL((corm_attend_gqa_kernel<8, LAZY>), grid, dim3(WG), 0, s, p); break;
    default: return CORM_EUNSUPPORTED;
  }
  return launch_status();
}

// grouped queries, bf16, d = 128: q.K^T on the matrix cores
bool attend_on_mfma(const corm_desc* d, const LaunchCtx& c) {
  return d->kv_dtype == CORM_BF16 && d->d == 128 && d->Hq > d->Hkv && c.path != 3;
}

template <bool LAZY>
int launch_attend_dt(const corm_desc* d, const Params& p, const LaunchCtx& c, int G, dim3 grid, hipStream_t s) {
  if (d->kv_dtype == CORM_F32)
    return d->d == 64 ? launch_attend_g<F32, 64, LAZY>(p, G, grid, s) : launch_attend_g<F32, 128, LAZY>(p, G, grid, s);
  if (attend_on_mfma(d, c)) return launch_attend_gqa<LAZY>(p, G, grid, s);
  return d->d == 64 ? launch_attend_g<BF16, 64, LAZY>(p, G, grid, s) : launch_attend_g<BF16, 128, LAZY>(p, G, grid, s);
}

int launch_attend(const corm_desc* d, const Params& p, const LaunchCtx& c, hipStream_t s) {
  const int G = d->Hq / d->Hkv / p.head_groups;
  const dim3 grid((d->Lcap + p.part_keys - 1) / p.part_keys, d->B * d->Hkv * p.head_groups);
  if (c.ev0 && hipEventRecord(c.ev0, s) != hipSuccess) return CORM_EHIP;
  const int rc = p.lazy ? launch_attend_dt<true>(d, p, c, G, grid, s) : launch_attend_dt<false>(d, p, c, G, grid, s);
  if (rc) return rc;
  if (c.ev1 && hipEventRecord(c.ev1, s) != hipSuccess) return CORM_EHIP;
  return CORM_OK;
}


size_t unit_lds_bytes(const corm_desc* d, int* lstride) {
  const int rowb = row_bytes(d);
  const int stage_rows = UNIT_WAVES * (64 / (rowb / 16)) * UNROLL;
  *lstride = (d->Lcap + 2 * stage_rows - 1) / (2 * stage_rows) * (2 * stage_rows);
  return (size_t)(d->Hq / d->Hkv) * (size_t)(*lstride) * sizeof(float);
}

// The unit kernel needs the unit's logits in LDS (48 KiB of dynamic LDS at most here, so that two
// workgroups fit a compute unit) and pays off once there are at least as many units as compute units.
bool use_unit_path(const corm_desc* d, const LaunchCtx& c) {
  int lstride;
  const bool fits = unit_lds_bytes(d, &lstride) <= 48 * 1024 && d->Hq / d->Hkv <= 4;  // G = 8 exceeds the register file
  if (c.path == 1 || c.path == 3 || !fits) return false;
  if (c.path == 2) return true;
  return d->B * d->Hkv >= c.cus;
}

template <typename DT, int D, bool LAZY>
int launch_unit_g(const Params& p, const LaunchCtx& c, int G, int units, size_t lds, int lstride, hipStream_t s) {
  // grouped queries: the small-stage instance (two workgroups per compute unit) once there are two units per
  // compute unit; measured on 32 query / 8 KV heads: 1024 units 161 -> 134 us per step, 512 units 139 -> 133 us,
  // but 256 units 81 -> 91 us
  const bool small = (long)p.B * p.Hkv >= 2L * c.cus;
  const dim3 grid(units), wg(UNIT_WG);
  switch (G) {
    case 1: hipLaunchKernelGGL((corm_unit_kernel<DT, D, 1, LAZY, UNROLL>), grid, wg, lds, s, p, lstride); break;
    case 2:
      if (small) hipLaunchKernelGGL((corm_unit_kernel<DT, D, 2, LAZY, UNROLL / 2>), grid, wg, lds, s, p, lstride);
      else hipLaunchKernelGGL((corm_unit_kernel<DT, D, 2, LAZY, UNROLL>), grid, wg, lds, s, p, lstride);
      break;
    case 4:
      if (small) hipLaunchKernelGGL((corm_unit_kernel<DT, D, 4, LAZY, UNROLL / 4>), grid, wg, lds, s, p, lstride);
      else hipLaunchKernelGGL((corm_unit_kernel<DT, D, 4, LAZY, UNROLL>), grid, wg, lds, s, p, lstride);
      break;
    default: return CORM_EUNSUPPORTED;
  }
  return launch_status();
}

template <bool LAZY>
int launch_unit_dt(const corm_desc* d, const Params& p, const LaunchCtx& c, int G, int units, size_t lds, int lstride,
                   hipStream_t s) {
  if (d->kv_dtype == CORM_F32)
    return d->d == 64 ? launch_unit_g<F32, 64, LAZY>(p, c, G, units, lds, lstride, s)
                      : launch_unit_g<F32, 128, LAZY>(p, c, G, units, lds, lstride, s);
  return d->d == 64 ? launch_unit_g<BF16, 64, LAZY>(p, c, G, units, lds, lstride, s)
                    : launch_unit_g<BF16, 128, LAZY>(p, c, G, units, lds, lstride, s);
}

int launch_unit(const corm_desc* d, const Params& p, const LaunchCtx& c, hipStream_t s) {
  int lstride;
  const size_t lds = unit_lds_bytes(d, &lstride);
  const int G = d->Hq / d->Hkv;
  const int units = (d->B * d->Hkv + UNIT_XCDS - 1) / UNIT_XCDS * UNIT_XCDS;   // grid: whole rounds over the XCDs
  if (c.ev0 && hipEventRecord(c.ev0, s) != hipSuccess) return CORM_EHIP;
  const int rc = p.lazy ? launch_unit_dt<true>(d, p, c, G, units, lds, lstride, s)
                        : launch_unit_dt<false>(d, p, c, G, units, lds, lstride, s);
  if (rc) return rc;
  if (c.ev1 && hipEventRecord(c.ev1, s) != hipSuccess) return CORM_EHIP;
  return CORM_OK;
}

// append (if p.do_append) + attend + record: one fused launch or the attend / record pair
int launch_attend_record(const corm_desc* d, const Params& p, const LaunchCtx& c, hipStream_t s);

template <int RC, int NT, bool APART>
int launch_record_rc(const corm_desc* d, const Params& p, int n_out, hipStream_t s) {
  const dim3 grid(d->B * d->Hkv, (p.nsplit + RC - 1) / RC + n_out);
  switch (d->Hq / d->Hkv) {
    case 1: hipLaunchKernelGGL((corm_record_kernel<1, RC, NT, APART>), grid, dim3(NT), 0, s, p, d->d, n_out); break;
    case 2: hipLaunchKernelGGL((corm_record_kernel<2, RC, NT, APART>), grid, dim3(NT), 0, s, p, d->d, n_out); break;
    case 4: hipLaunchKernelGGL((corm_record_kernel<4, RC, NT, APART>), grid, dim3(NT), 0, s, p, d->d, n_out); break;
    case 8: hipLaunchKernelGGL((corm_record_kernel<8, RC, NT, APART>), grid, dim3(NT), 0, s, p, d->d, n_out); break;
    default: return CORM_EUNSUPPORTED;
  }
  return launch_status();
}

int launch_record(const corm_desc* d, const Params& p, const LaunchCtx& c, hipStream_t s) {
  const int G = d->Hq / d->Hkv;
  const long units = (long)d->B * d->Hkv, want = 4L * c.cus;
  // the largest workgroup that still leaves about four workgroups per compute unit
  const int rc = units * ((p.nsplit + 3) / 4) >= want ? 4 : units * ((p.nsplit + 1) / 2) >= want ? 2 : 1;
  // A thread per key while the launch has at most two such workgroups per compute unit (eight heads a unit: three, if they can be more than half full),
  // else two keys a thread.  Whole steps, us, a thread per key | two keys: 256 workgroups of one head 16.5 | 16.9, 512 28.0 | 28.0, 640 36.0 | 35.0;
  // two heads 512 29.2 | 29.5, 640 37.6 | 36.6; four heads 512 32.5 | 33.2, 640 41.6 | 41.5, 800 52.3 | 51.3; eight heads 256 27.0 | 29.8, 512 39.9 | 41.6,
  // 768 65.6 | 66.0 and (384 units of two) 59.0 | 58.5, 840 68.0 | 67.5; 500 of 200 keys 31.0 | 31.2.
  const int nt = rc == 1 && units * p.nsplit <= (G == 8 && d->Lcap > CHUNK / 2 ? 3L : 2L) * c.cus ? CHUNK : WG;
  // workgroups that do a unit's out (record_out): an item a wave each or one, by the parts a full unit has
  const int items = G * (d->d / 64), nrec = (p.nsplit + rc - 1) / rc;
  const int n_out = (d->Lcap + p.part_keys - 1) / p.part_keys <= OUT_WAVE_PARTS ? (items + nt / 64 - 1) / (nt / 64) : items;
  // Where units have one record workgroup each and there are more of them than three and a half per compute unit, it does out itself: the chip
  // is full, and more workgroups only take longer to start (eight heads, us, apart | itself: 800 units x 450 keys 68.3 | 70.4, 1000 x 450
  // 76.5 | 76.2, 1000 x 196 53.7 | 52.3, 2000 x 450 147 | 137, 3000 x 450 211 | 194, 1500 x 2000 364 | 361).
  if (nrec == 1 && 2 * units > 7L * c.cus) return rc == 4 ? launch_record_rc<4, WG, false>(d, p, 0, s) : launch_record_rc<1, WG, false>(d, p, 0, s);
  if (rc == 4) return launch_record_rc<4, WG, true>(d, p, n_out, s);
  if (rc == 2) return launch_record_rc<2, WG, true>(d, p, n_out, s);
  return nt == WG ? launch_record_rc<1, WG, true>(d, p, n_out, s) : launch_record_rc<1, CHUNK, true>(d, p, n_out, s);
}

// Keys per attend workgroup on the split path: a whole chunk, or a half / a quarter of one while the
// launch would otherwise have fewer than about two workgroups per compute unit.  A part must hold whole
// pairs of pipeline stages of the kernel that runs.
int attend_part_keys(const corm_desc* d, const LaunchCtx& c) {
  const int stage_rows = attend_on_mfma(d, c) ? WAVES * 16 : WAVES * (64 / (row_bytes(d) / 16)) * UNROLL;
  const long want = 2L * c.cus;
  const long wgs = (long)d->B * d->Hkv * ((d->Lcap + CHUNK - 1) / CHUNK);
  int part = CHUNK;
  while (part / 2 >= 2 * stage_rows && CHUNK / (part / 2) <= MAX_PARTS_PER_CHUNK && wgs * (CHUNK / part) < want) part /= 2;
  return part;
}

// Workgroups that share a unit's query heads on the split path (vector-ALU kernel): while the launch would have fewer
// than two workgroups per compute unit, so that a part's dots and products of G heads do not run one after the
// other on a few of them (9 units of 8 heads, d 64, 840 keys: 63 workgroups 13.9 us, 504 of one head each 7.3 us).
// Each of them streams the part's rows.  With few heads left to each, a second workgroup per compute unit costs more in
// rows than it saves in products, with fp32 (more bytes a product) earlier than with bf16: about 200 -> 400 workgroups,
// fp32 d 128 of 2 heads 12.7 -> 16.2 us, of 4 heads 16.0 -> 17.6, of 8 heads 25.9 -> 22.6; fp32 d 64 of 2 heads 10.4 -> 11.8, of 4 12.6 ->
// 13.1; bf16 of 2 heads 11.4 -> 12.0 (d 64) and 11.8 -> 12.8 (d 128), of 4 heads 14.9 -> 14.2.
int attend_head_groups(const corm_desc* d, const LaunchCtx& c, int part_keys) {
  if (attend_on_mfma(d, c)) return 1;
  const int G = d->Hq / d->Hkv;
  const long wgs = (long)d->B * d->Hkv * ((d->Lcap + part_keys - 1) / part_keys);
  int n = 1;
  while (n < G && wgs * n * 2 <= 2L * c.cus && (long)d->B * d->Hkv * n * 2 <= 65535) {
    if (wgs * n * 2 > c.cus && G / (n * 2) < (d->kv_dtype == CORM_F32 ? 4 : 2)) break;
    n *= 2;
  }
  return n;
}

int launch_attend_record(const corm_desc* d, const Params& p0, const LaunchCtx& c, hipStream_t s) {
  if (use_unit_path(d, c)) return launch_unit(d, p0, c, s);
  Params p = p0;
  p.part_keys = attend_part_keys(d, c);
  p.head_groups = attend_head_groups(d, c, p.part_keys);
  const int rc = launch_attend(d, p, c, s);
  if (rc) return rc;
  return launch_record(d, p, c, s);
}

// A whole step in one launch (small.hpp)?  A unit is then one workgroup's alone, so only while its rows are few.  Whole steps in a
// captured graph, us, split launches | one, every slot in use, at which no key goes (in brackets: one does, at slot 0, so that every
// row moves).  fp32, rows of 256 bytes, 8 units: 64 slots 9.6 | 6.4 (12.3 | 7.4), 320 slots 9.9 | 7.7 (13.5 | 11.0), 640 slots
// 10.0 | 9.7 (14.9 | 15.1), 832 slots 10.0 | 11.6 (15.3 | 18.1); one unit of 640 slots 9.2 | 8.5 (13.3 | 14.5).  Two heads a
// unit, rows of 128 bytes: 640 slots 1.07 times as fast, 832 0.93; four heads: 256 slots 1.04, 320 0.97, 640 0.83.  From half the
// chip on the split launches share out less: 160 units of 1024 slots of 256 bytes 23.3 | 19.2, two heads 24.7 | 20.5, four
// 28.7 | 23.7.  What decides is the capacity, which the host knows: at the limits one launch is up to 8 % slower where every slot
// is in use, and with 52 keys in 576 slots (4 units that evict at every step) 14.0 | 11.2 as called from a program.  (Eight heads
// a unit, the deferred step and the two phases have no such kernel.)
bool small_step(const corm_desc* d, const LaunchCtx& c) {
  const int G = d->Hq / d->Hkv;
  if (c.path != 0 || c.ev0 || G > 4 || d->Lcap > SMALL_MAX_SLOTS || use_unit_path(d, c)) return false;
  if (attend_on_mfma(d, c)) return false;   // (the split launches form these logits on the matrix cores)
  const long kb = 2L * d->B * d->Hkv >= c.cus ? (G == 1 ? 256 : G == 2 ? 204 : 128) : (G == 1 ? 160 : G == 2 ? 104 : 40);
  return (long)d->Lcap * row_bytes(d) <= kb * 1024;
}

template <typename DT, int D, int G>
int launch_small_g(const Params& p, int units, hipStream_t s) {
  constexpr int stage_rows = Attend<DT, D, G, WAVES>::STAGE_ROWS;
  const int lstride = (p.Lcap + stage_rows - 1) / stage_rows * stage_rows, parts = (p.Lcap + p.part_keys - 1) / p.part_keys;
  hipLaunchKernelGGL((corm_small_kernel<DT, D, G>), dim3(units), dim3(SMALL_WG),
                     small_lds_floats(G, D, lstride, parts) * sizeof(float), s, p, lstride, parts);
  return launch_status();
}

template <typename DT, int D>
int launch_small_dt(const Params& p, int G, int units, hipStream_t s) {
  switch (G) {
    case 1: return launch_small_g<DT, D, 1>(p, units, s);
    case 2: return launch_small_g<DT, D, 2>(p, units, s);
    case 4: return launch_small_g<DT, D, 4>(p, units, s);
    default: return CORM_EUNSUPPORTED;
  }
}

int launch_small(const corm_desc* d, const Params& p0, const LaunchCtx& c, hipStream_t s) {
  const int G = d->Hq / d->Hkv, units = d->B * d->Hkv;
  Params p = p0;
  p.part_keys = attend_part_keys(d, c);
  if (d->kv_dtype == CORM_F32)
    return d->d == 64 ? launch_small_dt<F32, 64>(p, G, units, s) : launch_small_dt<F32, 128>(p, G, units, s);
  if (d->d == 64) return launch_small_dt<BF16, 64>(p, G, units, s);
  return G == 1 ? launch_small_g<BF16, 128, 1>(p, units, s) : CORM_EUNSUPPORTED;
}

// Policy of the compaction: exact mode compacts every unit that lost a key; lazy mode only
// units whose dead slots reach dead_num / dead_den of their slots.
struct CompactPolicy {
  int lazy = 0, dead_num = 0, dead_den = 1;
  unsigned long long* live = nullptr;   // lazy mode: the caller's live masks
  int32_t* nlive = nullptr;             // optional output: live keys per unit
  bool bulk = false;                    // prompt seeding: most of a unit may go at once
};

// One launch of column slabs, or two of chunks?  A slab is one serial walk over its unit: where units * slabs leave compute
// units idle, the chunks of a long unit share the work better (a hole at slot 0 of every unit, slabs | chunks, us, with
// the 2-3 us of the count launch; rows of 256 bytes): 1 unit x 2048 slots 11 | 13, 4096: 16 | 13, 16384: 53 | 14;
// 8 x 4096: 18 | 16, 16384: 56 | 30; 32 x 4096: 27 | 31, 16384: 136 | 94; 128 x 4096: 103 | 94; 512 x 4096: 441 | 443.  Where
// nothing is to be moved, and where a unit of many slots has few left, the slabs are a launch less (32 x 4096: 4.8 | 6.3),
// unless very many units pay for more workgroups (slabs + 1 each) than they have chunks (768 units x 512 slots of 512
// bytes 16.4 | 7.5).
// The limits are those of whole decode steps that evict at every step, now and then, and never (2 to 768 units, 300 to
// 16000 slots, 900 shapes): within them slabs are at worst 4 % slower than chunks and up to 45 % faster, beyond them up to 45 % slower
// (8 units x 11700 slots: 59 us a step by slabs, 34 by chunks).
// bulk: prompt seeding, whose eviction leaves few rows to walk (measured like that: 3 to 20 % faster by slabs); very many
// workgroups with nothing to walk cost the same there.
bool compact_by_slabs(int units, int Lcap, int rowb, bool bulk) {
  if (Lcap > SLAB_MAX_SLOTS) return false;
  const long slabs = 2 * rowb / slab_bytes(rowb), walks = units * slabs;
  const int nsplit = (Lcap + CHUNK - 1) / CHUNK;
  if (walks + units > 8192 && 2 * (slabs + 1) > 3 * nsplit) return false;
  if (bulk) return Lcap <= 5632 || walks >= 64;
  if (walks >= 1536) return true;
  if (rowb <= 128) return Lcap <= (walks > 128 && walks < 512 ? 2304 : 2816);
  return Lcap <= (rowb <= 256 && walks > 192 && walks < 320 ? 3072 : 4352);
}

template <int ROWB>
void launch_compact_rows(const CompactArgs& a, bool bulk, hipStream_t s) {
  if (compact_by_slabs(a.units, a.Lcap, ROWB, bulk)) {
    const int groups = (a.units + SLAB_XCDS - 1) / SLAB_XCDS * SLAB_XCDS;
    hipLaunchKernelGGL((corm_compact_slab_kernel<ROWB>), dim3(groups * (2 * ROWB / slab_bytes(ROWB) + 1)), dim3(SLAB_WG),
                       (size_t)a.Lcap * sizeof(uint16_t), s, a);
    return;
  }
  const dim3 grid(a.nsplit, a.units);
  hipLaunchKernelGGL((corm_compact_local_kernel<ROWB>), grid, dim3(CWG), 0, s, a);
  hipLaunchKernelGGL((corm_compact_boundary_kernel<ROWB>), grid, dim3(WG), 0, s, a);
}

// count_first: derive the per-split counts from the caller's mask
int launch_compact(const corm_desc* d, const WorkspaceLayout& wl, void* workspace, void* K, void* V, int32_t* pos,
                   int32_t* last_hit, int32_t* lens, const uint8_t* keep, int32_t* kept_idx, bool count_first,
                   const CompactPolicy& pol, hipStream_t s) {
  char* ws = reinterpret_cast<char*>(workspace);
  CompactArgs a;
  a.K = reinterpret_cast<char*>(K);
  a.V = reinterpret_cast<char*>(V);
  a.pos = pos; a.last_hit = last_hit; a.lens = lens; a.keep = keep; a.kept_idx = kept_idx;
  a.keepbits = reinterpret_cast<unsigned long long*>(ws + wl.keepbits_off);
  a.live = pol.live;
  a.kb_stride = wl.kb_stride;
  int32_t* counts = reinterpret_cast<int32_t*>(ws + wl.counts_off);
  a.counts = counts;
  a.unit_state = reinterpret_cast<int2*>(ws + wl.unit_state_off);
  a.nlive = pol.nlive;
  a.stage_k = ws + wl.stage_k_off;
  a.stage_v = ws + wl.stage_v_off;
  a.stage_meta = reinterpret_cast<int32_t*>(ws + wl.stage_meta_off);
  a.units = d->B * d->Hkv; a.nsplit = wl.nsplit; a.Lcap = d->Lcap;
  a.lazy = pol.lazy; a.dead_num = pol.dead_num; a.dead_den = pol.dead_den;
  const dim3 grid(wl.nsplit, d->B * d->Hkv);
  if (count_first) {
    hipLaunchKernelGGL(corm_count_kernel, grid, dim3(WG), 0, s, a, counts);
    if (launch_status()) return CORM_EHIP;
  }
  switch (row_bytes(d)) {
    case 128: launch_compact_rows<128>(a, pol.bulk, s); break;
    case 256: launch_compact_rows<256>(a, pol.bulk, s); break;
    case 512: launch_compact_rows<512>(a, pol.bulk, s); break;
    default: return CORM_EUNSUPPORTED;
  }
  return launch_status();
}

// How many workgroups share the query blocks of a key block (prompt seeding).
// bf16, where the latency of a block bounds the passes: a workgroup's time is its blocks and about one more (it loads its
// keys once, whatever the number of blocks), the launch takes that times the workgroups that each of two slots per
// compute unit gets, at least one; a split that gains less than a twentieth by this count is not made (4 units x 900
// keys, w 256: 49.6 us unsplit, 28.1; 8 units x 5000, w 700: 86.8, 60.3).
// fp32, where the matrix cores bound them: about SEED_WGS workgroups of at least two blocks, and no split in two, after
// which some compute units have two workgroups and others one (16 units x 2000 keys, 8 blocks: one workgroup 48 + 74
// us for the two passes, four 30 + 39 (two workgroups 45 us more than four); 16 units x 3000, 5 blocks: one 32 + 40, two 37 + 42).
constexpr int SEED_WGS = 1024;
void seed_segments(const corm_desc* d, const LaunchCtx& c, int m, long long key_blocks, int32_t* nseg,
                   int32_t* seg_blocks) {
  const int qt = (row_bytes(d) <= 256 ? PrefillGeom<256>::QT : PrefillGeom<512>::QT);
  const int blocks = ((m + 15) / 16 * (d->Hq / d->Hkv) + qt - 1) / qt;
  int n = 1;
  if (d->kv_dtype == CORM_F32) {
    n = (int)std::min((SEED_WGS + key_blocks - 1) / key_blocks, (long long)(blocks / 2));
    if (n < 3) n = 1;
  } else {
    double best = 0.;
    for (int i = 1; i <= std::min(blocks, 64); ++i) {
      const double cost = std::max(1., (double)key_blocks * i / (2. * c.cus)) * ((blocks + i - 1) / i + 1);
      if (i > 1 && cost > 0.95 * best) continue;
      best = cost;
      n = i;
    }
  }
  *seg_blocks = (blocks + n - 1) / n;
  *nseg = (blocks + *seg_blocks - 1) / *seg_blocks;
}

// Pass 1: query tiles per wave (max_qw, or 1) and how many workgroups share the keys of a query block (segments of whole
// key blocks; the partials have room for one per key block).  A launch takes its rounds over the chip (three workgroups per
// compute unit by registers, of the small ones four by LDS, which share it badly) times a segment's key tiles by the wave's query tiles and a fixed part
// (queries, first keys, the end).  Whole calls, us, one query tile and four per wave, each with its best number of segments, the rule's
// choice last: 512 heads x 1024 queries x 4096 keys 1892, 1666: 1671; 32 heads 147, 139: 139; 8 heads x 700 x 5000 66, 70: 65; 4 heads x
// 256 x 900 28, 36: 28; 64 heads x 48 x 20000 235, 252: 234.  Unsplit the last three take 103, 35 and 412.
constexpr double STATS_FIXED = 24., STATS_TILE = 1.5;
int stats_segments(const corm_desc* d, const LaunchCtx& c, const WorkspaceLayout& wl, int max_qw, PrefillArgs& a) {
  const int ntt = (a.m + 15) / 16 * (d->Hq / d->Hkv);
  const long long units = d->B * d->Hkv;
  double best = 0.;
  int qw = max_qw, n = 0;
  for (int w = max_qw; w >= 1; w -= w > 1 ? w - 1 : 1)
    for (int i = 1; i <= std::min(wl.seed_nkb, 64); ++i) {
      const long long wgs = units * ((ntt + WAVES * w - 1) / (WAVES * w)) * i, slots = (w > 1 ? 6LL : 7LL) * c.cus / 2;
      const int tiles = (wl.seed_nkb + i - 1) / i * (wl.seed_kb / 16);
      const double cost = (double)((wgs + slots - 1) / slots) * (tiles * (w + STATS_TILE) + STATS_FIXED);
      if (n > 0 && cost > 0.95 * best) continue;
      best = cost;
      qw = w;
      n = i;
    }
  a.nqb = (ntt + WAVES * qw - 1) / (WAVES * qw);
  a.kseg = (wl.seed_nkb + n - 1) / n * wl.seed_kb;
  a.nks = (d->Lcap + a.kseg - 1) / a.kseg;
  return qw;
}

template <typename DT, int D>
int launch_prefill_dt(const corm_desc* d, const LaunchCtx& c, const WorkspaceLayout& wl, PrefillArgs& a, dim3 grid,
                      dim3 mgrid, hipStream_t s) {
  constexpr int MAX_QW = stats_qw<DT>();
  const int qw = stats_segments(d, c, wl, MAX_QW, a);
  const long long wgs = (long long)PREFILL_XCDS * ((a.units + PREFILL_XCDS - 1) / PREFILL_XCDS) * a.nqb * a.nks;
  if (wgs > 2147483647LL) return CORM_EUNSUPPORTED;
  if (qw == MAX_QW) hipLaunchKernelGGL((corm_prefill_stats_kernel<DT, D, MAX_QW>), dim3((unsigned)wgs), dim3(WG), 0, s, a);
  else hipLaunchKernelGGL((corm_prefill_stats_kernel<DT, D, 1>), dim3((unsigned)wgs), dim3(WG), 0, s, a);
  hipLaunchKernelGGL(corm_prefill_merge_kernel, mgrid, dim3(256), 0, s, a);
  // (a head's ring of more than DEAD_OFFSET bytes, 8 heads x 4096 rows x 270336 bf16 positions: 1269 us by the general
  // blocks, 927 by the rows of a tile)
  const uint64_t row = a.ring_bits ? (uint64_t)a.ring_words * 4 : (uint64_t)a.Tcap * (a.ring_bf16 ? 2 : 4);
  const bool far = a.ring && a.w * row > DEAD_OFFSET;
  auto scores = [&](auto near_kernel, auto far_kernel) {
    if (far) hipLaunchKernelGGL(far_kernel, grid, dim3(WG), 0, s, a);
    else hipLaunchKernelGGL(near_kernel, grid, dim3(WG), 0, s, a);
  };
  if (a.ring_bits) scores(corm_prefill_scores_kernel<DT, D, SEED_BITS, false>, corm_prefill_scores_kernel<DT, D, SEED_BITS, true>);
  else if (a.ring_bf16) scores(corm_prefill_scores_kernel<DT, D, SEED_BF16, false>, corm_prefill_scores_kernel<DT, D, SEED_BF16, true>);
  else scores(corm_prefill_scores_kernel<DT, D, SEED_F32, false>, corm_prefill_scores_kernel<DT, D, SEED_F32, true>);
  return launch_status();
}

int check_step_pointers(const void* q, const void* k_new, const void* v_new, const void* K, const void* V,
                        const int32_t* lens, const int32_t* pos, const int32_t* last_hit, const int32_t* t,
                        const int32_t* t_first, const void* score_ring, const float* out, const int32_t* kept_idx,
                        const int32_t* status) {
  if (!q || !k_new || !v_new || !K || !V || !lens || !pos || !last_hit || !t || !t_first || !out)
    return CORM_EINVAL;   // (score_ring may be null: summary-only state)
  if (misaligned16(q) || misaligned16(k_new) || misaligned16(v_new) || misaligned16(K) || misaligned16(V) ||
      misaligned4(out) || misaligned4(score_ring))
    return CORM_EINVAL;
  if (misaligned4(lens) || misaligned4(pos) || misaligned4(last_hit) || misaligned4(t) || misaligned4(t_first) ||
      misaligned4(kept_idx) || misaligned4(status))
    return CORM_EINVAL;
  return CORM_OK;
}

}  // namespace

#endif  // CORM_HOST_HPP
