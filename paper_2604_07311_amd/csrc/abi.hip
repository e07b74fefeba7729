// C ABI: handles, plans, planning (tile choice, indexing-vector upload) and
// execution.  Errors are returned as famlies_status with a thread-local
// message (graceful error handling and bounds checking: Girder 1, "Code
// safety").
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "famlies.h"
#include "internal.hpp"
#include "launch.hpp"
#include "runtime.hpp"

// Device scratch of famlies_contract_noalloc: the indexing vectors and
// split-K partial sums of the call in flight, one copy per device, held until
// the process ends.  Host code never passes `scratch` itself to a kernel or
// a copy (in host code the name is only a stand-in): the device address is
// resolved per device with hipGetSymbolAddress and kept (g_scratch_addr).
static constexpr size_t kNoAllocScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace famlies {

static std::mutex g_scratch_mu;
static void* g_scratch_addr[64] = {};

// The scratch array's address on `device` (resolved once, with that device
// current).
static famlies_status scratch_address(int device, void** out) {
  if (device < 0 || device >= 64) return fail(FAMLIES_ERR_UNSUPPORTED, "device index above 63");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_addr[device]) {
    DeviceGuard dg(device);
    if (!dg.ok) return fail(FAMLIES_ERR_DEVICE, "cannot select the device");
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!ptr) return fail(FAMLIES_ERR_DEVICE, "hipGetSymbolAddress(scratch) returned null");
    g_scratch_addr[device] = ptr;
  }
  *out = g_scratch_addr[device];
  return FAMLIES_OK;
}

famlies_status hip_fail(hipError_t e, const char* what) {
  set_error(std::string(what) + ": " + hipGetErrorString(e));
  return e == hipErrorOutOfMemory ? FAMLIES_ERR_ALLOC : FAMLIES_ERR_DEVICE;
}

// Make `device` current for the scope, restoring the caller's device after.
DeviceGuard::DeviceGuard(int device) {
  ok = hipGetDevice(&prev) == hipSuccess;
  if (ok && prev != device) ok = hipSetDevice(device) == hipSuccess;
  else if (ok) prev = -1;
}
DeviceGuard::~DeviceGuard() {
  if (prev >= 0) (void)hipSetDevice(prev);
}

// Contracted offsets of an operand's pre-packed form -- block (tile, kb) of br x
// bk elements, [row][k] -- for the direct kernel, which then reads a packed
// operand like any other and sums in the same order (it works out the rows).
static void packed_ks(int64_t kd, int br, int bk, int64_t es, std::vector<uint32_t>* pk) {
  const int64_t n = ceil_div(kd, bk) * bk;
  for (int64_t k = 0; k < (int64_t)pk->size(); ++k)
    (*pk)[(size_t)k] = k < n ? (uint32_t)((k / bk * br * bk + k % bk) * es) : 0u;
}

template <typename OffT>
static famlies_status index_image(famlies_plan_s* p, const PlanUse& use, int64_t mp, int64_t np, int64_t kp,
                                  std::vector<char>* image) {
  const Analysis& an = p->an;
  std::vector<int64_t> v[9];
  offsets(an.I, 0, an.M, mp, v[0]);
  offsets(an.P, 0, an.K, std::max(an.K, kp), v[1]);
  offsets(an.P, 1, an.K, std::max(an.K, kp), v[2]);
  offsets(an.J, 1, an.N, np, v[3]);
  offsets(an.I, 2, an.M, mp, v[4]);
  offsets(an.J, 2, an.N, np, v[5]);
  offsets(an.Lm, 0, an.L, an.L, v[6]);
  offsets(an.Lm, 1, an.L, an.L, v[7]);
  offsets(an.Lm, 2, an.L, an.L, v[8]);
  // 32-bit forms rebase the row vectors to each operand's lowest element;
  // the byte form also scales every offset to bytes
  const bool rebase = sizeof(OffT) == 4, bytes = std::is_same<OffT, uint32_t>::value;
  const int64_t es = an.esize;
  vec_flags(an, p->cfg.bk, sizeof(OffT) == 4 ? 32 : 64, v, &p->x_vec, &p->y_vec);
  // host-side bounds check of the vectors against the descriptors' spans
  const int64_t x_lo = an.swapped ? an.b_lo : an.a_lo, x_hi = an.swapped ? an.b_hi : an.a_hi;
  const int64_t y_lo = an.swapped ? an.a_lo : an.b_lo, y_hi = an.swapped ? an.a_hi : an.b_hi;
  if ((an.K > 0 && (!offsets_in_span(v[0], an.M, v[1], an.K, v[6], an.L, x_lo, x_hi) ||
                    !offsets_in_span(v[3], an.N, v[2], an.K, v[7], an.L, y_lo, y_hi))) ||
      !offsets_in_span(v[4], an.M, v[5], an.N, v[8], an.L, an.c_lo, an.c_hi))
    return fail(FAMLIES_ERR_BOUNDS, "planner: an indexing vector addresses outside its tensor's span");
  p->xmode = an.x_kfast ? (p->x_vec ? 3 : 1) : 0;
  p->ymode = an.y_kfast ? (p->y_vec ? 3 : 1) : 0;
  // the kernels' contracted order (the plain one, or padded to 16-byte runs)
  // and its void mask, with byte offsets
  std::vector<uint32_t> kvoid;
  const int u = 16 / an.esize;
  if (bytes && !(use.scratch && use.lean)) {  // nothing reads the mask there: no runs, nothing pre-packed
    kvoid.assign((size_t)(ceil_div(kp, 32) + 1), 0);
    KRuns kr;
    const bool padded = p->kd != an.K;
    if (padded) {
      padded_k_runs(an, u, &kr);
      for (int i = 1; i <= 2; ++i) {
        std::vector<int64_t> w((size_t)kp, 0);
        for (int64_t k = 0; k < p->kd; ++k) w[(size_t)k] = v[i][(size_t)kr.index[(size_t)k]];
        v[i].swap(w);
      }
    }
    for (int64_t k = 0; k < (int64_t)kvoid.size() * 32; ++k)
      if (k >= p->kd || (padded && kr.skip[(size_t)k])) kvoid[(size_t)(k >> 5)] |= 1u << (k & 31);
    p->dx_vec = contiguous_k_runs(v[1], p->kd, u);
    p->dy_vec = contiguous_k_runs(v[2], p->kd, u);
    const int run = padded || p->kd % p->cfg.bk ? 4 : 3;
    if (an.x_kfast) p->xmode = p->dx_vec ? run : 1;
    if (an.y_kfast) p->ymode = p->dy_vec ? run : 1;
  }
  for (int i = 1; i <= 2; ++i) v[i].resize((size_t)kp);
  std::vector<uint32_t> packed[2];  // direct kernel: k's of a packed X, of a packed Y
  if (p->direct.bm && bytes && !use.scratch)
    for (int op = 0; op < 2; ++op) {
      const int64_t rows = op ? np : mp;
      const int br = op ? p->cfg.bn : p->cfg.bm;
      packed[op].resize((size_t)kp);
      packed_ks(p->kd, br, p->cfg.bk, es, &packed[op]);
      p->pk_fits[op] = rows * ceil_div(p->kd, p->cfg.bk) * p->cfg.bk * es < ((int64_t)1 << 32);
    }
  // rows and contracted offsets are rebased each by its own lowest, so every
  // entry of the byte form counts up from the operand's lowest element
  const int64_t shift[6] = {an.x_lo - an.xk_lo, an.xk_lo, an.yk_lo, an.y_lo - an.yk_lo, an.c_lo_mn, 0};
  size_t n6 = kvoid.size();
  for (int i = 0; i < 6; ++i) n6 += v[i].size();
  for (const auto& x : packed) n6 += x.size();
  const size_t b6 = (n6 * sizeof(OffT) + 7) & ~(size_t)7;
  const size_t total = b6 + 3 * (size_t)an.L * sizeof(int64_t);
  std::vector<char>& host = *image;
  host.assign(total, 0);
  OffT* o = reinterpret_cast<OffT*>(host.data());
  size_t pos = 0;
  for (int i = 0; i < 6; ++i) {
    p->off_pos[i] = pos;
    for (int64_t x : v[i]) {
      if (bytes)
        o[pos++] = (OffT)(uint64_t)((x - shift[i]) * es);  // wraps modulo 2^32 on purpose
      else if (rebase)
        o[pos++] = (OffT)(x - shift[i]);  // |value| < 2^31 (index_form)
      else
        o[pos++] = (OffT)x;
    }
  }
  for (int i = 0; i < 2; ++i) {
    p->pk_pos[i] = pos;
    for (uint32_t x : packed[i]) o[pos++] = (OffT)x;
  }
  p->kvoid_pos = pos;
  p->has_kvoid = !kvoid.empty();
  for (uint32_t x : kvoid) o[pos++] = (OffT)x;
  int64_t* lb = reinterpret_cast<int64_t*>(host.data() + b6);
  for (int i = 0; i < 3; ++i) {
    p->off_pos[6 + i] = (size_t)i * (size_t)an.L;
    for (int64_t l = 0; l < an.L; ++l) lb[i * an.L + l] = v[6 + i][(size_t)l];
  }
  p->batch_off_bytes = b6;
  return FAMLIES_OK;
}

template <typename OffT>
static PlainArgs<OffT> make_args(const famlies_plan_s* p, const void* x, const void* y, void* c,
                                 double alpha, double beta, bool extra) {
  PlainArgs<OffT> a;
  const OffT* o = static_cast<const OffT*>(p->d_off);
  const int64_t* lb = reinterpret_cast<const int64_t*>(static_cast<const char*>(p->d_off) + p->batch_off_bytes);
  const bool rebased = sizeof(OffT) == 4;
  const int64_t es = p->an.esize;
  // in the 32-bit forms the kernel addresses each operand from its lowest element
  a.x = x ? static_cast<const char*>(x) + (rebased ? p->an.x_lo * es : 0) : nullptr;
  a.y = y ? static_cast<const char*>(y) + (rebased ? p->an.y_lo * es : 0) : nullptr;
  a.c = static_cast<char*>(c) + (rebased ? p->an.c_lo_mn * es : 0);
  a.xmn = o + p->off_pos[0];
  a.xk = o + p->off_pos[1];
  a.yk = o + p->off_pos[2];
  a.ymn = o + p->off_pos[3];
  a.cm = o + p->off_pos[4];
  a.cn = o + p->off_pos[5];
  a.xl = lb + p->off_pos[6];
  a.yl = lb + p->off_pos[7];
  a.cl = lb + p->off_pos[8];
  a.M = (int32_t)p->an.M;
  a.N = (int32_t)p->an.N;
  a.kvoid = p->has_kvoid ? reinterpret_cast<const uint32_t*>(o + p->kvoid_pos) : nullptr;
  a.K = (int32_t)p->kd;
  a.L = (int32_t)p->an.L;
  a.x_nkb = 0;
  a.y_nkb = 0;
  a.tiles_m = (int32_t)ceil_div(p->an.M, p->cfg.bm);
  a.tiles_n = (int32_t)ceil_div(p->an.N, p->cfg.bn);
  a.splits = p->cfg.split;
  a.kchunk = p->kchunk;
  a.head = p->head;
  a.rem = extra ? p->level.rem : 0;
  if (a.rem) {
    a.splits = 1;
    a.head = p->level.head;
    a.lev_q = p->level.q;
    a.lev_part = p->level.part;
    a.lev_parts = p->level.parts;
  }
  a.alpha = alpha;
  a.beta = beta;
  a.work = p->d_work;
  return a;
}

// Planning decisions and the host image of the indexing vectors, touching no
// device memory: p->cfg, the split settlement, the loader flags, the vector
// positions and p->work_bytes (the split-K workspace the plan needs).
// *image is left empty when C has no elements.
static famlies_status prepare_plan(famlies_handle_s* h, famlies_plan_s* p, int dtype, int compute,
                                   const famlies_tensor* A, const famlies_tensor* B, const famlies_tensor* C,
                                   const PlanUse& use, std::vector<char>* image) {
  const TileCfg* force = use.force;
  const bool lean = use.lean;
  Analysis an;
  std::string err;
  int st = analyze(dtype, compute, A, B, C, &an, &err);
  if (st != FAMLIES_OK) return fail(st, err);
  const int64_t lim = kMaxGemmDim;
  if (an.M > lim || an.N > lim || an.K > lim || an.L > lim)
    return fail(FAMLIES_ERR_UNSUPPORTED, "a GEMM dimension exceeds 2^31 - 1024");
  p->h = h;
  p->an = an;
  const int i8 = int8_slices(compute);
  p->cfg = i8 ? int8_tile(i8, lean ? 64 : an.N) : force ? *force : choose_tiles(h, an, &p->table_hit, use.table);
  if (i8 && force) p->cfg.index_bits = force->index_bits;
  index_form(an, p->cfg.index_bits, &p->index_bits, &p->elem32);
  const int ns = split_parts(compute);
  // contracted order of the kernels: padded to 16-byte runs where that pays
  const int64_t runs =
      lean || p->index_bits != 32 || p->elem32 ? 0 : padded_k_length(an, 16 / an.esize);
  p->kd = runs && runs <= lim ? runs : an.K;
  if (i8) {
    // int8_tile (the narrow one in a lean plan: it pads N least), no tile table;
    // K ranges where tiles are few
    if (!lean && !use.bare && an.L == 1 && p->kd <= int8_exact_k(i8)) p->cfg.split = int8_split(h, an, p->cfg, p->kd);
  } else if (ns) {
    // the bf16 kernels split every tile or none: a tail split becomes none
    if (p->cfg.tail) {
      p->cfg.split = 1;
      p->cfg.tail = 0;
    }
    p->cfg.bk = split_slice_k(ns);
    if (!force && tall_tile(an, p->cfg, runs)) {
      p->cfg.bm = 256;
      p->cfg.bn = 128;
    }
    if (!split_tile_supported(ns, p->cfg.bm, p->cfg.bn)) p->cfg.bm = p->cfg.bn = 128;
  } else if (!plain_tile_supported(dtype, p->cfg.bm, p->cfg.bn, p->cfg.bk)) {
    p->cfg.bm = p->cfg.bn = 128;
    p->cfg.bk = dtype == FAMLIES_F64 ? 8 : 32;
  }
  if (an.L > 1) p->cfg.split = 1;  // batch modes already multiply the tile count
  const int64_t ntiles = ceil_div(an.M, p->cfg.bm) * ceil_div(an.N, p->cfg.bn);
  finalize_split(&p->cfg, p->kd, ntiles, &p->kchunk, &p->head);
  if (ntiles * p->cfg.split * an.L >= ((int64_t)1 << 31))
    return fail(FAMLIES_ERR_UNSUPPORTED, "the tile grid exceeds 2^31 workgroups");
  const ChainCfg chain = plan_chain(an, p->cfg, p->kd, ntiles, p->kchunk);
  double level_us = 1e30;
  if (!lean && !force && !p->table_hit && !i8) {
    bool unsplit = false;
    p->level = choose_level(h, an, p->cfg, p->kd, chain, &unsplit, &level_us);
    if (use.bare) p->level = LevelCfg();
    if (unsplit) {
      p->cfg.split = 1;
      p->cfg.tail = 0;
      finalize_split(&p->cfg, p->kd, ntiles, &p->kchunk, &p->head);
    }
  }
  LevelCfg planes_level;
  if (use.planes && !use.bare && !lean && !force && !p->table_hit && ns && p->index_bits == 32 && !p->elem32)
    p->planes = choose_planes(h, an, p->kd, chain, level_us, &planes_level, &p->planes_fold);
  if (!lean && !force && !p->table_hit && !i8 && !ns && p->index_bits == 32 && !p->elem32) {
    p->direct = choose_direct(h, an, p->cfg, chain, level_us);
    if (use.bare && p->direct.split > 1) p->direct = DirectCfg();
    if (p->direct.bm) {
      p->level = LevelCfg();
      const int ks = 64 / an.esize;
      DirectCfg& d = p->direct;
      if (an.L > 1) d.split = 1;
      d.kchunk = (int)(ceil_div(ceil_div(p->kd, d.split), ks) * ks);
      d.split = (int)ceil_div(p->kd, d.kchunk);
    }
  }
  image->clear();
  p->work_bytes = 0;
  if (an.M == 0 || an.N == 0) return FAMLIES_OK;
  const int64_t mp = ceil_div(std::max<int64_t>(an.M, 1), p->cfg.bm) * p->cfg.bm;
  const int64_t np = ceil_div(std::max<int64_t>(an.N, 1), p->cfg.bn) * p->cfg.bn;
  int64_t kp = ceil_div(std::max<int64_t>(p->kd, 1), p->cfg.bk) * p->cfg.bk + p->cfg.bk;
  if (p->planes) kp = std::max(kp, ceil_div(p->kd, 64) * 64);
  st = p->index_bits == 64 ? index_image<int64_t>(p, use, mp, np, kp, image)
       : p->elem32          ? index_image<int32_t>(p, use, mp, np, kp, image)
                            : index_image<uint32_t>(p, use, mp, np, kp, image);
  if (st != FAMLIES_OK) return st;
  if (i8 && an.K > 0) {
    p->work_bytes = int8_work_bytes(i8, an.M, an.N, p->kd, an.L, p->cfg.bn, p->cfg.split);  // digit planes and exponents
  } else if (p->cfg.split > 1 && an.K > 0) {
    // one BM x BN block per split tile and K slice (of FP64 sums in the bf16 kernels)
    p->work_bytes = ns ? (size_t)p->cfg.split * (size_t)mp * (size_t)np * 8
                       : (size_t)p->cfg.split * (size_t)(ntiles - p->head) * (size_t)p->cfg.bm *
                             (size_t)p->cfg.bn * (size_t)an.esize;
  }
  const size_t own = p->work_bytes;  // what the tile choice needs by itself
  if (p->planes) {
    p->planes_level = planes_level;
    p->work_bytes = std::max(p->work_bytes, planes_work_bytes(ns, an.M, an.N, p->kd, an.L, planes_level, p->planes_fold));
  }
  if (p->level.rem)
    p->work_bytes = std::max(p->work_bytes, (size_t)p->level.blocks() * 128 * 128 * (ns ? 8 : (size_t)an.esize));
  if (p->direct.bm && p->direct.split > 1)
    p->work_bytes = std::max(p->work_bytes, (size_t)p->direct.split * (size_t)ceil_div(an.M, p->direct.bm) *
                                                (size_t)ceil_div(an.N, p->direct.bn) *
                                                (size_t)(p->direct.bm * p->direct.bn) * (size_t)an.esize);
  p->extra_bytes = (int64_t)(p->work_bytes - own);
  p->choice_alone = own == 0 && p->extra_bytes > 0;
  return FAMLIES_OK;
}

famlies_status make_plan(famlies_handle h, famlies_plan* out, int dtype, int compute,
                         const famlies_tensor* A, const famlies_tensor* B, const famlies_tensor* C,
                         const TileCfg* force, bool table) {
  if (!out) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_plan_contract: null output pointer");
  *out = nullptr;
  if (!h) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_plan_contract: invalid handle");
  DeviceGuard dg(h->device);
  if (!dg.ok) return fail(FAMLIES_ERR_DEVICE, "cannot select the handle's device");
  famlies_plan_s* p = nullptr;
  struct Owner {  // frees the plan on every early return and if planning throws
    famlies_plan_s** q;
    ~Owner() {
      if (*q) delete *q;
    }
  } owner{&p};
  // Where the extra workspace of the routes past the tile choice does not fit
  // -- the handle's budget, or the device's memory -- the plan does without it,
  // a part at a time: without part planes, without any of it, and at last with
  // the smallest image too.
  PlanUse use;
  use.force = force;
  use.table = table;
  for (int step = 0;; ++step) {
    const bool last = step == 3 || force;
    use.planes = step < 1;
    use.bare = step >= 2;
    use.lean = step == 3;
    delete p;
    p = new (std::nothrow) famlies_plan_s();
    if (!p) return fail(FAMLIES_ERR_ALLOC, "out of host memory");
    std::vector<char> image;
    famlies_status st = prepare_plan(h, p, dtype, compute, A, B, C, use, &image);
    if (st != FAMLIES_OK) return st;
    if (p->extra_bytes) {
      if (h->extra_bytes->fetch_add(p->extra_bytes) + p->extra_bytes > kExtraBytesMax) {
        h->extra_bytes->fetch_sub(p->extra_bytes);
        continue;
      }
      p->extra_held = h->extra_bytes;
    }
    hipError_t e = hipSuccess;
    const char* what = "hipMalloc(indexing vectors)";
    if (!image.empty()) {
      e = hipMalloc(&p->d_off, image.size());
      if (e == hipSuccess) {
        e = hipMemcpy(p->d_off, image.data(), image.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpy(indexing vectors)");
      }
    }
    if (e == hipSuccess && p->work_bytes) {
      e = hipMalloc(&p->d_work, p->work_bytes);
      what = "hipMalloc(split-K workspace)";
    }
    if (e == hipSuccess) break;
    if (e != hipErrorOutOfMemory || last) return hip_fail(e, what);
    (void)hipGetLastError();
  }
  if (log_enabled()) log_plan(p);
  *out = p;
  p = nullptr;  // owned by the caller now
  return FAMLIES_OK;
}

void log_plan(const famlies_plan_s* p) {
  log_decision("plan", p->an, p->cfg, p->direct, p->planes ? p->planes_level : p->level, p->planes, p->planes_fold,
               p->elem32 ? -32 : p->index_bits, p->x_vec, p->y_vec, p->work_bytes, p->table_hit);
}

void destroy_plan(famlies_plan_s* p) {
  if (!p) return;
  DeviceGuard dg(p->h->device);
  delete p;
}

}  // namespace famlies

famlies_plan_s::~famlies_plan_s() {
  if (owns_device && d_off) (void)hipFree(d_off);
  if (owns_device && d_work) (void)hipFree(d_work);
  if (extra_held) extra_held->fetch_sub(extra_bytes);
  if (batch) famlies::destroy_batch(batch);
}

using namespace famlies;

extern "C" {

const char* famlies_version(void) { return "famlies-mi355x 0.1 (gfx950)"; }

famlies_status famlies_create(famlies_handle* out, int device) {
  if (!out) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_create: null output pointer");
  *out = nullptr;
  int n = 0;
  hipError_t e = hipGetDeviceCount(&n);
  if (e != hipSuccess) return hip_fail(e, "hipGetDeviceCount");
  if (device < 0 || device >= n) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_create: no such device");
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, device);
  if (e != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(FAMLIES_ERR_UNSUPPORTED, std::string("famlies_create: device is ") + prop.gcnArchName +
                                             ", this library is built for gfx950 only");
  auto* h = new (std::nothrow) famlies_handle_s();
  if (!h) return fail(FAMLIES_ERR_ALLOC, "famlies_create: out of host memory");
  h->device = device;
  h->num_cus = prop.multiProcessorCount;
  {
    famlies_status st = scratch_address(device, &h->scratch);
    if (st != FAMLIES_OK) {
      delete h;
      return st;
    }
  }
  const char* tt = std::getenv("FAMLIES_TUNE_TABLE");
  if (tt && *tt) {
    std::string err;
    if (!h->table.load(tt, &err)) {
      delete h;
      return fail(FAMLIES_ERR_INVALID_ARG, "FAMLIES_TUNE_TABLE: " + err);
    }
  }
  void* tok = registry_add(h, ObjKind::kHandle);
  if (!tok) {
    delete h;
    return fail(FAMLIES_ERR_ALLOC, "famlies_create: no free object slot");
  }
  *out = static_cast<famlies_handle>(tok);
  return FAMLIES_OK;
}

famlies_status famlies_destroy(famlies_handle tok) {
  auto* h = static_cast<famlies_handle_s*>(registry_take(tok, ObjKind::kHandle));
  if (!h) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_destroy: invalid handle");
  delete h;
  return FAMLIES_OK;
}

famlies_status famlies_plan_contract(famlies_handle htok, famlies_plan* out, int dtype, int compute,
                                     const famlies_tensor* A, const famlies_tensor* B,
                                     const famlies_tensor* C) {
  if (!out) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_plan_contract: null output pointer");
  *out = nullptr;
  famlies_plan_s* p = nullptr;
  famlies_status st = no_throw("famlies_plan_contract",
                               [&] { return make_plan(handle_of(htok), &p, dtype, compute, A, B, C, nullptr); });
  if (st != FAMLIES_OK) return st;
  void* tok = registry_add(p, ObjKind::kPlan);
  if (!tok) {
    destroy_plan(p);
    return fail(FAMLIES_ERR_ALLOC, "famlies_plan_contract: no free object slot");
  }
  *out = static_cast<famlies_plan>(tok);
  return FAMLIES_OK;
}

famlies_status famlies_plan_destroy(famlies_plan tok) {
  auto* p = static_cast<famlies_plan_s*>(registry_take(tok, ObjKind::kPlan));
  if (!p) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_plan_destroy: invalid plan");
  destroy_plan(p);
  return FAMLIES_OK;
}

famlies_status famlies_plan_get_info(famlies_plan tok, famlies_plan_info* info) {
  famlies_plan_s* p = plan_of(tok);
  if (!p || !info) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_plan_get_info: invalid argument");
  if (p->batch) {
    batch_info(p->batch, info);
    return FAMLIES_OK;
  }
  const int route = p->planes ? 256 : p->direct.bm ? 64 : p->level.rem ? 128 : 0;
  fill_info(p->an, p->cfg, p->index_bits, kernel_code(p->an, p->x_vec, p->y_vec) + route, info);
  info->index_elements = p->index_bits == 64 || p->elem32;
  return FAMLIES_OK;
}

static bool overlaps(const void* p, int64_t plo, int64_t phi, const void* q, int64_t qlo, int64_t qhi,
                     int es) {
  if (plo > phi || qlo > qhi) return false;
  const intptr_t a0 = (intptr_t)p + plo * es, a1 = (intptr_t)p + (phi + 1) * es;
  const intptr_t b0 = (intptr_t)q + qlo * es, b1 = (intptr_t)q + (qhi + 1) * es;
  return a0 < b1 && b0 < a1;
}

}  // extern "C"

namespace famlies {

// Whether an execution on stream s may use the plan's extra workspace: the
// first stream to ask has it, for good, and a stream that is captured counts
// as a stream of its own per capture (its graph may be launched anywhere).
// The per-thread default stream is a stream per thread and never has it.
static bool takes_extra(famlies_plan_s* p, hipStream_t s) {
  if (s == hipStreamPerThread) return false;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  if (hipStreamGetCaptureInfo(s, &st, &id) != hipSuccess) (void)hipGetLastError();  // the launch will report it
  if (st != hipStreamCaptureStatusActive) id = 0;
  if (!p->extra_taken) {
    p->extra_taken = true;
    p->extra_stream = s;
    p->extra_capture = id;
  }
  return p->extra_stream == s && p->extra_capture == id;
}

famlies_status execute_impl(famlies_plan_s* p, double alpha, const void* A, const void* B, double beta,
                            void* C, int packed, void* stream, bool ordered) {
  if (!p || p->batch) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_execute: invalid plan");
  const Analysis& an = p->an;
  if (an.M == 0 || an.N == 0) return FAMLIES_OK;
  const bool need_ab = alpha != 0.0 && an.K > 0;
  if (!C || (need_ab && (!A || !B))) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_execute: null data pointer");
  const uintptr_t al = (uintptr_t)an.esize - 1;
  if (((uintptr_t)C & al) || (need_ab && (((uintptr_t)A & al) || ((uintptr_t)B & al))))
    return fail(FAMLIES_ERR_ALIGN, "famlies_execute: data pointer not aligned to its element size");
  const bool pa = packed & 1, pb = packed & 2;
  size_t sza = 0, szb = 0;
  if (need_ab && pa) {
    famlies_status st = pack_size_impl(p, 0, &sza);
    if (st != FAMLIES_OK) return st;
    if ((uintptr_t)A & 15) return fail(FAMLIES_ERR_ALIGN, "famlies_execute_packed: packed A not 16-byte aligned");
  }
  if (need_ab && pb) {
    famlies_status st = pack_size_impl(p, 1, &szb);
    if (st != FAMLIES_OK) return st;
    if ((uintptr_t)B & 15) return fail(FAMLIES_ERR_ALIGN, "famlies_execute_packed: packed B not 16-byte aligned");
  }
  const int64_t es = an.esize;
  auto packed_overlap = [&](const void* q, size_t bytes) {
    return overlaps(C, an.c_lo, an.c_hi, q, 0, (int64_t)(bytes / (size_t)es) - 1, an.esize);
  };
  if (need_ab && ((pa ? packed_overlap(A, sza) : overlaps(C, an.c_lo, an.c_hi, A, an.a_lo, an.a_hi, an.esize)) ||
                  (pb ? packed_overlap(B, szb) : overlaps(C, an.c_lo, an.c_hi, B, an.b_lo, an.b_hi, an.esize))))
    return fail(FAMLIES_ERR_ALIAS, "famlies_execute: C overlaps A or B");
  DeviceGuard dg(p->h->device);
  if (!dg.ok) return fail(FAMLIES_ERR_DEVICE, "cannot select the plan's device");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const void* x = an.swapped ? B : A;
  const void* y = an.swapped ? A : B;
  const bool xp = an.swapped ? pb : pa, yp = an.swapped ? pa : pb;
  PlainLaunch L;
  L.bm = p->cfg.bm;
  L.bn = p->cfg.bn;
  L.bk = p->cfg.bk;
  L.xm = xp ? 2 : p->xmode;
  L.ym = yp ? 2 : p->ymode;
  L.kind = (an.K == 0 || alpha == 0.0) ? PlainLaunch::kScale : PlainLaunch::kMain;
  hipError_t e;
  const int ns = split_parts(an.compute);
  const int i8 = int8_slices(an.compute);
  // The launches of one execution through the workspace follow each other on
  // their stream (threads may share a plan and a stream), and a plan whose tile
  // choice needs no workspace stays free to run on several streams at once:
  // the others than the workspace's run that choice.
  std::unique_lock<std::mutex> in_order(p->work_mu, std::defer_lock);
  bool extra = true;
  if (p->work_bytes && L.kind == PlainLaunch::kMain) {
    in_order.lock();
    if (!ordered && p->choice_alone) extra = takes_extra(p, s);
    if (!extra && p->planes && xp != yp) {
      // no other kernel reads a packed operand of this plan, and the partner's
      // planes go to the workspace: wait until it is free, and take it over
      hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
      if (hipStreamIsCapturing(s, &st) == hipSuccess && st == hipStreamCaptureStatusNone) {
        e = hipDeviceSynchronize();
        if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
      }
      p->extra_taken = false;
      extra = takes_extra(p, s) || s == hipStreamPerThread;
    }
  }
  if (i8 && (pa || pb)) return fail(FAMLIES_ERR_UNSUPPORTED, "famlies_execute_packed: no packed operands for INT8 plans");
  if (i8 && L.kind == PlainLaunch::kMain) {
    const int xm = std::min(p->xmode, 2), ym = std::min(p->ymode, 2);  // 16-byte runs of any form: 2
    e = p->index_bits == 32
            ? launch_int8(make_args<uint32_t>(p, x, y, C, alpha, beta, extra), i8, p->cfg.bn, xm, ym, s)
            : launch_int8(make_args<int64_t>(p, x, y, C, alpha, beta, extra), i8, p->cfg.bn, xm, ym, s);
  } else if (ns && L.kind == PlainLaunch::kMain) {
    if (p->elem32) {
      e = launch_split(make_args<int32_t>(p, x, y, C, alpha, beta, extra), L, ns, s);
    } else if (p->index_bits == 32) {
      PlainArgs<uint32_t> a = make_args<uint32_t>(p, x, y, C, alpha, beta, extra);
      if (xp) {  // the packed buffer is addressed from its start, not through offsets
        a.x = x;
        a.x_nkb = (int32_t)((p->kd + L.bk - 1) / L.bk);
      }
      if (yp) {
        a.y = y;
        a.y_nkb = (int32_t)((p->kd + L.bk - 1) / L.bk);
      }
      if (p->planes && (extra || xp)) {  // (without the workspace: both operands pre-packed)
        const LevelCfg lv = extra ? p->planes_level : LevelCfg();
        a.tiles_m = (int32_t)ceil_div(an.M, 256);
        a.tiles_n = (int32_t)ceil_div(an.N, 128);
        a.splits = 1;
        a.head = lv.head;
        a.rem = lv.rem;
        a.lev_q = lv.q;
        a.lev_part = lv.part;
        a.lev_parts = lv.parts;
        e = launch_planes(a, ns, xp ? 3 : std::min(p->xmode, 2), yp ? 3 : std::min(p->ymode, 2),
                          p->planes_fold, s);
      } else {
        e = launch_split(a, L, ns, s);
      }
    } else {
      e = launch_split(make_args<int64_t>(p, x, y, C, alpha, beta, extra), L, ns, s);
    }
  } else if (p->elem32) {
    e = launch_plain(an.dtype, make_args<int32_t>(p, x, y, C, alpha, beta, extra), L, s);
  } else if (p->index_bits == 32) {
    PlainArgs<uint32_t> a = make_args<uint32_t>(p, x, y, C, alpha, beta, extra);
    if (xp) {
      a.x = x;
      a.x_nkb = (int32_t)((p->kd + L.bk - 1) / L.bk);
    }
    if (yp) {
      a.y = y;
      a.y_nkb = (int32_t)((p->kd + L.bk - 1) / L.bk);
    }
    if (p->direct.bm && (extra || p->direct.split == 1) && L.kind == PlainLaunch::kMain && (!xp || p->pk_fits[0]) &&
        (!yp || p->pk_fits[1])) {
      const DirectCfg& d = p->direct;
      const uint32_t* o = static_cast<const uint32_t*>(p->d_off);
      DirectPacked xd, yd;
      auto packed = [&](DirectPacked* q, int tiles, int nkb, int br) {
        q->plane = (int64_t)tiles * nkb * br * L.bk;
        q->shift = __builtin_ctz((unsigned)br);
        q->row = (uint32_t)(L.bk * an.esize);
        q->tile = (uint32_t)nkb * (uint32_t)br * q->row;
      };
      if (xp) {
        a.xk = o + p->pk_pos[0];
        packed(&xd, a.tiles_m, a.x_nkb, L.bm);
      }
      if (yp) {
        a.yk = o + p->pk_pos[1];
        packed(&yd, a.tiles_n, a.y_nkb, L.bn);
      }
      a.tiles_m = (int32_t)ceil_div(an.M, d.bm);
      a.tiles_n = (int32_t)ceil_div(an.N, d.bn);
      a.splits = d.split;
      a.kchunk = d.kchunk;
      a.head = 0;
      e = launch_direct(an.dtype, a, d, xp || p->dx_vec, yp || p->dy_vec, xd, yd, s);
      if (e == hipSuccess && d.split > 1) e = launch_splitk_reduce(an.dtype, false, a, d.bm, d.bn, s);
    } else {
      e = launch_plain(an.dtype, a, L, s);
    }
  } else {
    e = launch_plain(an.dtype, make_args<int64_t>(p, x, y, C, alpha, beta, extra), L, s);
  }
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  return FAMLIES_OK;
}

}  // namespace famlies

extern "C" {

famlies_status famlies_execute(famlies_plan tok, double alpha, const void* A, const void* B, double beta,
                               void* C, void* stream) {
  return execute_impl(plan_of(tok), alpha, A, B, beta, C, 0, stream);
}

famlies_status famlies_execute_packed(famlies_plan tok, double alpha, const void* A, const void* B, double beta,
                                      void* C, int packed, void* stream) {
  if (packed < 0 || packed > 3) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_execute_packed: packed must be 0..3");
  return execute_impl(plan_of(tok), alpha, A, B, beta, C, packed, stream);
}

}  // extern "C"

// The launch of contract_noalloc: the plan's device data go to the static
// scratch array.
static famlies_status run_noalloc(famlies_plan_s* p, const std::vector<char>& image, size_t off_bytes, double alpha,
                                  const void* a, const void* b, double beta, void* c, void* stream) {
  p->owns_device = false;
  if (off_bytes + p->work_bytes > kNoAllocScratchBytes)
    return fail(FAMLIES_ERR_UNSUPPORTED,
                "famlies_contract_noalloc: the call needs " + std::to_string(off_bytes + p->work_bytes) +
                    " bytes of scratch (indexing vectors and split-K partial sums); the maximum is " +
                    std::to_string(kNoAllocScratchBytes));
  p->d_off = p->h->scratch;
  p->d_work = p->work_bytes ? static_cast<char*>(p->h->scratch) + off_bytes : nullptr;
  if (log_enabled()) log_plan(p);
  if (!image.empty()) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    // stream-ordered after earlier work on the stream (which may still read
    // the scratch); the wait lets the host image go when the call returns
    hipError_t e = hipMemcpyAsync(p->d_off, image.data(), image.size(), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(indexing vectors to scratch)");
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  }
  return execute_impl(p, alpha, a, b, beta, c, 0, stream);
}

// famlies_plan_contract + famlies_execute in one call whose device data (the
// indexing vectors and any split-K partial sums) live in the static scratch
// array instead of plan-owned allocations.
static famlies_status contract_noalloc_impl(famlies_handle htok, int dtype, int compute, double alpha,
                                            const famlies_tensor* A, const void* a, const famlies_tensor* B,
                                            const void* b, double beta, const famlies_tensor* C, void* c,
                                            void* stream) {
  famlies_handle_s* h = handle_of(htok);
  if (!h || !h->scratch) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_contract_noalloc: invalid handle");
  DeviceGuard dg(h->device);
  if (!dg.ok) return fail(FAMLIES_ERR_DEVICE, "cannot select the handle's device");
  famlies_plan_s p, small;
  famlies_plan_s* use_plan = &p;
  std::vector<char> image;
  PlanUse use;
  use.scratch = true;
  famlies_status st = prepare_plan(h, &p, dtype, compute, A, B, C, use, &image);
  if (st != FAMLIES_OK) return st;
  size_t off_bytes = (image.size() + 255) & ~(size_t)255;
  if (off_bytes + p.work_bytes > kNoAllocScratchBytes) {
    use.lean = true;
    use_plan = &small;
    st = prepare_plan(h, &small, dtype, compute, A, B, C, use, &image);
    if (st != FAMLIES_OK) return st;
    off_bytes = (image.size() + 255) & ~(size_t)255;
  }
  return run_noalloc(use_plan, image, off_bytes, alpha, a, b, beta, c, stream);
}

extern "C" {

famlies_status famlies_contract_noalloc(famlies_handle h, int dtype, int compute, double alpha,
                                        const famlies_tensor* A, const void* a, const famlies_tensor* B,
                                        const void* b, double beta, const famlies_tensor* C, void* c,
                                        void* stream) {
  return no_throw("famlies_contract_noalloc", [&] {
    return contract_noalloc_impl(h, dtype, compute, alpha, A, a, B, b, beta, C, c, stream);
  });
}

}  // extern "C"
