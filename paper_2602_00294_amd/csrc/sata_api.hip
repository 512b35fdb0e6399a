// C ABI of the library: argument validation, per-device caches of feature
// tables and workspaces, and dispatch to the HIP kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "kernels.hpp"
#include "prefill_blocks.hpp"
#include "prefill_mfma.hpp"
#include "route.hpp"
#include "sata.h"
#include "sata_testing.h"
#include "state_table.hpp"
#include "table.hpp"

namespace {

thread_local std::string g_last_error;

sata_status fail(sata_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return s;
}

sata_status ok() {
  g_last_error.clear();
  return SATA_OK;
}

sata_status hip_fail(hipError_t e, const char* what) {
  return fail(SATA_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

struct TableEntry {
  sata::FeatureTable host;
  uint64_t* packed = nullptr;
  float* weight = nullptr;
  uint32_t* gen = nullptr;
  std::vector<uint32_t> host_gen;
};

// A state-sum work list on a device, one allocation.
struct StateTableEntry {
  char* ptr = nullptr;
  sata::DevStateTable dev;
};

struct Workspace {
  void* ptr = nullptr;
  size_t bytes = 0;
};

struct DeviceCache {
  std::map<std::pair<int, int>, TableEntry> tables;
  std::map<std::tuple<int, int, sata::StateShape>, StateTableEntry> state_tables;  // (d, P, shape)
  std::map<hipStream_t, Workspace> workspaces;
  std::map<hipStream_t, Workspace> counters;  // zeroed at allocation; kernels leave them zero
};

std::mutex g_mu;
std::map<int, DeviceCache> g_devices;

// Upper bound on features per head accepted by the kernels.
constexpr int64_t kMaxFeatures = (int64_t)1 << 26;
// Upper bound on B*H (one grid dimension per head).
constexpr int kMaxHeads = 65535;
// Upper bound on the partial-readout workspace of one segment of a call.
constexpr size_t kMaxWorkspace = (size_t)512 << 20;
// The same for the generated-feature kernel, whose segments each store and
// reload the whole state (at d = 64 a 4096-token call of 16 heads is one
// segment).
constexpr size_t kMaxFeatWorkspace = (size_t)2 << 30;
// The same for the backward, whose scan workgroups load and store their state
// slice at every segment.
constexpr size_t kMaxBackwardWorkspace = (size_t)2 << 30;
// The tuned matrix-core kernels hold the partial readouts of the whole call;
// beyond this much the call takes the segmented kernels instead.
constexpr size_t kMaxWholeCallWorkspace = (size_t)4 << 30;
// The flat decode kernel (the one that takes residuals) serves d_v up to this.
constexpr int kMaxCompensatedDv = 127;

// Scratch of sata_decode_step_noalloc: one array per device for the life of
// the process.  The first kScratchCounterBytes hold the per-head arrival
// counters of the split decode (zeroed once per device by a fill kernel; the
// kernels set each counter back to zero), the rest the pieces' partial sums.
// In host code `scratch` names a host-side stand-in: only the address that
// hipGetSymbolAddress returns for the current device may reach a kernel.
constexpr size_t kScratchBytes = (size_t)4 << 20;
constexpr size_t kScratchCounterBytes = sizeof(int) * 65536;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

struct ScratchSlot {
  bool ready = false;
  unsigned char* ptr = nullptr;  // the device address of `scratch` on that device
};
constexpr int kMaxDevices = 64;
ScratchSlot g_scratch[kMaxDevices];  // guarded by g_mu

sata_status get_table(int d, int P, hipStream_t stream, sata::DevTable* out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(g_mu);
  DeviceCache& dc = g_devices[dev];
  auto key = std::make_pair(d, P);
  auto it = dc.tables.find(key);
  if (it == dc.tables.end()) {
    TableEntry ent;
    ent.host = sata::build_table(d, P);
    ent.host_gen = sata::build_gen_program(ent.host, sata::kTablePad, sata::kGenBlock);
    // the device copy ends in kTablePad zero entries
    ent.host.packed.resize(ent.host.packed.size() + sata::kTablePad, 0);
    ent.host.weight.resize(ent.host.weight.size() + sata::kTablePad, 0.0f);
    const size_t D = (size_t)ent.host.D + sata::kTablePad;
    auto release = [&ent]() {
      hipFree(ent.packed);
      hipFree(ent.weight);
      hipFree(ent.gen);
    };
    if ((e = hipMalloc(&ent.packed, D * sizeof(uint64_t))) != hipSuccess ||
        (e = hipMalloc(&ent.weight, D * sizeof(float))) != hipSuccess ||
        (e = hipMalloc(&ent.gen, 2 * D * sizeof(uint32_t))) != hipSuccess) {
      release();
      return hip_fail(e, "hipMalloc(table)");
    }
    // The host copies live in the cache, so asynchronous copies are safe.
    e = hipMemcpyAsync(ent.packed, ent.host.packed.data(), D * sizeof(uint64_t), hipMemcpyHostToDevice, stream);
    if (e == hipSuccess)
      e = hipMemcpyAsync(ent.weight, ent.host.weight.data(), D * sizeof(float), hipMemcpyHostToDevice, stream);
    if (e == hipSuccess)
      e = hipMemcpyAsync(ent.gen, ent.host_gen.data(), 2 * D * sizeof(uint32_t), hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) {
      release();
      return hip_fail(e, "uploading feature table");
    }
    it = dc.tables.emplace(key, std::move(ent)).first;
  }
  out->packed = it->second.packed;
  out->weight = it->second.weight;
  out->gen = it->second.gen;
  out->D = it->second.host.D;
  out->d = d;
  out->P = P;
  return SATA_OK;
}

// The work list of the state sum for a block shape, uploaded once per device.
// It is built outside the lock: other calls go on meanwhile.
sata_status get_state_table(int d, int P, const sata::StateShape& shape, hipStream_t stream,
                            sata::DevStateTable* out) try {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  const auto key = std::make_tuple(d, P, shape);
  auto find = [&]() {
    DeviceCache& dc = g_devices[dev];
    auto it = dc.state_tables.find(key);
    if (it == dc.state_tables.end()) return false;
    *out = it->second.dev;
    return true;
  };
  {
    std::lock_guard<std::mutex> lock(g_mu);
    if (find()) return SATA_OK;
  }
  const sata::StateTable st = sata::make_state_table(d, P, shape);
  std::vector<char> host;
  auto put = [&host](const void* p, size_t bytes) {
    const size_t at = host.size();
    host.resize((at + bytes + 255) / 256 * 256);
    if (bytes) std::memcpy(host.data() + at, p, bytes);
    return at;
  };
  const size_t o_gsym = put(st.gsym.data(), st.gsym.size() * sizeof(st.gsym[0]));
  const size_t o_list = put(st.list.data(), st.list.size() * sizeof(st.list[0]));
  const size_t o_ftab = put(st.ftab.data(), st.ftab.size() * sizeof(st.ftab[0]));
  const size_t o_ztab = put(st.ztab.data(), st.ztab.size() * sizeof(st.ztab[0]));
  std::lock_guard<std::mutex> lock(g_mu);
  if (find()) return SATA_OK;
  StateTableEntry ent;
  if ((e = hipMalloc(&ent.ptr, host.size() + 256)) != hipSuccess) return hip_fail(e, "hipMalloc(state table)");
  e = hipMemcpyAsync(ent.ptr, host.data(), host.size(), hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    hipFree(ent.ptr);
    return hip_fail(e, "uploading the state table");
  }
  ent.dev.gsym = (const uint64_t*)(ent.ptr + o_gsym);
  ent.dev.list = (const sata::StateBlock*)(ent.ptr + o_list);
  ent.dev.ftab = (const int32_t*)(ent.ptr + o_ftab);
  ent.dev.ztab = (const int32_t*)(ent.ptr + o_ztab);
  ent.dev.zcols = st.zcols;
  ent.dev.tall = st.tall;
  ent.dev.blocks = st.blocks;
  ent.dev.zblocks = st.zblocks;
  *out = ent.dev;
  g_devices[dev].state_tables.emplace(key, ent);
  return SATA_OK;
} catch (const std::bad_alloc&) {
  return fail(SATA_ERR_HIP, "out of host memory for the state table of d_k=%d P=%d", d, P);
}

// The cached table of (d, P) on the current device, without creating one.
sata_status find_table(int d, int P, sata::DevTable* out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(g_mu);
  auto dc = g_devices.find(dev);
  if (dc != g_devices.end()) {
    auto it = dc->second.tables.find(std::make_pair(d, P));
    if (it != dc->second.tables.end()) {
      out->packed = it->second.packed;
      out->weight = it->second.weight;
      out->gen = it->second.gen;
      out->D = it->second.host.D;
      out->d = d;
      out->P = P;
      return SATA_OK;
    }
  }
  return fail(SATA_ERR_UNSUPPORTED,
              "no feature table for d_k=%d P=%d on device %d yet: make one sata_decode_step, sata_prefill or "
              "sata_feature_map call with these sizes first",
              d, P, dev);
}

// The device address of `scratch` on the current device; on the first call
// on a device it is looked up and the counter region cleared on `stream`.
sata_status get_scratch(hipStream_t stream, unsigned char** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return fail(SATA_ERR_UNSUPPORTED, "device %d beyond %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_mu);
  ScratchSlot& slot = g_scratch[dev];
  if (!slot.ready) {
    void* p = nullptr;
    if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess)
      return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if ((e = sata::launch_fill_zero((float*)p, (int64_t)(kScratchCounterBytes / sizeof(float)), stream)) !=
        hipSuccess)
      return hip_fail(e, "clearing the scratch counters");
    slot.ptr = (unsigned char*)p;
    slot.ready = true;
  }
  *out = slot.ptr;
  return SATA_OK;
}

// Returns a per-(device, stream) scratch buffer of at least `bytes`.
sata_status get_workspace(size_t bytes, hipStream_t stream, void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(g_mu);
  Workspace& ws = g_devices[dev].workspaces[stream];
  if (ws.bytes < bytes) {
    if (ws.ptr) {
      // earlier work on this stream may still read the old buffer
      if ((e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
      hipFree(ws.ptr);
      ws.ptr = nullptr;
      ws.bytes = 0;
    }
    size_t want = bytes < ((size_t)1 << 20) ? ((size_t)1 << 20) : bytes;
    if ((e = hipMalloc(&ws.ptr, want)) != hipSuccess) return hip_fail(e, "hipMalloc(workspace)");
    ws.bytes = want;
  }
  *out = ws.ptr;
  return SATA_OK;
}

// Returns a per-(device, stream) array of at least n ints, all zero.  It is
// cleared once, when allocated, by a fill kernel on the stream; the kernels
// that count in it set every counter back to zero.
sata_status get_counters(int64_t n, hipStream_t stream, int** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(g_mu);
  Workspace& ws = g_devices[dev].counters[stream];
  const size_t bytes = sizeof(int) * (size_t)n;
  if (ws.bytes < bytes) {
    if (ws.ptr) {
      if ((e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
      hipFree(ws.ptr);
      ws.ptr = nullptr;
      ws.bytes = 0;
    }
    size_t want = bytes < ((size_t)1 << 16) ? ((size_t)1 << 16) : bytes;
    if ((e = hipMalloc(&ws.ptr, want)) != hipSuccess) return hip_fail(e, "hipMalloc(counters)");
    if ((e = sata::launch_fill_zero((float*)ws.ptr, (int64_t)(want / sizeof(float)), stream)) != hipSuccess) {
      hipFree(ws.ptr);
      ws.ptr = nullptr;
      return hip_fail(e, "clearing counters");
    }
    ws.bytes = want;
  }
  *out = (int*)ws.ptr;
  return SATA_OK;
}

bool valid_dtype(sata_dtype t) { return t == SATA_F32 || t == SATA_BF16; }

sata_status check_dims(int d_k, int d_v, int P, int64_t* D) {
  if (d_k < 1 || d_k > sata::kMaxDim) return fail(SATA_ERR_INVALID_ARG, "d_k=%d outside 1..%d", d_k, sata::kMaxDim);
  if (d_v < 1 || d_v > sata::kMaxDim) return fail(SATA_ERR_INVALID_ARG, "d_v=%d outside 1..%d", d_v, sata::kMaxDim);
  if (P < 1 || P > sata::kMaxP) return fail(SATA_ERR_INVALID_ARG, "P=%d outside 1..%d", P, sata::kMaxP);
  const int64_t f = sata::feature_count(d_k, P);
  if (f < 0 || f > kMaxFeatures)
    return fail(SATA_ERR_TOO_LARGE, "C(d_k+P-1, P-1) features exceed %lld", (long long)kMaxFeatures);
  *D = f;
  return SATA_OK;
}

sata_status check_prefill_args(sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk,
                               int64_t* D) {
  if (!valid_dtype(dt)) return fail(SATA_ERR_INVALID_ARG, "unknown dtype %d", (int)dt);
  if (B < 1 || H < 1) return fail(SATA_ERR_INVALID_ARG, "B=%d H=%d must be >= 1", B, H);
  if (n < 0) return fail(SATA_ERR_INVALID_ARG, "n=%d < 0", n);
  sata_status st = check_dims(d_k, d_v, P, D);
  if (st != SATA_OK) return st;
  if (chunk != 16 && chunk != 32 && chunk != 64 && chunk != 128)
    return fail(SATA_ERR_UNSUPPORTED, "chunk=%d; supported: 16, 32, 64, 128", chunk);
  if ((int64_t)B * H > kMaxHeads) return fail(SATA_ERR_TOO_LARGE, "B*H=%lld exceeds %d", (long long)B * H, kMaxHeads);
  return SATA_OK;
}

enum class PrefillPath { kMfma32, kBlocks, kFeat, kFloat32 };

// The kernel family that serves a validated prefill request.
PrefillPath prefill_path(sata_dtype dt, int BH, int n, int d_k, int d_v, int P, int chunk) {
  sata::MfmaPrefillPlan mp;
  if (dt == SATA_BF16 && sata::plan_prefill_mfma(BH, n, d_k, d_v, P, chunk, &mp) &&
      mp.workspace_bytes <= kMaxWholeCallWorkspace)
    return PrefillPath::kMfma32;
  if (dt == SATA_BF16 && sata::plan_prefill_blocks(BH, n, d_k, d_v, P, chunk, &mp) &&
      mp.workspace_bytes <= kMaxWholeCallWorkspace)
    return PrefillPath::kBlocks;
  sata::FeatPrefillPlan fp;
  if (sata::plan_prefill_feat(sata::feature_count(d_k, P), BH, n, d_k, d_v, P, chunk, dt == SATA_F32, kMaxFeatWorkspace,
                              &fp))
    return PrefillPath::kFeat;
  return PrefillPath::kFloat32;
}

// Longest rows of one head that the pair-by-pair kernels address (32-bit byte
// offsets into a head's tensor, float32 at d = 64).
constexpr int64_t kMaxDirectTokens = (int64_t)1 << 22;

// Whether the pair-by-pair prefill covers a shape (query heads, for its grid).
bool direct_covers(sata_dtype dt, int query_heads, int n, int d_k, int d_v, int P, int64_t D) {
  return d_k <= 64 && d_v <= 64 && P >= 2 && D <= ((int64_t)1 << 22) && n <= kMaxDirectTokens &&
         sata::direct_blocks(dt == SATA_F32, d_v, query_heads, n) <= sata::kMaxPairBlocks;
}

// Whether a prefill computes its outputs pair by pair (prefill_direct.hip) and
// its state, where it is asked for, as one sum over the tokens
// (prefill_state.hip) rather than by the chunked scan: by the estimates of
// route.hpp.  A grouped call asks for its key/value heads alone: each member is
// bitwise the single-head prefill of its queries, so both take one way.
bool direct_pays(sata_dtype dt, int BH, int G, int n, int d_k, int d_v, int P, int chunk, int64_t D, bool want_state,
                 bool vectors) {
  if (!direct_covers(dt, BH * G, n, d_k, d_v, P, D)) return false;
  sata::RouteCall r;
  r.bf16 = dt == SATA_BF16;
  r.dk = d_k;
  r.dv = d_v;
  r.P = P;
  r.D = D;
  r.heads = BH;
  r.n = n;
  r.vectors = vectors;
  sata::ScanShape scan;
  const PrefillPath path = prefill_path(dt, BH, n, d_k, d_v, P, chunk);
  sata::FeatPrefillPlan fp;
  if (path == PrefillPath::kMfma32 || path == PrefillPath::kBlocks) {
    scan.tuned = true;
    scan.chunk = chunk;
  } else if (path == PrefillPath::kFeat &&
             sata::plan_prefill_feat(D, BH, n, d_k, d_v, P, chunk, !r.bf16, kMaxFeatWorkspace, &fp)) {
    scan.wave_features = fp.wave_features;
    scan.slices = fp.nslices;
    scan.parts = fp.parts;
  } else {
    return false;  // float32 arithmetic
  }
  double t = sata::pairs_us(r);
  if (want_state) {
    const double wgs = sata::state_workgroups(r);
    t = std::max(17.5, t + sata::state_us(r, wgs, sata::plan_prefill_state(D, BH, n, d_v, r.bf16, (int)(wgs + 0.5)).parts));
  }
  return t <= sata::scan_us(r, scan);
}

// Whether the rows of q, k and v are whole 16-byte vectors.
bool vector_rows(const void* q, const void* k, const void* v, sata_dtype dt, int d_k, int d_v) {
  const int elems = dt == SATA_BF16 ? 8 : 4;
  return d_k % elems == 0 && d_v % elems == 0 && (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v) & 15) == 0;
}

// Whether the gradients are computed pair by pair (backward_direct.hip) rather
// than by the scans over the states: c (n / 2 + 256) ps per head-token against
// a share of the state.  Measured, ns per head-token at 128 heads and n = 4096
// against the scans: bfloat16 d = 16, P = 3 2.9 / 9.8, d = 32, P = 2 3.2 / 12.9,
// d = 64, P = 2 5.3 / 31; float32 d = 16, P = 3 6.4 / 9.5, d = 32, P = 2
// 7.8 / 12.5, d = 64, P = 2 20 / 30.  The line errs towards the scans: of 4160
// calls timed both ways (1 to 1024 heads, 16 to 65536 tokens) it leaves 528 to
// scans that are slower by 5% and more, and gives none to slower pairs.
bool backward_direct_covers(sata_dtype dt, int BH, int n, int P) {
  return P >= 2 && n <= kMaxDirectTokens && sata::backward_blocks(dt == SATA_BF16, BH, n) <= sata::kMaxPairBlocks;
}
bool backward_direct_pays(sata_dtype dt, int BH, int n, int d_k, int d_v, int P, int64_t D) {
  if (!backward_direct_covers(dt, BH, n, P)) return false;
  const int tiles = (std::max(d_k, d_v) + 15) / 16;
  const double pair = (dt == SATA_BF16 ? (tiles <= 2 ? 1.75 : 2.6) : (tiles == 1 ? 3.0 : tiles == 2 ? 3.7 : 10.0)) +
                      0.3 * std::max(0, P - 4);
  const double scan = 1.5 + 0.26 * d_k + 0.9e-3 * (double)D * (d_v + 1);
  return 1.1 * 1e-3 * pair * (0.5 * n + 256.0) <= scan;
}

// The pair-by-pair ways allocate and upload other things than the scans (work
// lists by block shape; scratch for the parts' sums or the statistics), which a
// capturing stream cannot do.  There the state is summed in as many parts as
// the workspace holds, and a call without its list or statistics goes by the
// scans: what they need, an earlier call of other sizes may have left.
size_t workspace_bytes(hipStream_t stream) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  std::lock_guard<std::mutex> lock(g_mu);
  auto& spaces = g_devices[dev].workspaces;
  auto ws = spaces.find(stream);
  return ws == spaces.end() ? 0 : ws->second.bytes;
}
bool prefill_direct_in_place(sata_dtype dt, int d_k, int d_v, int P, bool want_state) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  std::lock_guard<std::mutex> lock(g_mu);
  DeviceCache& dc = g_devices[dev];
  return dc.tables.count(std::make_pair(d_k, P)) &&
         (!want_state || dc.state_tables.count(std::make_tuple(d_k, P, sata::state_shape(d_v, dt != SATA_BF16))));
}
bool captured(hipStream_t stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(stream, &status) == hipSuccess && status != hipStreamCaptureStatusNone;
}

// A prefill computed pair by pair: outputs for BH * G query heads, then the
// state of each of the BH key/value heads as one sum over the tokens.
sata_status prefill_direct(const void* q, const void* k, const void* v, sata_dtype dt, int BH, int G, int n, int d_k,
                           int d_v, int P, void* y, float* S_out, hipStream_t s, int64_t D) {
  sata_status st;
  hipError_t e;
  sata::DevTable t;
  if ((st = get_table(d_k, P, s, &t)) != SATA_OK) return st;
  const bool bf16 = dt == SATA_BF16;
  sata::StatePlan plan;
  sata::DevStateTable dst;
  float* partial = nullptr;
  // (without a state the list is uploaded all the same: a call with one may be
  // captured after this)
  if (S_out || (!prefill_direct_in_place(dt, d_k, d_v, P, true) && !captured(s))) {
    if ((st = get_state_table(d_k, P, sata::state_shape(d_v, !bf16), s, &dst)) != SATA_OK) return st;
  }
  if (S_out) {
    const int nwg = (dst.blocks + dst.zblocks) / 4;
    plan = sata::plan_prefill_state(D, BH, n, d_v, bf16, nwg);
    const size_t held = plan.parts > 1 ? workspace_bytes(s) : 0;
    if (plan.partial_bytes > held && captured(s)) plan = sata::plan_prefill_state(D, BH, n, d_v, bf16, nwg, held);
    if (plan.parts > 1) {
      void* ws = nullptr;
      if ((st = get_workspace(plan.partial_bytes, s, &ws)) != SATA_OK) return st;
      partial = (float*)ws;
    }
  }
  e = sata::launch_prefill_direct(q, k, v, y, bf16, BH * G, G, n, d_k, d_v, P, s);
  if (e != hipSuccess) return hip_fail(e, "prefill (pair by pair) launch");
  if (S_out) {
    e = sata::launch_prefill_state(k, v, bf16, BH, n, d_k, d_v, P, t, dst, plan, S_out, partial, s);
    if (e != hipSuccess) return hip_fail(e, "prefill (state) launch");
  }
  return ok();
}

// One prefill over BH key/value heads; q and y hold qg query heads per
// key/value head (head bh's queries start at head bh * qg of q).
sata_status prefill_dispatch(const void* q, const void* k, const void* v, sata_dtype dt, int BH, int n, int d_k,
                             int d_v, int P, int chunk, void* y, float* S_out, hipStream_t s, int64_t D, int qg) {
  const int E = d_v + 1;
  hipError_t e;
  sata_status st;
  if (n == 0) {
    if (S_out) {
      if ((e = sata::launch_fill_zero(S_out, (int64_t)BH * D * E, s)) != hipSuccess)
        return hip_fail(e, "fill launch");
    }
    return ok();
  }
  sata::DevTable t;
  if ((st = get_table(d_k, P, s, &t)) != SATA_OK) return st;

  // bf16 fast path on the matrix cores where a tuned kernel exists
  sata::MfmaPrefillPlan mp;
  const PrefillPath path = prefill_path(dt, BH, n, d_k, d_v, P, chunk);
  if (path == PrefillPath::kMfma32 && sata::plan_prefill_mfma(BH, n, d_k, d_v, P, chunk, &mp)) {
    void* ws = nullptr;
    if ((st = get_workspace(mp.workspace_bytes, s, &ws)) != SATA_OK) return st;
    e = sata::launch_prefill_mfma(q, k, v, y, S_out, BH, n, d_k, d_v, P, chunk, mp, ws, s, qg);
    if (e != hipSuccess) return hip_fail(e, "prefill (matrix-core) launch");
    return ok();
  }
  if (path == PrefillPath::kBlocks && sata::plan_prefill_blocks(BH, n, d_k, d_v, P, chunk, &mp)) {
    void* ws = nullptr;
    if ((st = get_workspace(mp.workspace_bytes, s, &ws)) != SATA_OK) return st;
    e = sata::launch_prefill_blocks(q, k, v, y, S_out, BH, n, d_k, d_v, P, chunk, mp, ws, s, qg);
    if (e != hipSuccess) return hip_fail(e, "prefill (matrix-core, per-block) launch");
    return ok();
  }

  sata::FeatPrefillPlan fp;
  if (path == PrefillPath::kFeat &&
      sata::plan_prefill_feat(D, BH, n, d_k, d_v, P, chunk, dt == SATA_F32, kMaxFeatWorkspace, &fp)) {
    const size_t state_bytes = S_out ? 0 : sizeof(float) * (size_t)BH * D * E;
    void* ws = nullptr;
    if ((st = get_workspace(fp.partial_bytes + state_bytes, s, &ws)) != SATA_OK) return st;
    float* partial = (float*)ws;
    float* S_state = S_out ? S_out : (float*)((char*)ws + fp.partial_bytes);
    e = sata::launch_prefill_feat(q, k, v, y, BH, n, d_k, d_v, P, t, fp, S_state, partial, s, qg);
    if (e != hipSuccess) return hip_fail(e, "prefill (matrix-core, generated features) launch");
    return ok();
  }

  sata::PrefillGenericPlan plan;
  if (!sata::plan_prefill_generic(D, BH, n, d_k, d_v, chunk, kMaxWorkspace, &plan))
    return fail(SATA_ERR_UNSUPPORTED, "no slice size fits on chip for d_k=%d d_v=%d chunk=%d", d_k, d_v, chunk);
  const size_t state_bytes = S_out ? 0 : sizeof(float) * (size_t)BH * D * E;
  void* ws = nullptr;
  if ((st = get_workspace(plan.partial_bytes + state_bytes, s, &ws)) != SATA_OK) return st;
  float* partial = (float*)ws;
  float* S_state = S_out ? S_out : (float*)((char*)ws + plan.partial_bytes);
  e = sata::launch_prefill_generic(q, k, v, y, dt == SATA_BF16, BH, n, d_k, d_v, chunk, t, plan, S_state,
                                   partial, s, qg);
  if (e != hipSuccess) return hip_fail(e, "prefill launch");
  return ok();
}

sata_status decode_step(float* S, float* R, const void* q, const void* k, const void* v, sata_dtype dt, int B,
                        int H, int d_k, int d_v, int P, void* y, void* stream) {
  if (!valid_dtype(dt)) return fail(SATA_ERR_INVALID_ARG, "unknown dtype %d", (int)dt);
  if (B < 1 || H < 1) return fail(SATA_ERR_INVALID_ARG, "B=%d H=%d must be >= 1", B, H);
  int64_t D = 0;
  sata_status st = check_dims(d_k, d_v, P, &D);
  if (st != SATA_OK) return st;
  if ((int64_t)B * H > kMaxHeads) return fail(SATA_ERR_TOO_LARGE, "B*H=%lld exceeds %d", (long long)B * H, kMaxHeads);
  if (!S || !q || !k || !v || !y) return fail(SATA_ERR_INVALID_ARG, "null tensor pointer");
  const int BH = B * H;
  hipStream_t s = (hipStream_t)stream;
  sata::DecodePlan plan = sata::plan_decode(D, d_k, d_v, BH);
  if (R && !sata::decode_supports_residuals(plan, S))
    return fail(SATA_ERR_UNSUPPORTED, "the compensated decode needs a 16-byte aligned state and d_v <= %d",
                kMaxCompensatedDv);
  sata::DevTable t;
  if ((st = get_table(d_k, P, s, &t)) != SATA_OK) return st;
  float* partial = nullptr;
  int* counters = nullptr;
  // partial sums: one row per slice (row-wise path) or per piece of a head (flat path)
  const int64_t rows = std::max<int64_t>(plan.nslices > 1 ? plan.nslices : 0, plan.flat_np > 1 ? plan.flat_np : 0);
  if (rows > 0) {
    void* ws = nullptr;
    const size_t bytes = sizeof(float) * (size_t)BH * rows * (d_v + 1);
    if ((st = get_workspace(bytes, s, &ws)) != SATA_OK) return st;
    partial = (float*)ws;
  }
  if (plan.flat_np > 1 && (st = get_counters(BH, s, &counters)) != SATA_OK) return st;
  hipError_t e =
      sata::launch_decode(S, q, k, v, y, dt == SATA_BF16, BH, d_k, d_v, t, plan, partial, counters, s, R);
  if (e != hipSuccess) return hip_fail(e, "decode launch");
  return ok();
}

// By which way a prefill or a backward is computed.
enum class Way { kEstimate, kPairs, kScan };

sata_status check_groups(int B, int H_kv, int G) {
  if (G < 1) return fail(SATA_ERR_INVALID_ARG, "G=%d must be >= 1", G);
  if (B >= 1 && H_kv >= 1 && (int64_t)B * H_kv * G > kMaxHeads)
    return fail(SATA_ERR_TOO_LARGE, "B*H_kv*G=%lld exceeds %d", (long long)B * H_kv * G, kMaxHeads);
  return SATA_OK;
}

// sata_prefill (G = 1) and sata_prefill_grouped.
sata_status prefill(Way way, const void* q, const void* k, const void* v, sata_dtype dt, int B, int H_kv, int G, int n,
                    int d_k, int d_v, int P, int chunk, void* y, float* S_out, void* stream) {
  int64_t D = 0;
  sata_status st = check_prefill_args(dt, B, H_kv, n, d_k, d_v, P, chunk, &D);
  if (st != SATA_OK) return st;
  if (n > 0 && (!q || !k || !v || !y)) return fail(SATA_ERR_INVALID_ARG, "null tensor pointer");
  if (way == Way::kPairs && !direct_covers(dt, B * H_kv * G, n, d_k, d_v, P, D))
    return fail(SATA_ERR_UNSUPPORTED, "no pair-by-pair prefill for n=%d d_k=%d d_v=%d P=%d", n, d_k, d_v, P);
  const hipStream_t s = (hipStream_t)stream;
  const bool want_state = S_out != nullptr;
  bool pairs = n > 0 && (way == Way::kPairs ||
                         (way == Way::kEstimate && direct_pays(dt, B * H_kv, G, n, d_k, d_v, P, chunk, D, want_state,
                                                               vector_rows(q, k, v, dt, d_k, d_v))));
  if (pairs && way == Way::kEstimate && !prefill_direct_in_place(dt, d_k, d_v, P, want_state) && captured(s))
    pairs = false;
  if (pairs) return prefill_direct(q, k, v, dt, B * H_kv, G, n, d_k, d_v, P, y, S_out, s, D);
  const size_t esz = dt == SATA_BF16 ? 2 : 4;
  // query head g + G h of each batch row is member g of key/value head h's
  // group: with the heads of the call numbered by key/value head, member g's
  // queries and outputs start g heads in and lie G heads apart
  for (int g = 0; g < G; ++g) {
    const void* qg = (const char*)q + esz * (size_t)g * (size_t)n * (size_t)d_k;
    void* yg = (char*)y + esz * (size_t)g * (size_t)n * (size_t)d_v;
    st = prefill_dispatch(qg, k, v, dt, B * H_kv, n, d_k, d_v, P, chunk, yg, g == 0 ? S_out : nullptr, s, D, G);
    if (st != SATA_OK) return st;
    if (n == 0) break;
  }
  return ok();
}

sata_status check_backward_args(sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk, int64_t* D) {
  if (!valid_dtype(dt)) return fail(SATA_ERR_INVALID_ARG, "unknown dtype %d", (int)dt);
  if (B < 1 || H < 1) return fail(SATA_ERR_INVALID_ARG, "B=%d H=%d must be >= 1", B, H);
  if (n < 0) return fail(SATA_ERR_INVALID_ARG, "n=%d < 0", n);
  sata_status st = check_dims(d_k, d_v, P, D);
  if (st != SATA_OK) return st;
  if ((int64_t)B * H > kMaxHeads) return fail(SATA_ERR_TOO_LARGE, "B*H=%lld exceeds %d", (long long)B * H, kMaxHeads);
  if (chunk != 16 && chunk != 32 && chunk != 64)
    return fail(SATA_ERR_UNSUPPORTED, "chunk=%d; the backward supports 16, 32, 64", chunk);
  if (d_k > sata::kMaxBackwardDim || d_v > sata::kMaxBackwardDim)
    return fail(SATA_ERR_UNSUPPORTED, "the backward supports d_k, d_v <= %d", sata::kMaxBackwardDim);
  return SATA_OK;
}

sata_status backward(Way way, const void* q, const void* k, const void* v, const void* dy, sata_dtype dt, int B, int H,
                     int n, int d_k, int d_v, int P, int chunk, void* dq, void* dk, void* dv, void* stream) {
  int64_t D = 0;
  sata_status st = check_backward_args(dt, B, H, n, d_k, d_v, P, chunk, &D);
  if (st != SATA_OK) return st;
  if (n == 0) return ok();
  if (!q || !k || !v || !dy || !dq || !dk || !dv) return fail(SATA_ERR_INVALID_ARG, "null tensor pointer");
  const int BH = B * H;
  sata::BackwardPlan plan;
  sata::PrefillGenericPlan fwd;
  if (!sata::plan_backward(D, BH, n, d_k, d_v, P, chunk, kMaxBackwardWorkspace, &plan, &fwd))
    return fail(SATA_ERR_UNSUPPORTED, "no backward slice fits on chip for d_k=%d d_v=%d chunk=%d", d_k, d_v, chunk);
  hipStream_t s = (hipStream_t)stream;
  if (way == Way::kPairs && !backward_direct_covers(dt, BH, n, P))
    return fail(SATA_ERR_UNSUPPORTED, "no pair-by-pair backward for n=%d P=%d", n, P);
  bool pairs = way == Way::kPairs || (way == Way::kEstimate && backward_direct_pays(dt, BH, n, d_k, d_v, P, D));
  if (pairs && way == Way::kEstimate && workspace_bytes(s) < sata::backward_direct_bytes(BH, n) && captured(s))
    pairs = false;
  if (pairs) {
    void* ws = nullptr;
    if ((st = get_workspace(sata::backward_direct_bytes(BH, n), s, &ws)) != SATA_OK) return st;
    hipError_t e = sata::launch_backward_direct(q, k, v, dy, dq, dk, dv, dt == SATA_BF16, BH, n, d_k, d_v, P,
                                                (float*)ws, s);
    if (e != hipSuccess) return hip_fail(e, "backward (pair by pair) launch");
    return ok();
  }
  sata::DevTable t;
  if ((st = get_table(d_k, P, s, &t)) != SATA_OK) return st;
  void* ws = nullptr;
  if ((st = get_workspace(plan.h_bytes + plan.state_bytes + plan.partial_bytes, s, &ws)) != SATA_OK) return st;
  float* h = (float*)ws;
  float* state = (float*)((char*)ws + plan.h_bytes);
  float* partial = (float*)((char*)ws + plan.h_bytes + plan.state_bytes);
  hipError_t e = sata::launch_backward(q, k, v, dy, dq, dk, dv, dt == SATA_BF16, BH, n, d_k, d_v, P, chunk, t, plan,
                                       fwd, h, state, partial, s);
  if (e != hipSuccess) return hip_fail(e, "backward launch");
  return ok();
}

}  // namespace

extern "C" {

int64_t sata_feature_count(int d, int P) {
  if (d < 1 || P < 1) return -1;
  return sata::feature_count(d, P);
}

int64_t sata_state_elems(int d_k, int d_v, int P) {
  if (d_k < 1 || d_v < 1 || P < 1) return -1;
  const int64_t f = sata::feature_count(d_k, P);
  if (f < 0 || f > INT64_MAX / (d_v + 1)) return -1;
  return f * (d_v + 1);
}

sata_status sata_feature_index(int d, int P, int64_t f, int* degree, int* idx) {
  if (!degree || !idx) return fail(SATA_ERR_INVALID_ARG, "null output pointer");
  if (d < 1 || d > sata::kMaxDim || P < 1 || P > sata::kMaxP)
    return fail(SATA_ERR_INVALID_ARG, "d=%d or P=%d out of range", d, P);
  const int64_t D = sata::feature_count(d, P);
  if (D < 0 || f < 0 || f >= D) return fail(SATA_ERR_INVALID_ARG, "feature %lld out of range", (long long)f);
  // skip whole degrees, then walk the tuples of the degree that holds f
  int64_t base = 0;
  for (int p = 0; p < P; ++p) {
    const int64_t m = sata::binom((int64_t)d + p - 1, p);
    if (f < base + m) {
      int64_t i = base;
      bool found = false;
      if (p == 0) found = true;
      else
        sata::for_each_tuple(d, p, [&](const int* t) {
          if (!found && i == f) {
            for (int j = 0; j < p; ++j) idx[j] = t[j];
            found = true;
          }
          ++i;
        });
      *degree = p;
      return ok();
    }
    base += m;
  }
  return fail(SATA_ERR_INVALID_ARG, "feature %lld out of range", (long long)f);
}

sata_status sata_feature_map(const void* x, sata_dtype xt, int64_t rows, int d, int P, float* phi,
                             void* stream) {
  if (!valid_dtype(xt)) return fail(SATA_ERR_INVALID_ARG, "unknown dtype %d", (int)xt);
  if (rows < 0) return fail(SATA_ERR_INVALID_ARG, "rows=%lld < 0", (long long)rows);
  int64_t D = 0;
  sata_status st = check_dims(d, 1, P, &D);
  if (st != SATA_OK) return st;
  if (rows == 0) return ok();
  if (!x || !phi) return fail(SATA_ERR_INVALID_ARG, "null tensor pointer");
  hipStream_t s = (hipStream_t)stream;
  sata::DevTable t;
  if ((st = get_table(d, P, s, &t)) != SATA_OK) return st;
  hipError_t e = sata::launch_feature_map(x, xt == SATA_BF16, rows, t, phi, s);
  if (e != hipSuccess) return hip_fail(e, "feature_map launch");
  return ok();
}

sata_status sata_prefill_operands(sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk,
                                  sata_operands* operands) {
  if (!operands) return fail(SATA_ERR_INVALID_ARG, "null output pointer");
  int64_t D = 0;
  sata_status st = check_prefill_args(dt, B, H, n, d_k, d_v, P, chunk, &D);
  if (st != SATA_OK) return st;
  if (prefill_path(dt, B * H, n, d_k, d_v, P, chunk) == PrefillPath::kFloat32)
    *operands = SATA_OPERANDS_F32;
  else
    *operands = dt == SATA_BF16 ? SATA_OPERANDS_BF16 : SATA_OPERANDS_SPLIT;
  return ok();
}

sata_status sata_prefill_parts(sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk, int* parts) {
  if (!parts) return fail(SATA_ERR_INVALID_ARG, "null output pointer");
  int64_t D = 0;
  sata_status st = check_prefill_args(dt, B, H, n, d_k, d_v, P, chunk, &D);
  if (st != SATA_OK) return st;
  *parts = 1;
  sata::FeatPrefillPlan fp;
  if (prefill_path(dt, B * H, n, d_k, d_v, P, chunk) == PrefillPath::kFeat &&
      sata::plan_prefill_feat(D, B * H, n, d_k, d_v, P, chunk, dt == SATA_F32, kMaxFeatWorkspace, &fp))
    *parts = fp.parts;
  return ok();
}

sata_status sata_prefill(const void* q, const void* k, const void* v, sata_dtype dt, int B, int H, int n,
                         int d_k, int d_v, int P, int chunk, void* y, float* S_out, void* stream) {
  return prefill(Way::kEstimate, q, k, v, dt, B, H, 1, n, d_k, d_v, P, chunk, y, S_out, stream);
}

sata_status sata_prefill_grouped(const void* q, const void* k, const void* v, sata_dtype dt, int B, int H_kv,
                                 int G, int n, int d_k, int d_v, int P, int chunk, void* y, float* S_out,
                                 void* stream) {
  sata_status st = check_groups(B, H_kv, G);
  if (st != SATA_OK) return st;
  return prefill(Way::kEstimate, q, k, v, dt, B, H_kv, G, n, d_k, d_v, P, chunk, y, S_out, stream);
}

sata_status sata_testing_prefill(int pairs, const void* q, const void* k, const void* v, sata_dtype dt, int B,
                                 int H_kv, int G, int n, int d_k, int d_v, int P, int chunk, void* y, float* S_out,
                                 void* stream) {
  sata_status st = check_groups(B, H_kv, G);
  if (st != SATA_OK) return st;
  return prefill(pairs ? Way::kPairs : Way::kScan, q, k, v, dt, B, H_kv, G, n, d_k, d_v, P, chunk, y, S_out, stream);
}

sata_status sata_testing_prefill_route(sata_dtype dt, int B, int H_kv, int G, int n, int d_k, int d_v, int P,
                                       int chunk, int want_state, sata_route* route) {
  if (!route) return fail(SATA_ERR_INVALID_ARG, "null output pointer");
  sata_status st = check_groups(B, H_kv, G);
  if (st != SATA_OK) return st;
  int64_t D = 0;
  if ((st = check_prefill_args(dt, B, H_kv, n, d_k, d_v, P, chunk, &D)) != SATA_OK) return st;
  if (direct_pays(dt, B * H_kv, G, n, d_k, d_v, P, chunk, D, want_state != 0,
                  vector_rows(nullptr, nullptr, nullptr, dt, d_k, d_v))) {
    *route = SATA_ROUTE_PAIRS;
    return ok();
  }
  return sata_testing_scan_route(dt, B, H_kv, n, d_k, d_v, P, chunk, route);
}

sata_status sata_testing_scan_route(sata_dtype dt, int B, int H_kv, int n, int d_k, int d_v, int P, int chunk,
                                    sata_route* route) {
  if (!route) return fail(SATA_ERR_INVALID_ARG, "null output pointer");
  int64_t D = 0;
  sata_status st = check_prefill_args(dt, B, H_kv, n, d_k, d_v, P, chunk, &D);
  if (st != SATA_OK) return st;
  static const sata_route kScans[] = {SATA_ROUTE_MFMA32, SATA_ROUTE_BLOCKS, SATA_ROUTE_FEATURES, SATA_ROUTE_FLOAT32};
  *route = kScans[(int)prefill_path(dt, B * H_kv, n, d_k, d_v, P, chunk)];
  return ok();
}

sata_status sata_backward(const void* q, const void* k, const void* v, const void* dy, sata_dtype dt, int B, int H,
                          int n, int d_k, int d_v, int P, int chunk, void* dq, void* dk, void* dv, void* stream) {
  return backward(Way::kEstimate, q, k, v, dy, dt, B, H, n, d_k, d_v, P, chunk, dq, dk, dv, stream);
}

sata_status sata_testing_backward(int pairs, const void* q, const void* k, const void* v, const void* dy,
                                  sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk, void* dq,
                                  void* dk, void* dv, void* stream) {
  return backward(pairs ? Way::kPairs : Way::kScan, q, k, v, dy, dt, B, H, n, d_k, d_v, P, chunk, dq, dk, dv, stream);
}

sata_status sata_testing_backward_route(sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk,
                                        sata_route* route) {
  if (!route) return fail(SATA_ERR_INVALID_ARG, "null output pointer");
  int64_t D = 0;
  sata_status st = check_backward_args(dt, B, H, n, d_k, d_v, P, chunk, &D);
  if (st != SATA_OK) return st;
  *route = backward_direct_pays(dt, B * H, n, d_k, d_v, P, D) ? SATA_ROUTE_PAIRS : SATA_ROUTE_FLOAT32;
  return ok();
}

sata_status sata_decode_step(float* S, const void* q, const void* k, const void* v, sata_dtype dt, int B,
                             int H, int d_k, int d_v, int P, void* y, void* stream) {
  return decode_step(S, nullptr, q, k, v, dt, B, H, d_k, d_v, P, y, stream);
}

sata_status sata_decode_step_noalloc(float* S, const void* q, const void* k, const void* v, sata_dtype dt, int B,
                                    int H, int d_k, int d_v, int P, void* y, void* stream) {
  if (!valid_dtype(dt)) return fail(SATA_ERR_INVALID_ARG, "unknown dtype %d", (int)dt);
  if (B < 1 || H < 1) return fail(SATA_ERR_INVALID_ARG, "B=%d H=%d must be >= 1", B, H);
  int64_t D = 0;
  sata_status st = check_dims(d_k, d_v, P, &D);
  if (st != SATA_OK) return st;
  if ((int64_t)B * H > kMaxHeads) return fail(SATA_ERR_TOO_LARGE, "B*H=%lld exceeds %d", (long long)B * H, kMaxHeads);
  if (!S || !q || !k || !v || !y) return fail(SATA_ERR_INVALID_ARG, "null tensor pointer");
  const int BH = B * H;
  sata::DecodePlan plan = sata::plan_decode(D, d_k, d_v, BH);
  const int64_t rows = std::max<int64_t>(plan.nslices > 1 ? plan.nslices : 0, plan.flat_np > 1 ? plan.flat_np : 0);
  const size_t partial_bytes = sizeof(float) * (size_t)BH * (size_t)rows * (size_t)(d_v + 1);
  if (partial_bytes > kScratchBytes - kScratchCounterBytes)
    return fail(SATA_ERR_TOO_LARGE, "partial sums of %zu bytes exceed the %zu-byte scratch", partial_bytes,
                kScratchBytes - kScratchCounterBytes);
  sata::DevTable t;
  if ((st = find_table(d_k, P, &t)) != SATA_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  unsigned char* base = nullptr;
  if ((st = get_scratch(s, &base)) != SATA_OK) return st;
  float* partial = rows > 0 ? (float*)(base + kScratchCounterBytes) : nullptr;
  int* counters = plan.flat_np > 1 ? (int*)base : nullptr;
  hipError_t e = sata::launch_decode(S, q, k, v, y, dt == SATA_BF16, BH, d_k, d_v, t, plan, partial, counters, s);
  if (e != hipSuccess) return hip_fail(e, "decode launch");
  return ok();
}

sata_status sata_decode_step_compensated(float* S, float* R, const void* q, const void* k, const void* v,
                                         sata_dtype dt, int B, int H, int d_k, int d_v, int P, void* y,
                                         void* stream) {
  if (!R) return fail(SATA_ERR_INVALID_ARG, "null residual pointer");
  return decode_step(S, R, q, k, v, dt, B, H, d_k, d_v, P, y, stream);
}

int64_t sata_residual_elems(int d_k, int d_v, int P) {
  if (d_k < 1 || d_v < 1 || P < 1) return -1;
  const int64_t f = sata::feature_count(d_k, P);
  if (f < 0) return -1;
  return f + (int64_t)(d_k + 1) * d_v;
}

sata_status sata_decode_step_grouped(float* S, const void* q, const void* k, const void* v, sata_dtype dt, int B,
                                     int H_kv, int G, int d_k, int d_v, int P, void* y, void* stream) {
  if (!valid_dtype(dt)) return fail(SATA_ERR_INVALID_ARG, "unknown dtype %d", (int)dt);
  if (B < 1 || H_kv < 1) return fail(SATA_ERR_INVALID_ARG, "B=%d H_kv=%d must be >= 1", B, H_kv);
  if (G < 1) return fail(SATA_ERR_INVALID_ARG, "G=%d must be >= 1", G);
  int64_t D = 0;
  sata_status st = check_dims(d_k, d_v, P, &D);
  if (st != SATA_OK) return st;
  if ((int64_t)B * H_kv * G > kMaxHeads)
    return fail(SATA_ERR_TOO_LARGE, "B*H_kv*G=%lld exceeds %d", (long long)B * H_kv * G, kMaxHeads);
  if (!S || !q || !k || !v || !y) return fail(SATA_ERR_INVALID_ARG, "null tensor pointer");
  if (G == 1) return sata_decode_step(S, q, k, v, dt, B, H_kv, d_k, d_v, P, y, stream);
  if (G != 2 && G != 4 && G != 8) return fail(SATA_ERR_UNSUPPORTED, "G=%d; supported: 1, 2, 4, 8", G);
  if (((uintptr_t)S & 15) != 0) return fail(SATA_ERR_UNSUPPORTED, "grouped decode needs a 16-byte aligned state");
  const int BH = B * H_kv;
  sata::GroupedDecodePlan plan = sata::plan_decode_grouped(D, d_k, d_v, BH, G);
  if (plan.tu <= 0)
    return fail(SATA_ERR_UNSUPPORTED, "no grouped decode plan fits on chip for d_k=%d d_v=%d P=%d G=%d", d_k, d_v, P,
                G);
  hipStream_t s = (hipStream_t)stream;
  sata::DevTable t;
  if ((st = get_table(d_k, P, s, &t)) != SATA_OK) return st;
  float* partial = nullptr;
  int* counters = nullptr;
  if (plan.np > 1) {
    void* ws = nullptr;
    const size_t bytes = sizeof(float) * (size_t)BH * plan.np * G * (d_v + 1);
    if ((st = get_workspace(bytes, s, &ws)) != SATA_OK) return st;
    partial = (float*)ws;
    if ((st = get_counters(BH, s, &counters)) != SATA_OK) return st;
  }
  hipError_t e = sata::launch_decode_grouped(S, q, k, v, y, dt == SATA_BF16, BH, d_k, d_v, t, plan, partial,
                                             counters, s);
  if (e != hipSuccess) return hip_fail(e, "grouped decode launch");
  return ok();
}

const char* sata_status_string(sata_status s) {
  switch (s) {
    case SATA_OK: return "ok";
    case SATA_ERR_INVALID_ARG: return "invalid argument";
    case SATA_ERR_UNSUPPORTED: return "unsupported";
    case SATA_ERR_TOO_LARGE: return "too large";
    case SATA_ERR_HIP: return "HIP error";
  }
  return "unknown status";
}

const char* sata_last_error(void) { return g_last_error.c_str(); }

void sata_release(void) {
  std::lock_guard<std::mutex> lock(g_mu);
  int cur = 0;
  hipGetDevice(&cur);
  for (auto& kv : g_devices) {
    hipSetDevice(kv.first);
    for (auto& t : kv.second.tables) {
      hipFree(t.second.packed);
      hipFree(t.second.weight);
      hipFree(t.second.gen);
    }
    for (auto& t : kv.second.state_tables) hipFree(t.second.ptr);
    for (auto& w : kv.second.workspaces) hipFree(w.second.ptr);
    for (auto& w : kv.second.counters) hipFree(w.second.ptr);
  }
  g_devices.clear();
  hipSetDevice(cur);
}

}  // extern "C"
