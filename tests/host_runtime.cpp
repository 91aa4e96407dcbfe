// A host stand-in for the HIP runtime and for the kernel launchers, so that
// the runtime of csrc/ee_api.hip (contexts, staging, buffers, error paths) runs
// and is tested on the CPU: device and pinned memory are malloc'd blocks, a
// launch does its job before it returns, and every pointer that a launch
// would hand to the device is checked against the live blocks (a launch with
// a bad range is counted and refused). The decoder itself is replaced by one
// whose outputs name their inputs: the cache entries of a position hold its
// input token, the token after t is (t + 1) % V, and a head's is that of its
// vector's first element.
// Test control: host_fail_alloc (fail the n-th next allocation of a kind),
// host_device_limit (bytes of device memory); host_bad_ranges counts the
// ranges refused.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "ee_internal.h"

namespace {

struct Block {
  size_t bytes;
  bool device;
};
std::map<const char*, Block> g_blocks;
size_t g_device_bytes = 0, g_limit = ~size_t(0);
int g_fail[2] = {0, 0};  // pinned, device: countdown to a failing allocation
int g_bad = 0;
int g_pinned_allocs = 0, g_tilings = 0;
int g_max_wgs = 1, g_grid = 0;

// hipMemset runs on the null stream, which the contexts' streams do not wait
// for: it happens with the next operation that does, and otherwise as late as
// after the first kernel or copy of another stream.
struct Pending {
  void* p;
  int v;
  size_t n;
};
std::vector<Pending> g_memsets;
void settle() {
  for (const Pending& m : g_memsets) memset(m.p, m.v, m.n);
  g_memsets.clear();
}

hipError_t host_alloc(void** p, size_t bytes, bool device) {
  *p = nullptr;
  if (g_fail[device] > 0 && --g_fail[device] == 0) return hipErrorOutOfMemory;
  if (device && bytes > g_limit - g_device_bytes) return hipErrorOutOfMemory;
  char* q = static_cast<char*>(malloc(bytes));
  if (!q) return hipErrorOutOfMemory;
  memset(q, 0xAB, bytes);  // a fresh allocation holds nothing useful
  g_blocks[q] = Block{bytes, device};
  if (device) g_device_bytes += bytes;
  else ++g_pinned_allocs;
  *p = q;
  return hipSuccess;
}

hipError_t host_free(void* p) {
  if (!p) return hipSuccess;
  settle();
  auto it = g_blocks.find(static_cast<char*>(p));
  if (it == g_blocks.end()) {
    ++g_bad;
    return hipErrorInvalidValue;
  }
  if (it->second.device) g_device_bytes -= it->second.bytes;
  memset(p, 0xCD, it->second.bytes);
  free(p);
  g_blocks.erase(it);
  return hipSuccess;
}

char g_params[sizeof(ee::DevParams) * ee::kParamSlots];
char g_scratch[ee::kScratchBytes];

bool live(const void* p, int64_t bytes) {
  const char* q = static_cast<const char*>(p);
  if (q >= g_scratch && q + bytes <= g_scratch + sizeof(g_scratch)) return bytes >= 0;
  if (q >= g_params && q + bytes <= g_params + sizeof(g_params)) return bytes >= 0;
  auto it = g_blocks.upper_bound(q);
  if (it == g_blocks.begin()) return false;
  --it;
  return bytes >= 0 && q >= it->first && q + bytes <= it->first + it->second.bytes;
}

bool ok(const void* p, int64_t bytes) {
  if (live(p, bytes)) return true;
  ++g_bad;
  return false;
}

void write_entry(const ee::DevParams& p, int wbf16, int pos, int tok) {
  const int page = p.block_table[pos >> p.page_shift], slot = pos & (p.page_size - 1);
  for (int l = 0; l < p.L; ++l)
    for (int h = 0; h < p.K; ++h) {
      const int64_t off = l * p.layer_stride + ((static_cast<int64_t>(page) * p.K + h) * p.page_size + slot) * p.D;
      for (int d = 0; d < p.D; ++d) {
        const float v = static_cast<float>(tok);  // exact in bf16 up to 256
        for (void* pool : {p.kpool, p.vpool}) {
          if (wbf16) {
            uint32_t u;
            memcpy(&u, &v, 4);
            static_cast<uint16_t*>(pool)[off + d] = static_cast<uint16_t>(u >> 16);
          } else {
            static_cast<float*>(pool)[off + d] = v;
          }
        }
      }
    }
}

hipError_t full_depth(const ee::DevParams& p, int wbf16, int pos0, const int32_t* tok, int n, bool head) {
  if (!ok(tok, 4ll * n) || !ok(p.hist_tok, 4ll * (pos0 + n)) || !ok(p.ctl, sizeof(ee::StepCtl))) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i) {
    int t = tok[i];
    if (t < 0 || t >= p.V) {
      p.ctl->error = ee::kErrToken;
      t = 0;
    }
    p.hist_tok[pos0 + i] = t;
    write_entry(p, wbf16, pos0 + i, t);
    if (head && i == n - 1) p.ctl->next_token = (t + 1) % p.V;
  }
  return hipSuccess;
}

hipError_t decode(const ee::DevParams& p, int wbf16, int pos0, int n) {
  if (p.force_tok && !ok(p.force_tok, 4ll * n)) return hipErrorInvalidValue;
  if (p.force_exit && !ok(p.force_exit, 4ll * n)) return hipErrorInvalidValue;
  if (!ok(p.ring_tok, 4ll * n) || !ok(p.ring_exit, 4ll * n) || !ok(p.ring_conf, 4ll * n)) return hipErrorInvalidValue;
  if (p.dbg_logits_r && (!ok(p.dbg_logits_r, 4ll * p.V) || !ok(p.dbg_logits_f, 4ll * p.V))) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i) {
    const int t = p.force_tok ? p.force_tok[i] : p.ctl->next_token;
    p.hist_tok[pos0 + i] = t;
    write_entry(p, wbf16, pos0 + i, t);
    const int next = (t + 1) % p.V, fe = p.force_exit ? p.force_exit[i] : -1;
    p.ring_tok[i] = next;
    p.ring_exit[i] = fe == 1;
    p.ring_conf[i] = 0.5f;
    if (p.ring_would) p.ring_would[i] = 0;
    if (p.ring_mass && p.nucleus) p.ring_mass[i] = 0.25f;
    p.ctl->next_token = next;
    p.ctl->readout_token = p.ctl->full_token = next;
    for (int v = 0; v < p.V && p.dbg_logits_r; ++v) p.dbg_logits_r[v] = p.dbg_logits_f[v] = static_cast<float>(v == next);
  }
  return hipSuccess;
}

}  // namespace

extern "C" {
void host_fail_alloc(int device, int nth) { g_fail[device] = nth; }
void host_device_limit(uint64_t bytes) { g_limit = bytes; }
uint64_t host_device_bytes() { return g_device_bytes; }
int host_bad_ranges() { return g_bad; }
int host_pinned_allocs() { return g_pinned_allocs; }
int host_tilings() { return g_tilings; }
void host_max_wgs(int n) { g_max_wgs = n; }
int host_last_grid() { return g_grid; }
int host_live_blocks() { return static_cast<int>(g_blocks.size()); }

hipError_t hipMalloc(void** p, size_t n) { return host_alloc(p, n, true); }
hipError_t hipFree(void* p) { return host_free(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) {
  if (!(flags & hipHostMallocCoherent)) ++g_bad;  // kernels read and write it in place
  return host_alloc(p, n, false);
}
hipError_t hipHostFree(void* p) { return host_free(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  settle();
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memmove(d, s, n);
  settle();
  return hipSuccess;
}
hipError_t hipMemcpy2D(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind) {
  settle();
  for (size_t i = 0; i < h; ++i) memcpy(static_cast<char*>(d) + i * dp, static_cast<const char*>(s) + i * sp, w);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  g_memsets.push_back(Pending{d, v, n});
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  settle();
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (!s) settle();
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(1);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "host"; }
}

namespace ee {

hipError_t launch_io(const IoBatch& b, hipStream_t) {
  if (b.n > IoBatch::kMax) ++g_bad;
  if (b.counters) memset(b.counters, 0, sizeof(Counters));
  if (b.tw_words) memset(b.tw, 0, b.tw_words * 8);
  if (b.ctl) {
    const int32_t next = b.ctl->next_token;
    const uint32_t keep = b.ctl->pad[0];
    memset(b.ctl, 0, sizeof(StepCtl));
    b.ctl->next_token = next;
    b.ctl->pad[0] = keep;
  }
  for (int j = 0; j < b.n; ++j) {
    const IoJob& q = b.job[j];
    if (!ok(q.dst, q.words * (q.form == kIoTag ? 8 : 4))) continue;
    if (!ok(q.src, q.words * (q.form == kIoUntag ? 8 : 4))) continue;
    for (int64_t i = 0; i < q.words; ++i) {
      const uint32_t v = q.form == kIoUntag ? static_cast<uint32_t>(static_cast<const uint64_t*>(q.src)[i])
                                            : static_cast<const uint32_t*>(q.src)[i];
      if (q.form == kIoTag) static_cast<uint64_t*>(q.dst)[i] = v;
      else static_cast<uint32_t*>(q.dst)[i] = v;
    }
  }
  settle();
  return hipSuccess;
}
hipError_t params_address(int slot, void** out) {
  *out = g_params + sizeof(DevParams) * slot;
  return hipSuccess;
}
hipError_t scratch_address(int, void** out) {
  *out = g_scratch;
  return hipSuccess;
}
hipError_t launch_decode_per_op(const DevParams& p, int wbf16, int pos0, int n, int, hipStream_t) {
  return decode(p, wbf16, pos0, n);
}
hipError_t launch_decode_persistent(const PersistentLaunch& L, int pos0, int n) {
  // every workgroup stores a head partial record
  g_grid = L.nwg;
  if (!ok(L.params_host->head_part, 4ll * kStatFloats * L.nwg)) return hipErrorInvalidValue;
  return decode(*L.params_host, L.wbf16, pos0, n);
}
hipError_t launch_prefill_per_op(const DevParams& p, int wbf16, int pos0, const int32_t* tok, int n, int, hipStream_t) {
  return full_depth(p, wbf16, pos0, tok, n, true);
}
hipError_t launch_prefill_persistent(const PersistentLaunch& L, int pos0, int n) {
  return full_depth(*L.params_host, L.wbf16, pos0, L.params_host->force_tok, n, true);
}
// A tiled copy names its matrix and holds its first bytes.
static void stamp(const void* W, void* T) {
  memcpy(T, &W, 8);
  memcpy(static_cast<char*>(T) + 8, W, 8);
}
static bool stamped(const void* W, const void* T) {
  if (!ok(T, 16)) return false;
  return memcmp(T, &W, 8) == 0 && memcmp(static_cast<const char*>(T) + 8, W, 8) == 0;
}

hipError_t launch_batched_pass(const BatchPass& bp, int pos0, const int32_t* tok, int n, hipStream_t s) {
  for (int l = 0; l < bp.p.L; ++l) {
    const LayerW& w = bp.layers[l];
    const int H = bp.p.H, AD = bp.p.A * bp.p.D, F = bp.p.F;
    const struct { const void* w; int n, k; } m[4] = {{w.wqkv, bp.p.qkv_rows, H}, {w.wo, H, AD}, {w.wgu, 2 * F, H}, {w.wd, H, F}};
    for (int i = 0; i < 4; ++i) {
      void* t = bp.spare;
      if (bp.tiled) {
        const LayerT& lt = bp.tiled[l];
        void* const kept[4] = {lt.wqkv, lt.wo, lt.wgu, lt.wd};
        t = kept[i];
      } else if (launch_tile_weights(bp.wbf16, m[i].w, m[i].n, m[i].k, t, s) != hipSuccess) {
        return hipErrorInvalidValue;
      }
      if (!stamped(m[i].w, t)) ++g_bad;  // a copy that is not there or not up to date
    }
  }
  const int row = (n - 1) % bp.buf.max_positions;
  if (!ok(bp.buf.X, 4ll * (row + 1) * bp.p.H)) return hipErrorInvalidValue;
  const hipError_t e = full_depth(bp.p, bp.wbf16, pos0, tok, n, false);
  if (e == hipSuccess && bp.head) bp.buf.X[static_cast<int64_t>(row) * bp.p.H] = static_cast<float>(tok[n - 1]);
  return e;
}
hipError_t launch_head_eval(const DevParams& p, int, const float* x, int, int, hipStream_t) {
  if (!ok(x, 4ll * p.H) || (p.dbg_logits_r && (!ok(p.dbg_logits_r, 4ll * p.V) || !ok(p.dbg_logits_f, 4ll * p.V))))
    return hipErrorInvalidValue;
  const int next = (static_cast<int>(fabsf(x[0])) + 1) % p.V;
  p.ctl->next_token = p.ctl->readout_token = p.ctl->full_token = next;
  for (int v = 0; v < p.V && p.dbg_logits_r; ++v) p.dbg_logits_r[v] = p.dbg_logits_f[v] = x[0];
  return hipSuccess;
}
hipError_t launch_tile_weights(int wbf16, const void* W, int N, int K, void* T, hipStream_t) {
  ++g_tilings;
  if (!ok(W, static_cast<int64_t>(N) * K * (wbf16 ? 2 : 4)) || !ok(T, batch_weight_bytes(wbf16, N, K)))
    return hipErrorInvalidValue;
  stamp(W, T);
  return hipSuccess;
}
size_t batch_weight_bytes(int wbf16, int N, int K) {
  return static_cast<size_t>((N + 15) / 16 * 16) * ((K + 63) / 64 * 64) * (wbf16 ? 2 : 4);
}
size_t batch_plane_bytes(int wbf16, int P, int K) {
  return static_cast<size_t>((P + 15) / 16 * 16) * ((K + 63) / 64 * 64) * (wbf16 ? 6 : 4);
}
hipError_t launch_stream_read(const void*, int64_t, int, uint32_t*, hipStream_t) { return hipSuccess; }
size_t lds_bytes(const DevParams&) { return 0; }
int fill_batch_slots(const DevParams&) { return 1; }
int chunks_per_lane(const DevParams& p, int wbf16) { return (p.H / (wbf16 ? 8 : 4) + 63) / 64; }
int persistent_max_wgs_per_cu(const DevParams&, int, size_t) { return g_max_wgs; }

}  // namespace ee
