// Launchers of the host-only build that checks the C ABI under sanitizers: nothing can be launched there, so each
// reports that there is no device.  (The real ones live next to their kernels.)  The two calls of the runtime with which the
// static scratch is looked up are answered here, so that flux_attn_decode_static gets as far as its launcher, which notes
// what it was given.
#include "flux_internal.h"

extern "C" {
hipError_t hipGetDevice(int* device) { *device = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { *p = const_cast<void*>(symbol); return hipSuccess; }
// of the last launch_decode
const void *hostcheck_status, *hostcheck_partials, *hostcheck_counters;
// what a decode call launches, and whether the rows that its parts leave behind end within what holds them: the small
// region or the partials of a context whose workspace is exactly what flux_workspace_needed says, and the static scratch
// where flux_attn_decode_static accepts the shape
int hostcheck_decode_wgs(const flux_attn_cfg* cfg, int batch, int max_kv_len) { return flux::plan_decode(*cfg, batch, max_kv_len).wgs; }
int hostcheck_decode_in_partials(const flux_attn_cfg* cfg, int batch, int max_kv_len) { return flux::plan_decode(*cfg, batch, max_kv_len).in_partials; }
// whether the blocks of all lists can be counted in 32 bits, each as up to 15 more where that is done
int hostcheck_decode_blocks_fit(const flux_attn_cfg* cfg, int batch, int max_kv_len) {
  const flux::DecodePlan p = flux::plan_decode(*cfg, batch, max_kv_len);
  const long long blocks = ((long long)max_kv_len + (1ll << p.block_shift) - 1) >> p.block_shift;
  return (__int128)batch * p.pps * (blocks + (p.aligned_shift < 0 ? 0 : 15)) <= INT32_MAX;
}
// how an append is launched
int hostcheck_append(int batch, int hkv, int d, int total_new, int max_new, int ring, int window, unsigned* wgs) {
  const flux::AppendPlan p = flux::plan_append(batch, hkv, d, total_new, max_new, ring, window);
  *wgs = p.wgs;
  return p.form;
}
int hostcheck_decode_rows_fit(const flux_attn_cfg* cfg, int batch, int max_kv_len) {
  const flux::DecodePlan p = flux::plan_decode(*cfg, batch, max_kv_len);
  const size_t rows = (size_t)2 * p.wgs * p.rpu * (cfg->head_dim + 2) * sizeof(float);
  const size_t partials = flux_workspace_needed(cfg, batch, max_kv_len) - flux::kHeaderBytes - flux::kSmallBytes;
  const bool context = p.in_partials ? flux::decode_rows_at(p, false) * sizeof(float) + rows <= partials : rows <= flux::kSmallBytes;
  const size_t scratch = FLUX_STATIC_SCRATCH_BYTES - 256;
  const bool fixed = flux::decode_static_bytes(*cfg, p) > scratch || flux::decode_rows_at(p, true) * sizeof(float) + rows <= scratch;
  return context && fixed;
}
}

namespace flux {

hipError_t launch_kv_append(const Ctx&, const flux_kv_cache&, int, int, const void*, const void*, const int32_t*, int, int, int,
                            int, int, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_kv_compact_ring(const flux_kv_cache&, const flux_kv_cache&, int, int, int, int, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_decode(const Ctx& c, const flux_attn_cfg&, const void*, int, const flux_kv_cache&, const uint8_t*, int, const void*,
                         const void*, void*, hipStream_t) {
  hostcheck_status = c.status;
  hostcheck_partials = c.partials;
  hostcheck_counters = c.counters ? c.counters : c.decode_counters ? c.decode_counters : c.router_counters;
  return hipErrorNoDevice;
}
hipError_t launch_prefill(const Ctx&, const flux_attn_cfg&, const void*, const int32_t*, int, int, const flux_kv_cache&,
                          const uint8_t*, const BlockMask*, void*, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_router(const Ctx&, const void*, const int32_t*, int, int, int, const void*, const void*, const void*,
                         const void*, int, uint8_t*, float*, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_xa_select(const Ctx&, const flux_attn_cfg&, const void*, const int32_t*, int, const flux_kv_cache&, float,
                            uint8_t*, int, int, hipStream_t) { return hipErrorNoDevice; }

}  // namespace flux
