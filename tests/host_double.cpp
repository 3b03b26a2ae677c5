// host_double.cpp -- a stand-in for the device under the library's host code.
//
// Linked with csrc/api.cpp (compiled for the host) into a library of its own:
// device memory is a byte count with a limit, streams and events do nothing,
// and every kernel launch of a ring product is written to a log with what its
// tables say.  The tests drive the C entry points with made-up device
// addresses and read which kernels a call would launch, over which tiles, and
// how its workspace was asked for.  The tile geometry comes from libmpc.so.
#include <rocblas/rocblas.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "internal.h"

namespace {
std::string g_log;
std::map<char*, size_t> g_blocks;  // device allocations
size_t g_used, g_limit = (size_t)288 << 30, g_mallocs, g_refused, g_frees, g_syncs;
char* g_next = (char*)((uintptr_t)1 << 44);  // addresses that are never read
constexpr size_t kReal = 4 << 20;            // small blocks (descriptor tables) hold what is copied there

void say(const char* f, ...) {
  char line[512];
  va_list v;
  va_start(v, f);
  std::vsnprintf(line, sizeof line, f, v);
  va_end(v);
  g_log += line;
  g_log += '\n';
}
long long at(const void* p) { return (long long)(uintptr_t)p; }
}  // namespace

extern "C" {
const char* double_log() { return g_log.c_str(); }
void double_clear() { g_log.clear(); g_mallocs = g_refused = g_frees = g_syncs = 0; }
void double_limit(size_t bytes) { g_limit = bytes; }
void double_counts(size_t out[5]) {
  const size_t v[5] = {g_mallocs, g_refused, g_frees, g_syncs, g_used};
  std::memcpy(out, v, sizeof v);
}

hipError_t hipMalloc(void** p, size_t n) {
  ++g_mallocs;
  if (n > g_limit || g_used > g_limit - n) {
    ++g_refused;
    return hipErrorOutOfMemory;
  }
  char* b = n <= kReal ? (char*)std::aligned_alloc(256, (n + 255) / 256 * 256) : g_next;
  if (n > kReal) g_next += (n + ((size_t)1 << 21)) / 256 * 256;
  g_blocks[b] = n;
  g_used += n;
  *p = b;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  ++g_frees;
  auto it = g_blocks.find((char*)p);
  if (it == g_blocks.end()) return p ? hipErrorInvalidValue : hipSuccess;
  g_used -= it->second;
  if (it->second <= kReal) std::free(p);
  g_blocks.erase(it);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) { std::memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)((uintptr_t)1 << 43); return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = g_limit - g_used; *t = g_limit; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)2; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++g_syncs; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = (hipGraph_t)3; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* g, hipGraph_t, hipGraphNode_t*, char*, size_t) { *g = (hipGraphExec_t)4; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
rocblas_status rocblas_create_handle(rocblas_handle*) { return rocblas_status_internal_error; }
rocblas_status rocblas_destroy_handle(rocblas_handle) { return rocblas_status_success; }
rocblas_status rocblas_set_stream(rocblas_handle, hipStream_t) { return rocblas_status_internal_error; }
rocblas_status rocblas_dgemm(rocblas_handle, rocblas_operation, rocblas_operation, rocblas_int, rocblas_int, rocblas_int, const double*,
                             const double*, rocblas_int, const double*, rocblas_int, const double*, double*, rocblas_int) {
  return rocblas_status_internal_error;
}
}  // extern "C"

namespace mpc {
hipError_t launch_prg_fill(hipStream_t, u64, u64*, size_t) { say("fill"); return hipSuccess; }
hipError_t launch_open(hipStream_t, const OpenJob*, const i64*, int n, i64) { say("open jobs=%d", n); return hipSuccess; }
hipError_t launch_im2col(hipStream_t, const u64*, const u64*, i64, i64, i64, i64, i64, i64, u64*) { say("im2col"); return hipSuccess; }
hipError_t launch_beaver_matmul_small(hipStream_t, const SmallMatmul& m) {
  say("small M=%lld N=%lld K=%lld", (long long)m.M, (long long)m.N, (long long)m.K);
  return hipSuccess;
}
hipError_t launch_plain_gemm(hipStream_t, const PlainProblem*, TileMap m, int tiles) { say("plain probs=%d tiles=%d", m.nprob, tiles); return hipSuccess; }
hipError_t launch_splitk_reduce_grouped(hipStream_t, const ReduceTables& t, i64) { say("reduce jobs=%d", t.njobs); return hipSuccess; }
hipError_t launch_mp_open(hipStream_t, const MpIn&, const MpIn&, int P, size_t, u64*) { say("mp_open P=%d", P); return hipSuccess; }
hipError_t launch_mp_fill_sum(hipStream_t, const MpKeys&, int, size_t, const MpOut&, u64*) { say("mp_fill"); return hipSuccess; }
hipError_t launch_pack(hipStream_t, const PackTables& t, i64, PackSet set) { say("limb_pack jobs=%d set=%d", t.njobs, (int)set); return hipSuccess; }
hipError_t launch_pack_party(hipStream_t, const PartyPackTables& t) { say("limb_pack_party P=%d", t.side[0].P); return hipSuccess; }
hipError_t launch_res_pack(hipStream_t, const PackTables& t, i64, PackSet set) { say("res_pack jobs=%d set=%d", t.njobs, (int)set); return hipSuccess; }
hipError_t launch_res_pack_party(hipStream_t, const PartyPackTables& t) { say("res_pack_party P=%d", t.side[0].P); return hipSuccess; }
hipError_t launch_limb_gemm(hipStream_t, const GemmTables& t, int tiles) {
  const LimbProblem* p = t.probs ? t.probs : t.iprobs;
  say("limb variant=%d group_m=%d remap=%d probs=%d tiles=%d", t.sched.variant, t.sched.group_m, t.sched.xcd_remap, t.map.nprob, tiles);
  for (int i = 0; i < t.map.nprob; ++i)
    say("limb_problem M=%lld N=%lld kb_begin=%d kb_end=%d slices=%d cls=%d", (long long)p[i].M, (long long)p[i].N, p[i].kb_begin, p[i].kb_end,
        p[i].slices, p[i].cls);
  return hipSuccess;
}
hipError_t launch_res_gemm(hipStream_t, const ResGemmTables& t, int tiles, int tile, int grid, bool conv) {
  const ResProblem* p = t.probs ? t.probs : t.iprobs;
  const int* start = t.probs ? t.tile_start : t.itile_start;
  int bm, bn;
  res_tile_shape(tile, &bm, &bn);
  say("res bm=%d bn=%d probs=%d tiles=%d grid=%d conv=%d", bm, bn, t.nprob, tiles, grid, (int)conv);
  for (int i = 0; i < t.nprob; ++i)
    say("res_problem bm=%d bn=%d R=%lld pr=%lld PA0=%lld pa=%lld pb=%lld kbs=%d kb_begin=%d kb_end=%d m0=%d nm=%d ntm=%d ntn=%d n64=%d start=%d end=%d "
        "ksz=%d stride=%d",
        bm, bn, at(p[i].R), (long long)p[i].pr, at(p[i].PA0), (long long)p[i].pa, (long long)p[i].pb, p[i].kbs, p[i].kb_begin, p[i].kb_end, p[i].m0,
        p[i].nm, p[i].ntm, p[i].ntn, p[i].n64, start[i], start[i + 1], p[i].cv.ksz, p[i].cv.stride);
  return hipSuccess;
}
hipError_t launch_res_combine(hipStream_t, const ResOutTables& t, i64 units) {
  const ResOut* o = t.outs ? t.outs : t.iouts;
  say("combine outs=%d units=%lld", t.nout, (long long)units);
  for (int i = 0; i < t.nout; ++i)
    say("combine_out M=%lld N=%lld nch=%d R=%lld pc=%lld", (long long)o[i].M, (long long)o[i].N, o[i].nch, at(o[i].R), (long long)o[i].pc);
  return hipSuccess;
}
}  // namespace mpc
