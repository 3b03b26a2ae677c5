// packed.h -- device helpers shared by the forms that pack their operands (the
// limb and the residue GEMM): descriptor tables read as constant memory, the
// pack jobs' arithmetic, buffer loads and the tile order.
#pragma once

#include "internal.h"

namespace mpc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr u64 kLimbBias = 0x8080808080808080ULL;

// Pointers into device global memory (global, not flat, instructions).
typedef __attribute__((address_space(1))) const u64 gcu64;
typedef __attribute__((address_space(1))) v4i gv4i;
__device__ __forceinline__ gcu64* gptr(const u64* p) { return (gcu64*)p; }


// Constant-memory views of a launch's descriptor tables (PackTables,
// GemmTables): inline entries are read from the kernel-argument segment,
// uploaded ones through the same constant address space, so that every
// access is a scalar load.  Each kernel takes its table struct as its only
// argument, so the struct starts the segment.  (The host compilation pass
// only parses the kernels; it gets plain pointers, which it can copy through.)
#if defined(__HIP_DEVICE_COMPILE__)
template <class T>
using cptr = __attribute__((address_space(4))) const T*;
#define MPC_KERNARG_PTR() __builtin_amdgcn_kernarg_segment_ptr()
#else
template <class T>
using cptr = const T*;
#define MPC_KERNARG_PTR() nullptr
#endif

struct PackView {
  cptr<PackJob> jobs;
  cptr<i64> bstart;
  int njobs;
};
__device__ __forceinline__ PackView pack_view() {
  const cptr<PackTables> t = (cptr<PackTables>)MPC_KERNARG_PTR();
  PackView v;
  v.njobs = t->njobs;
  v.jobs = t->jobs ? (cptr<PackJob>)(uintptr_t)t->jobs : t->ijobs;
  v.bstart = t->jobs ? (cptr<i64>)(uintptr_t)t->block_start : t->ibstart;
  return v;
}

// ------------------------------------------------------------------ packing
constexpr int kPackThreads = 256;  // 4 waves, one 32x32 block each
constexpr int kTPad = 33;          // LDS row stride (elements) of the transpose tile

__device__ __forceinline__ int find_job(cptr<i64> start, int njobs, i64 blk) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (start[mid] <= blk) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <int MODE> struct Mode;
template <> struct Mode<kModeCopy> {
  static constexpr int nin = 1, nout = 1;
  __device__ static u64 out(int, const u64* v) { return v[0]; }
};
template <> struct Mode<kModeSum2> {
  static constexpr int nin = 2, nout = 1;
  __device__ static u64 out(int, const u64* v) { return v[0] + v[1]; }
};
template <> struct Mode<kModePrgSum2> {  // v0, v1 drawn from the PRG -> v0 + v1
  static constexpr int nin = 2, nout = 1;
  __device__ static u64 out(int, const u64* v) { return v[0] + v[1]; }
};
template <> struct Mode<kModeOpenLeft> {  // x0, x1, a0, a1 -> eps, g0 = a0 + eps, a1
  static constexpr int nin = 4, nout = 3;
  __device__ static u64 out(int o, const u64* v) {
    return o == 0 ? v[0] + v[1] - v[2] - v[3] : o == 1 ? v[0] + v[1] - v[3] : v[3];
  }
};
template <> struct Mode<kModeOpenRight> {  // y0, y1, b0, b1 -> delta, b0, b1
  static constexpr int nin = 4, nout = 3;
  __device__ static u64 out(int o, const u64* v) {
    return o == 0 ? v[0] + v[1] - v[2] - v[3] : o == 1 ? v[2] : v[3];
  }
};
template <> struct Mode<kModePrgSum2A> {  // PRG v0, v1 -> v0 + v1, v1
  static constexpr int nin = 2, nout = 2;
  __device__ static u64 out(int o, const u64* v) { return o == 0 ? v[0] + v[1] : v[1]; }
};
template <> struct Mode<kModePrgSum2B> {  // PRG v0, v1 -> v0 + v1, v0, v1
  static constexpr int nin = 2, nout = 3;
  __device__ static u64 out(int o, const u64* v) { return o == 0 ? v[0] + v[1] : o == 1 ? v[0] : v[1]; }
};
template <> struct Mode<kModeOpenLeft2> {  // x0, x1, a0, a1 -> eps, g0 = a0 + eps
  static constexpr int nin = 4, nout = 2;
  __device__ static u64 out(int o, const u64* v) { return o == 0 ? v[0] + v[1] - v[2] - v[3] : v[0] + v[1] - v[3]; }
};
template <> struct Mode<kModeOpenRight1> {  // y0, y1, b0, b1 -> delta
  static constexpr int nin = 4, nout = 1;
  __device__ static u64 out(int, const u64* v) { return v[0] + v[1] - v[2] - v[3]; }
};

// The (kind, mode) pairs of one pack kernel: its waves' jobs each have one of them.
constexpr int km(int kind, int mode) { return kind * 16 + mode; }
template <int... KM>
struct PackPairs {
  static constexpr bool has(int kind) { return ((KM / 16 == kind) || ...); }
};
template <PackSet S> struct SetPairs;
template <> struct SetPairs<kPackMatmul> { using T = PackPairs<km(kPackRow, kModeOpenLeft), km(kPackCol, kModeOpenRight)>; };
template <> struct SetPairs<kPackMatmulPre> { using T = PackPairs<km(kPackRow, kModeOpenLeft2), km(kPackCol, kModeOpenRight1)>; };
template <> struct SetPairs<kPackConv> { using T = PackPairs<km(kPackRow, kModeOpenRight), km(kPackIm2col, kModeOpenLeft)>; };
template <> struct SetPairs<kPackConvDirect> { using T = PackPairs<km(kPackConvRow, kModeOpenRight), km(kPackChan, kModeOpenLeft)>; };
template <> struct SetPairs<kPackDeal> { using T = PackPairs<km(kPackRow, kModePrgSum2), km(kPackCol, kModePrgSum2)>; };
template <> struct SetPairs<kPackDealPre> { using T = PackPairs<km(kPackRow, kModePrgSum2A), km(kPackCol, kModePrgSum2B)>; };
template <> struct SetPairs<kPackDealConv> { using T = PackPairs<km(kPackRow, kModePrgSum2), km(kPackIm2col, kModeSum2)>; };
template <> struct SetPairs<kPackDealConvDirect> { using T = PackPairs<km(kPackConvRow, kModePrgSum2), km(kPackChan, kModeSum2)>; };
template <> struct SetPairs<kPackMatmulLeft> { using T = PackPairs<km(kPackRow, kModeOpenLeft)>; };
template <> struct SetPairs<kPackMatmulRight> { using T = PackPairs<km(kPackCol, kModeOpenRight)>; };
template <> struct SetPairs<kPackMatmulPreLeft> { using T = PackPairs<km(kPackRow, kModeOpenLeft2)>; };
template <> struct SetPairs<kPackMatmulPreRight> { using T = PackPairs<km(kPackCol, kModeOpenRight1)>; };
template <> struct SetPairs<kPackParties> { using T = PackPairs<km(kPackRow, kModeCopy), km(kPackRow, kModeSum2), km(kPackCol, kModeCopy)>; };
template <> struct SetPairs<kPackRing> { using T = PackPairs<km(kPackRow, kModeCopy), km(kPackCol, kModeCopy)>; };

// One block of one side of a P-party open: every party's two shares are read
// once, its triple share is packed at once and the opened value at the end, so
// no opened value is written to memory and read back (512 x 1024 x 1024 among
// three parties: 21 us; two opens and three packs of their own 17 + 23).
// emit(dst, w) packs a lane's 16 elements.
template <bool LEFT, class Emit>
__device__ __forceinline__ void party_block(cptr<PartyPack> s, const i64 (&off)[16], const bool (&ok)[16], bool interior, Emit emit) {
  u64 open[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) open[q] = 0;
  const int P = s->P;
#pragma unroll 1
  for (int p = P - 1; p >= 0; --p) {
    gcu64 *x = gptr(s->x[p]), *a = gptr(s->a[p]);
    u64 xv[16], av[16];
    if (interior) {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        xv[q] = x[off[q]];
        av[q] = a[off[q]];
      }
    } else {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        xv[q] = ok[q] ? x[off[q]] : 0;
        av[q] = ok[q] ? a[off[q]] : 0;
      }
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      open[q] += xv[q] - av[q];
      if (LEFT && p == 0) av[q] += open[q];  // the last party read: eps is whole
    }
    emit(s->dst[p], av);
  }
  emit(s->dst[P], open);
}

// ------------------------------------------------------------------ GEMM
__device__ __forceinline__ int find_problem(cptr<int> start, int nprob, int t) {
  int lo = 0, hi = nprob - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (start[mid] <= t) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Buffer resource over `bytes` bytes at `base` (raw, no stride).  Loads go
// through the scalar descriptor with a per-lane byte offset in one VGPR, a
// per-step scalar offset and the plane offset in the instruction's immediate.
constexpr int kBufferWord3 = 0x00020000;  // 32-bit raw data format, gfx9 family

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const uint8_t* base, i64 bytes) {
  const int n = bytes > 0x7fffffff ? 0x7fffffff : (int)bytes;
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, n, kBufferWord3);
}

__device__ __forceinline__ v4i ld_buf(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, soff, 0);
}

// Output tile of this workgroup.  One workgroup per tile.  Workgroups are
// dispatched to the 8 XCDs round-robin in index order, so index b runs on XCD
// b % 8 as that XCD's (b / 8)-th workgroup.  With the remap, each XCD takes
// runs of `run` consecutive tiles, the tiles it holds at one time (its 32
// compute units times the workgroups per unit), the runs going round the XCDs
// in turn: the tiles an XCD runs together are neighbours that share operand
// blocks in its L2, and when tiles differ in cost (a grouped launch lists its
// longest problems first) every XCD gets its share of each kind.  Inside a
// problem the tiles follow a grouped raster: runs of group_m tile rows, column
// by column.
constexpr int kXcds = 8, kXcdCUs = 32;

__device__ __forceinline__ int remap_tile(int b, int G, int run) {
  const int span = kXcds * run;
  if (b >= G / span * span) return b;  // the last partial round keeps dispatch order
  const int x = b % kXcds, j = b / kXcds;
  return ((j / run) * kXcds + x) * run + j % run;
}

}  // namespace
}  // namespace mpc
