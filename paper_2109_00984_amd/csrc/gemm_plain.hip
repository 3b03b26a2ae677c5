// gemm_plain.hip -- ring GEMM over Z/2^64 on the vector ALUs (the "plain" form).
//
// C = [A0 (+A0add) | A1] @ [B0 (+B0add) ; B1] mod 2^64 for a list of problems
// in one launch.  A 256-thread workgroup computes a 128x64 tile; each thread
// owns an 8x4 register block.  Operand tiles of 16 k are staged through LDS
// (the left tile stored k-major) with the next tile prefetched into registers;
// the LDS tiles are double-buffered, so one barrier per step hands them over.
//
// One ring multiply-accumulate a*b on 32-bit halves a = aL + 2^32 aH,
// b = bL + 2^32 bH:  a*b = aL*bL + 2^32 (aL*bH + aH*bL)  (mod 2^64).  The full
// aL*bL goes into a 64-bit accumulator (v_mad_u64_u32); the cross terms only
// matter modulo 2^32 and go into a 32-bit accumulator that is shifted in once
// at the end.
#include <utility>

#include "packed.h"

namespace mpc {
namespace {

constexpr int BM = 128, BN = 64, BK = kPlainBK;
constexpr int TM = 8, TN = 4;
constexpr int kThreads = 256;

__device__ __forceinline__ u64 load_a(const PlainProblem& p, i64 m, i64 k) {
  if (m >= p.M) return 0;
  if (k < p.K0) {
    u64 v = p.A0[m * p.lda0 + k];
    if (p.A0add) v += p.A0add[m * p.lda0 + k];
    return v;
  }
  if (k < p.K0 + p.K1) return p.A1[m * p.lda1 + (k - p.K0)];
  return 0;
}

__device__ __forceinline__ u64 load_b(const PlainProblem& p, i64 k, i64 n) {
  if (n >= p.N) return 0;
  if (k < p.K0) {
    u64 v = p.B0[k * p.ldb0 + n];
    if (p.B0add) v += p.B0add[k * p.ldb0 + n];
    return v;
  }
  if (k < p.K0 + p.K1) return p.B1[(k - p.K0) * p.ldb1 + n];
  return 0;
}

__global__ void __launch_bounds__(kThreads, 2)
    k_plain_gemm(const PlainProblem* __restrict__ probs, TileMap map) {
  // two buffers: a step computes from one while the next step's tiles are
  // stored into the other, so one barrier per step hands them over
  __shared__ u64 As[2][BK][BM];
  __shared__ u64 Bs[2][BK][BN];

  const int t = blockIdx.x;
  const int pi = find_problem((cptr<int>)(uintptr_t)map.tile_start, map.nprob, t);
  const PlainProblem p = probs[pi];
  const int local = t - map.tile_start[pi];
  const int ntn = (int)((p.N + BN - 1) / BN);
  const int tiles_mn = (int)((p.M + BM - 1) / BM) * ntn;
  const int slice = local / tiles_mn, lt = local % tiles_mn;
  const i64 m0 = (i64)(lt / ntn) * BM, n0 = (i64)(lt % ntn) * BN;
  // this workgroup's k range: one slice of a split problem, else all of k
  const i64 kbeg = (i64)slice * p.kslice;
  const i64 Ktot = min(p.K0 + p.K1, kbeg + p.kslice);

  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  // loader coordinates
  const int la_row = tid >> 1, la_k = (tid & 1) * 8;  // 8 consecutive k of one row
  const int lb_k = tid >> 4, lb_n = (tid & 15) * 4;   // 4 consecutive n of one k

  u64 ra[8], rb[4];
  auto fetch = [&](i64 k0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) ra[q] = load_a(p, m0 + la_row, k0 + la_k + q);
#pragma unroll
    for (int q = 0; q < 4; ++q) rb[q] = load_b(p, k0 + lb_k, n0 + lb_n + q);
  };

  u64 lo[TM][TN];
  u32 cr[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      lo[i][j] = 0;
      cr[i][j] = 0;
    }

  auto store = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 8; ++q) As[buf][la_k + q][la_row] = ra[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) Bs[buf][lb_k][lb_n + q] = rb[q];
  };
  if (kbeg < Ktot) {
    fetch(kbeg);
    store(0);
  }
  __syncthreads();
  int cur = 0;
  for (i64 k0 = kbeg; k0 < Ktot; k0 += BK) {
    // the next step's loads go out first and land during this step's
    // multiply-adds; they are then stored into the other buffer, which every
    // thread finished reading before the previous barrier
    const bool more = k0 + BK < Ktot;
    if (more) fetch(k0 + BK);
#pragma unroll 4
    for (int kk = 0; kk < BK; ++kk) {
      u64 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[cur][kk][ty + 16 * i];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = Bs[cur][kk][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const u32 al = (u32)a[i], ah = (u32)(a[i] >> 32);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const u32 bl = (u32)b[j], bh = (u32)(b[j] >> 32);
          lo[i][j] += (u64)al * (u64)bl;
          cr[i][j] += al * bh + ah * bl;
        }
      }
    }
    if (more) store(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }

  if (p.ksplit > 1) {
    // raw slice sum; the reduction adds the slices and applies the epilogue
    u64* part = p.partial + (i64)slice * p.M * p.N;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const i64 m = m0 + ty + 16 * i;
      if (m >= p.M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const i64 n = n0 + tx + 16 * j;
        if (n < p.N) part[m * p.N + n] = lo[i][j] + ((u64)cr[i][j] << 32);
      }
    }
    return;
  }
  const Epilogue& ep = p.ep;
  i64 coff[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const i64 n = n0 + tx + 16 * j;
    coff[j] = (n / ep.view.n_div) * ep.view.ld_q + (n % ep.view.n_div);
  }
  // Every added term is loaded before any store, unconditionally (a thread
  // past the product's edge reads its first element, and stores nothing): with
  // a store between two loads, each load would wait for the store before it,
  // since the compiler cannot tell the output from the added terms.  Four
  // rows (16 outputs) at a time, to stay within the registers of two
  // workgroups per compute unit.
  auto ok = [&](int i, int j) { return m0 + ty + 16 * i < p.M && n0 + tx + 16 * j < p.N; };
  auto at = [&](int i, int j) { return ok(i, j) ? (m0 + ty + 16 * i) * ep.view.ld_m + coff[j] : (i64)0; };
  const u64 neg = ep.csign < 0 ? ~(u64)0 : 0;  // -c as (c ^ ~0) + 1
  constexpr int kRows = 4;
#pragma unroll
  for (int i0 = 0; i0 < TM; i0 += kRows) {
    u64 v[kRows][TN];
#pragma unroll
    for (int i = 0; i < kRows; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) v[i][j] = lo[i0 + i][j] + ((u64)cr[i0 + i][j] << 32);
    if (ep.accumulate) {
#pragma unroll
      for (int i = 0; i < kRows; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) v[i][j] += ep.Out[at(i0 + i, j)];
    }
    if (ep.Cadd) {
#pragma unroll
      for (int i = 0; i < kRows; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          v[i][j] += (ep.Cadd[at(i0 + i, j)] ^ neg) + (neg & 1);
    }
#pragma unroll
    for (int i = 0; i < kRows; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        if (ok(i0 + i, j))
          ep.Out[at(i0 + i, j)] = ep.trunc_bits ? (u64)((i64)v[i][j] >> ep.trunc_bits) : v[i][j];
  }
}

__device__ __forceinline__ void reduce_one(const u64* __restrict__ partial, int ks, i64 total, i64 N,
                                           const Epilogue& ep, i64 e) {
  // four independent sums keep several loads in flight (the ring sum does
  // not depend on the order)
  u64 v0 = 0, v1 = 0, v2 = 0, v3 = 0;
  int s = 0;
  for (; s + 4 <= ks; s += 4) {
    v0 += partial[(i64)s * total + e];
    v1 += partial[(i64)(s + 1) * total + e];
    v2 += partial[(i64)(s + 2) * total + e];
    v3 += partial[(i64)(s + 3) * total + e];
  }
  for (; s < ks; ++s) v0 += partial[(i64)s * total + e];
  u64 v = (v0 + v1) + (v2 + v3);
  const i64 m = e / N, n = e % N;
  const i64 off = m * ep.view.ld_m + (n / ep.view.n_div) * ep.view.ld_q + (n % ep.view.n_div);
  if (ep.accumulate) v += ep.Out[off];
  if (ep.Cadd) v += (ep.csign < 0) ? (u64)0 - ep.Cadd[off] : ep.Cadd[off];
  if (ep.trunc_bits) v = (u64)((i64)v >> ep.trunc_bits);
  ep.Out[off] = v;
}

__global__ void __launch_bounds__(kThreads) k_splitk_reduce_grouped(ReduceTables) {
  const cptr<ReduceTables> t = (cptr<ReduceTables>)MPC_KERNARG_PTR();
  const cptr<ReduceJob> jobs = t->jobs ? (cptr<ReduceJob>)(uintptr_t)t->jobs : t->ijobs;
  const cptr<i64> chunk_start = t->jobs ? (cptr<i64>)(uintptr_t)t->chunk_start : t->ichunk_start;
  const i64 c = blockIdx.x;
  const int lo = find_job(chunk_start, t->njobs, c);
  const ReduceJob jb = jobs[lo];
  const i64 total = jb.M * jb.N;
  const i64 base = (c - chunk_start[lo]) * kReduceChunk;
  const i64 end = min(base + kReduceChunk, total);
  for (i64 e = base + threadIdx.x; e < end; e += kThreads) reduce_one(jb.partial, jb.ks, total, jb.N, jb.ep, e);
}

}  // namespace

hipError_t launch_splitk_reduce_grouped(hipStream_t s, const ReduceTables& t, i64 total_chunks) {
  if (total_chunks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_splitk_reduce_grouped, dim3((unsigned)total_chunks), dim3(kThreads), 0, s, t);
  return hipGetLastError();
}

// Whole Beaver matmul of a small product in one launch, for k below
// kSmallMatmulShortK.  A workgroup owns a 4x4 block of outputs of both parties'
// shares; its 256 threads are those 16 outputs times 16 lanes of k.  Bound by
// the launch and the workgroups' own latency (4 us up to some 4000 outputs,
// then 0.75 us per 1024 workgroups at k of 16 and less): the kernel below, with
// 128 lanes of k and 512 threads, has most of them idle here.  This one against
// that one: 256 x 256 x 1 5.5 / 16.2 us, 512 x 512 x 1 13.6 / 56.8, 256 x 256 x
// 16 7.4 / 16.9, 256 x 256 x 32 10.9 / 18.3, 128 x 128 x 64 6.9 / 7.6, 128 x 128 x
// 96 8.7 / 8.8, 2048 x 8 x 104 9.1 / 8.7; over 18 shapes even at k of 112, where
// its lanes' loops of eight begin to diverge (14 x 649 x 120 8.5 / 7.7, x 127 10.8 /
// 7.8), and behind from there on (128 x 128 x 128 10.7 / 9.8, x 192 14.2 / 11.9).
constexpr int kShortSide = 4, kShortOut = kShortSide * kShortSide, kShortKl = kThreads / kShortOut;

__global__ void __launch_bounds__(kThreads) k_beaver_matmul_short(SmallMatmul s) {
  __shared__ u64 part[2][kShortKl][kShortOut];
  const int o = threadIdx.x % kShortOut, kl = threadIdx.x / kShortOut;
  const i64 ntn = (s.N + kShortSide - 1) / kShortSide;
  const i64 m = (blockIdx.x / ntn) * kShortSide + o / kShortSide;
  const i64 n = (blockIdx.x % ntn) * kShortSide + o % kShortSide;
  const bool ok = m < s.M && n < s.N;
  u64 z0 = 0, z1 = 0;
  if (ok) {
#pragma unroll 8
    for (i64 k = kl; k < s.K; k += kShortKl) {
      const i64 ia = m * s.K + k, ib = k * s.N + n;
      const u64 a0 = s.a0[ia], a1 = s.a1[ia], b0 = s.b0[ib], b1 = s.b1[ib];
      const u64 eps = (s.x0[ia] - a0) + (s.x1[ia] - a1);
      const u64 del = (s.y0[ib] - b0) + (s.y1[ib] - b1);
      z0 += eps * b0 + (a0 + eps) * del;
      z1 += eps * b1 + a1 * del;
    }
  }
  part[0][kl][o] = z0;
  part[1][kl][o] = z1;
  __syncthreads();
  if (kl == 0 && ok) {
    u64 v0 = 0, v1 = 0;
#pragma unroll
    for (int q = 0; q < kShortKl; ++q) {
      v0 += part[0][q][o];
      v1 += part[1][q][o];
    }
    const i64 off = m * s.N + n;
    v0 += s.c0[off];
    v1 += s.c1[off];
    if (s.trunc) {
      v0 = (u64)((i64)v0 >> s.trunc);
      v1 = (u64)((i64)v1 >> s.trunc);
    }
    s.z0[off] = v0;
    s.z1[off] = v1;
  }
}

// The same for k of kSmallMatmulShortK and more.  A workgroup owns a 4x4 block
// of outputs of both parties' shares.  Each of its 512 threads takes
// one column of the block and every 128th k: it forms the opened eps = x - a
// and delta = y - b of the elements it reads from the shares themselves (an
// open pass and its workspace would cost more than the product at this size)
// and accumulates
//   z_0 = eps b_0 + (a_0 + eps) delta,  z_1 = eps b_1 + a_1 delta
// for the column's four rows.  Bound by the number of load instructions (some
// 16 cycles each, and more where they touch more than 16 lines): 20 per 4
// outputs and k, where a thread of one output has 8 per output (128 x 10 x 1024
// 12.0 us, that form 16.8; the plain form's open, GEMM and reduction 25 to 31,
// the limb form 19 to 20), and one of all 16, 2 per output, reads the right
// operand in 64 lines an instruction (11.8 there, but 64 x 64 x 512 13.2 against
// 7.7, 9.7 with one output; 64 x 32 x 128 5.7, 3.9 and 4.1).  The eight sums of
// a wave's 16 threads of one column meet by a butterfly that halves the values
// a lane holds with every step, then in LDS across the waves, before c_p and
// the truncation.  Ring sums do not depend on their order.
constexpr int kSmallSide = 4, kSmallOut = kSmallSide * kSmallSide, kSmallThreads = 512;

__global__ void __launch_bounds__(kSmallThreads) k_beaver_matmul_small(SmallMatmul s) {
  constexpr int S = kSmallSide;
  __shared__ u64 part[kSmallThreads / 64][2][kSmallOut];
  const i64 ntn = (s.N + S - 1) / S;
  const i64 m0 = (blockIdx.x / ntn) * S, n0 = (blockIdx.x % ntn) * S;
  // rows and columns past the product's read its last one
  const i64 nc = min(n0 + threadIdx.x % S, s.N - 1);
  i64 row[S];
#pragma unroll
  for (int i = 0; i < S; ++i) row[i] = min(m0 + i, s.M - 1) * s.K;
  u64 v[2 * S] = {};
#pragma unroll 1
  for (i64 k = threadIdx.x / S; k < s.K; k += kSmallThreads / S) {
    const i64 ib = k * s.N + nc;
    const u64 b0 = s.b0[ib], b1 = s.b1[ib];
    const u64 del = (s.y0[ib] - b0) + (s.y1[ib] - b1);
#pragma unroll
    for (int i = 0; i < S; ++i) {
      if (i && m0 + i >= s.M) break;
      const i64 ia = row[i] + k;
      const u64 a0 = s.a0[ia], a1 = s.a1[ia];
      const u64 eps = (s.x0[ia] - a0) + (s.x1[ia] - a1);
      v[i] += eps * b0 + (a0 + eps) * del;
      v[S + i] += eps * b1 + a1 * del;
    }
  }
  // lanes 32, 16 and 8 apart split the values they both hold: each ends with
  // one, of party lane / 32 and row lane / 8 % 4
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  [&]<int... B>(std::integer_sequence<int, B...>) {
    (
        [&] {
          constexpr int half = S >> B, d = 32 >> B;
          const bool up = lane & d;
#pragma unroll
          for (int q = 0; q < half; ++q) {
            const u64 keep = up ? v[q + half] : v[q], send = up ? v[q] : v[q + half];
            v[q] = keep + __shfl_xor(send, d);
          }
        }(),
        ...);
  }(std::make_integer_sequence<int, 3>{});
  v[0] += __shfl_xor(v[0], 4);
  if (!(lane & 4)) part[wave][lane >> 5][(lane >> 3 & 3) * S + lane % S] = v[0];
  __syncthreads();
  const int o = threadIdx.x;
  const i64 m = m0 + o / S, n = n0 + o % S;
  if (o < kSmallOut && m < s.M && n < s.N) {
    u64 v0 = 0, v1 = 0;
#pragma unroll
    for (int w = 0; w < kSmallThreads / 64; ++w) {
      v0 += part[w][0][o];
      v1 += part[w][1][o];
    }
    const i64 off = m * s.N + n;
    v0 += s.c0[off];
    v1 += s.c1[off];
    if (s.trunc) {
      v0 = (u64)((i64)v0 >> s.trunc);
      v1 = (u64)((i64)v1 >> s.trunc);
    }
    s.z0[off] = v0;
    s.z1[off] = v1;
  }
}

int plain_tiles(i64 M, i64 N) { return (int)(((M + BM - 1) / BM) * ((N + BN - 1) / BN)); }

hipError_t launch_beaver_matmul_small(hipStream_t s, const SmallMatmul& m) {
  static_assert(kShortSide == kSmallMatmulSide && kSmallSide == kSmallMatmulSide, "one grid for both");
  const i64 tiles = small_matmul_groups(m.M, m.N);
  if (tiles <= 0) return hipSuccess;
  if (m.K < kSmallMatmulShortK) hipLaunchKernelGGL(k_beaver_matmul_short, dim3((unsigned)tiles), dim3(kThreads), 0, s, m);
  else hipLaunchKernelGGL(k_beaver_matmul_small, dim3((unsigned)tiles), dim3(kSmallThreads), 0, s, m);
  return hipGetLastError();
}

hipError_t launch_plain_gemm(hipStream_t s, const PlainProblem* probs, TileMap map,
                             int total_tiles) {
  if (total_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_plain_gemm, dim3(total_tiles), dim3(kThreads), 0, s, probs, map);
  return hipGetLastError();
}

}  // namespace mpc
