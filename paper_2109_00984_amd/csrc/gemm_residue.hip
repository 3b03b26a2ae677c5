// gemm_residue.hip -- bit-exact ring GEMM over Z/2^64 through residues on INT8
// matrix cores.
//
// Method.  Read every operand element as the integer v = sum_j d_j 2^(8j) of
// its signed limbs (gemm_limb.hip): v is congruent to the element mod 2^64 and
// |v| <= V = 0x80..80.  A sum x of K products then satisfies |x| <= K V^2, and
// for K <= kResMaxKBlocks * 64 it is smaller than half of M, the product of
// 18 coprime moduli m_i <= 256.  So x is determined by its residues, each of
// which is one int8 GEMM over residues in [-128, 127], exact in int32
// (K 2^14 < 2^31): 18 int8 GEMMs per ring GEMM instead of the 36 limb pairs,
// and integers throughout, so the result is the same bits.  (Chinese remainder
// theorem; residue arithmetic for matrix products on int8 units is the scheme
// of Ozaki, Uchino and Imamura, "Ozaki scheme II", 2025, here over integers.)
//   pack      v -> v mod m_i, by two 4-way byte dot products with the weights
//             2^(8j) mod m_i and one reduction.  A right operand's weights also
//             hold inv_i = (M/m_i)^-1 mod m_i, so that the GEMM's result is
//             c_i = x inv_i mod m_i, the coefficient that the combine needs.
//   GEMM      c_i mod m_i, one byte per output and modulus.
//   combine   x = sum_i c_i (M/m_i) - q M with q = round(sum_i c_i / m_i), the
//             sum in 24-bit fractions: |x| < M/2 (1 - 2^-8) keeps the rounding
//             away from its ties by more than the fractions' error
//             (18 * 128 * 2^-25 < 2^-13).  Only x mod 2^64 is formed, from byte
//             dot products of the c_i and q with the bytes of M/m_i and -M.
#include <utility>

#include "packed.h"

namespace mpc {
namespace {

// ------------------------------------------------------------------ constants
constexpr u64 mod_pow256(int j, u64 m) {
  u64 v = 1 % m;
  for (int i = 0; i < j; ++i) v = v * 256 % m;
  return v;
}
// (M / m_i) mod m, over all the other moduli
constexpr u64 cofactor_mod(int i, u64 m) {
  u64 v = 1 % m;
  for (int k = 0; k < kRes; ++k)
    if (k != i) v = v * (u64)kResModuli[k] % m;
  return v;
}
constexpr u64 cofactor_inv(int i) {
  const u64 m = (u64)kResModuli[i], c = cofactor_mod(i, m);
  for (u64 v = 1; v < m; ++v)
    if (c * v % m == 1) return v;
  return 0;
}
// M / m_i mod 2^64 (i < kRes), or M mod 2^64 (i = kRes)
constexpr u64 cofactor_64(int i) {
  u64 v = 1;
  for (int k = 0; k < kRes; ++k)
    if (k != i) v *= (u64)kResModuli[k];
  return v;
}
constexpr int gcd(int a, int b) { return b ? gcd(b, a % b) : a; }
constexpr bool moduli_ok() {
  for (int i = 0; i < kRes; ++i) {
    if (kResModuli[i] > 256 || cofactor_inv(i) == 0) return false;
    for (int k = 0; k < i; ++k)
      if (gcd(kResModuli[i], kResModuli[k]) != 1) return false;
  }
  return kResModuli[0] == 256;
}
static_assert(moduli_ok(), "pairwise coprime moduli of at most 256, 256 first");
// kResK * V^2 < M/2 (1 - 2^-8), in doubles with room to spare (the exact bound is 11082)
constexpr double moduli_product() {
  double v = 1;
  for (int i = 0; i < kRes; ++i) v *= kResModuli[i];
  return v;
}
static_assert(64.0 * kResMaxKBlocks * (double)kLimbBias * (double)kLimbBias < moduli_product() * 0.5 * (1 - 1.0 / 256) * (1 - 1e-9),
              "a chunk's exact sum fits the moduli");

// Signed byte j (balanced base 256, mod 2^64) of w, as an unsigned byte.
constexpr u32 sbyte(u64 w, int j) { return (u32)((((w + kLimbBias) ^ kLimbBias) >> (8 * j)) & 0xff); }
constexpr u32 quad(u32 a, u32 b, u32 c, u32 d) { return a | b << 8 | c << 16 | d << 24; }
constexpr u32 bal(u64 r, u64 m) { return (u32)((r > (m - 1) / 2 ? r - m : r) & 0xff); }

// Per modulus: the byte weights of a left and of a right operand, -m and 1/m.
struct ResConst {
  int wl[2], wr[2], neg_m, fold;  // fold: 256 mod m where the epilogue folds the high bits down, else 0
  float inv;
  // The packing's byte sums start from the bits of the float `bias`, a multiple
  // of 256 m next to 1.5 * 2^23, and so come out as the bits of bias + t: their
  // quotient needs no conversion, and the bias drops out of the low byte.
  int bias;
  float back;  // 1.5 * 2^23 - bias / m
};
constexpr ResConst res_const(int i) {
  ResConst c{};
  const u64 m = (u64)kResModuli[i], inv = cofactor_inv(i);
  for (int h = 0; h < 2; ++h) {
    u32 l[4] = {}, r[4] = {};
    for (int b = 0; b < 4; ++b) {
      const u64 p = mod_pow256(4 * h + b, m);
      l[b] = bal(p, m);
      r[b] = bal(p * inv % m, m);
    }
    c.wl[h] = (int)quad(l[0], l[1], l[2], l[3]);
    c.wr[h] = (int)quad(r[0], r[1], r[2], r[3]);
  }
  c.neg_m = -(int)m;
  c.fold = m >= 216 && m < 256 ? (int)(256 - m) : 0;
  c.inv = (float)(1.0 / (double)m);
  const u64 step = 256 * m, bias = (((u64)3 << 22) + step / 2) / step * step;  // t below 2^18 keeps it in [2^23, 2^24)
  c.bias = (int)(0x4b000000 + (u32)(bias - ((u64)1 << 23)));
  c.back = (float)(12582912.0 - (double)(bias / m));
  return c;
}
struct ResConsts {
  ResConst c[kRes];
};
template <int... I>
constexpr ResConsts res_consts(std::integer_sequence<int, I...>) {
  return ResConsts{{res_const(I)...}};
}
__constant__ const ResConsts g_res = res_consts(std::make_integer_sequence<int, kRes>());

// t reduced mod m: an integer congruent to t whose low byte, read as int8, is
// that integer.  q = round(t / m) comes out of one fma against 1.5 * 2^23,
// whose low 23 bits then hold q + 2^22; only the low byte of t - m q matters
// and m 2^22 does not reach it.
constexpr float kMagic = 12582912.0f;
__device__ __forceinline__ u32 reduce(int t, float inv, int neg_m) {
  const int q = __float_as_int(__builtin_fmaf((float)t, inv, kMagic));
  return (u32)(__mul24(q, neg_m) + t);
}
// Bytes 0 of four words as one word.
__device__ __forceinline__ u32 low_bytes(u32 a, u32 b, u32 c, u32 d) {
  const u32 ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u), cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
  return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

// ------------------------------------------------------------------ packing
constexpr int kResTPad = 65;  // LDS row stride (elements) of the transpose tile

// Element offsets of a lane's 16 loads and whether each is inside the operand.
// A wave packs one block of 16 rows (columns) x 64 k.
template <int KIND>
__device__ __forceinline__ void res_offsets(const PackJob& jb, i64 rb, i64 kb, int lane, i64 (&off)[16], bool (&ok)[16]) {
  if (KIND == kPackRow) {
    // load layout: load q covers row q of the block, k = lane
    const i64 k = kb * 64 + lane;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const i64 r = rb * 16 + q;
      ok[q] = r < jb.rows && k < jb.K;
      off[q] = r * jb.ld + k;
    }
    return;
  }
  // packed lane order: column n = rb * 16 + lane % 16, k = kb * 64 + (lane / 16) * 16 + q
  const i64 n = rb * 16 + (lane & 15), k0 = kb * 64 + (lane >> 4) * 16;
  if (KIND == kPackCol) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      ok[q] = n < jb.rows && k0 + q < jb.K;
      off[q] = (k0 + q) * jb.ld + n;
    }
  } else {
    // im2col: column n = (b, l), k = (c, j); (c, j) advances incrementally
    const bool n_ok = n < jb.rows;
    const i64 nn = n_ok ? n : 0;
    const i64 b = nn / jb.lout, l = nn % jb.lout;
    i64 c = k0 / jb.ksz, j = k0 % jb.ksz;
    const i64 base = b * jb.cin * jb.len + l * jb.stride;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      ok[q] = n_ok && k0 + q < jb.K;
      off[q] = base + c * jb.len + j;
      if (++j == jb.ksz) {
        j = 0;
        ++c;
      }
    }
  }
}

// One lane's 16 elements -> 16 residues per modulus, one 16-byte store each.
template <bool RIGHT>
__device__ __forceinline__ void write_residues(uint8_t* dst, i64 plane, const u64 (&v)[16]) {
  int lo[16], hi[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const u64 d = (v[q] + kLimbBias) ^ kLimbBias;
    lo[q] = (int)(u32)d;
    hi[q] = (int)(u32)(d >> 32);
  }
  {
    // modulus 256: the low limb (times inv for a right operand)
    v4i w;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      u32 r[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) r[b] = RIGHT ? (u32)__builtin_amdgcn_sdot4(lo[4 * x + b], g_res.c[0].wr[0], 0, false) : (u32)lo[4 * x + b];
      w[x] = (int)low_bytes(r[0], r[1], r[2], r[3]);
    }
    *(gv4i*)dst = w;
  }
  ResConst k = g_res.c[1];
#pragma unroll 1
  for (int i = 1; i < kRes; ++i) {
    const int w0 = RIGHT ? k.wr[0] : k.wl[0], w1 = RIGHT ? k.wr[1] : k.wl[1], neg_m = k.neg_m, bias = k.bias;
    const float inv = k.inv, back = k.back;
    k = g_res.c[i + 1 < kRes ? i + 1 : i];  // the next modulus' constants arrive behind this one's work
    v4i w;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      u32 r[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int t = __builtin_amdgcn_sdot4(hi[4 * x + b], w1, __builtin_amdgcn_sdot4(lo[4 * x + b], w0, bias, false), false);
        r[b] = (u32)(__mul24(__float_as_int(__builtin_fmaf(__int_as_float(t), inv, back)), neg_m) + t);
      }
      w[x] = (int)low_bytes(r[0], r[1], r[2], r[3]);
    }
    *(gv4i*)(dst + i * plane) = w;
  }
}

// A wave's 16 x 64 block from load layout (64 lanes along a row) to packed order.
__device__ __forceinline__ void res_turn_rows(u64 (&w)[16], u64* t, int lane) {
#pragma unroll
  for (int q = 0; q < 16; ++q) t[q * kResTPad + lane] = w[q];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int q = 0; q < 16; ++q) w[q] = t[(lane & 15) * kResTPad + (lane >> 4) * 16 + q];
  __builtin_amdgcn_wave_barrier();
}

// Bound by HBM: 32 bytes read and 54 written per element of a Beaver operand
// (4096 x 4096: 0.29 ms, 5.0 TB/s; a copy of 2 GiB reaches 4.9).
// One wave packs one 16 x 64 block of every output of a job; all loads of a
// lane are issued before any is used.  Left operands (ROW) are read with 64
// lanes along a row and transposed through LDS, right ones in packed order (16
// lanes along n: whole 128-byte lines).
template <int KIND, int MODE>
__device__ __forceinline__ void res_pack_block(const PackJob& jb, i64 local, u64* tiles, int wave, int lane) {
  using Md = Mode<MODE>;
  u64* tile = tiles + wave * 16 * kResTPad;
  // the waves of a workgroup take neighbouring blocks along the operand's rows in memory
  constexpr bool left = KIND == kPackRow || KIND == kPackConvRow;
  const i64 rb = left ? local / jb.kblocks : local % jb.rreal;
  const i64 kb = left ? local % jb.kblocks : local / jb.rreal;
  const i64 plane = jb.rblocks * jb.kblocks * kResBlockBytes;
  size_t boff = (size_t)(rb * jb.kblocks + kb) * kResBlockBytes + (size_t)lane * 16;

  i64 off[16];
  bool ok[16], interior, skip = false;
  if constexpr (KIND == kPackChan) {
    // 16 channels of 64 neighbouring positions, one position per lane: the four
    // waves of a workgroup take the quarters of one 64-channel group
    const i64 groups = (jb.cin + 63) / 64, runs = (jb.len + 63) / 64;
    const i64 quarter = local % 4, run = local / 4 % runs, bg = local / 4 / runs, g = bg % groups, b = bg / groups;
    const i64 pos = run * 64 + lane, c0 = g * 64 + quarter * 16;
    if (pos >= jb.len) return;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      ok[q] = c0 + q < jb.cin;
      off[q] = (b * jb.cin + c0 + q) * jb.len + pos;
    }
    interior = c0 + 16 <= jb.cin;
    boff = (size_t)((bg * jb.len + pos) * 64 + quarter * 16);
  } else if constexpr (KIND == kPackConvRow) {
    // A workgroup packs 16 rows x 64 channels x 4 taps, wave w the block of tap
    // w.  Loads run along the taps, as the weight does, and turn through LDS: a
    // 2000 x 250 x 32 weight takes 0.33 ms (reading in packed order, which uses
    // 8 bytes of each line, 0.65; writing from that order in 16-byte pieces 0.54).
    const i64 chunks = (jb.ksz + 3) / 4, groups = (jb.cin + 63) / 64, rg = local / 4 / chunks;
    const i64 tap0 = local / 4 % chunks * 4, g = rg % groups, rb16 = rg / groups;
    const i64 c = g * 64 + (threadIdx.x >> 2), j = tap0 + (threadIdx.x & 3);
    const bool in = c < jb.cin && j < jb.ksz;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      ok[q] = in && rb16 * 16 + q < jb.rows;
      off[q] = (rb16 * 16 + q) * jb.ld + c * jb.ksz + j;
    }
    interior = (rb16 + 1) * 16 <= jb.rows && (g + 1) * 64 <= jb.cin && tap0 + 4 <= jb.ksz;
    skip = tap0 + wave >= jb.ksz;
    boff = (size_t)((rb16 * jb.kblocks + g * jb.ksz + tap0 + wave) * kResBlockBytes + lane * 16);
  } else {
    res_offsets<KIND>(jb, rb, kb, lane, off, ok);
    interior = (rb + 1) * 16 <= jb.rows && (kb + 1) * 64 <= jb.K;
  }
  gcu64* in[Md::nin];
#pragma unroll
  for (int i = 0; i < Md::nin; ++i) in[i] = gptr(jb.in[i]);
  u64 v[16][Md::nin];
  if constexpr (MODE == kModePrgSum2) {
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        v[q][i] = ok[q] ? sm_out(jb.key[i], (u64)off[q]) : 0;
        if (ok[q]) jb.share[i][off[q]] = v[q][i];
      }
  } else if (interior) {
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int i = 0; i < Md::nin; ++i) v[q][i] = in[i][off[q]];
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int i = 0; i < Md::nin; ++i) v[q][i] = ok[q] ? in[i][off[q]] : 0;
  }

#pragma unroll
  for (int o = 0; o < Md::nout; ++o) {
    u64 w[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) w[q] = Md::out(o, v[q]);
    if constexpr (KIND == kPackRow) res_turn_rows(w, tile, lane);
    if constexpr (KIND == kPackConvRow) {
      u64* t = tiles;
#pragma unroll
      for (int q = 0; q < 16; ++q) t[((threadIdx.x & 3) * 16 + q) * kResTPad + (threadIdx.x >> 2)] = w[q];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 16; ++q) w[q] = t[(wave * 16 + (lane & 15)) * kResTPad + (lane >> 4) * 16 + q];
      __syncthreads();
    }
    if (!skip) write_residues<!left>(jb.dst[o] + boff, plane, w);
  }
}

// One launch packs both operands of a call.
template <int... KM>
__global__ void __launch_bounds__(kPackThreads) k_res_pack(PackTables, PackPairs<KM...>) {
  using P = PackPairs<KM...>;
  const PackView tv = pack_view();
  const cptr<i64> start = tv.bstart;
  const int njobs = tv.njobs;
  __shared__ u64 tiles[P::has(kPackRow) || P::has(kPackConvRow) ? 4 * 16 * kResTPad : 1];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // (CONV_ROW: neighbouring workgroups share lines, so an XCD takes runs of
  // them: 0.33 ms for a 2000 x 250 x 32 weight, 0.46 without)
  const i64 unit = (i64)(P::has(kPackConvRow) ? remap_tile(blockIdx.x, gridDim.x, 32) : (int)blockIdx.x) * 4 + wave;
  // A whole wave leaves; only CONV_ROW, whose job comes first and in whole
  // workgroups, syncs beyond the wave.
  if (unit >= start[njobs]) return;
  const int ji = find_job(start, njobs, unit);
  const PackJob jb = tv.jobs[ji];
  const int pair = km(jb.kind, jb.mode);
  ((pair == KM ? res_pack_block<KM / 16, KM % 16>(jb, unit - start[ji], tiles, wave, lane) : (void)0), ...);
}

template <int KIND>
__device__ __forceinline__ void res_party_block(cptr<PartyPack> s, i64 local, u64* tile, int lane) {
  const PackJob jb = s->job;
  const i64 rb = KIND == kPackRow ? local / jb.kblocks : local % jb.rreal;
  const i64 kb = KIND == kPackRow ? local % jb.kblocks : local / jb.rreal;
  const i64 plane = jb.rblocks * jb.kblocks * kResBlockBytes;
  const size_t boff = (size_t)(rb * jb.kblocks + kb) * kResBlockBytes + (size_t)lane * 16;
  i64 off[16];
  bool ok[16];
  res_offsets<KIND>(jb, rb, kb, lane, off, ok);
  party_block<KIND == kPackRow>(s, off, ok, (rb + 1) * 16 <= jb.rows && (kb + 1) * 64 <= jb.K, [&](uint8_t* dst, u64 (&w)[16]) {
    if constexpr (KIND == kPackRow) res_turn_rows(w, tile, lane);
    write_residues<KIND != kPackRow>(dst + boff, plane, w);
  });
}
__global__ void __launch_bounds__(kPackThreads) k_res_pack_party(PartyPackTables) {
  const cptr<PartyPackTables> t = (cptr<PartyPackTables>)MPC_KERNARG_PTR();
  __shared__ u64 tile[4][16 * kResTPad];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const i64 unit = (i64)blockIdx.x * 4 + wave, n0 = t->side[0].job.units;
  if (unit < n0) res_party_block<kPackRow>(&t->side[0], unit, tile[wave], lane);
  else if (unit < n0 + t->side[1].job.units) res_party_block<kPackCol>(&t->side[1], unit - n0, tile[wave], lane);
}

template <int... KM>
hipError_t launch_res_pack_set(hipStream_t s, const PackTables& t, i64 units, PackPairs<KM...> pairs) {
  hipLaunchKernelGGL((k_res_pack<KM...>), dim3((unsigned)((units + 3) / 4)), dim3(kPackThreads), 0, s, t, pairs);
  return hipGetLastError();
}

// ------------------------------------------------------------------ GEMM
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) v4i lds_v4i;

// Workgroup of four waves in a 2 x 2 grid, each with HA x HB blocks of 16x16
// outputs: a 32HA x 32HB tile.  One modulus of one product is an ordinary int8
// GEMM, so unlike in the limb form (8 diagonals an output) the accumulators
// leave room for a 256x256 tile, half of the register file at one workgroup per
// compute unit; it fetches 128 bytes per MFMA, no more than the limb form's
// 64x64 tile.  Steps of 64 k go through DEPTH LDS buffers, filled AHEAD steps
// ahead by buffer loads that write LDS directly (32 KiB a step at 256x256; two
// steps ahead instead of three take 1.37 times as long, four ahead no less).
// What bounds it is the board's power: 4096 x 4096 x 8192 runs in 1.73 ms (2850
// TOP/s int8, 18 products; the limb form 3.04 ms at 3250 TOP/s for 36) at 1385 W,
// matrix cores busy 0.75 of the cycles at 1.87 GHz, the same rate of matrix
// work as the limb form's 0.91 at 1.55 GHz.  A scalar instruction less or more
// in the loop, or another place of the barrier, changes nothing there.
template <int HA_, int HB_, int DEPTH, int AHEAD, int PER_CU>
struct RGeo {
  static constexpr int HA = HA_, HB = HB_, BM = 32 * HA, BN = 32 * HB;
  static constexpr int SA = 2 * HA, SB = 2 * HB;  // strips of 16 rows per operand
  static constexpr int kDepth = DEPTH, kAhead = AHEAD, kPerCU = PER_CU;
  static constexpr int kStepBytes = (SA + SB) * kResBlockBytes;
  static constexpr int CA = SA / 4, CB = SB / 4, kCopies = CA + CB;  // 1 KiB copies per wave and step
  static constexpr int kNM = HA * HB;              // MFMAs per wave and step
  static constexpr int kReads = HA + HB;
  // One barrier per step, after MFMA kBarrier; behind it come the reads of the
  // next step's fragments.  The copies are spread evenly over the step, behind
  // the barrier only where they would overwrite what was read last.
  static constexpr int kBarrier = DEPTH == AHEAD ? kNM / 4 - 1 : 2;
  static constexpr int reads_upto(int i) {  // reads issued after MFMA i or before
    if (i < kBarrier) return 0;
    const int n = (kNM - kBarrier) * 3 / 4;
    const int r = ((i - kBarrier + 1) * kReads + n - 1) / n;
    return r < kReads ? r : kReads;
  }
  static constexpr int copies_upto(int i) {
    const int first = DEPTH == AHEAD ? kBarrier : 0;
    return i < first ? 0 : ((i - first + 1) * kCopies) / (kNM - first);
  }
  static constexpr int kPending = (kAhead - 2) * kCopies + copies_upto(kBarrier - 1);  // copies of later steps
  static_assert(kDepth * kStepBytes * kPerCU <= 160 * 1024, "step buffers must fit in LDS");
  static_assert(HB % 4 == 0 && HA % 2 == 0, "whole units and even copies");
  static_assert(copies_upto(kNM - 1) == kCopies && reads_upto(kNM - 1) == kReads && kPending < 64, "schedule");
};
using R256x256 = RGeo<8, 8, 4, 3, 1>;
using R256x128 = RGeo<8, 4, 3, 3, 2>;
using R128x256 = RGeo<4, 8, 3, 3, 2>;
using R128x128 = RGeo<4, 4, 4, 3, 2>;

__device__ __forceinline__ void mfma_acc(v4i& acc, const v4i& a, const v4i& b) {
  asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_new(v4i& acc, const v4i& a, const v4i& b) {
  asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, 0" : "=a"(acc) : "v"(a), "v"(b));
}

template <int PENDING>
__device__ __forceinline__ void step_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PENDING) : "memory");
}

// One wave's copies: CA neighbouring strips of the left operand and CB of the
// right one, 1 KiB each per step.  The second segment's left pointer is moved
// back by one segment, so that block kg of the concatenation is at kg KiB of
// either; so is the right one's, unless it is a convolution's activation, whose
// steps follow its channel groups and taps.
template <class G, bool CONV>
struct CopySrc {
  const uint8_t *a0, *a1, *b0, *b1;  // first strip (or plane) of each operand in segment 0 and 1
  int kbs;                           // blocks per segment
  int kg, kend;                      // the next block to copy, and the end of the tile's
  int tap, boff, ksz, wrap;          // CONV: the block's tap, its offset, and the step back to the next group's tap 0
  unsigned vb[CONV ? G::CB : 1];     // CONV: this lane's bytes in each strip's columns
};
// The copies of one step.
struct Copies {
  const uint8_t *a, *b;
  int n;            // bytes that the descriptors cover: past the last step 0, and the loads return zeros without a fetch
  int aoff, boff;   // the block's offsets
  int next;         // from strip to strip, less the 1 KiB that the instruction's offset adds on both sides
};
template <class G, bool CONV>
__device__ __forceinline__ Copies next_copies(CopySrc<G, CONV>& s) {
  const bool seg0 = s.kg < s.kbs;
  const Copies c{seg0 ? s.a0 : s.a1, seg0 ? s.b0 : s.b1, s.kg < s.kend ? 0x7fffffff : 0, s.kg * kResBlockBytes,
                 CONV ? s.boff : s.kg * kResBlockBytes, (s.kbs - 1) * kResBlockBytes};
  ++s.kg;
  if constexpr (CONV) {
    const bool last = ++s.tap == s.ksz;
    s.boff += last ? s.wrap : 64;
    s.tap = last ? 0 : s.tap;
    s.boff = s.kg == s.kbs ? 0 : s.boff;
  }
  return c;
}
// Copy J of a wave's step: the immediate offset moves source and destination
// alike, so up to four strips share one LDS base.
template <class G, bool CONV, int J>
__device__ __forceinline__ void copy_one(const CopySrc<G, CONV>& s, const Copies& c, lds_u8* buf, int wave, unsigned lane16) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only parses the kernels
  using lds_void = __attribute__((address_space(3))) void;
  constexpr bool left = J < G::CA;
  constexpr int q = left ? J : J - G::CA;
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(left ? c.a : c.b), 0, c.n, kBufferWord3);
  lds_u8* base = buf + (left ? wave * G::CA : G::SA + wave * G::CB) * kResBlockBytes;
  if constexpr (CONV && !left)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(base + q * kResBlockBytes), 16, s.vb[q], c.boff, 0, 0);
  else
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)base, 16, lane16, (left ? c.aoff : c.boff) + q * c.next, q * kResBlockBytes, 0);
#endif
}

template <class G>
struct RFrags {
  v4i a[G::HA], b[G::HB];
};

// What one step touches besides its accumulators and fragments.
template <class G, bool CONV>
struct RStep {
  const CopySrc<G, CONV>& src;
  Copies c;
  const lds_u8 *ra, *rb;  // the next step's fragments
  lds_u8* wbuf;        // where the copies go
  int wave;
  unsigned lane16;
};

// MFMA number I of a step and what follows it.
template <class G, bool CONV, bool FIRST, int I>
__device__ __forceinline__ void res_mfma(v4i (&acc)[G::HA][G::HB], const RFrags<G>& cur, RFrags<G>& nxt, const RStep<G, CONV>& st) {
  constexpr int HA = G::HA, HB = G::HB;
  if constexpr (I < G::kNM) {
    constexpr int x = I / HB, y = I % HB;
    // columns on the MFMA's row side: a lane then holds four neighbouring columns of one row
    if constexpr (FIRST) mfma_new(acc[x][y], cur.b[y], cur.a[x]);
    else mfma_acc(acc[x][y], cur.b[y], cur.a[x]);
    if constexpr (I == G::kBarrier) {
      __builtin_amdgcn_sched_barrier(0);
      step_barrier<G::kPending>();
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr int r0 = G::reads_upto(I - 1), c0 = G::copies_upto(I - 1);
    [&]<int... Q>(std::integer_sequence<int, Q...>) {
      ([&] {
        // in the order of their first use: a[0], all of b, the rest of a
        constexpr int rd = r0 + Q;
        if constexpr (rd >= 1 && rd <= HB) nxt.b[(rd - 1) % HB] = *(const lds_v4i*)(st.rb + (rd - 1) * kResBlockBytes);
        else nxt.a[rd ? (rd - HB) % HA : 0] = *(const lds_v4i*)(st.ra + (rd ? rd - HB : 0) * kResBlockBytes);
      }(), ...);
    }(std::make_integer_sequence<int, G::reads_upto(I) - r0>{});
    [&]<int... Q>(std::integer_sequence<int, Q...>) {
      (copy_one<G, CONV, c0 + Q>(st.src, st.c, st.wbuf, st.wave, st.lane16), ...);
    }(std::make_integer_sequence<int, G::copies_upto(I) - c0>{});
    __builtin_amdgcn_sched_barrier(0);
    res_mfma<G, CONV, FIRST, I + 1>(acc, cur, nxt, st);
  }
}

struct ResView {
  cptr<ResProblem> probs;
  cptr<int> tile_start;
  int nprob, tiles;
};
__device__ __forceinline__ ResView res_view() {
  const cptr<ResGemmTables> t = (cptr<ResGemmTables>)MPC_KERNARG_PTR();
  ResView v;
  v.nprob = t->nprob;
  v.tiles = t->tiles;
  v.probs = t->probs ? (cptr<ResProblem>)(uintptr_t)t->probs : t->iprobs;
  v.tile_start = t->probs ? (cptr<int>)(uintptr_t)t->tile_start : t->itile_start;
  return v;
}

constexpr int kResGroupM = 8;  // tile rows per raster group

// Tile t of the launch.
struct ResPos {
  int pi, mi, tm, tn;
};
template <class G>
__device__ __forceinline__ ResPos res_pos(const ResView& tv, int idx) {
  ResPos q;
  const int t = remap_tile(idx, tv.tiles, kXcdCUs * G::kPerCU);
  q.pi = find_problem(tv.tile_start, tv.nprob, t);
  const cptr<ResProblem> pp = tv.probs + q.pi;
  // modulus, then a grouped raster
  const int local = t - tv.tile_start[q.pi], ntm = pp->ntm, ntn = pp->ntn, per = ntm * ntn;
  q.mi = pp->m0 + local / per;
  const int in_mod = local % per, first_m = in_mod / (kResGroupM * ntn) * kResGroupM;
  const int gsize = min(ntm - first_m, kResGroupM), in_group = in_mod % (kResGroupM * ntn);
  q.tm = first_m + in_group % gsize;
  q.tn = in_group / gsize;
  return q;
}

template <class G, bool CONV>
__device__ __forceinline__ CopySrc<G, CONV> res_source(cptr<ResProblem> pp, const ResPos& q, int wave, int lane) {
  CopySrc<G, CONV> c;
  c.kbs = pp->kbs;
  c.kg = pp->kb_begin;
  c.kend = pp->kb_end;
  const i64 seg = (i64)c.kbs * kResBlockBytes;  // one strip's bytes in a segment
  const i64 oa = q.mi * pp->pa + ((i64)q.tm * G::SA + wave * G::CA) * seg;
  c.a0 = pp->PA0 + oa;
  c.a1 = pp->PA1 + oa - seg;
  if constexpr (CONV) {
    c.b0 = pp->PB0 + q.mi * pp->pb;
    c.b1 = pp->PB1 + q.mi * pp->pb;
    const cptr<ResConv> cv = &pp->cv;
    const int ksz = cv->ksz, len = cv->len, kk = c.kg < c.kbs ? c.kg : c.kg - c.kbs;
    c.ksz = ksz;
    c.wrap = (len - ksz + 1) * 64;
    c.tap = kk % ksz;
    c.boff = (kk / ksz * len + c.tap) * 64;
#pragma unroll
    for (int j = 0; j < G::CB; ++j) {
      // columns past the product's read its last one
      const int n = min((q.tn * G::SB + wave * G::CB + j) * 16 + (lane & 15), cv->n - 1);
      const int b = n / cv->lout, l = n % cv->lout;
      c.vb[j] = (unsigned)((b * cv->groups * len + l * cv->stride) * 64 + (lane >> 4) * 16);
    }
  } else {
    const i64 ob = q.mi * pp->pb + ((i64)q.tn * G::SB + wave * G::CB) * seg;
    c.b0 = pp->PB0 + ob;
    c.b1 = pp->PB1 + ob - seg;
  }
  return c;
}

// The copies of a tile's first kAhead steps.
template <class G, bool CONV>
__device__ __forceinline__ void res_prefetch(CopySrc<G, CONV>& src, lds_u8* lds, int wave, unsigned lane16) {
#pragma unroll
  for (int s = 0; s < G::kAhead; ++s) {
    const Copies c = next_copies(src);
    [&]<int... J>(std::integer_sequence<int, J...>) {
      (copy_one<G, CONV, J>(src, c, lds + s * G::kStepBytes, wave, lane16), ...);
    }(std::make_integer_sequence<int, G::kCopies>{});
  }
}

template <class G, bool CONV>
__global__ void __launch_bounds__(256, G::kPerCU) k_res_gemm(ResGemmTables) {
  constexpr int HA = G::HA, HB = G::HB;
  __shared__ v4i lds_words[G::kDepth * G::kStepBytes / 16];
  lds_u8* lds = (lds_u8*)&lds_words[0];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const ResView tv = res_view();
  const unsigned lane16 = lane * 16;
  const unsigned roff_a = wr * HA * kResBlockBytes + lane16, roff_b = (G::SA + wc * HB) * kResBlockBytes + lane16;
  ResPos pos = res_pos<G>(tv, blockIdx.x);
  cptr<ResProblem> pp = tv.probs + pos.pi;
  CopySrc<G, CONV> src = res_source<G, CONV>(pp, pos, wave, lane);
  int nsteps = pp->kb_end - pp->kb_begin;
  res_prefetch(src, lds, wave, lane16);
  for (int idx = blockIdx.x;;) {
    v4i acc[HA][HB];
    // step 0's copies (and the previous tile's stores: loads and stores share the counter)
    step_barrier<0>();
    if (nsteps > 0) {
      RFrags<G> f0, f1;
#pragma unroll
      for (int h = 0; h < HB; ++h) f0.b[h] = *(const lds_v4i*)(lds + roff_b + h * kResBlockBytes);
#pragma unroll
      for (int h = 0; h < HA; ++h) f0.a[h] = *(const lds_v4i*)(lds + roff_a + h * kResBlockBytes);
      __builtin_amdgcn_sched_barrier(0);
      // step s: MFMAs on its fragments; reads of step s + 1's (past the last
      // step they return what an empty copy left: unused); copies of step
      // s + kAhead, into the buffer that step s's fragments were read from
      // (kDepth == kAhead) or step s - 1's
      auto step = [&]<bool FIRST>(int s, const RFrags<G>& cur, RFrags<G>& nxt) {
        lds_u8* rbuf = lds + ((s + 1) % G::kDepth) * G::kStepBytes;
        lds_u8* wbuf = lds + ((s + G::kAhead) % G::kDepth) * G::kStepBytes;
        const Copies c = next_copies(src);
        res_mfma<G, CONV, FIRST, 0>(acc, cur, nxt, RStep<G, CONV>{src, c, rbuf + roff_a, rbuf + roff_b, wbuf, wave, lane16});
      };
      step.template operator()<true>(0, f0, f1);
      int s = 1;
      for (; s + 1 < nsteps; s += 2) {
        step.template operator()<false>(s, f1, f0);
        step.template operator()<false>(s + 1, f0, f1);
      }
      if (s < nsteps) step.template operator()<false>(s, f1, f0);
    } else {
#pragma unroll
      for (int x = 0; x < HA; ++x)
#pragma unroll
        for (int y = 0; y < HB; ++y) acc[x][y] = v4i{0, 0, 0, 0};
    }
    // no (empty) copy may still write LDS when the next tile's start to, or when the workgroup ends
    step_barrier<0>();
    const ResPos done = pos;
    const cptr<ResProblem> dp = pp;
    idx += gridDim.x;
    const bool more = idx < tv.tiles;
    if (more) {
      // the next tile's first steps travel during this one's epilogue
      pos = res_pos<G>(tv, idx);
      pp = tv.probs + pos.pi;
      src = res_source<G, CONV>(pp, pos, wave, lane);
      nsteps = pp->kb_end - pp->kb_begin;
      res_prefetch(src, lds, wave, lane16);
    }
    // wait states between the last MFMAs and the reads of their results
#pragma unroll
    for (int x = 0; x < HA; ++x)
#pragma unroll
      for (int y = 0; y < HB; ++y) asm volatile("s_nop 3" : "+a"(acc[x][y]));

    // Epilogue: int32 sums -> residues mod m, four columns per word, four words
    // (64 columns) per 16-byte store.  |sum| < 2^27.5: for the moduli near 256,
    // whose balanced range nearly fills a byte, the high bits are folded down
    // first (2^8 = fold mod m) so that the quotient's float error stays far
    // below the range's slack; the smaller ones have slack for it as it is.
    const int mi = done.mi, neg_m = g_res.c[mi].neg_m, fold = g_res.c[mi].fold;
    const float inv = g_res.c[mi].inv;
    const int n64 = dp->n64;
    uint8_t* R = dp->R + mi * dp->pr + lane * 16;
    auto finish = [&]<int KINDM>() {
#pragma unroll
      for (int x = 0; x < HA; ++x)
#pragma unroll
        for (int u = 0; u < HB / 4; ++u) {
          v4i w;
#pragma unroll
          for (int y = 0; y < 4; ++y) {
            u32 r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int c = acc[x][4 * u + y][e];
              if constexpr (KINDM == 0) r[e] = (u32)c;
              else if constexpr (KINDM == 1) r[e] = reduce(__mul24(c >> 8, neg_m) + c, inv, neg_m);  // (c >> 8) fold + (c & 255)
              else r[e] = reduce(c, inv, neg_m);
            }
            w[y] = (int)low_bytes(r[0], r[1], r[2], r[3]);
          }
          const i64 rb = (i64)done.tm * G::SA + wr * HA + x, cb = (i64)done.tn * (G::BN / 64) + wc * (HB / 4) + u;
          *(gv4i*)(R + (rb * n64 + cb) * kResBlockBytes) = w;
        }
    };
    if (mi == 0) finish.template operator()<0>();
    else if (fold) finish.template operator()<1>();
    else finish.template operator()<2>();
    if (!more) break;
  }
}

// ------------------------------------------------------------------ combine
// Byte weights: slot i < kRes is c_i, slot kRes is q.
constexpr int kSlots4 = (kRes + 1 + 3) / 4;
struct CombineWeights {
  u32 w[8][kSlots4];  // byte j of M/m_i (and of -M), four slots a word
  u32 f[3][kSlots4];  // byte j of round(2^24 / m_i)
};
constexpr CombineWeights combine_weights() {
  CombineWeights c{};
  for (int i = 0; i <= kRes; ++i) {
    const u64 w = i < kRes ? cofactor_64(i) : (u64)0 - cofactor_64(kRes);
    for (int j = 0; j < 8; ++j) c.w[j][i / 4] |= sbyte(w, j) << (8 * (i % 4));
    if (i == kRes) continue;
    const u64 m = (u64)kResModuli[i], f = (((u64)1 << 24) + m / 2) / m;
    for (int j = 0; j < 3; ++j) c.f[j][i / 4] |= sbyte(f, j) << (8 * (i % 4));
  }
  return c;
}
constexpr CombineWeights kComb = combine_weights();

// x mod 2^64 from the 18 residues of one output (four to a word; byte 2 of the
// last word is free for q).
__device__ __forceinline__ u64 combine_one(const u32 (&c)[kSlots4]) {
  int d[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    d[j] = 0;
#pragma unroll
    for (int g = 0; g < kSlots4; ++g) d[j] = __builtin_amdgcn_sdot4((int)c[g], (int)kComb.f[j][g], d[j], false);
  }
  const int q = (d[0] + (d[1] << 8) + (d[2] << 16) + (1 << 23)) >> 24;
  const u32 last = c[kSlots4 - 1] | (u32)(q & 0xff) << (8 * (kRes % 4));
  int s[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    s[j] = 0;
#pragma unroll
    for (int g = 0; g < kSlots4; ++g)
      s[j] = __builtin_amdgcn_sdot4((int)(g + 1 < kSlots4 ? c[g] : last), (int)kComb.w[j][g], s[j], false);
  }
  // |s_j| < 2^19: neighbouring bytes pair up within 32 bits
  const i64 p0 = s[0] + (s[1] << 8), p1 = s[2] + (s[3] << 8);
  const u32 hi = (u32)(s[4] + (s[5] << 8)) + ((u32)(s[6] + (s[7] << 8)) << 16);
  return (u64)p0 + ((u64)p1 << 16) + ((u64)hi << 32);
}
static_assert(kRes % 4 != 0, "q takes a free slot of the last word");

struct ResOutView {
  cptr<ResOut> outs;
  cptr<i64> unit_start;
  int nout;
};

// Bound by HBM: 18 bytes of residues, 8 of the added term and 8 stored an
// output (two shares of 4096 x 4096: 0.23 ms, 4.9 TB/s).
// One wave combines one unit of 16 rows x 64 columns: 18 loads of 16 bytes a
// lane and chunk, all in flight before the first is used.  The residues come in
// the GEMM's lane order (a lane holds 4 x 4 columns of one row); the outputs turn
// through LDS so that the added term and the stores run along rows, 512
// contiguous bytes an access (without, 16 rows of 8-byte pieces each: 0.28 ms).
constexpr int kCombPad = 66;
__global__ void __launch_bounds__(256) k_res_combine(ResOutTables) {
  __shared__ u64 turn[4][16 * kCombPad];
  const cptr<ResOutTables> tp = (cptr<ResOutTables>)MPC_KERNARG_PTR();
  const cptr<ResOut> outs = tp->outs ? (cptr<ResOut>)(uintptr_t)tp->outs : tp->iouts;
  const cptr<i64> us = tp->outs ? (cptr<i64>)(uintptr_t)tp->unit_start : tp->iunit_start;
  const int nout = tp->nout;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const i64 un = (i64)blockIdx.x * 4 + wave;
  if (un >= us[nout]) return;  // whole wave leaves; only wave-level sync below
  const int oi = find_job(us, nout, un);
  const cptr<ResOut> o = outs + oi;
  const i64 local = un - us[oi], real64 = (o->N + 63) / 64;
  const i64 ur = local / real64, uc = local % real64;
  const uint8_t* R = o->R + (ur * o->n64 + uc) * kResBlockBytes + lane * 16;
  // after the turn: this lane's column, row by row; lanes past the edge read the first element
  const Epilogue ep = o->ep;
  const i64 m0 = ur * 16, n = uc * 64 + lane, M = o->M;
  const bool n_ok = n < o->N;
  const i64 coff = ep.view.ld_q ? n / ep.view.n_div * ep.view.ld_q + n % ep.view.n_div : n;
  u64 z[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) z[k] = 0;
  const int nch = o->nch;
  for (int ch = 0; ch < nch; ++ch) {
    v4i p[kRes];
#pragma unroll
    for (int i = 0; i < kRes; ++i) p[i] = *(const gv4i*)(R + ch * o->pc + i * o->pr);
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      u32 c[4][kSlots4];
#pragma unroll
      for (int g = 0; g < kSlots4; ++g) {
        const u32 w0 = (u32)p[4 * g][y], w1 = 4 * g + 1 < kRes ? (u32)p[(4 * g + 1) % kRes][y] : 0;
        const u32 w2 = 4 * g + 2 < kRes ? (u32)p[(4 * g + 2) % kRes][y] : 0, w3 = 4 * g + 3 < kRes ? (u32)p[(4 * g + 3) % kRes][y] : 0;
        const u32 a0 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), a1 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
        const u32 b0 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), b1 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
        c[0][g] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
        c[1][g] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
        c[2][g] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
        c[3][g] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) z[4 * y + e] += combine_one(c[e]);
    }
  }
  u64* t = turn[wave];
#pragma unroll
  for (int k = 0; k < 16; ++k) t[(lane & 15) * kCombPad + (k >> 2) * 16 + (lane >> 4) * 4 + (k & 3)] = z[k];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < 16; ++k) z[k] = t[k * kCombPad + lane];
  // the shared epilogue: added term, truncation, store (loads before stores)
  if (ep.Cadd) {
    const u64 neg = ep.csign < 0 ? ~(u64)0 : 0;  // -c as (c ^ ~0) + 1
    u64 cv[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) cv[k] = ep.Cadd[n_ok && m0 + k < M ? (m0 + k) * ep.view.ld_m + coff : 0];
#pragma unroll
    for (int k = 0; k < 16; ++k) z[k] += (cv[k] ^ neg) + (neg & 1);
  }
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (n_ok && m0 + k < M) ep.Out[(m0 + k) * ep.view.ld_m + coff] = ep.trunc_bits ? (u64)((i64)z[k] >> ep.trunc_bits) : z[k];
}

}  // namespace

i64 res_rblocks(i64 rows) { return ((rows + 15) / 16 + kResRowPad - 1) / kResRowPad * kResRowPad; }
i64 res_kblocks(i64 K) { return (K + 63) / 64; }
void res_tile_shape(int tile, int* bm, int* bn) {
  static const int rows[kResTiles] = {R256x256::BM, R256x128::BM, R128x256::BM, R128x128::BM};
  static const int cols[kResTiles] = {R256x256::BN, R256x128::BN, R128x256::BN, R128x128::BN};
  *bm = rows[tile];
  *bn = cols[tile];
}

hipError_t launch_res_pack(hipStream_t s, const PackTables& t, i64 total_units, PackSet set) {
  if (total_units <= 0) return hipSuccess;
  switch (set) {
    case kPackMatmul: return launch_res_pack_set(s, t, total_units, SetPairs<kPackMatmul>::T{});
    case kPackConv: return launch_res_pack_set(s, t, total_units, SetPairs<kPackConv>::T{});
    case kPackConvDirect: return launch_res_pack_set(s, t, total_units, SetPairs<kPackConvDirect>::T{});
    case kPackDeal: return launch_res_pack_set(s, t, total_units, SetPairs<kPackDeal>::T{});
    case kPackDealConv: return launch_res_pack_set(s, t, total_units, SetPairs<kPackDealConv>::T{});
    case kPackDealConvDirect: return launch_res_pack_set(s, t, total_units, SetPairs<kPackDealConvDirect>::T{});
    case kPackRing: return launch_res_pack_set(s, t, total_units, SetPairs<kPackRing>::T{});
    case kPackMatmulLeft: return launch_res_pack_set(s, t, total_units, SetPairs<kPackMatmulLeft>::T{});
    case kPackMatmulRight: return launch_res_pack_set(s, t, total_units, SetPairs<kPackMatmulRight>::T{});
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_res_pack_party(hipStream_t s, const PartyPackTables& t) {
  const i64 units = t.side[0].job.units + t.side[1].job.units;
  if (units <= 0) return hipSuccess;
  if (t.side[0].P > kMaxParties || t.side[1].P > kMaxParties) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_res_pack_party, dim3((unsigned)((units + 3) / 4)), dim3(kPackThreads), 0, s, t);
  return hipGetLastError();
}

int res_tile_per_cu(int tile) {
  static const int per[kResTiles] = {R256x256::kPerCU, R256x128::kPerCU, R128x256::kPerCU, R128x128::kPerCU};
  return per[tile];
}

hipError_t launch_res_gemm(hipStream_t s, const ResGemmTables& tables, int total_tiles, int tile, int grid, bool conv) {
  if (total_tiles <= 0) return hipSuccess;
  if (grid < 1 || grid > total_tiles) return hipErrorInvalidValue;
  ResGemmTables t = tables;
  t.tiles = total_tiles;
#define MPC_RES_CASE(T, G)                                                                      \
  case T:                                                                                       \
    if (conv) hipLaunchKernelGGL((k_res_gemm<G, true>), dim3(grid), dim3(256), 0, s, t);        \
    else hipLaunchKernelGGL((k_res_gemm<G, false>), dim3(grid), dim3(256), 0, s, t);            \
    break;
  switch (tile) {
    MPC_RES_CASE(kRes256x256, R256x256)
    MPC_RES_CASE(kRes256x128, R256x128)
    MPC_RES_CASE(kRes128x256, R128x256)
    MPC_RES_CASE(kRes128x128, R128x128)
    default: return hipErrorInvalidValue;
  }
#undef MPC_RES_CASE
  return hipGetLastError();
}

hipError_t launch_res_combine(hipStream_t s, const ResOutTables& t, i64 total_units) {
  if (total_units <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_res_combine, dim3((unsigned)((total_units + 3) / 4)), dim3(256), 0, s, t);
  return hipGetLastError();
}

}  // namespace mpc
