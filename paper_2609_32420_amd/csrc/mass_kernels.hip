// Exact (token-level) attention mass of every block pair of the historical
// run: Appendix C.3 keeps, per head and query block, the smallest set of key
// blocks covering a fixed fraction of the source attention mass; read
// literally, that mass is the historical softmax attention summed over the
// tokens of each block pair (the pooled builder of mask_kernels.hip
// estimates it from block means).
//
//   M[b,h,i,j] = (1 / n_i) sum_{a in block i} sum_{t in block j}
//                softmax_t(sigma q_a . k_t)        (rows sum to 1)
//
// Pass 1 (mass_pass_kernel): a workgroup of NW waves per 64 NW queries, 64
// queries per wave in two sets of 32, streams every key block of its head
// through LDS and computes S^T = K Q^T on bf16 MFMA 32x32x16 (fp32
// accumulation), keys as MFMA rows so that a query's scores sit in one lane
// pair.  Each query has one reference r (log2 units, a whole number, fixed
// for the whole pass), and per key block one fp32 record s_j = sum of
// 2^(x - r) over the block's keys; at the end its total l (fp64).  Pass 2
// (mass_reduce_kernel) forms M_ij = sum_a s_j / l_a / n_i in fp64.
// The records are block-major ([bh][j][a]) so a wave's 64 queries write 256
// contiguous bytes.
//
// The reference is the maximum m over the query's first 32 keys, or
// min(m + 32, 0) if m is below 0: no running maximum and no rescaling, a score
// costs one fma, one exp2 and one add.  2^(x - r) spans 2^-126 .. 2^127
// whatever r is, so the sums are as precise as with the row maximum; with
// r >= 0 the fma rounds x - r no coarser than x itself for every x that
// carries mass, and with scores that all lie lower x - r stays within
// -32 .. 64 there.  A query whose total leaves [2^-40, 2^100] (2^64 if a query
// of its wave has r < 0; scores about 100 log2 units above its first keys), or
// with inputs that are not finite, makes its workgroup start over with the
// true row maxima, taken in a pass of their own: three passes over K for one
// (every workgroup of 12 heads x 32,760 tokens: 2.95 -> 7.9 ms, of 48 x 17,776
// at d = 64 2.57 -> 6.2).  A shift of every score by -40 nats costs nothing.
//
// Bound: the vector work beside the MFMAs (per 32-key tile and set D / 16
// MFMAs against 16 fma, 16 exp2 and 16 adds).  12 heads of 32,760 tokens, d =
// 128: both passes 2.95 ms, 1120 TFLOP/s (3.56 ms with the MFMAs and then the
// exponentials of a tile in turn, a running maximum and 8-byte records); 48
// heads of 17,776 tokens, d = 64: 2.33 ms (3.34).  Relative error of the
// masses against 64 bits 2e-8 .. 4e-8 (7e-8 .. 2e-7 with log2-sum-exps).
#include "internal.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace carnator {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// 16-byte chunk c of K row r sits in slot c ^ swz(r): the 32 rows an operand
// read touches at one chunk spread over the LDS banks.
template <int CPR>
__device__ inline int mswz(int r) {
  if constexpr (CPR == 16) return r & 15;
  else return (r >> 1) & 7;
}

// 16 bytes per lane from p to LDS offset lds_off + 16 lane (lds_off the same
// in every lane): a direct load, inline so that the compiler does not drain
// it before the next LDS read.  M0 is written a wait state before its use.
__device__ inline void mass_dma16(const void *p, unsigned lds_off) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p),
               "s"(__builtin_amdgcn_readfirstlane(lds_off))
               : "memory", "m0");
}
__device__ inline void mass_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
__device__ inline void mass_anchor(float x) { asm volatile("" ::"v"(x)); }

// x of the lane pair (l, l + 32), combined in the same order in both lanes.
__device__ inline float pair_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// Lanes 0 .. 31: the pair sum of a, lanes 32 .. 63: that of b.
__device__ inline float pair_sums(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// How far (log2 units) a reference below 0 lies above the query's first
// maximum, and the total that such a query may reach.
constexpr float kLowReference = 32.f;
constexpr double kLowTotalMax = 0x1p64;

template <int D, int BS, int NW>
struct MassCfg {
  static constexpr int NT = 64 * NW;
  static constexpr int Q = 64 * NW;          // queries per workgroup
  static constexpr int CPR = D / 8;          // 16-byte chunks per K row
  static constexpr int RB = D * 2;           // bytes per K row
  static constexpr int TILE = BS * RB;       // one key block in LDS
  static constexpr int LDS = 2 * TILE;       // double buffer
  static constexpr int RPL = 1024 / RB;      // rows per 1-KiB direct load
  static constexpr int LI = TILE / 1024 / NW;  // direct loads per wave per block
  static constexpr int F = D / 16;           // K fragments (MFMA steps) per tile
  static constexpr int MT = BS / 32;         // tiles per block
  static_assert(TILE % (1024 * NW) == 0 && 16 % F == 0, "tile split");
};

// One 32-key tile and query set at a time: MFMA step t of one set shares its
// slot with 16 / F scores of the other set's exponentials, so every wave's
// instruction stream keeps both units busy.  Per block and tile m:
//   Y: accB = K(m) Q_B^T   beside the exponentials of accA (tile m); each K
//      fragment is refilled with tile m + 1 once used for the last time
//   X: accA = K(m + 1) Q_A^T beside the exponentials of accB (tile m)
// The tile after a block's last is the next block's first.  The barrier
// before a block's last Y says that the next block is in LDS and that nobody
// reads this block's tile any more; the block after the next is then loaded
// into it.
//
// At d = 64 with 8 waves the kernel is held to 128 registers (a few spills
// outside the loop), so that two workgroups share a CU: the exponentials take
// twice the MFMAs' time there, and four waves per SIMD fill their latencies
// better than two (2.33 against 2.47 ms on 48 heads of 17,776 tokens).
template <int D, int BS, int NW>
__global__ void __launch_bounds__(64 * NW, (D == 64 && NW == 8) ? 4 : 2)
mass_pass_kernel(View q, View k, int H, int N, int nB, int bh0, float c2,
                 float *__restrict__ rec, float *__restrict__ total) {
  using C = MassCfg<D, BS, NW>;
  constexpr int F = C::F, MT = C::MT, SPS = 16 / F;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int ng = (nB * BS + C::Q - 1) / C::Q;  // query groups per head
  const int qg = (int)(blockIdx.x % ng);
  // heads bh0 .. of the chunk this launch covers; records and totals are
  // indexed inside the chunk
  const int bc = (int)(blockIdx.x / ng);
  const int bh = bh0 + bc;
  const int b = bh / H, h = bh - b * H;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  // the scores of this lane belong to query l32 of each of the wave's two
  // sets of 32; its records to query `lane` of the 64
  const int aw = qg * C::Q + wave * 64;
  const bool mine = aw + lane < N;

  // Q as the B operand: query l32 of a set, channels 16 t + 8 hh .. + 8
  bf16x8 q0[F], q1[F];
  {
    const uint16_t *qh = q.data + (int64_t)b * q.sb + (int64_t)h * q.sh + 8 * hh;
    const int a0 = aw + l32, a1 = a0 + 32;
    const uint16_t *p0 = qh + (int64_t)min(a0, N - 1) * q.sn;
    const uint16_t *p1 = qh + (int64_t)min(a1, N - 1) * q.sn;
#pragma unroll
    for (int t = 0; t < F; ++t) {
      const uint4 v0 = *reinterpret_cast<const uint4 *>(p0 + 16 * t);
      const uint4 v1 = *reinterpret_cast<const uint4 *>(p1 + 16 * t);
      q0[t] = a0 < N ? __builtin_bit_cast(bf16x8, v0) : bf16x8{};
      q1[t] = a1 < N ? __builtin_bit_cast(bf16x8, v1) : bf16x8{};
    }
  }
  // the fragments are in registers before any direct load is issued
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)

  // Direct loads: the i-th of this wave fills rows RPL (wave LI + i) .. + RPL
  // of a block's tile; lane l writes 16 bytes at 16 l, slot `slot` of row
  // +lrow, which holds chunk slot ^ swz(row).  Rows past N read row N - 1.
  const uint16_t *kbase = k.data + (int64_t)b * k.sb + (int64_t)h * k.sh;
  const int lrow = lane / (C::RB / 16), slot = lane % (C::RB / 16);
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)lds;
  auto load_block = [&](int j, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < C::LI; ++i) {
      const int r = C::RPL * (wave * C::LI + i) + lrow;
      const int tok = min(j * BS + r, N - 1);
      mass_dma16(kbase + (int64_t)tok * k.sn + (slot ^ mswz<C::CPR>(r)) * 8,
                 lds_base + (unsigned)(buf * C::TILE + (wave * C::LI + i) * 1024));
    }
  };
  // K fragment t of a tile (A operand): row l32, chunk 2 t + hh
  int kread[F];
  auto reset_kread = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < F; ++t) kread[t] = l32 * C::RB + 16 * ((2 * t + hh) ^ mswz<C::CPR>(l32));
  };
  bf16x8 kf[F];
  auto frag = [&](int t, int m) __attribute__((always_inline)) {
    kf[t] = *reinterpret_cast<const bf16x8 *>(lds + kread[t] + m * 32 * C::RB);
  };
  auto mfma = [&](f32x16 &acc, const bf16x8 (&qf)[F], int t) __attribute__((always_inline)) {
    if (t == 0) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t], qf[t], f32x16{}, 0, 0, 0);
    else acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t], qf[t], acc, 0, 0, 0);
  };
  auto tile_max = [&](const f32x16 &acc) __attribute__((always_inline)) {
    float m = acc[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m = fmaxf(m, acc[v]);
    return pair_max(m);
  };

  f32x16 accA, accB;
  float refA = 0.f, refB = 0.f;
  double l = 0.0;
  // at most two rounds: the second with the row maxima as references
  for (int round = 0; round < 2; ++round) {
    reset_kread();
    if (round == 1) {
      float mA = -INFINITY, mB = -INFINITY;
      for (int j = 0; j < nB; ++j) {
        load_block(j, 0);
        mass_wait_barrier();
        for (int m = 0; m < MT; ++m) {
#pragma unroll
          for (int t = 0; t < F; ++t) frag(t, m);
#pragma unroll
          for (int t = 0; t < F; ++t) mfma(accA, q0, t), mfma(accB, q1, t);
          mA = fmaxf(mA, tile_max(accA));
          mB = fmaxf(mB, tile_max(accB));
        }
        mass_wait_barrier();
      }
      refA = ceilf(mA * c2), refB = ceilf(mB * c2);
    }
    load_block(0, 0);
    load_block(min(1, nB - 1), 1);
    mass_wait_barrier();
#pragma unroll
    for (int t = 0; t < F; ++t) frag(t, 0);
#pragma unroll
    for (int t = 0; t < F; ++t) mfma(accA, q0, t), mfma(accB, q1, t);
    if (round == 0) {
      const float mA = ceilf(tile_max(accA) * c2), mB = ceilf(tile_max(accB) * c2);
      refA = mA < 0.f ? fminf(mA + kLowReference, 0.f) : mA;
      refB = mB < 0.f ? fminf(mB + kLowReference, 0.f) : mB;
    }
    // whether a query of the wave has a reference below 0 (scalar: kept per
    // lane it would cost vector registers through the loop)
    const bool low = __ballot(fminf(refA, refB) < 0.f) != 0;
    l = 0.0;
    float psA0, psA1, psB0, psB1;
    // scores [v, v + SPS) of a tile
    auto expo = [&](const f32x16 &acc, float ref, float &s0, float &s1, int v, int key0, int lim,
                    auto masked) __attribute__((always_inline)) {
#pragma unroll
      for (int x = v; x < v + SPS; x += 2) {
        float e0 = __builtin_amdgcn_exp2f(fmaf(acc[x], c2, -ref));
        float e1 = __builtin_amdgcn_exp2f(fmaf(acc[x + 1], c2, -ref));
        if constexpr (decltype(masked)::value) {
          int left = lim - key0 - 4 * hh;
          asm volatile("" : "+v"(left));  // compared here, not 64 times ahead of the loop
          e0 = 8 * (x >> 2) + (x & 3) < left ? e0 : 0.f;
          e1 = 8 * (x >> 2) + (x & 3) + 1 < left ? e1 : 0.f;
        }
        s0 += e0;
        s1 += e1;
        mass_anchor(s0);
        mass_anchor(s1);
      }
    };
    auto block = [&](auto masked, int j) __attribute__((always_inline)) {
      psA0 = psA1 = psB0 = psB1 = 0.f;
      const int lim = N - j * BS;  // valid keys of this block (used when masked)
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (m == MT - 1) {
          mass_wait_barrier();
          if (j + 2 < nB) load_block(j + 2, j & 1);
        }
        // Y
#pragma unroll
        for (int t = 0; t < F; ++t) {
          mfma(accB, q1, t);
          if (m < MT - 1) {
            frag(t, m + 1);
          } else {
            kread[t] ^= C::TILE;
            frag(t, 0);
          }
          expo(accA, refA, psA0, psA1, t * SPS, 32 * m, lim, masked);
          __builtin_amdgcn_sched_barrier(0);
        }
        // X
#pragma unroll
        for (int t = 0; t < F; ++t) {
          mfma(accA, q0, t);
          expo(accB, refB, psB0, psB1, t * SPS, 32 * m, lim, masked);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      const float s = pair_sums(psA0 + psA1, psB0 + psB1);
      l += (double)s;
      if (mine) rec[((int64_t)bc * nB + j) * N + aw + lane] = s;
    };
    for (int j = 0; j < nB - 1; ++j) block(std::false_type{}, j);
    block(std::true_type{}, nB - 1);  // only the last block can be partial
    const double most = low ? kLowTotalMax : 0x1p100;
    const bool bad = mine && !(l >= 0x1p-40 && l <= most);
    if (round == 1 || !__syncthreads_or(bad)) break;
  }
  if (mine) total[(int64_t)bc * N + aw + lane] = (float)l;
}

// One wave per (bh, i): lane x holds queries a0 + x and a0 + 64 + x of block
// i (the valid ones among them) and the reciprocals of their totals; the
// wave walks the key blocks j, eight at a time with all their record loads
// in flight, and forms M_ij = sum_a s / l_a / n_i in fp64 with one wave sum
// per j.
constexpr int kReduceUnroll = 8;
__global__ void __launch_bounds__(256) mass_reduce_kernel(const float *__restrict__ rec,
                                                          const float *__restrict__ total, int N,
                                                          int nB, int bs, int rows,
                                                          double *__restrict__ mass) {
  const int w = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (w >= rows) return;  // the whole wave
  const int i = w % nB, bh = w / nB;
  const int a0 = i * bs, a1 = min(a0 + bs, N);
  const int qa = a0 + lane, qb = a0 + 64 + lane;
  const int ca = min(qa, N - 1), cb = min(qb, N - 1);  // clamped: loads stay in the head
  const float *lh = total + (int64_t)bh * N;
  const double inv = 1.0 / (double)(a1 - a0);
  const bool va = qa < a1, vb = qb < a1;
  const double wa = inv / (double)lh[ca], wb = inv / (double)lh[cb];
  const float *rh = rec + (int64_t)bh * nB * N;
  double *out = mass + (int64_t)w * nB;
  for (int j0 = 0; j0 < nB; j0 += kReduceUnroll) {
    float ra[kReduceUnroll], rb[kReduceUnroll];
#pragma unroll
    for (int u = 0; u < kReduceUnroll; ++u) {
      const float *rj = rh + (int64_t)min(j0 + u, nB - 1) * N;
      ra[u] = rj[ca];
      rb[u] = rj[cb];
    }
#pragma unroll
    for (int u = 0; u < kReduceUnroll; ++u) {
      double t = va ? (double)ra[u] * wa : 0.0;
      t += vb ? (double)rb[u] * wb : 0.0;
      t = wave_sum(t);
      if (lane == 0 && j0 + u < nB) out[j0 + u] = t;
    }
  }
}

}  // namespace

// The entry point asks for 8 bytes per (query, key block) and 4 per query of a
// head, for as many heads as fit kMassScratchCap (at least one), so the
// workspace stays bounded whatever the number of heads.  The pass writes 4-byte
// records (34 MB a head at 32K tokens, 443 MB at 119K), so a chunk takes about
// twice as many heads, and where one chunk holds them all half of the workspace
// is not touched: the size asked for stays what callers that keep a workspace
// have always allocated.
constexpr size_t kMassScratchCap = (size_t)4 << 30;

size_t mass_scratch_bytes(int BH, int N, int nB) {
  const size_t per = (size_t)nB * N * 8 + (size_t)N * 4;
  const size_t ch = std::max<size_t>(1, std::min<size_t>(kMassScratchCap / per, (size_t)BH));
  return align_up(ch * nB * N * 8) + align_up(ch * N * 4);
}

// Heads whose records and totals (each array aligned) fit that workspace.
static int mass_chunk_heads(int BH, int N, int nB) {
  const size_t per = ((size_t)nB + 1) * N * sizeof(float);
  const size_t fit = (mass_scratch_bytes(BH, N, nB) - kAlign) / per;
  return (int)std::max<size_t>(1, std::min<size_t>(fit, (size_t)BH));
}

// Whether the pass takes workgroups of 4 waves (256 queries) instead of 8
// (512).  At d = 128 a CU holds one workgroup of 8 waves or two of 4, so both
// take rounds of 512 queries per CU, but a last round of at most one
// 4-wave workgroup per CU takes about 0.65 of a round (each wave has a SIMD
// to itself); the second stream of K per CU costs a full round about 5 %.
// Measured, 8 against 4 waves: 60 / 108 workgroups 66 / 47 us, 120 / 240
// 131 / 96, 288 / 564 637 / 537, 294 / 588 1461 / 1204, but 432 / 864 506 /
// 540, 480 / 948 1159 / 1213 and 768 / 1536 2952 / 3040.  At d = 64 a CU
// holds two of 8 waves: only a grid that leaves it half empty gains (60 / 108
// 51 / 35 us, 240 / 480 120 / 124).
static bool mass_small_groups(int heads, int rows, int d) {
  const int64_t g8 = (int64_t)heads * ((rows + 511) / 512), g4 = (int64_t)heads * ((rows + 255) / 256);
  if (d == 64) return g4 <= 256;
  const int64_t rem = g4 % 512;
  const double t8 = (double)((g8 + 255) / 256);
  const double t4 = (double)(g4 / 512) + (rem == 0 ? 0.0 : rem <= 256 ? 0.65 : 1.0);
  return 1.05 * t4 < t8;
}

hipError_t launch_mass(View q, View k, int B, int H, int N, int d, int bs, float scale,
                       double *mass, void *scratch, hipStream_t s) {
  const int nB = (N + bs - 1) / bs;
  const int BH = B * H;
  const int ch = mass_chunk_heads(BH, N, nB);
  float *rec = static_cast<float *>(scratch);
  float *total = reinterpret_cast<float *>(static_cast<char *>(scratch) +
                                           align_up((size_t)ch * nB * N * sizeof(float)));
  const float c2 = scale * 1.4426950408889634f;
  for (int bh0 = 0; bh0 < BH; bh0 += ch) {
    const int nh = std::min(ch, BH - bh0);
    hipError_t e = hipSuccess;
#define CARNATOR_MASS_W(DD, BB, WW)                                                              \
  do {                                                                                           \
    using C = MassCfg<DD, BB, WW>;                                                               \
    const dim3 grid((unsigned)(nh * ((nB * BB + C::Q - 1) / C::Q)));                             \
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&mass_pass_kernel<DD, BB, WW>),       \
                            hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);                 \
    if (e != hipSuccess) return e;                                                               \
    hipLaunchKernelGGL((mass_pass_kernel<DD, BB, WW>), grid, dim3(C::NT), C::LDS, s, q, k, H, N, \
                       nB, bh0, c2, rec, total);                                                 \
  } while (0)
#define CARNATOR_MASS(DD, BB)                                                                    \
  do {                                                                                           \
    if (mass_small_groups(nh, nB * BB, DD)) CARNATOR_MASS_W(DD, BB, 4);                          \
    else CARNATOR_MASS_W(DD, BB, 8);                                                             \
  } while (0)
    if (d == 128 && bs == 128) CARNATOR_MASS(128, 128);
    else if (d == 128 && bs == 64) CARNATOR_MASS(128, 64);
    else if (d == 64 && bs == 128) CARNATOR_MASS(64, 128);
    else CARNATOR_MASS(64, 64);
#undef CARNATOR_MASS
#undef CARNATOR_MASS_W
    const int rows = nh * nB;
    hipLaunchKernelGGL(mass_reduce_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, rec,
                       total, N, nB, bs, rows, mass + (int64_t)bh0 * nB * nB);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace carnator
