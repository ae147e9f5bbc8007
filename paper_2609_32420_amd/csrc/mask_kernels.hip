// Historical block-connectivity mask (Appendix C.3): block pooling of the
// historical Q/K, pooled logits, softmax over key blocks and the smallest
// prefix of key blocks (descending logit) whose mass reaches the threshold,
// with logits within 1e-6 of the cut handed to the lower block indices.
// Everything here runs in fp64.
#include "internal.h"

#include <math.h>

#include <type_traits>

namespace carnator {
namespace {

constexpr double kTieEps = 1e-6;

__device__ inline double bf16_to_f64(uint32_t bits16) {
  return (double)__uint_as_float(bits16 << 16);
}

// One workgroup per (tensor, bh, block).  Thread t owns 8 consecutive
// channels (one 16-byte chunk) of every G-th token of the block.  The G
// partial sums are combined in a fixed order (first across the lanes of a
// wave that share a chunk, then across waves), so the result does not depend
// on timing.
template <int D>
__global__ void __launch_bounds__(256) pool_kernel(View q, View k, int H, int N, int bs, int nB,
                                                   double *__restrict__ qbar,
                                                   double *__restrict__ kbar) {
  constexpr int CPR = D / 8;         // 16-byte chunks per token
  constexpr int G = 256 / CPR;       // token groups
  __shared__ double part[4][D];      // one partial per wave
  const int blk = blockIdx.x;
  const int bh = blockIdx.y;
  const int which = blockIdx.z;  // 0: Q_hist, 1: K_hist
  const View v = which ? k : q;
  const int b = bh / H, h = bh - b * H;
  const int t0 = blk * bs;
  const int n = min(bs, N - t0);
  const int c = threadIdx.x % CPR;
  const int g = threadIdx.x / CPR;
  const uint16_t *base = v.data + (int64_t)b * v.sb + (int64_t)h * v.sh + (int64_t)t0 * v.sn + c * 8;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  // All of this thread's tokens (at most RPT) are loaded before any is added,
  // so a wave keeps RPT 16-byte loads in flight instead of one.
  constexpr int RPT = 128 / G;
  uint4 w[RPT];
#pragma unroll
  for (int u = 0; u < RPT; ++u) {
    const int r = g + u * G;
    w[u] = r < n ? *reinterpret_cast<const uint4 *>(base + (int64_t)r * v.sn) : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < RPT; ++u) {
    const uint32_t ww[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += bf16_to_f64(ww[e] & 0xffffu);
      acc[2 * e + 1] += bf16_to_f64(ww[e] >> 16);
    }
  }
  // lanes l, l + CPR, l + 2 CPR, ... of a wave hold the same channels
#pragma unroll
  for (int o = CPR; o < 64; o <<= 1)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane < CPR) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[wave][c * 8 + e] = acc[e];
  }
  __syncthreads();
  for (int ch = threadIdx.x; ch < D; ch += 256) {
    const double s = ((part[0][ch] + part[1][ch]) + part[2][ch]) + part[3][ch];
    const double mean = s / (double)n;
    (which ? kbar : qbar)[((int64_t)bh * nB + blk) * D + ch] = mean;
  }
}

// ---- selection --------------------------------------------------------------
//
// Selection keys: an order-preserving map of the fp64 logit onto uint64 whose
// low 11 bits are replaced by (2047 - block index).  Descending key order is
// descending logit with the lower index first among logits equal in their
// top 53 bits; logits closer than that (2^-42 relative) lie deep inside the
// 1e-6 tie band, where the final choice is made by block index anyway.  The
// keys are unique; the selection finds the k-th largest by bisection and
// reads back the exact logit of its block.
__device__ inline uint64_t sel_key(double s, int j) {
  const uint64_t b = (uint64_t)__double_as_longlong(s);
  const uint32_t hi = (uint32_t)(b >> 32);
  const uint32_t neg = (uint32_t)((int32_t)hi >> 31);  // all ones for a negative logit
  const uint32_t kh = hi ^ (neg | 0x80000000u);
  const uint32_t kl = (((uint32_t)b ^ neg) & ~0x7ffu) | (uint32_t)(2047 - j);
  return ((uint64_t)kh << 32) | kl;
}
__device__ inline int sel_index(uint64_t k) { return 2047 - (int)(k & 0x7ff); }
// The logit a selection key stands for, up to its low 11 bits (used only to pick
// bisection points).
__device__ inline double key_value(uint64_t k) {
  const uint64_t b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
  return __longlong_as_double((long long)b);
}

// exp(x) for x <= 0 (NaN gives NaN, anything below the subnormals 0): x = n ln 2 + r
// with n the nearest integer (ln 2 in two parts), the Taylor series of exp(r)
// to r^13 (|r| <= 0.347: truncation 4e-18, 0.02 ulp) and a scaling by 2^n.
// Free of branches and with its coefficients in scalar registers, so the
// exponentials of a lane's positions interleave: through the library's exp
// each position was a predicated block of its own that first moved every
// coefficient into vector registers (42 vector instructions against 22).
struct ExpCoef {
  double c[12];  // 1 / 13!, ..., 1 / 2!
  double log2e, ln2hi, ln2lo;
};
__device__ inline double in_sgpr(double x) {
  asm("" : "+s"(x));
  return x;
}
__device__ inline ExpCoef exp_coef() {
  ExpCoef e;
  constexpr double f[12] = {1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0,
                            1.0 / 362880.0,     1.0 / 40320.0,     1.0 / 5040.0,     1.0 / 720.0,
                            1.0 / 120.0,        1.0 / 24.0,        1.0 / 6.0,        1.0 / 2.0};
#pragma unroll
  for (int i = 0; i < 12; ++i) e.c[i] = in_sgpr(f[i]);
  e.log2e = in_sgpr(1.4426950408889634074);
  e.ln2hi = in_sgpr(0x1.62e42fefa0000p-1);        // ln 2 to 36 bits: n ln2hi is exact
  e.ln2lo = in_sgpr(0x1.cf79abc9e3b3ap-40);       // ln 2 - ln2hi
  return e;
}
__device__ inline double exp_neg(double x, const ExpCoef &e) {
  x = x < -800.0 ? -800.0 : x;
  const double n = __builtin_rint(x * e.log2e);
  double r = __builtin_fma(-n, e.ln2hi, x);
  r = __builtin_fma(-n, e.ln2lo, r);
  double p = e.c[0];
#pragma unroll
  for (int i = 1; i < 12; ++i) p = __builtin_fma(p, r, e.c[i]);
  p = __builtin_fma(p, r, 1.0);
  p = __builtin_fma(p, r, 1.0);
  return __builtin_ldexp(p, (int)n);
}

// Bisection state of one row (the same in every lane): mass(key >= lo) >=
// tau Z > mass(key >= hi), cnt_* the numbers of keys >= lo and >= hi.
struct Bisect {
  uint64_t lo, hi;
  int cnt_lo, cnt_hi;
  double m_hi;  // mass of the keys >= hi
  bool trie;
  int it;
};

// Bisection steps over EE positions per lane until at most `until` keys lie
// in [lo, hi).  The keys counted are those of the positions plus c_off, the
// mass their weights plus m_off (the keys above the positions' range).
// Split at the midpoint of the values while that separates keys; once it
// does not (a run of equal logits), split at the highest bit in which the
// interval's smallest and largest keys differ, which leaves keys on both
// sides and resolves equal logits by their index bits.
template <int EE>
__device__ inline void bisect_steps(const uint64_t (&key)[EE], const double (&pl)[EE], int c_off,
                                    double m_off, double tauZ, int until, Bisect &b) {
  for (; b.it < 192 && b.cnt_lo - b.cnt_hi > until; ++b.it) {
    uint64_t K = 0;
    if (!b.trie) {
      const double lv = key_value(b.lo), hv = key_value(b.hi - 1);
      K = sel_key(uniform(lv + 0.5 * (hv - lv)), 2047);
      b.trie = !(K > b.lo && K < b.hi);
    }
    if (b.trie) {
      uint64_t a = ~0ull, z = 0ull;
#pragma unroll
      for (int u = 0; u < EE; ++u) {
        const bool in = key[u] >= b.lo && key[u] < b.hi;
        a = in && key[u] < a ? key[u] : a;
        z = in && key[u] > z ? key[u] : z;
      }
      a = wave_min_u64(a);
      z = wave_max_u64(z);
      // a < z: the interval holds at least two (distinct) keys
      K = z & ~((1ull << (63 - __clzll((long long)(a ^ z)))) - 1ull);
    }
    double m = 0.0;
    int c = c_off;
#pragma unroll
    for (int u = 0; u < EE; ++u) {
      const bool ge = key[u] >= K;
      m += ge ? pl[u] : 0.0;
      c += __popcll(__ballot(ge));
    }
    m = m_off + wave_sum(m);
    const int before = b.cnt_lo - b.cnt_hi;
    if (m >= tauZ) {
      b.lo = K;
      b.cnt_lo = c;
    } else {
      b.hi = K;
      b.cnt_hi = c;
      b.m_hi = m;
    }
    if (b.cnt_lo - b.cnt_hi == before) b.trie = true;
  }
}

// The k-th largest key once the bisection has ended: the one key in [lo, hi)
// (k = cnt_lo), or, if the step cap was hit, the largest key in [lo, hi) and
// the number of keys at or above it.
template <int EE>
__device__ inline uint64_t bisect_result(const uint64_t (&key)[EE], int c_off, const Bisect &b,
                                         int &k) {
  uint64_t kstar = 0ull;
  if (b.cnt_lo - b.cnt_hi == 1) {
#pragma unroll
    for (int u = 0; u < EE; ++u) {
      const unsigned long long hit = __ballot(key[u] >= b.lo && key[u] < b.hi);
      if (hit) kstar = read_lane(key[u], __ffsll((long long)hit) - 1);
    }
    k = b.cnt_lo;
  } else {
    uint64_t kl = 0ull;
#pragma unroll
    for (int u = 0; u < EE; ++u)
      if (key[u] >= b.lo && key[u] < b.hi && key[u] > kl) kl = key[u];
    kstar = wave_max_u64(kl);
    k = c_off;
#pragma unroll
    for (int u = 0; u < EE; ++u) k += __popcll(__ballot(key[u] >= kstar));
  }
  return kstar;
}

// The positions per lane that select_kernel is instantiated for; the one
// before E (rows taken by E have more than 64 sel_prev(E) blocks).
constexpr int kSelE[] = {0, 1, 2, 3, 4, 6, 8, 10, 12, 16, 24, 32};
constexpr int sel_prev(int e) {
  int p = 0;
  for (int x : kSelE) p = x < e ? x : p;
  return p;
}

// One workgroup of W = R waves per (bh, R consecutive query blocks).
//
// Phase 1, s_ij = sigma <qbar_i, kbar_j>: the R pooled query rows sit in LDS;
// a wave takes 16 key blocks at a time and forms the 16 x 16 tile of dot
// products on the fp64 matrix cores (16x16x4 steps over the channels).  The
// contraction visits the channels in an order that suits the loads: in
// 16-channel group g, lane (i, k) = (lane & 15, lane >> 4) holds channels
// 16 g + 4 k .. 16 g + 4 k + 3 of key block i (one 32-byte piece of its kbar
// row) and feeds channel 16 g + 4 k + t to step t, and the query side takes
// its channels in the same order.  With R = 8 the upper half of the tile
// repeats row R - 1 and is not stored.  Phase 2: wave w selects row w of the
// workgroup (E = positions per lane, 64 E >= nB).
//
// Bound: at nB = 591 (40 heads) 192 us, was 244 us: the score tiles with
// their kbar loads (0.9 GB through the L2) 119 us, 74 us of it the fp64
// matrix cores (2048 cycles a tile), and the selection 73 us of dependent
// vector work, ~1330 vector instructions a row; one workgroup per CU, so the
// two do not overlap: by its LDS from 385 blocks on, below by the registers of
// its 16 waves (75 a lane at d = 64 and 119 at 128, where two would need 64).
// The gain is one row per wave on 16 waves (244 -> 215 us) and a selection
// free of branches per position: rows padded to 64 E so that every logit is
// loaded at once, exp_neg, and the tie ranks taken on whole 64-bit words.  At
// nB <= 256 one workgroup's latency (20 us), twice that where there are more
// workgroups than CUs (48 heads of 139 blocks: 432).
// MASS: the rows are given, as block masses [BH][nB][nB] at qbar (kbar and
// sigma unused): phase 1 copies the workgroup's rows into LDS and phase 2
// selects on the masses themselves instead of the softmax of logits.
template <int D, int E, int R, int W, bool MASS>
__global__ void __launch_bounds__(64 * W) select_kernel(const double *__restrict__ qbar,
                                                        const double *__restrict__ kbar, int nB,
                                                        double sigma, double tau,
                                                        uint8_t *__restrict__ mask,
                                                        uint64_t *__restrict__ bits, int BH) {
  // LDS: [R][NP] logits (NP = 64 E, -inf past nB), then the R pooled query rows, QS doubles apart (a
  // 16-byte pad spreads the 16 rows read by one MFMA step over the banks),
  // at least W * 128 doubles
  constexpr int QS = D + 2, NP = 64 * E;
  extern __shared__ double sc[];
  // Workgroups are dealt to the 8 XCDs in turn.  Logical workgroup
  // (L mod 8) ceil(G / 8) + L / 8 gives each XCD a contiguous run of
  // (head, row block) pairs, so an XCD's L2 fetches the kbar of about
  // BH / 8 heads instead of all of them.
  static_assert(W == R, "one row per wave in phase 2");
  const int nbx = (nB + R - 1) / R;
  const int G = nbx * BH;
  const int per = (G + 7) / 8;
  const int T = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (T >= G) return;  // the whole workgroup, before any barrier
  const int bh = T / nbx;
  const int r0 = (T - bh * nbx) * R;
  const int nr = min(R, nB - r0);
  const double *qb = qbar + ((int64_t)bh * nB + r0) * D;
  const double *kb = kbar + (int64_t)bh * nB * D;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  // phase 2's candidate buffers (64 keys and weights per wave) reuse the
  // pooled-row area, which phase 1's last barrier frees
  uint64_t *cbuf = reinterpret_cast<uint64_t *>(sc + R * NP);

  if constexpr (MASS) {
    const double *src = qbar + ((int64_t)bh * nB + r0) * nB;
    if (wave < nr)
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const int p = u * 64 + lane;
        const double m = src[wave * nB + min(p, nB - 1)];
        sc[wave * NP + p] = p < nB ? m : -INFINITY;
      }
    __syncthreads();
  } else {
    double *qs = sc + R * NP;
    {
      constexpr int SPT = R * D / (64 * W);  // staged values per thread (all loads in flight)
      double sv[SPT];
  #pragma unroll
      for (int i = 0; i < SPT; ++i) {
        const int x = threadIdx.x + i * 64 * W, r = x / D, c = x - r * D;
        sv[i] = qb[min(r, nr - 1) * D + c];
      }
  #pragma unroll
      for (int i = 0; i < SPT; ++i) {
        const int x = threadIdx.x + i * 64 * W, r = x / D, c = x - r * D;
        qs[r * QS + c] = sv[i];
      }
    }
    if (wave < nr)
      for (int p = nB + lane; p < NP; p += 64) sc[wave * NP + p] = -INFINITY;
    __syncthreads();
    {
      typedef double f64x4 __attribute__((ext_vector_type(4)));
      constexpr int NG = D / 16;  // 16-channel groups
      const int li = lane & 15, lk = lane >> 4;
      const double *qr = qs + min(li, R - 1) * QS + 4 * lk;
      // The groups start at a different place in every wave: walking them in
      // lockstep sends every wave of the chip to the same few L2 channels.
      const int rot = (wave * 5 + T * 3) & (NG - 1);
      // All of a wave's first tile is loaded before its first product (left to
      // itself the compiler keeps two loads in flight, and a tile then costs
      // D / 8 L2 round trips instead of one); after that each channel group
      // is loaded for the next tile as soon as its products are issued, so
      // the loads of one tile run under the products of the other without a
      // second set of registers.
      double2 kv[NG][2];
      const double *kr = kb + 4 * lk;
      auto load = [&](int g, int j) __attribute__((always_inline)) {
        const int gr = (g + rot) & (NG - 1);
        const double *p = kr + (int64_t)min(j + li, nB - 1) * D + 16 * gr;
        kv[g][0] = *reinterpret_cast<const double2 *>(p);
        kv[g][1] = *reinterpret_cast<const double2 *>(p + 2);
      };
      auto tile = [&](auto next, int j0) __attribute__((always_inline)) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const int gr = (g + rot) & (NG - 1);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qr[16 * gr + 0], kv[g][0].x, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qr[16 * gr + 1], kv[g][0].y, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qr[16 * gr + 2], kv[g][1].x, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qr[16 * gr + 3], kv[g][1].y, acc, 0, 0, 0);
          if constexpr (decltype(next)::value) {
            load(g, j0 + 16 * W);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        const int j = j0 + li;
        if (j < nB) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int r = lk + 4 * v;
            if (r < nr) sc[r * NP + j] = sigma * acc[v];
          }
        }
      };
      int j0 = wave * 16;
      if (j0 < nB) {
#pragma unroll
        for (int g = 0; g < NG; ++g) load(g, j0);
        __builtin_amdgcn_sched_barrier(0);
        for (; j0 + 16 * W < nB; j0 += 16 * W) tile(std::true_type{}, j0);
        tile(std::false_type{}, j0);
      }
    }
    __syncthreads();
  }

  // ---- phase 2: selection, one row per wave.  Lane l holds positions
  // u 64 + l.  The k-th largest selection key K* (k the shortest prefix whose
  // mass reaches tau) is found by bisection over the keys, keeping
  // mass(key >= lo) >= tau > mass(key >= hi) until [lo, hi) holds one key.
  // The bisection state is the same in every lane and lives in scalar
  // registers; the vector work per step is one compare and add per position
  // and one wave sum.
  const ExpCoef ec = exp_coef();
  if (const int r = wave; r < nr) {
    const double *row = sc + r * NP;
    const int64_t grow = (int64_t)bh * nB + r0 + r;
    double pl[E];
    uint64_t key[E];
    double smax = -INFINITY, smin = INFINITY;
    // (positions below 64 EP are always valid: the launcher takes the
    // smallest E with 64 E >= nB)
    constexpr int EP = sel_prev(E);
#pragma unroll
    for (int u = 0; u < E; ++u) pl[u] = row[u * 64 + lane];  // the logit until the softmax below
#pragma unroll
    for (int u = 0; u < E; ++u) {
      const int p = u * 64 + lane;
      const bool ok = u < EP || p < nB;
      const double s = pl[u];
      key[u] = ok ? sel_key(s, p) : 0ull;  // valid keys are > 2047
      smax = fmax(smax, s);
      smin = ok ? fmin(smin, s) : smin;
    }
    smax = wave_max(smax);
    smin = wave_min(smin);
    // softmax weights exp(s - max): a set's mass p = weight / Z reaches tau
    // when its weight reaches tau Z (Z the sum of all weights)
    double lsum = 0.0;
#pragma unroll
    for (int u = 0; u < E; ++u) {
      const bool ok = u < EP || u * 64 + lane < nB;
      if constexpr (MASS) pl[u] = ok ? pl[u] : 0.0;
      else pl[u] = ok ? exp_neg(pl[u] - smax, ec) : 0.0;
      lsum += pl[u];
    }
    const double Z = wave_sum(lsum);
    const double tauZ = tau * Z;

    // every key lies in [smallest key of value smin, largest key of smax],
    // and together they hold the whole mass Z
    Bisect bs{sel_key(smin, 2047), sel_key(smax, 0) + 1, nB, 0, 0.0, false, 0};
    const bool reach = Z >= tauZ;
    int k;
    double cut;
    if (!reach) {
      k = bs.cnt_lo;  // the whole row falls short of tau: keep every block
      cut = smin;
    } else {
      uint64_t kstar;
      if constexpr (E == 1) {
        bisect_steps<1>(key, pl, 0, 0.0, tauZ, 1, bs);
        kstar = bisect_result<1>(key, 0, bs, k);
      } else {
        // all positions until at most 64 keys are left in [lo, hi); those
        // keys and weights then go one per lane (through this wave's LDS
        // area), and the remaining steps touch one position per lane
        bisect_steps<E>(key, pl, 0, 0.0, tauZ, 64, bs);
        if (bs.cnt_lo - bs.cnt_hi > 64) {
          kstar = bisect_result<E>(key, 0, bs, k);  // the step cap was hit
        } else {
          uint64_t *ck = cbuf + wave * 128;
          double *cw = reinterpret_cast<double *>(ck + 64);
          int base = 0;
#pragma unroll
          for (int u = 0; u < E; ++u) {
            const bool in = key[u] >= bs.lo && key[u] < bs.hi;
            const unsigned long long hit = __ballot(in);
            if (in) {
              const int x = base + __popcll(hit & ((1ull << lane) - 1ull));
              ck[x] = key[u];
              cw[x] = pl[u];
            }
            base += __popcll(hit);
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          // empty lanes hold key 0, below every valid key (> 2047)
          uint64_t k1[1] = {lane < base ? ck[lane] : 0ull};
          double p1[1] = {lane < base ? cw[lane] : 0.0};
          const int c_off = bs.cnt_hi;
          const double m_off = bs.m_hi;
          bisect_steps<1>(k1, p1, c_off, m_off, tauZ, 1, bs);
          kstar = bisect_result<1>(k1, c_off, bs, k);
        }
      }
      cut = row[sel_index(kstar)];
    }
    const double hiT = cut + kTieEps;

    // Lane u takes over chunk u (positions 64 u .. 64 u + 63) as two words:
    // the blocks above the tie band (S+) and the tied ones.
    uint64_t above = 0, tied = 0;
    {
      double sv[E];
#pragma unroll
      for (int u = 0; u < E; ++u) sv[u] = row[u * 64 + lane];
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const bool ok = u < EP || u * 64 + lane < nB;
        const uint64_t a = __ballot(ok && sv[u] > hiT);
        const uint64_t t = __ballot(ok && fabs(sv[u] - cut) <= kTieEps);
        above = lane == u ? a : above;
        tied = lane == u ? t : tied;
      }
    }
    // the first `need` tied blocks in index order are kept
    const int need = k - wave_sum_i32(__popcll(above));
    const int nt = __popcll(tied);
    int left = min(max(need - (wave_incl_scan(nt) - nt), 0), nt);  // of this chunk
    uint64_t word = above | (left == nt ? tied : 0ull);
    if (left < nt)
      for (; left > 0; --left) {
        word |= tied & (0ull - tied);
        tied &= tied - 1ull;
      }
    // write the row: word u from lane u, or as bytes, chunk by chunk
    if (bits != nullptr) {
      const int nw = (nB + 63) / 64;
      if (lane < nw) bits[grow * nw + lane] = word;
    } else {
      uint8_t *mrow = mask + grow * nB;
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const uint64_t w = read_lane(word, u);
        const int jj = u * 64 + lane;
        if (u < EP || jj < nB) mrow[jj] = (uint8_t)((w >> lane) & 1ull);
      }
    }
  }
}

__global__ void fill_ones_kernel(uint8_t *p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 1;
}

}  // namespace

hipError_t launch_pool(View q, View k, int B, int H, int N, int d, int bs, double *qbar,
                       double *kbar, hipStream_t s) {
  const int nB = (N + bs - 1) / bs;
  dim3 grid(nB, B * H, 2);
  if (d == 128)
    hipLaunchKernelGGL(pool_kernel<128>, grid, dim3(256), 0, s, q, k, H, N, bs, nB, qbar, kbar);
  else
    hipLaunchKernelGGL(pool_kernel<64>, grid, dim3(256), 0, s, q, k, H, N, bs, nB, qbar, kbar);
  return hipGetLastError();
}

template <int D, int R, int W, bool MASS>
static hipError_t launch_select_dr(const double *qbar, const double *kbar, int BH, int nB,
                                   double sigma, double tau, uint8_t *mask, uint64_t *bits,
                                   hipStream_t s) {
  const int G = (nB + R - 1) / R * BH;
  dim3 grid((G + 7) / 8 * 8);
  const int need = (nB + 63) / 64;  // positions per lane
  // the logits (rows padded to 64 E), then the pooled rows or phase 2's
  // candidate buffers
  const auto lds_of = [](int e) { return ((size_t)R * 64 * e + (size_t)max(R * (D + 2), W * 128)) * sizeof(double); };
#define CARNATOR_SEL(EE)                                                                          \
  do {                                                                                            \
    const size_t lds = lds_of(EE);                                                                \
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&select_kernel<D, EE, R, W, MASS>), \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);     \
    if (e != hipSuccess) return e;                                                                \
    hipLaunchKernelGGL((select_kernel<D, EE, R, W, MASS>), grid, dim3(64 * W), lds, s, qbar, kbar, nB, \
                       sigma, tau, mask, bits, BH);                                               \
  } while (0)
  if constexpr (R == 16) {  // serves nB <= 1024
    if (need <= 1) CARNATOR_SEL(1);
    else if (need <= 2) CARNATOR_SEL(2);
    else if (need <= 3) CARNATOR_SEL(3);
    else if (need <= 4) CARNATOR_SEL(4);
    else if (need <= 6) CARNATOR_SEL(6);
    else if (need <= 8) CARNATOR_SEL(8);
    else if (need <= 10) CARNATOR_SEL(10);
    else if (need <= 12) CARNATOR_SEL(12);
    else if (need <= 16) CARNATOR_SEL(16);
    else return hipErrorInvalidValue;
  } else {  // longer rows
    if (need <= 24) CARNATOR_SEL(24);
    else if (need <= 32) CARNATOR_SEL(32);
    else return hipErrorInvalidValue;
  }
#undef CARNATOR_SEL
  return hipGetLastError();
}

// R query blocks per workgroup: their logits (rows padded to 64 E) and pooled
// rows (or the selection's candidate buffers, 1 KiB per wave) take
// 8 (64 E R + max(R (d + 2), 128 W)) bytes of LDS, within 160 KiB for R = 16 up
// to nB = 1024 and for R = 8 up to nB = 2048.  R = 16 fills the 16-row fp64
// MFMA tiles and halves the kbar re-reads; W = R waves, one row each: with one
// workgroup per CU (its LDS) the waves of that workgroup are all there is to
// hide the phases' latencies (at nB = 591 244 us with 8 waves of two rows
// each, 215 us with 16 waves).
template <int D>
static hipError_t launch_select_d(const double *qbar, const double *kbar, int BH, int nB,
                                  double sigma, double tau, uint8_t *mask, uint64_t *bits,
                                  hipStream_t s) {
  if (nB <= 1024) return launch_select_dr<D, 16, 16, false>(qbar, kbar, BH, nB, sigma, tau, mask, bits, s);
  return launch_select_dr<D, 8, 8, false>(qbar, kbar, BH, nB, sigma, tau, mask, bits, s);
}

hipError_t launch_select(const double *qbar, const double *kbar, int BH, int nB, int d,
                         double sigma, double tau, uint8_t *mask, uint64_t *bits,
                         hipStream_t s) {
  if (d == 128) return launch_select_d<128>(qbar, kbar, BH, nB, sigma, tau, mask, bits, s);
  return launch_select_d<64>(qbar, kbar, BH, nB, sigma, tau, mask, bits, s);
}

hipError_t launch_select_mass(const double *mass, int BH, int nB, double tau, uint8_t *mask,
                              uint64_t *bits, hipStream_t s) {
  // the pooled-row area of the LDS layout is not used: the smallest D
  if (nB <= 1024) return launch_select_dr<64, 16, 16, true>(mass, nullptr, BH, nB, 1.0, tau, mask, bits, s);
  return launch_select_dr<64, 8, 8, true>(mass, nullptr, BH, nB, 1.0, tau, mask, bits, s);
}

hipError_t launch_fill_ones(uint8_t *p, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_ones_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace carnator
