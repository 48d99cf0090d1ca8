// Window scoring, Eq. (4), with a unit's keys resident in LDS and every
// weight in fp32: the kernel for windows whose keys fit (bf16 d = 64 up to
// 1152 keys, bf16 d = 128 and fp32 d = 64 up to 512, fp32 d = 128 up to 256).
//
// A workgroup of 8 waves copies the unit's N keys into LDS once and takes its
// query rows 32 per wave at a time.  KS waves share a set of rows and split
// the keys, so that a wave's 32 rows x (NTW*16) keys of weights fit in
// registers (NTW*8 of the 256 that two waves per SIMD leave each).  Every
// logit is formed and exponentiated once; the weights e = 2^(x - m) wait in
// registers, in fp32, for the row sums, and then each is multiplied by its
// row's 1/L and added to its key's column sum: one more multiply-add instead
// of a second sweep's matrix product, multiply-add, exponential and add.  The
// reference m is the maximum over the wave's own first 16 keys; the waves
// that share rows exchange (m, L) once per 32 rows and each folds
// 2^(m - M) into its weights.
//
// Bound by the vector instructions (four per logit, one an exponential, and
// a third as many again for the row sums, exchanges and addresses; the vector
// port is two thirds busy); in fp32 by the matrix instructions, which the
// single sweep halves.  More waves do not help: 16 waves of 16 rows (four per
// SIMD, 128 registers) took 4 % to 40 % longer, the work per 16-row step being
// the same for half the logits.  Against two sweeps, scoring alone: 21 x 6
// layers x 8 heads, 701/33 keys, d = 64, two heads a group 703 -> 337 us; 64
// units x 8 of 512 keys, d = 128, four heads 348 -> 199 us; fp32 d = 64, 64 x 8
// units of 512 keys 579 -> 330 us.
#include <type_traits>

#include "kara_lds.h"
#include "kara_score.h"
#include "kara_score_dpp.h"

namespace kara {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegInf = -__builtin_huge_valf();
constexpr float kMaxFloor = -1e30f;   // finite, so that 2^(-inf - m) is 0 and not NaN
// Row sums past this run again from the exact maximum.  At most 2^60, so that
// 1 / sum and a weight's share stay normal numbers (v_rcp_f32 and v_exp_f32
// flush those below 2^-126) and the sum of four key parts cannot overflow; and
// where two parts' references differ by more than 2^126, which flushes the
// lower part's factor, its weights are below 2^-66 of the row's sum.
constexpr float kSumMax = 0x1p60f;

template <int DT, int D, int NTW, int KS>
struct RCfg {
  static constexpr int kRowBytes = D * (DT == KARA_BF16 ? 2 : 4);
  static constexpr int kCPR = kRowBytes / 16;       // 16-byte chunks per row
  static constexpr int kKC = kCPR / 4;              // chunks per lane of an operand
  static constexpr int kKeys = KS * NTW * 16;
  static constexpr int kCopies = kKeys * kRowBytes / (kThreads * 16);
  static constexpr int kRG = kWaves / KS;           // row groups of 32
  static constexpr int kRows = 32 * kRG;            // rows per iteration
  static constexpr int kNT4 = (NTW + 3) / 4 * 4;
  static_assert(kCopies * kThreads * 16 == kKeys * kRowBytes, "whole copies");
  static_assert(kKeys * kRowBytes + kKeys * 4 + 2 * KS * kRows * 8 + 64 <= 160 * 1024, "LDS budget");
  static_assert(kWaves * kNT4 * 16 * 4 <= kKeys * kRowBytes, "the column sums reuse the keys' LDS");
  // XOR swizzle of a row's chunks, conflict-free for 16 rows x 16 bytes per
  // lane group (the row's two low bits moved to the top)
  static __device__ __forceinline__ int swz(int row) {
    if constexpr (kCPR == 8) return ((row & 3) << 1) | ((row >> 2) & 1);
    return ((row & 3) << 2) | ((row >> 2) & 3);
  }
};

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// lane I's value, in every lane of its 16-lane row
template <int I>
__device__ __forceinline__ float row_bcast(float v) {
  return dpp<0x150 + I>(v);
}

template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

template <int DT, int D, int NTW, int KS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void score_res_kernel(ScoreArgs a) {
  using C = RCfg<DT, D, NTW, KS>;
  constexpr int KC = C::kKC, RB = C::kRowBytes;
  __shared__ __attribute__((aligned(16))) char kbuf[C::kKeys * RB];
  __shared__ uint32_t key_off[C::kKeys];          // 16-byte units from the pool; past N: key 0
  __shared__ float2 xch[2][KS][C::kRows];         // (m, L) of each key part's rows
  __shared__ __attribute__((aligned(16))) int sbad[2][kWaves];

  const Geom& g = a.g;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gq = lane >> 4, li = lane & 15;
  const int kq = wave % KS, rg = wave / KS;

  // the row splits of one unit run together on one XCD (its L2 keeps the keys)
  int64_t bid = blockIdx.x;
  if ((a.n_blocks & 7) == 0) bid = (bid & 7) * (a.n_blocks >> 3) + (bid >> 3);
  const int64_t u = bid / a.n_splits;
  const int split = (int)(bid % a.n_splits);
  const int h = (int)(u % g.Hkv);
  const int tw = (int)((u / g.Hkv) % ((int64_t)g.n_trig * g.n_win));
  const int t = tw / g.n_win;
  const int wi = tw - t * g.n_win;
  const int l = (int)(u / ((int64_t)g.Hkv * g.n_trig * g.n_win));
  const int N = g.N;
  float* out = a.n_splits == 1 ? a.scores + u * (int64_t)N : a.partials + (u * a.n_splits + split) * (int64_t)N;
  if (a.status[t] != 0) {
    for (int j = tid; j < N; j += kThreads) out[j] = 0.f;
    return;
  }
  const int s = a.trig[t];
  const int p0 = a.win_start[s] + wi * N;
  const char* kpool = (const char*)a.k.p[l];
  const char* qunit = a.q + (((int64_t)l * g.n_trig + t) * g.n_win + wi) * g.Wq * g.Hq * (int64_t)RB;
  const int r0 = split * a.rows_split;
  const int r1 = min(g.G * g.Wq, r0 + a.rows_split);
  const float c = g.scale * kLog2e;

  // ---- the unit's keys into LDS ----
  {
    const int32_t* row_pages = a.bt + (int64_t)s * g.max_blocks;
    for (int j = tid; j < C::kKeys; j += kThreads) {
      const int pos = p0 + (j < N ? j : 0);
      const int b = pos / g.bs;
      const uint64_t row = ((uint64_t)row_pages[b] * g.Hkv + h) * g.bs + (pos - b * g.bs);
      key_off[j] = (uint32_t)(row * C::kCPR);
    }
  }
  lds_barrier();
#pragma unroll
  for (int r = 0; r < C::kCopies; ++r) {
    const int slot = r * kThreads + tid;
    const int kr = slot / C::kCPR;
    const int chunk = (slot % C::kCPR) ^ C::swz(kr);
    copy16(kpool + ((uint64_t)key_off[kr] + chunk) * 16, kbuf + (r * kWaves + wave) * 1024);
  }

  // This wave's 32 query rows of an iteration: row r = w*G + gi is position w,
  // query head h*G + gi.  qoff: the rows' offsets (16-byte units) and qgi
  // their gi, stepped from one iteration to the next without a division.
  // Rows past r1 repeat row r0 and weigh nothing.
  uint32_t qoff[2], qoff0;
  int qgi[2];
  const int step_w = C::kRows / g.G, step_gi = C::kRows - step_w * g.G;
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const int r = r0 + rg * 32 + rt * 16 + li;
    const int w = r / g.G;
    qgi[rt] = r - w * g.G;
    qoff[rt] = (uint32_t)(w * g.Hq + h * g.G + qgi[rt]) * C::kCPR;
  }
  qoff0 = (uint32_t)(r0 / g.G * g.Hq + h * g.G + r0 % g.G) * C::kCPR;
  uint4 qa[2][KC];
  auto load_q = [&](int row, const uint32_t (&off)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const uint4* src = (const uint4*)(qunit + (uint64_t)(row + rt * 16 + li < r1 ? off[rt] : qoff0) * 16) + gq * KC;
#pragma unroll
      for (int ks = 0; ks < KC; ++ks) qa[rt][ks] = src[ks];
    }
  };
  auto step_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      qoff[rt] += (uint32_t)(step_w * g.Hq + step_gi) * C::kCPR;
      qgi[rt] += step_gi;
      if (qgi[rt] >= g.G) {
        qgi[rt] -= g.G;
        qoff[rt] += (uint32_t)(g.Hq - g.G) * C::kCPR;
      }
    }
  };
  load_q(r0 + rg * 32, qoff);
  wait_vm<0>();
  lds_barrier();

  int koff[KC];
#pragma unroll
  for (int ks = 0; ks < KC; ++ks) koff[ks] = li * RB + (((gq * KC + ks) ^ C::swz(li)) * 16);
  const char* kpart = kbuf + kq * NTW * 16 * RB;
  const int key0 = kq * NTW * 16;

  // key operands, read kAhead tiles ahead (two where the registers allow)
  constexpr int kAhead = KC == 2 ? 2 : 1;
  uint4 kb[kAhead + 1][KC];
  auto kread = [&](int tile, int b) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) kb[b][ks] = *(const uint4*)(kpart + tile * 16 * RB + koff[ks]);
  };
  // logits of 16 rows x 16 keys: rows 4gq + q, key li, added to z
  auto dot = [&](const uint4 (&q)[KC], const uint4 (&k)[KC], floatx4 acc) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) {
      if constexpr (DT == KARA_BF16) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, q[ks]), __builtin_bit_cast(bf16x8, k[ks]),
                                                      acc, 0, 0, 0);
      } else {
        const floatx4 x = __builtin_bit_cast(floatx4, q[ks]), y = __builtin_bit_cast(floatx4, k[ks]);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], acc, 0, 0, 0);
      }
    }
    return acc;
  };

  floatx4 e[NTW][2];         // logits, then weights: [tile][row tile]
  float m[8], L[8];          // rows (i >> 2)*16 + 4gq + (i & 3)
  float m_own = kMaxFloor;   // row li & 7's reference
  float colacc[C::kNT4];
#pragma unroll
  for (int j = 0; j < C::kNT4; ++j) colacc[j] = 0.f;

  // the logits start from zq: 0, and -inf for keys past N (weight 0).  The
  // keys past N are a tail of the tiles, so zq changes at most twice a sweep.
  // (n_keys: N, opaque to the compiler, which would otherwise hoist every
  // tile's zq out of the row loop into registers of its own)
  floatx4 zq;
  int n_keys = N;
  auto form = [&](int tile, int b) __attribute__((always_inline)) {
    if (key0 + tile * 16 + 16 > n_keys) {
      const float z = key0 + tile * 16 + li >= n_keys ? kNegInf : 0.f;
      zq = floatx4{z, z, z, z};
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) e[tile][rt] = dot(qa[rt], kb[b], zq);
  };
  auto share_max = [&](float (&mx)[8]) __attribute__((always_inline)) {
    m_own = fmaxf(reduce_scatter8<true>(mx, li) * c, kMaxFloor);
    static_for<0, 8>([&](auto i) __attribute__((always_inline)) { m[decltype(i)::value] = row_bcast<decltype(i)::value>(m_own); });
  };
  auto vexp = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float v = __builtin_amdgcn_exp2f(fmaf(e[tile][rt][q], c, -m[rt * 4 + q]));
        e[tile][rt][q] = v;
        L[rt * 4 + q] += v;
      }
  };
  // One pass over the wave's tiles: logits of tile it beside the weights of
  // tile it-1, the next tile's operands read ahead.  Tiles past N weigh
  // nothing but are worked like the others (a second, masked copy of the pass
  // or branches around the tiles cost registers that spill).
  auto sweep = [&](bool m_given) __attribute__((always_inline)) {
    asm volatile("" : "+s"(n_keys));
    zq = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) L[i] = 0.f;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) kread(i, i);
    static_for<0, NTW>([&](auto it_c) __attribute__((always_inline)) {
      constexpr int it = decltype(it_c)::value;
      if constexpr (it + kAhead < NTW) kread(it + kAhead, (it + kAhead) % (kAhead + 1));
      form(it, it % (kAhead + 1));
      if constexpr (it == 0) {
        if (!m_given) {
          float mx[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) mx[i] = e[0][i >> 2][i & 3];
          share_max(mx);
        }
      } else {
        vexp(it - 1);
      }

    });
    vexp(NTW - 1);
  };
  // the exact row maxima over this wave's keys
  auto exact_max = [&]() {
    float mx[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) mx[i] = kNegInf;
#pragma unroll 1
    for (int tile = 0; tile < NTW; ++tile) {
      kread(tile, 0);
      asm volatile("" : "+s"(n_keys));
      const float z = key0 + tile * 16 + li >= n_keys ? kNegInf : 0.f;
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const floatx4 x = dot(qa[rt], kb[0], floatx4{z, z, z, z});
#pragma unroll
        for (int q = 0; q < 4; ++q) mx[rt * 4 + q] = fmaxf(mx[rt * 4 + q], x[q]);
      }
    }
    share_max(mx);
  };

  int par = 0;
  const int own_row = ((li >> 2) & 1) * 16 + 4 * gq + (li & 3);   // of the wave's 32
  const int n_it = (r1 - r0 + C::kRows - 1) / C::kRows;
  for (int it = 0; it < n_it; ++it) {
    const int row = r0 + it * C::kRows + rg * 32;
    if (KS == 1 && row >= r1) break;   // (with shared rows every wave meets the barriers)

    const uint32_t qcur[2] = {qoff[0], qoff[1]};
    step_q();
    float w_own = 0.f;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
      sweep(pass != 0);
      // the next rows' queries arrive behind the exchange and the column sums
      if (it + 1 < n_it) load_q(row + C::kRows, qoff);
      const float l_own = reduce_scatter8<false>(L, li);
      // a logit 60 log2-units above the reference: once more, from the exact
      // maximum
      bool bad = __builtin_amdgcn_ballot_w64(!(l_own <= kSumMax)) != 0;
      float m_all = m_own, l_all = l_own;
      if constexpr (KS > 1) {
        if (li < 8) xch[par][kq][rg * 32 + own_row] = float2{m_own, l_own};
        if (lane == 0) sbad[par][wave] = bad;
        lds_barrier();
        const int4 f0 = *(const int4*)&sbad[par][0], f1 = *(const int4*)&sbad[par][4];
        bad = __builtin_amdgcn_readfirstlane(f0.x | f0.y | f0.z | f0.w | f1.x | f1.y | f1.z | f1.w) != 0;
        float2 v[KS];
#pragma unroll
        for (int x = 0; x < KS; ++x) v[x] = xch[par][x][rg * 32 + own_row];
        m_all = v[0].x;
#pragma unroll
        for (int x = 1; x < KS; ++x) m_all = fmaxf(m_all, v[x].x);
        l_all = 0.f;
#pragma unroll
        for (int x = 0; x < KS; ++x) l_all += v[x].y * __builtin_amdgcn_exp2f(v[x].x - m_all);
        par ^= 1;
      }
      if (!bad || pass == 1) {
        w_own = __builtin_amdgcn_rcpf(l_all);
        if constexpr (KS > 1) w_own *= __builtin_amdgcn_exp2f(m_own - m_all);
        break;
      }
      load_q(row, qcur);
      exact_max();
    }
    if (row + own_row >= r1) w_own = 0.f;
    float w[8];
    static_for<0, 8>([&](auto i) __attribute__((always_inline)) { w[decltype(i)::value] = row_bcast<decltype(i)::value>(w_own); });
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int tile = 0; tile < NTW; ++tile) colacc[tile] = fmaf(e[tile][i >> 2][i & 3], w[i], colacc[tile]);
  }

  // ---- column sums over the four lane groups, then the row groups ----
  lds_barrier();   // every wave is done with the keys
  float* col = (float*)kbuf + wave * C::kNT4 * 16;
#pragma unroll
  for (int j = 0; j < C::kNT4; j += 4) {
    const float x0 = swap32_add(colacc[j], colacc[j + 2]);
    const float x1 = swap32_add(colacc[j + 1], colacc[j + 3]);
    col[(j + gq) * 16 + li] = swap16_add(x0, x1);   // lane group gq: tile j + gq
  }
  lds_barrier();
  for (int j = tid; j < N; j += kThreads) {
    const int part = j / (NTW * 16), x = j - part * NTW * 16;
    float v = 0.f;
#pragma unroll
    for (int r = 0; r < C::kRG; ++r) v += ((const float*)kbuf)[(r * KS + part) * C::kNT4 * 16 + x];
    out[j] = v;
  }
}

// (NTW, KS) instance: the fewest key parts whose tiles hold the keys and
// whose weights and operands fit the registers (512-byte rows: 8 tiles)
struct ResShape {
  int ntw, ks;
};
ResShape res_shape(const Geom& g) {
  const int T = (g.N + 15) / 16;
  const bool wide = g.d * g.esize == 512;
  if (T <= (wide ? 8 : 16)) return {(T + 3) / 4 * 4, 1};
  if (wide) return {8, 2};
  if (T <= 32) return {T <= 20 ? 10 : T <= 24 ? 12 : T <= 28 ? 14 : 16, 2};
  return {T <= 40 ? 10 : T <= 48 ? 12 : T <= 56 ? 14 : T <= 64 ? 16 : 18, 4};
}

template <int DT, int D>
hipError_t launch_d(const ScoreArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)a.n_blocks), block(kThreads);
  const ResShape r = res_shape(a.g);
#define KARA_RES(NTW, KS) \
  if (r.ntw == NTW && r.ks == KS) hipLaunchKernelGGL((score_res_kernel<DT, D, NTW, KS>), grid, block, 0, stream, a)
  KARA_RES(4, 1);
  else KARA_RES(8, 1);
  if constexpr (D * (DT == KARA_BF16 ? 2 : 4) == 512) {
    KARA_RES(8, 2);
  } else {
    KARA_RES(12, 1);
    else KARA_RES(16, 1);
    else KARA_RES(10, 2);
    else KARA_RES(12, 2);
    else KARA_RES(14, 2);
    else KARA_RES(16, 2);
  }
  if constexpr (D * (DT == KARA_BF16 ? 2 : 4) == 128) {
    KARA_RES(10, 4);
    else KARA_RES(12, 4);
    else KARA_RES(14, 4);
    else KARA_RES(16, 4);
    else KARA_RES(18, 4);
  }
#undef KARA_RES
  return hipGetLastError();
}

}  // namespace

bool resident_fits(const Geom& g) {
  const int row = g.d * g.esize;
  return g.N <= (row == 128 ? 1152 : row == 256 ? 512 : 256);
}

int resident_rows(const Geom& g, int64_t n_units) {
  const int64_t rows = (int64_t)g.G * g.Wq;
  const int64_t chunks = (rows + 31) / 32;
  const ResShape r = res_shape(g);
  const int rg = kWaves / r.ks;
  // Time of a launch with s splits per unit: rounds of one workgroup per CU,
  // each its start (the key copies and column sums, about `fixed`) and its
  // iterations, in units of about 0.27 us (measured at d = 64).  Split only
  // while the launch stays within kSplitMaxWgs.
  const int64_t per_it = g.dtype == KARA_BF16 ? 2 + r.ntw : 2 + r.ntw * (g.d / 16), fixed = 20, sum_launch = 5;
  int64_t best = chunks, best_t = -1;
  for (int64_t s = 1; s <= chunks && (s == 1 || s * n_units <= kSplitMaxWgs); ++s) {
    const int64_t c = (chunks + s - 1) / s;
    const int64_t used = (chunks + c - 1) / c;
    // (a step's time is that of two waves on a SIMD; of one, half)
    const int64_t waves = (c < rg ? c : rg) * r.ks;
    const int64_t step = waves > 4 ? per_it : (per_it + 1) / 2;
    const int64_t t = (used * n_units + kScoreCUs - 1) / kScoreCUs * (fixed + (c + rg - 1) / rg * step) +
                      (used > 1 ? sum_launch : 0);
    if (best_t < 0 || t < best_t) best_t = t, best = c;
  }
  return (int)(best * 32);
}

hipError_t launch_score_resident(const ScoreArgs& a, hipStream_t stream) {
  if (a.g.dtype == KARA_BF16)
    return a.g.d == 128 ? launch_d<KARA_BF16, 128>(a, stream) : launch_d<KARA_BF16, 64>(a, stream);
  return a.g.d == 128 ? launch_d<KARA_F32, 128>(a, stream) : launch_d<KARA_F32, 64>(a, stream);
}

}  // namespace kara
