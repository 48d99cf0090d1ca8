// Decoding-side helpers for long-running workloads (kara_harness.h): token
// append into the paged cache, and split-key decode attention of one query
// per (layer, sequence, query head) over the compressed cache.  Not part of
// the compression step; same paged layout.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kara_harness.h"
#include "kara_internal.h"

namespace kara {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegInf = -__builtin_huge_valf();
// Lower end of a running maximum: finite, so that a logit of -inf weighs 0 and
// not 2^(-inf + inf) where a wave has met no other yet; below any finite logit.
constexpr float kMaxFloor = -3.402823466e38f;
constexpr int kSplitKeys = KARA_HARNESS_SPLIT_KEYS;
constexpr int kDecWgTarget = 4096;   // workgroups a launch keeps when its splits grow (16 per CU)

// ---------------------------------------------------------------- append

constexpr int kAppendThreads = 256;
constexpr int kAppendUnroll = 8;       // 16-byte pieces per thread
// Appends of up to this many tokens check their sequence in the copying
// workgroups and in the committing one: a launch less (8 sequences, one token:
// a decoding step 43 -> 39 us of host time).  Longer ones have a table row to
// read per check and keep it in a kernel of its own.
constexpr int kAppendFusedTokens = 32;

// Status of listed sequence j, by all threads of a workgroup; the same value
// in each.
__device__ int append_status(const Geom& g, int n, const int32_t* __restrict__ seqs, int n_new,
                             const int32_t* __restrict__ bt, const int32_t* __restrict__ seq_lens, int j) {
  const int s = seqs[j];
  if (s < 0 || s >= g.n_seqs) return KARA_SEQ_BAD_INDEX;
  int dup = 0;
  for (int o = threadIdx.x; o < n; o += kAppendThreads) dup |= o != j && seqs[o] == s;
  const int64_t len = seq_lens[s];
  const int64_t new_len = len + n_new;
  const bool fits = len >= 0 && new_len <= (int64_t)g.max_blocks * g.bs;
  int bad = 0;
  if (fits) {
    const int32_t* row = bt + (int64_t)s * g.max_blocks;
    for (int b = (int)(len / g.bs) + threadIdx.x; b < (int)((new_len + g.bs - 1) / g.bs); b += kAppendThreads) {
      const int pg = row[b];
      bad |= pg < 0 || pg >= g.num_pages;
    }
  }
  const int any = __syncthreads_or(dup | (bad << 1));
  // (the two flags come back as one "any": told apart by a second vote only
  // when something is wrong)
  if (!any) return fits ? KARA_SEQ_OK : KARA_SEQ_BAD_WINDOW;
  const int d = __syncthreads_or(dup) ? KARA_SEQ_DUP_TRIGGER : 0;
  const int p = __syncthreads_or(bad) ? KARA_SEQ_BAD_PAGE : 0;
  return d | p | (fits ? 0 : KARA_SEQ_BAD_WINDOW);
}

__global__ __launch_bounds__(kAppendThreads) void append_check_kernel(Geom g, int n, const int32_t* __restrict__ seqs,
                                                                      int n_new, const int32_t* __restrict__ bt,
                                                                      const int32_t* __restrict__ seq_lens,
                                                                      int32_t* __restrict__ status) {
  const int st = append_status(g, n, seqs, n_new, bt, seq_lens, blockIdx.x);
  if (threadIdx.x == 0) status[blockIdx.x] = st;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One workgroup per `toks` tokens of a listed sequence: grid (sequences x token
// chunks, layer, K|V), kAppendUnroll pieces of 16 bytes per thread, all loaded
// before the first is stored.  The new rows are read once (nontemporal); the
// pool rows are stored to stay cached, as scoring reads the keys next (stored
// nontemporally, the append of 4 x 4 layers of 16,893 tokens gained 30 us and
// the scoring after it lost 95 us).  128 sequences x 4 layers of 1,280 tokens
// (5.4 GB): 1093 us with one piece per thread, 1006 us so.
template <bool CHECK>
__global__ __launch_bounds__(kAppendThreads) void append_kernel(Geom g, int n, const int32_t* __restrict__ seqs, int n_new,
                                                                int toks, int chunks, const char* __restrict__ k_new,
                                                                const char* __restrict__ v_new, PoolPtrs kp, PoolPtrs vp,
                                                                const int32_t* __restrict__ bt,
                                                                const int32_t* __restrict__ seq_lens,
                                                                const int32_t* __restrict__ status) {
  const int j = blockIdx.x / chunks;
  const int tok0 = (blockIdx.x - j * chunks) * toks;
  const int l = blockIdx.y;
  const int kv = blockIdx.z;
  if constexpr (CHECK) {
    if (append_status(g, n, seqs, n_new, bt, seq_lens, j) != KARA_SEQ_OK) return;
  } else {
    if (status[j] != 0) return;
  }
  const int s = seqs[j];
  const int row_bytes = g.d * g.esize;
  const int cpr = row_bytes / 16;
  const int per_tok = g.Hkv * cpr;              // pieces of one token
  const int count = min(toks, n_new - tok0) * per_tok;
  const int pos0 = seq_lens[s] + tok0;
  const int32_t* row_pages = bt + (int64_t)s * g.max_blocks;
  const char* src = (kv ? v_new : k_new) + (((int64_t)l * n + j) * n_new + tok0) * per_tok * 16;
  char* pool = (char*)(kv ? vp.p[l] : kp.p[l]);
  for (int i0 = threadIdx.x; i0 < count; i0 += kAppendThreads * kAppendUnroll) {
    u32x4 v[kAppendUnroll];
    int64_t dst[kAppendUnroll];
#pragma unroll
    for (int k = 0; k < kAppendUnroll; ++k) {
      const int i = i0 + k * kAppendThreads;
      if (i < count) {
        v[k] = __builtin_nontemporal_load((const u32x4*)(src + (int64_t)i * 16));
        const int tok = i / per_tok, x = i - tok * per_tok;
        const int h = x / cpr, c = x - h * cpr;
        const int pos = pos0 + tok, b = pos / g.bs;
        dst[k] = (((int64_t)row_pages[b] * g.Hkv + h) * g.bs + (pos - b * g.bs)) * row_bytes + c * 16;
      }
    }
#pragma unroll
    for (int k = 0; k < kAppendUnroll; ++k)
      if (i0 + k * kAppendThreads < count) *(u32x4*)(pool + dst[k]) = v[k];
  }
}

// CHECK: a workgroup per listed sequence, which finds and writes its status
// and waits for every thread to have read the length; else a thread each.
// (Distinct sequences: a duplicate is flagged and its length left alone, so no
// workgroup's check sees another's new length.)
template <bool CHECK>
__global__ __launch_bounds__(kAppendThreads) void append_commit_kernel(Geom g, int n, const int32_t* __restrict__ seqs,
                                                                       int n_new, const int32_t* __restrict__ bt,
                                                                       int32_t* __restrict__ seq_lens,
                                                                       int32_t* __restrict__ status) {
  if constexpr (CHECK) {
    const int j = blockIdx.x;
    const int st = append_status(g, n, seqs, n_new, bt, seq_lens, j);
    __syncthreads();
    if (threadIdx.x == 0) {
      status[j] = st;
      if (st == KARA_SEQ_OK) seq_lens[seqs[j]] += n_new;
    }
  } else {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n && status[j] == 0) seq_lens[seqs[j]] += n_new;
  }
}

// ---------------------------------------------------------------- decode

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / 64;
constexpr int kDecMaxSplit = 1024;   // keys per split, at most

// Geometry of one instance: element type DT, head dim D, GP query heads.
template <int DT, int D, int GP>
struct DCfg {
  static constexpr int kES = DT == KARA_BF16 ? 2 : 4;
  static constexpr int kRowBytes = D * kES;
  // 16-key tiles per block, and buffers of its keys: a block of 16 rows of 256
  // bytes or more leaves registers for a third wave per SIMD (G <= 5), 4 % on
  // launches of a few workgroups per CU against 32; half as long rows take 32.
  static constexpr int kTB = DT == KARA_BF16 && D == 64 ? 2 : 1;
  static constexpr int kKBuf = DT == KARA_F32 && D == 128 && GP == 16 ? 1 : 2;
  static constexpr int kBlock = 16 * kTB;                  // keys per block
  static constexpr int kKC = kRowBytes / 64;               // 16-byte chunks of a key row per lane
  static constexpr int kE = D / 16;                        // output columns per lane
  static constexpr int kVBytes = kE * kES;                 // a lane's bytes of a value row: 8, 16 or 32
  static constexpr int kVW = kVBytes / 4;
};

// p of lane `I` of the 16-lane row, in every lane of the row
template <int I>
__device__ __forceinline__ float row_bcast(float p) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, p), 0x150 + I, 0xf, 0xf, false));
}

template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// sums over the four 16-lane rows, of two values at once: row 0/1 lanes end
// with a's sum, row 2/3 lanes with b's
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

// One workgroup of four waves per (layer, sequence, KV head, split of
// split_keys keys): for the KV head's G query heads, the split's maximum m,
// exponential sum l and unnormalised output o, in log2 units and fp32.
//
// Bound by the K and V bytes.  The rows' pool offsets are formed once per
// split into LDS, so no load waits on the block table, and the waves take
// the split's 16-key blocks (32 for bf16 at d = 64) in turn, each with the
// next block's keys and this block's values in flight while it works: 8 to 12
// KB per wave.  S^T = K Q^T on the matrix cores puts query li of lane (gq, li)
// against keys 16t + 4gq + r, and the value rows are loaded so that row gq of
// the wave holds exactly those keys: a weight reaches the 16 lanes that hold
// its key's columns by one DPP row broadcast, and P V runs in fp32 on the
// vector units (about a quarter of the time the bytes take), with no LDS
// exchange.  The reference m is raised only past a headroom of 2^8.
// 128 sequences x 4 layers of 8K tokens, 40/8 heads, bf16 (15.9 GB): 8.0 ms
// with one wave per 256 keys and loads that waited on the table, 2.8 ms here
// (5.6 TB/s); 8 sequences of 300-4000 tokens, one layer: 138 -> 21 us.
//
// One split in the launch, or a sequence that ends inside its first: out
// is written here.  Otherwise a record per (layer, j, query head, split) in
// ws, strided as n_splits: m, l, o[d].
template <int DT, int D, int GP>
__global__ __launch_bounds__(kDecThreads, 2) void decode_split_kernel(
    Geom g, int n, const int32_t* __restrict__ seqs, const char* __restrict__ q, PoolPtrs kp, PoolPtrs vp,
    const int32_t* __restrict__ bt, const int32_t* __restrict__ seq_lens, int max_len, int split_keys, int n_splits,
    float* __restrict__ ws, float* __restrict__ out) {
  using C = DCfg<DT, D, GP>;
  constexpr int TB = C::kTB, KC = C::kKC, E = C::kE, VW = C::kVW;
  __shared__ __attribute__((aligned(16))) uint32_t row_of[kDecMaxSplit];   // pool row of the split's keys
  __shared__ __attribute__((aligned(16))) float red_o[kDecWaves][GP][D];
  __shared__ float red_m[kDecWaves][16], red_l[kDecWaves][16];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gq = lane >> 4, li = lane & 15;
  const int split = blockIdx.x % n_splits;
  const int64_t rest = blockIdx.x / n_splits;
  const int h = (int)(rest % g.Hkv);
  const int j = (int)((rest / g.Hkv) % n);
  const int l = (int)(rest / ((int64_t)g.Hkv * n));
  const int s = seqs[j];
  const int G = g.G;
  const int64_t orow = ((int64_t)l * n + j) * g.Hq + h * G;   // first query head's output row
  const int len = s >= 0 && s < g.n_seqs ? seq_lens[s] : 0;
  const int k0 = split * split_keys;
  if (len <= 0 || len > max_len || k0 >= len) {
    // no keys: zero rows where no combine kernel follows
    if (n_splits == 1)
      for (int i = tid; i < G * D; i += kDecThreads) out[orow * D + i] = 0.f;
    return;
  }
  const int nk = min(len - k0, split_keys);                   // keys of this split
  const float c = g.scale * kLog2e;

  {
    const int32_t* row_pages = bt + (int64_t)s * g.max_blocks;
    // (padding keys of the last block repeat its last key, with no weight)
    const int npad = (nk + C::kBlock - 1) / C::kBlock * C::kBlock;
    for (int i = tid; i < npad; i += kDecThreads) {
      const int pos = k0 + min(i, nk - 1);
      const int b = pos / g.bs;
      row_of[i] = (uint32_t)(((int64_t)row_pages[b] * g.Hkv + h) * g.bs + (pos - b * g.bs));
    }
  }
  // lane (gq, li): 16-byte chunks gq + 4x of row li (any assignment of chunks
  // to lane groups gives the same dot product; this one makes each load
  // instruction read 64 contiguous bytes of a row)
  uint4 qa[KC];
  {
    const uint4* src = (const uint4*)(q + (orow + (li < G ? li : 0)) * C::kRowBytes) + gq;
#pragma unroll
    for (int x = 0; x < KC; ++x) qa[x] = li < G ? src[4 * x] : uint4{0, 0, 0, 0};
  }
  __syncthreads();

  const char* kbase = (const char*)kp.p[l] + gq * 16;
  const char* vbase = (const char*)vp.p[l] + li * (C::kVBytes < 16 ? C::kVBytes : 16);
  uint4 kb[C::kKBuf][TB][KC];
  uint32_t vb[TB][4][VW];
  auto load_k = [&](int blk, int b) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const char* src = kbase + (uint64_t)row_of[blk * C::kBlock + t * 16 + li] * C::kRowBytes;
#pragma unroll
      for (int x = 0; x < KC; ++x) kb[b][t][x] = *(const uint4*)(src + x * 64);
    }
  };
  auto load_v = [&](int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const uint4 rows = *(const uint4*)&row_of[blk * C::kBlock + t * 16 + 4 * gq];
      const uint32_t rw[4] = {rows.x, rows.y, rows.z, rows.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const char* src = vbase + (uint64_t)rw[r] * C::kRowBytes;
        if constexpr (VW == 2) {
          const uint2 v = *(const uint2*)src;
          vb[t][r][0] = v.x, vb[t][r][1] = v.y;
        } else {
          // (32 bytes per lane: columns 4li.. and 64 + 4li..)
#pragma unroll
          for (int y = 0; y < VW / 4; ++y) {
            const uint4 v = *(const uint4*)(src + y * 256);
            vb[t][r][4 * y] = v.x, vb[t][r][4 * y + 1] = v.y, vb[t][r][4 * y + 2] = v.z, vb[t][r][4 * y + 3] = v.w;
          }
        }
      }
    }
  };

  float m = kMaxFloor, lsum = 0.f;   // query li's reference, and this lane's part of its sum
  float o[GP][E];                  // query i, this lane's columns, over its row's keys
#pragma unroll
  for (int i = 0; i < GP; ++i)
#pragma unroll
    for (int e = 0; e < E; ++e) o[i][e] = 0.f;

  const int nblk = (nk + C::kBlock - 1) / C::kBlock;
  auto work = [&](int blk, int b) __attribute__((always_inline)) {
    floatx4 sv[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = 0; x < KC; ++x) {
        if constexpr (DT == KARA_BF16) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kb[b][t][x]),
                                                        __builtin_bit_cast(bf16x8, qa[x]), acc, 0, 0, 0);
        } else {
          const floatx4 ka = __builtin_bit_cast(floatx4, kb[b][t][x]), qx = __builtin_bit_cast(floatx4, qa[x]);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[i], qx[i], acc, 0, 0, 0);
        }
      }
      sv[t] = acc;
    }
    // Wait states between the last product and the first read of its result:
    // the branch below comes between, and past it the compiler gave 1 where 8
    // (bf16) or 10 (fp32) are needed, so with three waves per SIMD the maximum
    // read what the registers held before.  12 cycles per block.
    asm volatile("s_nop 7\n\ts_nop 3" : "+v"(sv[TB - 1]));
    const int left = nk - blk * C::kBlock;
    if (left < C::kBlock) {
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t * 16 + 4 * gq + r >= left) {
            sv[t][r] = kNegInf;
#pragma unroll
            for (int x = 0; x < VW; ++x) vb[t][r][x] = 0;   // its weight is 0, its value must be finite
          }
    }
    float mx = sv[0][0];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sv[t][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c;
    if (__ballot(mx > m + 8.f) != 0ull) {
      const float mn = fmaxf(m, mx);
      const float f = __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      lsum *= f;
      static_for<0, GP>([&](auto i) __attribute__((always_inline)) {
        const float fi = row_bcast<decltype(i)::value>(f);
#pragma unroll
        for (int e = 0; e < E; ++e) o[decltype(i)::value][e] *= fi;
      });
    }
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sv[t][r], c, -m));
        lsum += p;
        float v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if constexpr (DT == KARA_BF16)
            v[e] = __uint_as_float((e & 1) ? vb[t][r][e >> 1] & 0xffff0000u : vb[t][r][e >> 1] << 16);
          else
            v[e] = __uint_as_float(vb[t][r][e]);
        }
        static_for<0, GP>([&](auto i) __attribute__((always_inline)) {
          const float pi = row_bcast<decltype(i)::value>(p);
#pragma unroll
          for (int e = 0; e < E; ++e) o[decltype(i)::value][e] = fmaf(pi, v[e], o[decltype(i)::value][e]);
        });
      }
  };
  // (next block's keys after this block's values, so that waiting for the
  // values leaves the keys in flight)
  if constexpr (C::kKBuf == 1) {
    for (int blk = wave; blk < nblk; blk += kDecWaves) {
      load_k(blk, 0);
      load_v(blk);
      work(blk, 0);
    }
  } else if (wave < nblk) {
    load_k(wave, 0);
    int blk = wave;
    for (;;) {
      load_v(blk);
      const int n1 = blk + kDecWaves;
      if (n1 < nblk) load_k(n1, 1);
      work(blk, 0);
      if (n1 >= nblk) break;
      load_v(n1);
      blk = n1 + kDecWaves;
      if (blk < nblk) load_k(blk, 0);
      work(n1, 1);
      if (blk >= nblk) break;
    }
  }

  // ---- the wave's sums over its four rows, then the four waves' ----
  lsum = swap32_add(lsum, lsum);
  lsum = swap16_add(lsum, lsum);
  if (gq == 0) {
    red_m[wave][li] = m;
    red_l[wave][li] = lsum;
  }
  // columns of a lane: bf16 E*li + e; fp32 at d = 128 4li + e and 64 + 4li + e - 4
  auto column = [&](int e) { return DT == KARA_F32 && E == 8 ? (e >> 2) * 64 + 4 * li + (e & 3) : E * li + e; };
#pragma unroll
  for (int i = 0; i < GP; ++i)
#pragma unroll
    for (int e = 0; e < E; e += 4) {
      // rows 0..3 of the wave end with columns e, e+1, e+2, e+3
      const float x0 = swap32_add(o[i][e], o[i][e + 2]);
      const float x1 = swap32_add(o[i][e + 1], o[i][e + 3]);
      const float y = swap16_add(x0, x1);
      // (the 32-lane swap leaves a in rows 0,1 and b in rows 2,3; the 16-lane
      // one a in rows 0,2 and b in rows 1,3)
      red_o[wave][i][column(e + (gq >> 1) * 2 + (gq & 1))] = y;
    }
  __syncthreads();
  const int nw = min(nblk, kDecWaves);   // waves that had keys
  const bool direct = len <= split_keys;
  float* rec = ws + (orow * n_splits + split) * (D + 2);
  for (int x = tid; x < G * D; x += kDecThreads) {
    const int i = x / D, e = x - i * D;
    float M = red_m[0][i];
    for (int w = 1; w < nw; ++w) M = fmaxf(M, red_m[w][i]);
    float L = 0.f, O = 0.f;
    for (int w = 0; w < nw; ++w) {
      const float f = __builtin_amdgcn_exp2f(red_m[w][i] - M);
      L += red_l[w][i] * f;
      O += red_o[w][i][e] * f;
    }
    if (direct) {
      out[orow * D + x] = O / L;
    } else {
      float* r = rec + (int64_t)i * n_splits * (D + 2);
      if (e == 0) r[0] = M, r[1] = L;
      r[2 + e] = O;
    }
  }
}

// One wave per (layer, sequence, query head) of a sequence longer than one
// split: its splits' factors are formed 64 at a time, its records added one by
// one (the shuffles keep the compiler from unrolling that loop).
template <int D>
__global__ __launch_bounds__(256) void decode_combine_kernel(Geom g, int n, const int32_t* __restrict__ seqs,
                                                             const int32_t* __restrict__ seq_lens, int max_len,
                                                             int split_keys, int n_splits, int64_t n_rows,
                                                             const float* __restrict__ ws, float* __restrict__ out) {
  constexpr int kDPerLane = D / 64;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // (l, j, hq)
  if (row >= n_rows) return;
  const int j = (int)((row / g.Hq) % n);
  const int s = seqs[j];
  const int len = s >= 0 && s < g.n_seqs ? seq_lens[s] : 0;
  float* dst = out + row * D + lane * kDPerLane;
  if (len <= 0 || len > max_len) {
#pragma unroll
    for (int e = 0; e < kDPerLane; ++e) dst[e] = 0.f;
    return;
  }
  if (len <= split_keys) return;   // the split kernel wrote it
  const int ns = (len + split_keys - 1) / split_keys;
  const int rec = D + 2;
  const float* w = ws + row * n_splits * rec;
  // lane i: split i's maximum and sum (64 at a time)
  float M = kNegInf;
  for (int sp = lane; sp < ns; sp += 64) M = fmaxf(M, w[sp * rec]);
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) M = fmaxf(M, __shfl_xor(M, x, 64));
  float L = 0.f, acc[kDPerLane] = {};
  for (int sp0 = 0; sp0 < ns; sp0 += 64) {
    const int sp = sp0 + lane;
    const float f = sp < ns ? __builtin_amdgcn_exp2f(w[sp * rec] - M) : 0.f;
    const float lf = sp < ns ? w[sp * rec + 1] * f : 0.f;
    const int cnt = min(64, ns - sp0);
    for (int i = 0; i < cnt; ++i) {
      L += __shfl(lf, i, 64);
      const float fi = __shfl(f, i, 64);
#pragma unroll
      for (int e = 0; e < kDPerLane; ++e) acc[e] += w[(sp0 + i) * rec + 2 + lane * kDPerLane + e] * fi;
    }
  }
#pragma unroll
  for (int e = 0; e < kDPerLane; ++e) dst[e] = acc[e] / L;
}

// Keys per split: 256 (the workspace's records are sized for that) while
// the launch has few workgroups, up to 1024 where 16 per CU remain: fewer
// records and prologues.
int decode_split_keys(const Geom& g, int n, int n_layers, int max_len) {
  const int64_t units = (int64_t)n_layers * n * g.Hkv;
  int keys = kSplitKeys;
  while (keys < kDecMaxSplit && units * ((max_len + 2 * keys - 1) / (2 * keys)) >= kDecWgTarget) keys *= 2;
  return keys;
}

template <int DT, int D, int GP>
hipError_t launch_decode_g(const Geom& g, int n, const int32_t* seqs, int n_layers, const void* q, const PoolPtrs& kp,
                           const PoolPtrs& vp, const int32_t* bt, const int32_t* seq_lens, int max_len, float* out,
                           float* ws, hipStream_t stream) {
  const int keys = decode_split_keys(g, n, n_layers, max_len);
  const int n_splits = (max_len + keys - 1) / keys;
  const int64_t blocks = (int64_t)n_layers * n * g.Hkv * n_splits;
  hipLaunchKernelGGL((decode_split_kernel<DT, D, GP>), dim3((unsigned)blocks), dim3(kDecThreads), 0, stream, g, n, seqs,
                     (const char*)q, kp, vp, bt, seq_lens, max_len, keys, n_splits, ws, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || n_splits == 1) return e;
  const int64_t rows = (int64_t)n_layers * n * g.Hq;
  hipLaunchKernelGGL((decode_combine_kernel<D>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream, g, n, seqs,
                     seq_lens, max_len, keys, n_splits, rows, (const float*)ws, out);
  return hipGetLastError();
}

// query heads per KV head, rounded up to an instance's accumulators
template <int DT, int D>
hipError_t launch_decode(const Geom& g, int n, const int32_t* seqs, int n_layers, const void* q, const PoolPtrs& kp,
                         const PoolPtrs& vp, const int32_t* bt, const int32_t* seq_lens, int max_len, float* out,
                         float* ws, hipStream_t stream) {
#define KARA_DECODE_G(GP) \
  return launch_decode_g<DT, D, GP>(g, n, seqs, n_layers, q, kp, vp, bt, seq_lens, max_len, out, ws, stream)
  if (g.G == 1) KARA_DECODE_G(1);
  if (g.G == 2) KARA_DECODE_G(2);
  if (g.G <= 4) KARA_DECODE_G(4);
  if (g.G == 5) KARA_DECODE_G(5);
  if (g.G <= 8) KARA_DECODE_G(8);
  KARA_DECODE_G(16);
#undef KARA_DECODE_G
}

// the step's window fields are irrelevant here; validate the rest
kara_status_t harness_geom(const kara_params_t* p, int32_t n, Geom* g) {
  kara_status_t st = make_geom(p, n, g);
  if (st != KARA_OK) return st;
  return KARA_OK;
}

}  // namespace
}  // namespace kara

using namespace kara;

extern "C" {

kara_status_t kara_harness_kv_append(const kara_params_t* p, int32_t n, const int32_t* seqs, int32_t n_new,
                                     int32_t n_layers, const void* k_new, const void* v_new, void* const* k_pools,
                                     void* const* v_pools, const int32_t* block_table, int32_t* seq_lens,
                                     int32_t* status, void* stream) {
  Geom g;
  kara_status_t st = harness_geom(p, n, &g);
  if (st != KARA_OK) return st;
  if (n < 0 || n_new < 0 || n_layers < 1 || n_layers > kMaxLayersPerLaunch) return KARA_ERR_INVALID_ARG;
  if (n == 0 || n_new == 0) return KARA_OK;
  if (!seqs || !k_new || !v_new || !block_table || !seq_lens || !status ||
      !pools_ok((const void* const*)k_pools, n_layers) || !pools_ok((const void* const*)v_pools, n_layers))
    return KARA_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  PoolPtrs kp{}, vp{};
  for (int i = 0; i < n_layers; ++i) {
    kp.p[i] = k_pools[i];
    vp.p[i] = v_pools[i];
  }
  // tokens per workgroup: enough pieces for its threads' loads in flight
  const int per_tok = g.Hkv * (g.d * g.esize / 16);
  const int toks = std::min(n_new, std::max(1, 2 * kAppendThreads * kAppendUnroll / per_tok));
  const int64_t chunks = ((int64_t)n_new + toks - 1) / toks;
  const dim3 copy_grid((unsigned)(n * chunks), (unsigned)n_layers, 2), block(kAppendThreads);
  if (n_new <= kAppendFusedTokens) {
    hipLaunchKernelGGL((append_kernel<true>), copy_grid, block, 0, s, g, n, seqs, n_new, toks, (int)chunks,
                       (const char*)k_new, (const char*)v_new, kp, vp, block_table, seq_lens, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_status(e);
    hipLaunchKernelGGL((append_commit_kernel<true>), dim3((unsigned)n), block, 0, s, g, n, seqs, n_new, block_table,
                       seq_lens, status);
    return hip_status(hipGetLastError());
  }
  hipLaunchKernelGGL(append_check_kernel, dim3((unsigned)n), block, 0, s, g, n, seqs, n_new, block_table, seq_lens,
                     status);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_status(e);
  hipLaunchKernelGGL((append_kernel<false>), copy_grid, block, 0, s, g, n, seqs, n_new, toks, (int)chunks,
                     (const char*)k_new, (const char*)v_new, kp, vp, block_table, seq_lens, status);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_status(e);
  hipLaunchKernelGGL((append_commit_kernel<false>), dim3((n + kAppendThreads - 1) / kAppendThreads), block, 0, s, g, n,
                     seqs, n_new, block_table, seq_lens, status);
  return hip_status(hipGetLastError());
}

kara_status_t kara_harness_decode_workspace_size(const kara_params_t* p, int32_t n, int32_t n_layers,
                                                 int32_t max_len, size_t* bytes) {
  Geom g;
  kara_status_t st = harness_geom(p, n, &g);
  if (st != KARA_OK) return st;
  if (!bytes || n_layers < 1 || max_len < 1 || (int64_t)max_len > (int64_t)g.max_blocks * g.bs)
    return KARA_ERR_INVALID_ARG;
  const int64_t n_splits = (max_len + kSplitKeys - 1) / kSplitKeys;
  *bytes = (size_t)n_layers * n * g.Hq * n_splits * (g.d + 2) * sizeof(float);
  return KARA_OK;
}

kara_status_t kara_harness_decode_attention(const kara_params_t* p, int32_t n, const int32_t* seqs,
                                            int32_t n_layers, const void* q, const void* const* k_pools,
                                            const void* const* v_pools, const int32_t* block_table,
                                            const int32_t* seq_lens, int32_t max_len, float* out,
                                            void* workspace, size_t workspace_bytes, void* stream) {
  Geom g;
  kara_status_t st = harness_geom(p, n, &g);
  if (st != KARA_OK) return st;
  if (g.G > KARA_HARNESS_MAX_GROUP) return KARA_ERR_UNSUPPORTED;
  size_t need = 0;
  st = kara_harness_decode_workspace_size(p, n, n_layers, max_len, &need);
  if (st != KARA_OK) return st;
  if (n_layers > kMaxLayersPerLaunch) return KARA_ERR_INVALID_ARG;
  if (n == 0) return KARA_OK;
  if (!seqs || !q || !block_table || !seq_lens || !out || !pools_ok(k_pools, n_layers) ||
      !pools_ok(v_pools, n_layers))
    return KARA_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < need) return KARA_ERR_WORKSPACE;
  PoolPtrs kp{}, vp{};
  for (int i = 0; i < n_layers; ++i) {
    kp.p[i] = const_cast<void*>(k_pools[i]);
    vp.p[i] = const_cast<void*>(v_pools[i]);
  }
  hipStream_t s = (hipStream_t)stream;
  float* ws = (float*)workspace;
  hipError_t e;
  if (g.dtype == KARA_BF16)
    e = g.d == 128 ? launch_decode<KARA_BF16, 128>(g, n, seqs, n_layers, q, kp, vp, block_table, seq_lens, max_len,
                                                  out, ws, s)
                   : launch_decode<KARA_BF16, 64>(g, n, seqs, n_layers, q, kp, vp, block_table, seq_lens, max_len,
                                                 out, ws, s);
  else
    e = g.d == 128 ? launch_decode<KARA_F32, 128>(g, n, seqs, n_layers, q, kp, vp, block_table, seq_lens, max_len,
                                                 out, ws, s)
                   : launch_decode<KARA_F32, 64>(g, n, seqs, n_layers, q, kp, vp, block_table, seq_lens, max_len,
                                                out, ws, s);
  return hip_status(e);
}

}  // extern "C"
