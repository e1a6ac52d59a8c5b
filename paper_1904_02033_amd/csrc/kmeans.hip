// k-means of the balanced clustering (Section 3.3; Lloyd's k-means, Section
// 2) on int8 points with centres on a grid of 2^-8, in exact integer
// arithmetic:
//   assignment  argmin_j ||2^8 x - C_j||^2 = argmin_j ( ||C_j||^2 - 2^9 <x, C_j> ),
//               ties to the lower index.  <x, C_j> is an int8 matrix product
//               of the points with the two signed base-256 digits of C_j (C =
//               256 hi + lo, lo in [-128, 127]) on the matrix cores; every
//               partial sum stays within int32 for d <= 256.  A centre with a
//               coordinate outside [-2^15, 2^15 - 129] (no mean of points is
//               one) has no such digits and is compared by itself.
//   update      centre j = floor(2^8 S_j / n_j + 1/2) from exact 64-bit
//               sums (integer atomics, so the order of the additions does
//               not matter); an empty cluster keeps its centre.
#include <hip/hip_runtime.h>
#include "kernels.h"
#include "launch.h"
#include "mfma.h"

namespace sanns {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kKmStage = 64;       // centres staged in LDS at a time
constexpr int kKmTiles = 4;        // 16-point column tiles per wave
constexpr int kKmWgPoints = 4 * 16 * kKmTiles;  // points per workgroup (4 waves)
constexpr int kKmIdxBits = 22;     // centre index bits of a packed candidate

// One wave per centre j: its digit words hi[w], then lo[w], w < dw <= 64 (4
// coordinates per word, zero past d), and ||C_j||^2; zero digits and -1 for one
// beyond the digits' range.  (A thread per centre, walking its row alone, took 21
// us for 2,000 centres of 96 coordinates; the wave reads the row in one load.)
__global__ void __launch_bounds__(256)
k_km_pack(const int32_t* __restrict__ C, int k, int d, int dw, int32_t* __restrict__ packed,
          int64_t* __restrict__ cnorm) {
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), w = threadIdx.x & 63;
  if (j >= k) return;
  const int32_t* c = C + (size_t)j * d;
  uint32_t h = 0, l = 0;
  int64_t nrm = 0;
  bool far = false;
  if (w < dw) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = 4 * w + b;
      const int v = i < d ? c[i] : 0;
      far |= v < -32768 || v > 32639;
      const int lv = ((v + 128) & 255) - 128;
      const int hv = (v - lv) / 256;
      l |= (uint32_t)(uint8_t)(int8_t)lv << (8 * b);
      h |= (uint32_t)(uint8_t)(int8_t)hv << (8 * b);
      nrm += (int64_t)v * v;
    }
  }
  far = __any(far);
  if (w < dw) {
    packed[(size_t)j * 2 * dw + w] = far ? 0 : (int32_t)h;
    packed[(size_t)j * 2 * dw + dw + w] = far ? 0 : (int32_t)l;
  }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) nrm += __shfl_xor(nrm, s);
  if (w == 0) cnorm[j] = far ? -1 : nrm;
}

// Closest centres on the int8 matrix cores.  A tile is 16 centres (rows) x 16
// points (columns); a wave keeps the fragments of 4 column tiles (64 points) in
// registers for the whole launch, the workgroup's 4 waves share the centres'
// digits, staged in LDS 64 at a time (the next stage's words are loaded into
// registers behind the current one's products).  For centre j and point x the
// key ||C_j||^2 - 2^9 <x, C_j> = 2^9 (n_j - <x, C_j>) + r_j with ||C_j||^2 =
// 2^9 n_j + r_j, so the smallest key is the largest
//     G = 256 <x, hi_j> + (<x, lo_j> - n_j)     (an int32; the accumulator of the
//                                               low digits starts at -n_j),
// among those the smallest r_j, then the smallest j.  A lane holds 4 centres of
// a tile for one point and keeps the maximum of the 64-bit candidate (G, ~(r_j,
// j)), five instructions per pair (shift and add, a copy of the tag, compare, two
// selects); the four lanes of a point are compared at the end.  Per pair and 64
// coordinates the products take a quarter of a cycle of a SIMD's matrix core for
// each digit, the selection a quarter of a cycle per instruction, so the selection
// bounds it for d <= 128.  Centre
// indices beyond 22 bits are taken in blocks, whose winners are compared in 64
// bits.  At n = 200,000, d = 96, k = 2,000: 1.18 ms by 4-way dot products on the
// vector units, 0.13 ms here.
// (At least two waves per SIMD: with all 512 registers of one the compiler puts
// the sums in the accumulation half and copies each out, 32 more instructions
// for 64 candidates.)
template <int DW>
__global__ void __launch_bounds__(256, DW <= 24 ? 4 : DW <= 40 ? 3 : 2)
k_km_assign(const int8_t* __restrict__ X, long n, int d, int words_ok,
            const int32_t* __restrict__ C, const int32_t* __restrict__ packed, const int64_t* __restrict__ cnorm, int k,
            const int32_t* __restrict__ prev, int32_t* __restrict__ assign,
            uint32_t* __restrict__ changed) {
  constexpr int NS = DW / 16;             // steps of 64 coordinates
  constexpr bool HALF = DW % 16 != 0;     // and a last one of 32
  constexpr int RU = DW / 2;              // 16-byte units of a centre's digits
  constexpr int RS = RU + 1;              // with one of padding (LDS banks)
  constexpr int NU = DW / 8;              // units a thread stages (64 RU / 256)
  __shared__ uint4 cw[kKmStage * RS];
  __shared__ int32_t cng[kKmStage];       // -n_j
  __shared__ uint32_t ctag[kKmStage];     // ~(r_j, j)
  const int tid = threadIdx.x, lane = tid & 63, m16 = lane & 15, g = lane >> 4;
  const long base = (long)blockIdx.x * kKmWgPoints + (tid >> 6) * 16 * kKmTiles;
  v4i bx[kKmTiles][NS > 0 ? NS : 1];
  int64_t bh[kKmTiles];
#pragma unroll
  for (int t = 0; t < kKmTiles; ++t) {
    const long pt = base + 16 * t + m16;
    const int8_t* row = X + (pt < n ? pt : 0) * (long)d;
    // the word at coordinates 4w .. 4w + 3, zero past d
    auto word = [&](int w) -> uint32_t {
      if (words_ok) return 4 * w < d ? reinterpret_cast<const uint32_t*>(row)[w] : 0u;
      uint32_t v = 0;
      for (int b = 0; b < 4; ++b)
        if (4 * w + b < d) v |= (uint32_t)(uint8_t)row[4 * w + b] << (8 * b);
      return v;
    };
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int b = 0; b < 4; ++b) bx[t][s][b] = (int)word(16 * s + 4 * g + b);
    if (HALF)
      bh[t] = (int64_t)((uint64_t)word(16 * NS + 2 * g) |
                        (uint64_t)word(16 * NS + 2 * g + 1) << 32);
  }
  int64_t bkey[kKmTiles];
  int bidx[kKmTiles];
#pragma unroll
  for (int t = 0; t < kKmTiles; ++t) {
    bkey[t] = INT64_MAX;
    bidx[t] = 0;
  }
  const uint4* src = reinterpret_cast<const uint4*>(packed);
  const long n_units = (long)k * RU;
  uint4 nx[NU];
  int64_t ncn = 0;
  auto fetch = [&](int c0) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const long e = (long)c0 * RU + tid + 256 * u;
      nx[u] = e < n_units ? src[e] : make_uint4(0, 0, 0, 0);
    }
    if (tid < kKmStage && c0 + tid < k) ncn = cnorm[c0 + tid];
  };
  constexpr int kBlock = 1 << kKmIdxBits;
  bool far = false;
  fetch(0);
  for (int k0 = 0; k0 < k; k0 += kBlock) {
    const int k1 = k - k0 < kBlock ? k : k0 + kBlock;
    int64_t best[kKmTiles];
#pragma unroll
    for (int t = 0; t < kKmTiles; ++t) best[t] = INT64_MIN;
    for (int c0 = k0; c0 < k1; c0 += kKmStage) {
      __syncthreads();  // the previous stage has been read
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int e = tid + 256 * u;
        cw[e / RU * RS + e % RU] = nx[u];
      }
      if (tid < kKmStage) {
        // padding centres and those beyond the digits' range never win: G =
        // INT32_MIN, tag 0, the candidate that best[] starts from
        const bool real = c0 + tid < k && ncn >= 0;
        far |= c0 + tid < k && ncn < 0;
        cng[tid] = real ? -(int32_t)(ncn >> 9) : INT32_MIN;
        ctag[tid] = real ? ~(((uint32_t)ncn & 511u) << kKmIdxBits | (uint32_t)(c0 + tid - k0)) : 0u;
      }
      __syncthreads();
      if (c0 + kKmStage < k) fetch(c0 + kKmStage);
      const int nc = k1 - c0 < kKmStage ? k1 - c0 : kKmStage;
      for (int ct = 0; ct < nc; ct += 16) {
        const char* ab = reinterpret_cast<const char*>(cw + (ct + m16) * RS);
        v4i ah[NS > 0 ? NS : 1], al[NS > 0 ? NS : 1];
        int64_t ahh = 0, alh = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          ah[s] = *reinterpret_cast<const v4i*>(ab + 64 * s + 16 * g);
          al[s] = *reinterpret_cast<const v4i*>(ab + 4 * DW + 64 * s + 16 * g);
        }
        if (HALF) {
          ahh = *reinterpret_cast<const int64_t*>(ab + 64 * NS + 8 * g);
          alh = *reinterpret_cast<const int64_t*>(ab + 4 * DW + 64 * NS + 8 * g);
        }
        const v4i ng = *reinterpret_cast<const v4i*>(cng + ct + 4 * g);
        const v4i tag = *reinterpret_cast<const v4i*>(ctag + ct + 4 * g);
        // The products of all four tiles, step by step, then the selection of
        // each: a product's successor in its sum is eight products away.  Where
        // the last step is the 32-coordinate shape, mfma_shape_change keeps it
        // clear of the 64-coordinate one (tile by tile, each right behind the
        // other, half of the centres' sums were wrong at 96 coordinates).
        v4i hs[kKmTiles], ls[kKmTiles];
#pragma unroll
        for (int t = 0; t < kKmTiles; ++t) {
          hs[t] = v4i{0, 0, 0, 0};
          ls[t] = ng;
        }
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int t = 0; t < kKmTiles; ++t) {
            hs[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah[s], bx[t][s], hs[t], 0, 0, 0);
            ls[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[s], bx[t][s], ls[t], 0, 0, 0);
          }
        if (HALF && NS > 0) mfma_shape_change();
        if (HALF) {
#pragma unroll
          for (int t = 0; t < kKmTiles; ++t) {
            hs[t] = __builtin_amdgcn_mfma_i32_16x16x32_i8(ahh, bh[t], hs[t], 0, 0, 0);
            ls[t] = __builtin_amdgcn_mfma_i32_16x16x32_i8(alh, bh[t], ls[t], 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < kKmTiles; ++t) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int32_t G = (int32_t)(((uint32_t)hs[t][e] << 8) + (uint32_t)ls[t][e]);
            const int64_t cand = (int64_t)((uint64_t)(uint32_t)G << 32 | (uint32_t)tag[e]);
            best[t] = cand > best[t] ? cand : best[t];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kKmTiles; ++t) {
      int64_t b = best[t];
      int64_t o = __shfl_xor(b, 16);
      b = o > b ? o : b;
      o = __shfl_xor(b, 32);
      b = o > b ? o : b;
      const uint32_t tag = ~(uint32_t)b;
      const int64_t key = (int64_t)(tag >> kKmIdxBits) - 512 * (int64_t)(int32_t)(b >> 32);
      if (b != INT64_MIN && key < bkey[t]) {
        bkey[t] = key;
        bidx[t] = k0 + (int)(tag & (kBlock - 1));
      }
    }
  }
  // lanes g = t write tile t
  int mine = bidx[0];
#pragma unroll
  for (int t = 1; t < kKmTiles; ++t) mine = g == t ? bidx[t] : mine;
  const long pt = base + 16 * g + m16;
  const bool in = pt < n;
  if (__syncthreads_or(far)) {
    // the centres beyond the digits' range, coordinate by coordinate
    int64_t key0 = bkey[0];
#pragma unroll
    for (int t = 1; t < kKmTiles; ++t) key0 = g == t ? bkey[t] : key0;
    __int128 key = key0 == INT64_MAX ? (__int128)1 << 100 : (__int128)key0;
    const int8_t* row = X + (in ? pt : 0) * (long)d;
    for (int j = 0; j < k; ++j) {
      if (cnorm[j] >= 0) continue;
      __int128 f = 0;
      for (int i = 0; i < d; ++i) {
        const int64_t c = C[(size_t)j * d + i];
        f += c * (c - 512 * (int64_t)row[i]);
      }
      if (f < key || (f == key && j < mine)) {
        key = f;
        mine = j;
      }
    }
  }
  if (prev && changed) {
    const uint64_t diff = __ballot(in && prev[in ? pt : 0] != mine);
    if (lane == 0 && diff) atomicAdd(changed, (uint32_t)__popcll(diff));
  }
  if (in) assign[pt] = mine;
}

__global__ void __launch_bounds__(256) k_km_zero(uint64_t* __restrict__ p, long cnt) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < cnt) p[g] = 0;
}

// Exact sums and counts of every cluster.  Thread per (point, two
// coordinates): both, shifted to [0, 255], ride in one 64-bit atomic add, low
// and high half, which the launcher keeps from carrying (255 n < 2^32).  The
// adds bound it (19 M of one coordinate each took 124 us at n = 200,000, d = 96,
// k = 2,000; half as many take 73 us).  Assignments outside [0, k) are skipped.
__global__ void __launch_bounds__(256)
k_km_accum2(const int8_t* __restrict__ X, long n, int d, const int32_t* __restrict__ assign,
            int k, uint64_t* __restrict__ sums, uint64_t* __restrict__ counts) {
  const int h = (d + 1) / 2;
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n * h) return;
  const long pt = g / h;
  const int i = (int)(g % h);
  const int a = assign[pt];
  if (a < 0 || a >= k) return;
  const int8_t* x = X + pt * d + 2 * i;
  const uint64_t v = (uint64_t)(uint32_t)(x[0] + 128) |
                     (2 * i + 1 < d ? (uint64_t)(uint32_t)(x[1] + 128) << 32 : 0);
  atomicAdd((unsigned long long*)&sums[(size_t)a * h + i], (unsigned long long)v);
  if (i == 0) atomicAdd((unsigned long long*)&counts[a], 1ull);
}

// The same with the adds gathered in LDS first: a workgroup takes one part of
// the points and PAIRS coordinate pairs, adds into its own table of every
// cluster (k PAIRS words, then k counts that the workgroups of the first pairs
// keep), and then adds the table to the global sums.  Few atomics leave the
// workgroup, and clusters that many points share do not queue in the L2.
constexpr int kKmAccThreads = 1024;
template <int PAIRS>
__global__ void __launch_bounds__(kKmAccThreads)
k_km_accum_lds(const int8_t* __restrict__ X, long n, int d, const int32_t* __restrict__ assign,
               int k, int slices, long part_len, uint64_t* __restrict__ sums,
               uint64_t* __restrict__ counts) {
  extern __shared__ uint64_t tab[];
  uint32_t* cnt = reinterpret_cast<uint32_t*>(tab + (size_t)k * PAIRS);
  const int h = (d + 1) / 2, tid = threadIdx.x;
  const int slice = blockIdx.x % slices;
  const long p0 = (blockIdx.x / slices) * part_len;
  const long p1 = p0 + part_len < n ? p0 + part_len : n;
  for (int u = tid; u < k * PAIRS; u += kKmAccThreads) tab[u] = 0;
  for (int u = tid; u < k; u += kKmAccThreads) cnt[u] = 0;
  __syncthreads();
  const int j = tid % PAIRS, i = slice * PAIRS + j;
  if (i < h) {
    constexpr int U = 8, STEP = kKmAccThreads / PAIRS;  // points in flight per thread
    const bool two = 2 * i + 1 < d;
    for (long pt = p0 + tid / PAIRS; pt < p1; pt += U * STEP) {
      int a[U];
      uint64_t v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long q = pt + u * STEP < p1 ? pt + u * STEP : pt;
        const int8_t* x = X + q * d + 2 * i;
        a[u] = pt + u * STEP < p1 ? assign[q] : -1;
        v[u] = (uint64_t)(uint32_t)(x[0] + 128) |
               (uint64_t)(two ? (uint32_t)(x[two] + 128) : 0u) << 32;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (a[u] < 0 || a[u] >= k) continue;
        atomicAdd((unsigned long long*)&tab[a[u] * PAIRS + j], (unsigned long long)v[u]);
        if (i == 0) atomicAdd(&cnt[a[u]], 1u);
      }
    }
  }
  __syncthreads();
  for (int u = tid; u < k * PAIRS; u += kKmAccThreads) {
    const int a = u / PAIRS, ii = slice * PAIRS + u % PAIRS;
    if (tab[u]) atomicAdd((unsigned long long*)&sums[(size_t)a * h + ii], (unsigned long long)tab[u]);
  }
  if (slice == 0)
    for (int a = tid; a < k; a += kKmAccThreads)
      if (cnt[a]) atomicAdd((unsigned long long*)&counts[a], (unsigned long long)cnt[a]);
}

// Parts of the points for that form, 0 where it is not the one to take: the
// tables must fit a CU's LDS (k up to 7,680 with two pairs each), a part needs
// points enough that few adds leave it (n >= 64 k, four for each table entry and
// 16 parts), and with fewer than 32 workgroups the chip would idle.  Whole
// updates, global adds / LDS tables: n = 200,000, d = 96, k = 30: 670 / 29 us, k =
// 300: 198 / 35, k = 2,000: 81 / 52; n = 1,000,000, k = 1,000: 446 / 106; below
// the line n = 100,000, d = 128, k = 2,500: 60 / 65 and n = 200,000, k = 5,000:
// 78 / 90.
static int km_accum_parts(long n, int d, int k, int* pairs) {
  constexpr size_t kLds = 150 * 1024;
  *pairs = 0;
  for (int p : {8, 4, 2})
    if (!*pairs && (size_t)k * (8 * p + 4) <= kLds) *pairs = p;
  if (!*pairs || n < 64l * k) return 0;
  const int slices = ((d + 1) / 2 + *pairs - 1) / *pairs;
  const long most = slices >= 256 ? 1 : 256 / slices;
  const long parts = n / (4l * k) < most ? n / (4l * k) : most;
  return parts * slices < 32 ? 0 : (int)parts;
}

template <int PAIRS>
static bool launch_km_accum_lds(const int8_t* X, long n, int d, const int32_t* assign, int k,
                                int parts, uint64_t* sums, uint64_t* counts, hipStream_t st) {
  const int slices = ((d + 1) / 2 + PAIRS - 1) / PAIRS;
  const size_t lds = (size_t)k * (8 * PAIRS + 4);
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute((const void*)k_km_accum_lds<PAIRS>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();  // the other form takes the call
    return false;
  }
  hipLaunchKernelGGL(k_km_accum_lds<PAIRS>, dim3((unsigned)(slices * parts)), dim3(kKmAccThreads), lds, st,
                     X, n, d, assign, k, slices, (n + parts - 1) / parts, sums, counts);
  return true;
}

// The sums for n where a pair could carry: thread per (point, coordinate), two's
// complement 64-bit sums.
__global__ void __launch_bounds__(256)
k_km_accum(const int8_t* __restrict__ X, long n, int d, const int32_t* __restrict__ assign,
           int k, uint64_t* __restrict__ sums, uint64_t* __restrict__ counts) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n * d) return;
  const long pt = g / d;
  const int i = (int)(g % d);
  const int a = assign[pt];
  if (a < 0 || a >= k) return;
  atomicAdd((unsigned long long*)&sums[(size_t)a * d + i],
            (unsigned long long)(int64_t)X[pt * d + i]);
  if (i == 0) atomicAdd((unsigned long long*)&counts[a], 1ull);
}

// Thread per (centre, coordinate): C = floor((2^9 S + n) / (2 n)) for n > 0
// (paired: the sums of k_km_accum2).
__global__ void __launch_bounds__(256)
k_km_centers(const uint64_t* __restrict__ sums, const uint64_t* __restrict__ counts, int k,
             int d, int paired, int32_t* __restrict__ C) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (long)k * d) return;
  const int j = (int)(g / d);
  const int64_t cnt = (int64_t)counts[j];
  if (cnt == 0) return;
  int64_t S;
  if (paired) {
    const int i = (int)(g - (long)j * d);
    const uint64_t v = sums[(size_t)j * ((d + 1) / 2) + i / 2];
    S = (int64_t)(uint32_t)(i & 1 ? v >> 32 : v) - 128 * cnt;
  } else {
    S = (int64_t)sums[g];
  }
  const int64_t num = S * 512 + cnt, den = 2 * cnt;
  int64_t q = num / den;
  if (num % den != 0 && num < 0) q -= 1;  // floor
  C[g] = (int32_t)q;
}

// Initial centres: C_j = 2^8 x_{idx[j]}.
__global__ void __launch_bounds__(256)
k_km_init(const int8_t* __restrict__ X, long n, int d, const int64_t* __restrict__ idx, int k,
          int32_t* __restrict__ C, uint32_t* __restrict__ bad) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (long)k * d) return;
  const int j = (int)(g / d), i = (int)(g % d);
  long p = idx[j];
  if (p < 0 || p >= n) {
    if (i == 0) atomicOr(bad, 1u);
    p = 0;
  }
  C[g] = 256 * (int32_t)X[p * d + i];
}

int km_words(int d) { return (d + 3) / 4; }

size_t km_workspace(int k, int d) {
  const size_t dw = km_words(d) <= 8 ? 8 : (size_t)(km_words(d) + 7) / 8 * 8;
  return (size_t)k * 2 * dw * 4 + (size_t)k * 8 + (size_t)k * d * 8 + (size_t)k * 8 + 256;
}

static int km_dw(int d) {
  const int w = km_words(d);
  return w <= 8 ? 8 : (w + 7) / 8 * 8;  // 8, 16, ..., 64
}

hipError_t launch_km_init(const int8_t* X, long n, int d, const int64_t* idx, int k, int32_t* C,
                          uint32_t* bad, hipStream_t st) {
  const long t = (long)k * d;
  hipLaunchKernelGGL(k_km_init, dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st, X, n, d, idx,
                     k, C, bad);
  return hipGetLastError();
}

hipError_t launch_km_assign(const int8_t* X, long n, int d, const int32_t* C, int k,
                            const int32_t* prev, int32_t* assign, uint32_t* changed, void* ws,
                            hipStream_t st) {
  const int dw = km_dw(d);
  int32_t* packed = (int32_t*)ws;
  int64_t* cnorm = (int64_t*)((char*)ws + (size_t)k * 2 * dw * 4);
  hipLaunchKernelGGL(k_km_pack, dim3((unsigned)((k + 3) / 4)), dim3(256), 0, st, C, k, d, dw,
                     packed, cnorm);
  const unsigned grid = (unsigned)((n + kKmWgPoints - 1) / kKmWgPoints);
  // points are read as 32-bit words where every row starts on one
  const int words_ok = d % 4 == 0 && (uintptr_t)X % 4 == 0;
  switch (dw) {
#define SANNS_KM(DWV)                                                                       \
  case DWV:                                                                                 \
    hipLaunchKernelGGL(k_km_assign<DWV>, dim3(grid), dim3(256), 0, st, X, n, d, words_ok, C,   \
                       packed, cnorm, k, prev, assign, changed);                            \
    break;
    SANNS_KM(8) SANNS_KM(16) SANNS_KM(24) SANNS_KM(32) SANNS_KM(40) SANNS_KM(48) SANNS_KM(56)
    SANNS_KM(64)
#undef SANNS_KM
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_km_update(const int8_t* X, long n, int d, const int32_t* assign, int k,
                            int32_t* C, int64_t* counts_out, void* ws, hipStream_t st) {
  const int dw = km_dw(d);
  uint64_t* sums = (uint64_t*)((char*)ws + (size_t)k * 2 * dw * 4 + (size_t)k * 8);
  uint64_t* counts = sums + (size_t)k * d;
  const long zc = (long)k * d + k;
  hipLaunchKernelGGL(k_km_zero, dim3((unsigned)((zc + 255) / 256)), dim3(256), 0, st, sums, zc);
  // two coordinates per add while their halves cannot carry; not for one or two
  // coordinates by global adds, where a pair's denser lines queue longer than an add
  // less is worth (n = 137,778, k = 1,966, d = 2: 28 us in pairs, 24 apart)
  int pairs = 0, paired = n < (1l << 32) / 255;
  const int parts = paired ? km_accum_parts(n, d, k, &pairs) : 0;
  if (parts == 0 && d <= 2) paired = 0;
  const long t = n * (paired ? (d + 1) / 2 : d);
  const bool done =
      parts > 0 &&
      (pairs == 8   ? launch_km_accum_lds<8>(X, n, d, assign, k, parts, sums, counts, st)
       : pairs == 4 ? launch_km_accum_lds<4>(X, n, d, assign, k, parts, sums, counts, st)
                    : launch_km_accum_lds<2>(X, n, d, assign, k, parts, sums, counts, st));
  if (!done && t > 0) {
    if (paired)
      hipLaunchKernelGGL(k_km_accum2, dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st, X, n,
                         d, assign, k, sums, counts);
    else
      hipLaunchKernelGGL(k_km_accum, dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st, X, n,
                         d, assign, k, sums, counts);
  }
  const long tc = (long)k * d;
  hipLaunchKernelGGL(k_km_centers, dim3((unsigned)((tc + 255) / 256)), dim3(256), 0, st, sums,
                     counts, k, d, paired, C);
  if (counts_out)
    (void)hipMemcpyAsync(counts_out, counts, (size_t)k * 8, hipMemcpyDeviceToDevice, st);
  return hipGetLastError();
}

}  // namespace sanns
