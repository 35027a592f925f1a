// Index construction of the wave index: segmented spherical k-means over the
// keys of every (sequence, KV head) unit and the meta index / cluster-contiguous
// KV layout that results (paper: "Index Organization", "Lightweight Index
// Construction and Updates"; value sums and sizes from the estimation section).
//
// Per segment of L tokens:
//   mean        fp64 mean of the segment's keys
//   normalise   xhat = quant((K - mean) / |K - mean|)             (fp64, one rounding)
//   init        k seeded distinct points of the segment become the first centroids
//   T times:    assign  (MFMA similarities, fp32 accumulate; running best and
//                        second best per point; near-ties re-decided with fp64
//                        similarities)
//               update  (centroid = quant(member sum / |member sum|), fp64)
//   sort        stable counting sort of the segment's points by cluster, after the
//               last round and wherever an update reads members by cluster
// Three forms of the T rounds, same results: bf16 segments of a few clusters in one
// workgroup each (kmeans_small_kernel); bf16 with a segment's centroids in LDS and four
// points per cluster or more: later rounds compare changed centroids and sum moved
// points (assign_delta_kernel, update_moves_kernel); else assign, refine, sort and update
// of the touched clusters, a launch each (f32: assign with its near-ties, and sort with update).
//   finalize    sizes, offsets, mean of raw keys, value sums, permuted K/V rows
#include <stdlib.h>

#include <type_traits>

#include "wave_common.h"

namespace wave {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float floatx16;

constexpr float kNegHuge = -3.0e38f;
// Two similarities closer than this are re-decided in fp64.  It covers the fp32
// accumulation error of a unit-vector dot product (<= (d + 1) * 2^-24 < 8e-6; in the
// MFMA path the sums run near 2, so 8 steps of 2^-23) on both values plus the 5 low
// mantissa bits the MFMA path overwrites with the row code (<= 2^-18 relative each).
constexpr float kAssignGuard = 4.0e-5f;

struct SegInfo {
  int unit, s, seg_start, L_s, k_s;
};
__device__ __forceinline__ SegInfo seg_info(int sg, int S, int L, int kk, int N_idx) {
  SegInfo r;
  r.unit = sg / S;
  r.s = sg - r.unit * S;
  r.seg_start = r.s * L;
  r.L_s = min(L, N_idx - r.seg_start);
  r.k_s = min(kk, r.L_s);
  return r;
}

// a / b for many a and one b: with r the correctly rounded 1 / b, one multiply
// and one fused residual correction give the correctly rounded quotient (the
// classic Newton step on the quotient), three instructions instead of a full
// division each.
__device__ __forceinline__ double div_shared(double a, double b, double r) {
  const double q = a * r;
  return fma(fma(-q, b, a), r, q);
}

// ============================================================================
// Segment mean (fp64).  `pieces` workgroups per segment sum a run of its rows each, in a fixed order; with more than
// one they leave their sums in `mean` for normalise_kernel to add up in order, [segment, piece, D].
// (A few segments: 32 of 8192 points 70 us with one workgroup each, 14 us with eight and four rows in flight, 11 us with
// sixteen and eight; 128 of 1024 points 10 and 7.7 us.  Behind the eights a batch of four: without it 31 of 1000 points
// 8.8 us, 8.0 so, 4192 of 100 26.3 and 25.2.)
// ============================================================================
template <typename T, int D>
__global__ __launch_bounds__(256) void seg_mean_kernel(const T* __restrict__ K, double* __restrict__ mean,
                                                       int32_t* __restrict__ flag_count,
                                                       int32_t* __restrict__ range,
                                                       int32_t* __restrict__ nchanged,
                                                       int32_t* __restrict__ nlisted, int S, int L,
                                                       int kk, int N, int N_idx, int n_sink, int pieces) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = 256 / LPR;
  const int sg = blockIdx.x / pieces, piece = blockIdx.x - sg * pieces;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const int sub = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  if (blockIdx.x == 0 && threadIdx.x == 0) *flag_count = 0;
  if (range && piece == 0 && threadIdx.x < 2) range[2 * sg + threadIdx.x] = threadIdx.x ? 0 : 255;  // for normalise_kernel
  if (range && piece == 0 && threadIdx.x == 0) nchanged[sg] = nlisted[sg] = 0;  // for update_moves_kernel, assign_listed_kernel
  const T* Ku = K + ((size_t)si.unit * N + n_sink + si.seg_start) * D + sub * EPC;
  double acc[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) acc[e] = 0.0;
  const int per = (si.L_s + pieces - 1) / pieces, hi = min(si.L_s, (piece + 1) * per);
  int i = min(si.L_s, piece * per) + grp;
  auto add = [&](auto batch) {  // rows in flight, added in row order
    constexpr int U = decltype(batch)::value;
    for (; i + (U - 1) * GROUPS < hi; i += U * GROUPS) {
      uint4 raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = load16(Ku + (size_t)(i + u * GROUPS) * D);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float f[EPC];
        unpack<T>(raw[u], f);
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] += (double)f[e];
      }
    }
  };
  add(std::integral_constant<int, 8>{});
  add(std::integral_constant<int, 4>{});
  add(std::integral_constant<int, 1>{});
  __shared__ double red[GROUPS][D];
#pragma unroll
  for (int e = 0; e < EPC; ++e) red[grp][sub * EPC + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    double s = 0.0;
    for (int g = 0; g < GROUPS; ++g) s += red[g][threadIdx.x];
    mean[(size_t)blockIdx.x * D + threadIdx.x] = pieces == 1 ? s / (double)si.L_s : s;
  }
}

// Exponent fields of the nonzero elements of a 16-byte chunk: their smallest and largest
// (a subnormal counts as exponent field 1, which has the same unit in the last place).
template <typename T>
__device__ __forceinline__ void exponent_range(const uint4& raw, int& emin, int& emax);
template <>
__device__ __forceinline__ void exponent_range<bf16_t>(const uint4& raw, int& emin, int& emax) {
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t v = h ? w[i] >> 16 : w[i] & 0xffffu;
      if (v & 0x7fffu) {
        const int e = max(1, (int)((v >> 7) & 0xffu));
        emin = min(emin, e);
        emax = max(emax, e);
      }
    }
  }
}
template <>
__device__ __forceinline__ void exponent_range<float>(const uint4& raw, int& emin, int& emax) {
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (w[i] & 0x7fffffffu) {
      const int e = max(1, (int)((w[i] >> 23) & 0xffu));
      emin = min(emin, e);
      emax = max(emax, e);
    }
}
// The same of many chunks of bf16, two elements at a time: add() each chunk, then range().
struct ExponentRange {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  u16x2 least = {0xffff, 0xffff}, most = {0, 0};  // magnitude bits - 1 (zero: the largest), magnitude bits
  __device__ __forceinline__ void add(const uint4& raw) {
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u16x2 mag = __builtin_bit_cast(u16x2, w[i] & 0x7fff7fffu);
      most = __builtin_elementwise_max(most, mag);
      least = __builtin_elementwise_min(least, mag - (unsigned short)1);
    }
  }
  __device__ __forceinline__ void range(int& emin, int& emax) const {
    const int lo = min(least.x, least.y);
    emin = lo == 0xffff ? 255 : max(1, (lo + 1) >> 7);
    emax = max(most.x, most.y) >> 7;
  }
};
template <typename T>
struct MantissaBits;
template <>
struct MantissaBits<bf16_t> {
  static constexpr int value = 7;
};
template <>
struct MantissaBits<float> {
  static constexpr int value = 23;
};

// ============================================================================
// Centre, normalise, round to the storage type.  A workgroup takes `row_step` rows of one
// segment and keeps the mean in registers; HBM-bound (16 sequences x 120K tokens 1.48 ms, 5.4 TB/s; with
// every quotient and rounding in fp64 1.88 ms; with rows of any segment in a workgroup, every lane reading its 64
// bytes of the fp64 mean again for each 16 bytes of key, 2.16 ms).  Four rows of a group in flight where
// that many are left, else one by one: four with repeats of the last one took 485 us for 65536
// segments of 16 rows, 172 us so.
// row_step: 128; 64 where that leaves CUs without a workgroup (2 fp32 segments of 2048 rows 4.8 and 4.0 us, 31 bf16 ones
// of 1000 11.9 and 10.6; 5200 of 100 rows 51.8, in two pieces each 60.9); 256 where these workgroups are all resident
// at once (6 per CU) and those of 128 are not: 32 segments of 8192 rows 42 and 33 us; 1920 of them 1.48 and 1.51 ms.
// With `range` 64 only up to a workgroup a CU, and where the four rows in flight fit: every workgroup adds to the few lines
// of range (d = 128: one segment of 4096 rows 11.3 and 9.3 us, six 15.5 and 17.2; d = 64, 128 rows in flight: three of
// 4096 9.9 and 11.2).
// ============================================================================
constexpr int NORM_ROWS = 128, NORM_RESIDENT = 6 * 256;

template <typename T, int D>
__global__ __launch_bounds__(256) void normalise_kernel(const T* __restrict__ K,
                                                        const double* __restrict__ mean,
                                                        double* __restrict__ mean_out,
                                                        T* __restrict__ xhat, int32_t* __restrict__ range, int S, int L, int kk, int N,
                                                        int N_idx, int n_sink, int chunks, int row_step, int pieces) {
  // mean: of every segment, or with pieces > 1 the sums of its pieces (a segment's first workgroup then leaves
  // the mean in mean_out, where it is without pieces: the workspace holds the same in either form; no later step reads it)
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = 256 / LPR, U = 4;
  const int sub = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  const int sg = blockIdx.x / chunks, chunk = blockIdx.x - sg * chunks;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const int lo = chunk * row_step, hi = min(si.L_s, lo + row_step);
  if (lo >= hi) return;
  // (range: the smallest and the largest exponent field of the segment's nonzero elements)
  __shared__ int seg_emin, seg_emax;
  if (threadIdx.x == 0) {
    seg_emin = 255;
    seg_emax = 0;
  }
  ExponentRange seen;
  __shared__ double mean_s[D];
  if (pieces > 1) {
    if (threadIdx.x < D) {
      double m = 0.0;
#pragma unroll 8
      for (int j = 0; j < pieces; ++j) m += mean[((size_t)sg * pieces + j) * D + threadIdx.x];
      m /= (double)si.L_s;
      mean_s[threadIdx.x] = m;
      if (chunk == 0) mean_out[(size_t)sg * D + threadIdx.x] = m;
    }
    __syncthreads();
  }
  double mu[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) mu[e] = pieces == 1 ? mean[(size_t)sg * D + sub * EPC + e] : mean_s[sub * EPC + e];
  const T* Ku = K + ((size_t)si.unit * N + n_sink + si.seg_start) * D + sub * EPC;
  T* Xu = xhat + ((size_t)si.unit * N_idx + si.seg_start) * D + sub * EPC;
  auto rows = [&](auto batch, int r0) {  // rows r0, r0 + GROUPS, ... below hi, in flight together
    constexpr int N = decltype(batch)::value;
    uint4 raw[N];
#pragma unroll
    for (int u = 0; u < N; ++u) raw[u] = load16(Ku + (size_t)(r0 + u * GROUPS) * D);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      float f[EPC];
      unpack<T>(raw[u], f);
      double x[EPC], n2 = 0.0;
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        x[e] = (double)f[e] - mu[e];
        n2 = fma(x[e], x[e], n2);
      }
      n2 = group_sum_f64<LPR>(n2);
      const double nrm = sqrt(n2);
      const double dv = nrm > 0.0 ? nrm : 1.0;
      const double rdv = 1.0 / dv;
      T o[EPC];
      bool exact = true;  // (the same for the wave)
      if constexpr (sizeof(T) == 2) {
        // In fp32 the quotient is off by three roundings at most (x, 1 / |x|, their product): where that
        // cannot reach the middle between two bf16 values, it rounds as the fp64 quotient does.
        // A zero, as of a channel that is constant in the segment, is one; looked at only where something is unsure
        // (16 sequences x 120K tokens with one such channel: 2.27 ms with both quotients of every row, 1.64 so).
        const float rf = (float)rdv;
        const bool scale_unsure = !(dv > 0x1p-20 && dv < 0x1p100);  // (so that no operand below is subnormal)
        bool unsure = scale_unsure;
        auto quotient_unsure = [](uint32_t u) {
          return (u & 0xffffu) - 0x7ffcu <= 8u ||                               // 4 steps around the middle
                 (u & 0x7fffffffu) - 0x0d800000u >= 0x7f800000u - 0x0d800000u;  // below 2^-100, no number
        };
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
          const uint32_t u = __float_as_uint((float)x[e] * rf);
          unsure |= quotient_unsure(u);
          o[e].bits = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
        }
        exact = __ballot(unsure) != 0;
        if (exact) {
          unsure = scale_unsure;
#pragma unroll
          for (int e = 0; e < EPC; ++e) {
            if (x[e] == 0.0) o[e].bits = 0;
            else unsure |= quotient_unsure(__float_as_uint((float)x[e] * rf));
          }
          exact = __ballot(unsure) != 0;
        }
      }
      if (exact) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) o[e] = quant_store<T>(div_shared(x[e], dv, rdv));
      }
      store16(Xu + (size_t)(r0 + u * GROUPS) * D, *reinterpret_cast<uint4*>(o));
      if (range) seen.add(*reinterpret_cast<uint4*>(o));
    }
  };
  int r0 = lo;
  for (; r0 + U * GROUPS <= hi; r0 += U * GROUPS) rows(std::integral_constant<int, U>{}, r0 + grp);
  for (r0 += grp; r0 < hi; r0 += GROUPS) rows(std::integral_constant<int, 1>{}, r0);
  if (range) {
    int emin, emax;
    seen.range(emin, emax);
    for (int off = 32; off >= 1; off >>= 1) {
      emin = min(emin, __shfl_xor(emin, off));
      emax = max(emax, __shfl_xor(emax, off));
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
      atomicMin(&seg_emin, emin);
      atomicMax(&seg_emax, emax);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      atomicMin(&range[2 * sg], seg_emin);
      atomicMax(&range[2 * sg + 1], seg_emax);
    }
  }
}

// ============================================================================
// Seeded initial centroids: the first k entries of a Fisher-Yates shuffle of the
// segment's positions, without running the shuffle.  The generator's state
// advances by a constant per draw, so draw i is a function of i alone, and so is
// its target j_i = i + draw_i mod (L_s - i).  Step i picks the value found at
// position j_i and leaves position i's value there.  The value at position p
// just before step b (p >= b) is p itself unless an earlier step targeted p; if
// t < b is the latest such step, it is the value position t held before step t.
// Every thread follows that chain for its own i (chains are short: k << L).  The steps are found through
// buckets of their targets.  `pieces` workgroups a segment each know all targets and take a share of the draws;
// eight rows of a group in flight.  (Every earlier step compared, rows one by one, one workgroup for 512 draws: 41 us
// for 32 segments, 127 for 1920; 5.8 and 106 us so, the latter at the rate of its row reads.)
// ============================================================================

template <typename T, int D>
__global__ __launch_bounds__(256) void init_kernel(const T* __restrict__ xhat, T* __restrict__ chat,
                                                   int S, int L, int kk, int N_idx, int Hkv,
                                                   uint64_t seed, int seg_id_base, int pieces, int buckets) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = 256 / LPR;
  const int sg = blockIdx.x / pieces, piece = blockIdx.x - sg * pieces;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  extern __shared__ int init_lds[];  // 3 * kk + buckets ints
  int* target = init_lds;
  int* chosen = target + kk;
  int* next = chosen + kk;           // the steps of a bucket of targets, in no order
  int* head = next + kk;
  for (int i = threadIdx.x; i < buckets; i += 256) head[i] = -1;
  __syncthreads();
  // (seg_id_base: the segments of an index update continue the numbering of the build)
  const uint64_t st0 = init_stream_state(seed, si.unit / Hkv, si.unit % Hkv, si.s + seg_id_base);
  for (int i = threadIdx.x; i < si.k_s; i += 256) {
    uint64_t st = st0 + (uint64_t)i * 0x9E3779B97F4A7C15ull;  // state before draw i
    const uint64_t draw = splitmix64_next(st);
    const int t = i + (int)(draw % (uint64_t)(si.L_s - i));
    target[i] = t;
    next[i] = atomicExch(&head[t & (buckets - 1)], i);
  }
  __syncthreads();
  const int per = (si.k_s + pieces - 1) / pieces, c_lo = min(si.k_s, piece * per), c_hi = min(si.k_s, c_lo + per);
  for (int i = c_lo + threadIdx.x; i < c_hi; i += 256) {
    int cur = target[i], bound = i;
    while (true) {
      int t = -1;  // the latest step before `bound` onto cur
      for (int u = head[cur & (buckets - 1)]; u >= 0; u = next[u])
        if (u < bound && u > t && target[u] == cur) t = u;
      if (t < 0) break;
      cur = t;
      bound = t;
    }
    chosen[i] = cur;
  }
  __syncthreads();
  const int sub = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  const T* X = xhat + ((size_t)si.unit * N_idx + si.seg_start) * D + sub * EPC;
  T* Cs = chat + (size_t)sg * kk * D + sub * EPC;
  constexpr int U = 8;
  for (int c = c_lo + grp; c < c_hi; c += U * GROUPS) {
    uint4 raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u] = load16(X + (size_t)chosen[min(c + u * GROUPS, c_hi - 1)] * D);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u * GROUPS < c_hi) store16(Cs + (size_t)(c + u * GROUPS) * D, raw[u]);
  }
}

// ============================================================================
// Assign, MFMA path (bf16).  A workgroup of NW waves takes NW * 32 * NF points
// of one segment.  Each wave keeps its points as B operands (K x N = 16 x 32 per
// instruction) in registers for the whole kernel and streams the centroids,
// 32 at a time, through a padded LDS tile as A operands (M x K = 32 x 16), so
// D[centroid][point] accumulates in v_mfma_f32_32x32x16_bf16 and a lane holds
// 16 centroid rows of ONE point: the running best / second best never leave the
// lane.  Four of the five bits of the centroid's row inside the tile are written
// over low mantissa bits of the similarity (the fifth is the lane's half), so
// one v_med3 pair carries value and index: 3 VALU instructions per similarity.
// ============================================================================
// Similarities of unit vectors lie in [-1, 1]; the accumulators start at
// kAssignBias so every value is a positive float, whose bit pattern orders like
// a signed integer: max and median then run on the integer pipes, free of the
// NaN handling a float max drags in.
constexpr float kAssignBias = 2.0f;

__device__ __forceinline__ int med3_i32(int a, int b, int c) {
  int r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Difference of two biased similarities (a key of 0: no centroid).
__device__ __forceinline__ float key_gap(int a, int b) { return __int_as_float(a) - __int_as_float(b); }

template <int NF, bool TAIL>
__device__ __forceinline__ void assign_epilogue(const floatx16 (&acc)[NF], int (&best)[NF],
                                                int (&second)[NF], int (&btile)[NF], int t, int half,
                                                int k_s) {
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int before = best[f];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      constexpr uint32_t kClear = ~27u;               // bits 0,1,3,4 carry the row code
      const uint32_t code = 8u * (v / 4) + (v % 4);   // row = code | 4 * half
      int key = (int)((__float_as_uint(acc[f][v]) & kClear) | code);
      if (TAIL && 32 * t + (int)code + 4 * half >= k_s) key = 0;
      second[f] = med3_i32(best[f], second[f], key);
      best[f] = max(best[f], key);
    }
    btile[f] = (best[f] != before) ? t : btile[f];
  }
}

// Lanes l and l ^ 32 hold the same point over disjoint centroid rows: the point's best row
// (returned) and its best and second-best keys over both.
__device__ __forceinline__ int merge_halves(int& best, int& second, int btile, int half) {
  int row = btile * 32 + ((best & 27) | (4 * half));
  const int ob = __shfl_xor(best, 32), os = __shfl_xor(second, 32), orow = __shfl_xor(row, 32);
  second = max(min(best, ob), max(second, os));
  row = ob > best ? orow : row;
  best = max(best, ob);
  return row;
}

template <int D, int NF, int NW>
__global__ __launch_bounds__(64 * NW) void assign_mfma_kernel(
    const bf16_t* __restrict__ xhat, const bf16_t* __restrict__ chat, int32_t* __restrict__ assign,
    int32_t* __restrict__ flag_list, int32_t* __restrict__ flag_count, int S, int L, int kk, int N_idx,
    int wgs_per_seg) {
  constexpr int KS = D / 16;            // MFMA k-steps per tile
  constexpr int PW = 32 * NF;           // points per wave
  constexpr int PWG = NW * PW;          // points per workgroup
  constexpr int NT = 64 * NW;           // threads
  constexpr int ROWB = D * 2 + 16;      // LDS row pitch: 16 B pad keeps 16 lanes on 64 distinct banks
  constexpr int CPR = D / 8;            // 16-byte chunks per centroid row
  constexpr int CHUNKS = 32 * CPR;      // chunks per tile
  constexpr int CPT = (CHUNKS + NT - 1) / NT;  // chunks each thread moves per tile
  __shared__ __attribute__((aligned(16))) char lds[2][32 * ROWB];

  const int wg = xcd_logical_block(blockIdx.x, gridDim.x);
  const int sg = wg / wgs_per_seg, piece = wg - sg * wgs_per_seg;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const int p0 = piece * PWG;
  if (p0 >= si.L_s) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const bf16_t* X = xhat + ((size_t)si.unit * N_idx + si.seg_start) * D;
  const bf16_t* Cs = chat + (size_t)sg * kk * D;

  uint4 bfrag[NF][KS];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int row = min(p0 + wave * PW + 32 * f + col, si.L_s - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) bfrag[f][s] = load16(X + (size_t)row * D + (2 * s + half) * 8);
  }
  int best[NF], second[NF], btile[NF];  // biased similarities as integers; 0 is below all of them
#pragma unroll
  for (int f = 0; f < NF; ++f) best[f] = second[f] = btile[f] = 0;

  const int ntiles = (si.k_s + 31) / 32;
  // Centroid tiles travel global -> registers -> LDS.  Two register stages keep
  // the loads two tiles ahead of the MFMAs that consume them.
  uint4 stage[2][CPT];
  auto gload = [&](int t, uint4 (&st)[CPT]) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int id = tid + NT * i, row = id / CPR, ch = id - row * CPR;
      if (CHUNKS % NT == 0 || id < CHUNKS) {
        const int crow = min(32 * t + row, si.k_s - 1);
        st[i] = load16(Cs + (size_t)crow * D + ch * 8);
      }
    }
  };
  auto sstore = [&](int buf, const uint4 (&st)[CPT]) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int id = tid + NT * i, row = id / CPR, ch = id - row * CPR;
      if (CHUNKS % NT == 0 || id < CHUNKS) store16(&lds[buf][row * ROWB + ch * 16], st[i]);
    }
  };
  auto tile_step = [&](int t, uint4 (&st_next)[CPT], uint4 (&st_load)[CPT]) {
    // st_next holds tile t + 1 (requested one step ago); st_load receives tile t + 2
    if (t + 2 < ntiles) gload(t + 2, st_load);
    floatx16 acc[NF];
    const char* tile = lds[t & 1];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, load16(tile + col * ROWB + (2 * s + half) * 16));
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const bf16x8 bv = __builtin_bit_cast(bf16x8, bfrag[f][s]);
        if (s == 0) {
          constexpr float B0 = kAssignBias;
          const floatx16 bias = {B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0};
          acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bv, bias, 0, 0, 0);
        } else {
          acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bv, acc[f], 0, 0, 0);
        }
      }
    }
    if (32 * t + 32 > si.k_s)
      assign_epilogue<NF, true>(acc, best, second, btile, t, half, si.k_s);
    else
      assign_epilogue<NF, false>(acc, best, second, btile, t, half, si.k_s);
    if (t + 1 < ntiles) sstore((t + 1) & 1, st_next);
    __syncthreads();
  };
  gload(0, stage[0]);
  if (ntiles > 1) gload(1, stage[1]);
  sstore(0, stage[0]);
  __syncthreads();
  for (int t = 0; t < ntiles; t += 2) {
    tile_step(t, stage[1], stage[0]);
    if (t + 1 < ntiles) tile_step(t + 1, stage[0], stage[1]);
  }

#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int crow = merge_halves(best[f], second[f], btile[f], half);
    const int point = p0 + wave * PW + 32 * f + col;
    if (half == 0 && point < si.L_s) {
      const size_t gp = (size_t)si.unit * N_idx + si.seg_start + point;
      assign[gp] = crow;
      if (key_gap(best[f], second[f]) < kAssignGuard) flag_list[atomicAdd(flag_count, 1)] = (int32_t)gp;
    }
  }
}

// ============================================================================
// Assign, MFMA path with the segment's centroids resident in LDS: one workgroup
// of 16 waves copies all k_s centroid rows into LDS once (padded rows, at most
// ~136 KiB) and then every wave works through fragments of 32 * NF points on
// its own: no barrier and no global centroid traffic inside the loop.
// ============================================================================
template <int D>
struct ResidentTile {
  static constexpr int KS = D / 16;        // MFMA k-steps per tile
  static constexpr int ROWB = D * 2 + 16;  // LDS row pitch: 16 B pad keeps 16 lanes on 64 distinct banks
  static constexpr int CPR = D / 8;        // 16-byte chunks per centroid row
};

// `rows` (a multiple of 32) of the centroids Cs into padded LDS rows, row i the centroid source(i), four requests
// of a thread in flight (a request and its store one after the other are a round trip each).
template <int D, int NT, typename Source>
__device__ __forceinline__ void copy_centroids(const bf16_t* Cs, int rows, char* cent, Source&& source) {
  using RT = ResidentTile<D>;
  constexpr int U = 4;
  const int chunks = rows * RT::CPR;
  for (int id0 = threadIdx.x; id0 < chunks; id0 += U * NT) {
    uint4 raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int id = min(id0 + u * NT, chunks - 1);
      raw[u] = load16(Cs + (size_t)source(id / RT::CPR) * D + id % RT::CPR * 8);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int id = min(id0 + u * NT, chunks - 1);
      store16(cent + id / RT::CPR * RT::ROWB + id % RT::CPR * 16, raw[u]);
    }
  }
}

// The segment's k_s centroid rows into the padded LDS tiles (rows beyond k_s repeat the
// last one; the epilogue ignores them).  All NT threads call this; the caller's barrier follows.
template <int D, int NT>
__device__ __forceinline__ void resident_load_centroids(const bf16_t* Cs, int k_s, char* cent) {
  copy_centroids<D, NT>(Cs, 32 * ((k_s + 31) / 32), cent, [&](int row) { return min(row, k_s - 1); });
}

// Wave `wave` of NW takes the fragments f_lo + wave * NF, + NW * NF, ... below f_hi of the
// segment's points X against the centroids in `cent`; emit(point, row, best, second, state) is
// called once per point by the lane that holds it (the keys of its two best rows and the best one's
// number; state: what fetch(point) returned when the point's row was requested).
struct NoState {};
template <int D, int NF, int NW, typename Fetch, typename Emit>
__device__ __forceinline__ void resident_assign_fragments(const bf16_t* X, const char* cent, int L_s, int k_s,
                                                          int f_lo, int f_hi, Fetch&& fetch, Emit&& emit) {
  using RT = ResidentTile<D>;
  constexpr int KS = RT::KS, ROWB = RT::ROWB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int ntiles = (k_s + 31) / 32;
  const int nfull = k_s / 32;  // tiles without rows beyond k_s
  constexpr float B0 = kAssignBias;
  floatx16 bias = {B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0};
  asm volatile("" : "+v"(bias));  // kept in registers: one accumulator-start operand for every tile
  for (int fb = f_lo + wave * NF; fb < f_hi; fb += NW * NF) {
    uint4 bfrag[NF][KS];
    decltype(fetch(0)) state[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int row = min(32 * (fb + f) + col, L_s - 1);
      state[f] = fetch(row);
#pragma unroll
      for (int s = 0; s < KS; ++s) bfrag[f][s] = load16(X + (size_t)row * D + (2 * s + half) * 8);
    }
    int best[NF], second[NF], btile[NF];  // biased similarities as integers; 0 is below all of them
#pragma unroll
    for (int f = 0; f < NF; ++f) best[f] = second[f] = btile[f] = 0;
    auto mfma_tile = [&](int t, floatx16 (&acc)[NF]) {
      const char* tile = cent + (size_t)(32 * t + col) * ROWB + half * 16;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, load16(tile + s * 32));
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          const bf16x8 bv = __builtin_bit_cast(bf16x8, bfrag[f][s]);
          acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bv, s == 0 ? bias : acc[f], 0, 0, 0);
        }
      }
    };
    // One tile's MFMAs are issued between the integer epilogue instructions of
    // the tile before it (two accumulator sets): the matrix pipe works while the
    // vector ALU ranks the previous results.
    auto interleave = [&]() {
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // the first two LDS reads
#pragma unroll
      for (int i = 0; i < KS * NF; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // the LDS read two MFMAs ahead
        __builtin_amdgcn_sched_group_barrier(0x002, 48 / KS, 0);  // a share of the epilogue
      }
    };
    floatx16 accA[NF], accB[NF];
    if (nfull > 0) {
      mfma_tile(0, accA);
      int t = 1;
      for (; t + 1 < nfull; t += 2) {
        mfma_tile(t, accB);
        assign_epilogue<NF, false>(accA, best, second, btile, t - 1, half, k_s);
        interleave();
        mfma_tile(t + 1, accA);
        assign_epilogue<NF, false>(accB, best, second, btile, t, half, k_s);
        interleave();
      }
      if (t < nfull) {
        mfma_tile(t, accB);
        assign_epilogue<NF, false>(accA, best, second, btile, t - 1, half, k_s);
        interleave();
        assign_epilogue<NF, false>(accB, best, second, btile, t, half, k_s);
      } else {
        assign_epilogue<NF, false>(accA, best, second, btile, t - 1, half, k_s);
      }
    }
    if (nfull < ntiles) {  // the last tile has rows beyond k_s
      mfma_tile(nfull, accA);
      assign_epilogue<NF, true>(accA, best, second, btile, nfull, half, k_s);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int row = merge_halves(best[f], second[f], btile[f], half);
      const int point = 32 * (fb + f) + col;
      if (half == 0 && fb + f < f_hi && point < L_s) emit(point, row, best[f], second[f], state[f]);
    }
  }
}

// The same step for few centroid tiles (short segments): one accumulator set and no
// instruction interleaving, the next fragment's rows requested before the current one is
// worked on.  Same similarities, same epilogue, same fetch and emit.  (fetch belongs to the
// requests made ahead: a load issued behind them and used at once would wait for all of them.)
// stage() fills `cent` once the first rows are requested; all threads of the workgroup call this.
template <int D, int NW, typename Fetch, typename Emit, typename Stage>
__device__ __forceinline__ void lean_assign_fragments(const bf16_t* X, const char* cent, int L_s, int k_s,
                                                      int f_lo, int f_hi, Fetch&& fetch, Emit&& emit, Stage&& stage) {
  using RT = ResidentTile<D>;
  constexpr int KS = RT::KS, ROWB = RT::ROWB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int ntiles = (k_s + 31) / 32, nfull = k_s / 32;
  constexpr float B0 = kAssignBias;
  const floatx16 bias = {B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0};
  decltype(fetch(0)) state, next_state;
  auto load_frag = [&](int fb, uint4 (&dst)[KS], decltype(fetch(0))& st) {
    const int row = min(32 * fb + col, L_s - 1);
    st = fetch(row);
#pragma unroll
    for (int s = 0; s < KS; ++s) dst[s] = load16(X + (size_t)row * D + (2 * s + half) * 8);
  };
  uint4 cur[KS], nxt[KS];
  if (f_lo + wave < f_hi) load_frag(f_lo + wave, cur, state);
  stage();
  for (int fb = f_lo + wave; fb < f_hi; fb += NW) {
    if (fb + NW < f_hi) load_frag(fb + NW, nxt, next_state);
    int best[1] = {0}, second[1] = {0}, btile[1] = {0};
    for (int t = 0; t < ntiles; ++t) {
      const char* tile = cent + (size_t)(32 * t + col) * ROWB + half * 16;
      floatx16 acc[1];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, load16(tile + s * 32));
        const bf16x8 bv = __builtin_bit_cast(bf16x8, cur[s]);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bv, s == 0 ? bias : acc[0], 0, 0, 0);
      }
      if (t < nfull) assign_epilogue<1, false>(acc, best, second, btile, t, half, k_s);
      else assign_epilogue<1, true>(acc, best, second, btile, t, half, k_s);
    }
    const int row = merge_halves(best[0], second[0], btile[0], half);
    const int point = 32 * fb + col;
    if (half == 0 && point < L_s) emit(point, row, best[0], second[0], state);
#pragma unroll
    for (int s = 0; s < KS; ++s) cur[s] = nxt[s];
    state = next_state;
  }
}

// The same for segments whose points a workgroup holds in registers from round to round: KEEP fragments
// per wave, fragment f of wave w is the segment's f * NW + w.
template <int D, int KEEP, int NW>
__device__ __forceinline__ void load_kept_fragments(const bf16_t* X, int L_s, uint4 (&kept)[KEEP][D / 16]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int f = 0; f < KEEP; ++f) {
    const int row = min(32 * (f * NW + wave) + (lane & 31), L_s - 1);
#pragma unroll
    for (int s = 0; s < D / 16; ++s) kept[f][s] = load16(X + (size_t)row * D + (2 * s + (lane >> 5)) * 8);
  }
}

// Fragments f0 and f0 + NW of the segment against all centroids: a pair shares the reads of a tile (with
// one fragment at a time the reads take as long as the matrix instructions).
template <int D, int NW, typename Emit>
__device__ __forceinline__ void assign_pair(const uint4 (&x0)[D / 16], const uint4 (&x1)[D / 16], int f0,
                                            const char* cent, int L_s, int k_s, Emit&& emit) {
  using RT = ResidentTile<D>;
  constexpr int KS = RT::KS, ROWB = RT::ROWB;
  const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int ntiles = (k_s + 31) / 32, nfull = k_s / 32;
  constexpr float B0 = kAssignBias;
  const floatx16 bias = {B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0};
  int best[2] = {}, second[2] = {}, btile[2] = {};
  for (int t = 0; t < ntiles; ++t) {
    const char* tile = cent + (size_t)(32 * t + col) * ROWB + half * 16;
    floatx16 acc[2];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, load16(tile + s * 32));
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, x0[s]), s == 0 ? bias : acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, x1[s]), s == 0 ? bias : acc[1], 0, 0, 0);
    }
    if (t < nfull) assign_epilogue<2, false>(acc, best, second, btile, t, half, k_s);
    else assign_epilogue<2, true>(acc, best, second, btile, t, half, k_s);
  }
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int row = merge_halves(best[f], second[f], btile[f], half);
    const int point = 32 * (f0 + f * NW) + col;
    if (half == 0 && point < L_s) emit(point, row, best[f], second[f], NoState{});
  }
}

template <int D, int KEEP, int NW, typename Emit>
__device__ __forceinline__ void assign_kept_fragments(const uint4 (&kept)[KEEP][D / 16], const char* cent, int L_s,
                                                      int k_s, Emit&& emit) {
  const int wave = threadIdx.x >> 6;
  static_assert(KEEP % 2 == 0, "whole pairs");
#pragma unroll
  for (int f = 0; f < KEEP; f += 2) {
    if (32 * (f * NW + wave) >= L_s) break;
    assign_pair<D, NW>(kept[f], kept[f + 1], f * NW + wave, cent, L_s, k_s, emit);
  }
}

// What the assign step of one round leaves for the next about a point: the key of its cluster's
// similarity and a key that no other centroid's similarity exceeds (both up to the fp32 error).
// (A unit's bounds start `bounds_skip` entries further on than the units' points are counted.)
struct __attribute__((aligned(8))) PointBounds {
  int own, others;
};

struct PointState {
  int cluster;
  PointBounds bounds;
};

// A point that changed its cluster in round t carries (t, the cluster it left) in prev[].
constexpr int PREV_CLUSTER_BITS = 11;  // (at most 1024 centroids are resident)
constexpr int PREV_ROUNDS = 1 << (31 - PREV_CLUSTER_BITS);  // rounds that fit beside them in an int

// The round's outcome for a point that was in cluster `before`.  bounds: null when no later round
// needs it (nor prev, nor `before`).
__device__ __forceinline__ void settle_point(int32_t* assign, int32_t* prev, PointBounds* bounds, int round,
                                             size_t gp, int before, int cluster, int own, int others) {
  if (bounds) {
    bounds[gp] = PointBounds{own, others};
    if (before != cluster)
      prev[gp] = round << PREV_CLUSTER_BITS | before;
    else if (round == 1)
      prev[gp] = 0;  // (the first round to leave marks: every point's are set)
    if (before == cluster) return;
  }
  assign[gp] = cluster;
}

constexpr int ASSIGN_POINTS = 4096;  // most points of a workgroup of the resident kernels
// A workgroup's list of points for assign_listed_kernel goes behind what is there of its segment's.
__device__ __forceinline__ void publish_list(const uint16_t* left, int n, int first, int32_t* list, int32_t* count) {
  __shared__ int at;
  if (n == 0) return;  // (the same for the whole workgroup)
  if (threadIdx.x == 0) at = atomicAdd(count, n);
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) list[at + i] = first + left[i];
}

// ============================================================================
// Points that need every centroid (near-ties of a full pass; what a later round's bounds leave open): up to
// LIST_POINTS of a segment at a time, by the NW waves of a workgroup.  point(i) is the i-th of n points.
// The points' rows are staged in LDS, the waves share out the centroid tiles, read from the
// cache, and the tiles' best two are merged per point.  A point whose two best are closer than the
// guard gets fp64 similarities (exact for the stored operands up to fp64 rounding, ties to
// the lowest centroid) of the centroids in every tile whose best is that close, one lane per
// centroid; the bound on its other similarities is then `best` too.
// ============================================================================
constexpr int LIST_POINTS = 64;

// (the rows, then per (tile, point): best, second, row)
template <int D>
constexpr size_t listed_lds(int kmax) {
  return (size_t)LIST_POINTS * ResidentTile<D>::ROWB + sizeof(int) * 3 * LIST_POINTS * (size_t)((kmax + 31) / 32);
}

template <int D, int NW, typename Point, typename Settle>
__device__ __forceinline__ void assign_listed_batch(const bf16_t* X, const bf16_t* Cs, int k_s, int n, char* rows,
                                                    Point&& point, Settle&& settle) {
  using RT = ResidentTile<D>;
  constexpr int KS = RT::KS, ROWB = RT::ROWB, CPR = RT::CPR, FRAGS = LIST_POINTS / 32;
  int* part = reinterpret_cast<int*>(rows + LIST_POINTS * ROWB);
  __shared__ int near_p[LIST_POINTS], near_best[LIST_POINTS], near_row[LIST_POINTS], nnear;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int ntiles = (k_s + 31) / 32;
  if (tid == 0) nnear = 0;
  uint4 a[KS];
  auto load_tile = [&](int t) {
    const bf16_t* cr = Cs + (size_t)min(32 * t + col, k_s - 1) * D + half * 8;
#pragma unroll
    for (int s = 0; s < KS; ++s) a[s] = load16(cr + 16 * s);
  };
  if (wave < ntiles) load_tile(wave);
  for (int id = tid; id < LIST_POINTS * CPR; id += 64 * NW) {
    const int p = id / CPR, ch = id - p * CPR;
    store16(rows + p * ROWB + ch * 16, load16(X + (size_t)point(min(p, n - 1)) * D + ch * 8));
  }
  __syncthreads();
  for (int t = wave; t < ntiles; t += NW) {
    constexpr float B0 = kAssignBias;
    floatx16 acc[FRAGS];
#pragma unroll
    for (int f = 0; f < FRAGS; ++f) acc[f] = {B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0, B0};
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int f = 0; f < FRAGS; ++f)
        acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, a[s]),
            __builtin_bit_cast(bf16x8, load16(rows + (32 * f + col) * ROWB + (2 * s + half) * 16)), acc[f], 0, 0, 0);
    if (t + NW < ntiles) load_tile(t + NW);
    int best[FRAGS] = {}, second[FRAGS] = {}, btile[FRAGS] = {};
    assign_epilogue<FRAGS, true>(acc, best, second, btile, t, half, k_s);
#pragma unroll
    for (int f = 0; f < FRAGS; ++f) {
      const int row = merge_halves(best[f], second[f], btile[f], half);
      if (half == 0) {
        int* o = part + (t * LIST_POINTS + 32 * f + col) * 3;
        o[0] = best[f];
        o[1] = second[f];
        o[2] = row;
      }
    }
  }
  __syncthreads();
  if (tid < LIST_POINTS && tid < n) {
    const int* mine = part + tid * 3;
    int best = mine[0], second = mine[1], row = mine[2];
#pragma unroll 4
    for (int t = 1; t < ntiles; ++t) {
      const int* o = mine + t * LIST_POINTS * 3;
      second = max(max(second, o[1]), min(best, o[0]));
      row = o[0] > best ? o[2] : row;
      best = max(best, o[0]);
    }
    if (key_gap(best, second) < kAssignGuard) {
      const int q = atomicAdd(&nnear, 1);
      near_p[q] = tid;
      near_best[q] = best;
      near_row[q] = row;
    } else {
      settle(point(tid), row, best, second);
    }
  }
  __syncthreads();
  for (int q = wave; q < nnear; q += NW) {
    const int p = near_p[q], best = near_best[q];
    uint64_t close = __ballot(lane < ntiles &&
                              key_gap(best, part[(min(lane, ntiles - 1) * LIST_POINTS + p) * 3]) < kAssignGuard);
    double bv = -1.0e300;
    int bc = 0x7fffffff;
    while (close) {  // two tiles at a time, one per half of the wave
      const int t0 = __ffsll((unsigned long long)close) - 1;
      close &= close - 1;
      const int t1 = close ? __ffsll((unsigned long long)close) - 1 : t0;
      close &= close - 1;
      const int c = 32 * (half ? t1 : t0) + col;
      const bf16_t* cr = Cs + (size_t)min(c, k_s - 1) * D;
      double acc = 0.0;
#pragma unroll D / 16
      for (int e0 = 0; e0 < D; e0 += 8) {
        float xf[8], cf[8];
        unpack<bf16_t>(load16(rows + p * ROWB + e0 * 2), xf);
        unpack<bf16_t>(load16(cr + e0), cf);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = fma((double)xf[e], (double)cf[e], acc);
      }
      if (c < k_s && acc > bv) {  // (c ascends within a lane: strict > keeps the lowest)
        bv = acc;
        bc = c;
      }
    }
    for (int off = 32; off >= 1; off >>= 1) {
      const double ov = __shfl_xor(bv, off);
      const int oc = __shfl_xor(bc, off);
      if (ov > bv || (ov == bv && oc < bc)) {
        bv = ov;
        bc = oc;
      }
    }
    // (nothing comparable: the fp32 decision stands)
    if (lane == 0) settle(point(p), bc < k_s ? bc : near_row[q], best, best);
  }
  __syncthreads();
}

// The n points of a workgroup's own list (from point `first` of the segment on).
template <int D, int NW, typename Settle>
__device__ __forceinline__ void settle_left(const bf16_t* X, const bf16_t* Cs, int k_s, const uint16_t* left, int n,
                                            int first, char* rows, Settle&& settle) {
  for (int b0 = 0; b0 < n; b0 += LIST_POINTS)  // (the same for the whole workgroup)
    assign_listed_batch<D, NW>(X, Cs, k_s, n - b0, rows, [&](int i) { return first + left[b0 + i]; }, settle);
}

// `rows` padded centroid rows, with room for a batch of listed points in their place (at_once).
template <int D>
constexpr size_t rows_lds(int rows, int kmax, bool at_once) {
  const size_t held = (size_t)rows * ResidentTile<D>::ROWB, batch = at_once ? listed_lds<D>(kmax) : 0;
  return held > batch ? held : batch;
}

template <int D>
inline size_t resident_lds(int kmax, bool at_once) {
  return rows_lds<D>(32 * ((kmax + 31) / 32), kmax, at_once) + sizeof(uint16_t) * ASSIGN_POINTS;
}

template <int D, int NF, int NW, bool AT_ONCE>
__global__ __launch_bounds__(64 * NW) void assign_resident_kernel(
    const bf16_t* __restrict__ xhat, const bf16_t* __restrict__ chat, int32_t* __restrict__ assign,
    int32_t* __restrict__ prev, PointBounds* bounds, long long bounds_skip, int32_t* __restrict__ listed,
    int32_t* __restrict__ nlisted, int32_t* __restrict__ nflag, int round, int S, int L, int kk, int N_idx,
    int pieces_per_seg) {
  // Near-ties are decided here (AT_ONCE), or go to a list per segment in `listed`, for assign_listed_kernel, or
  // (nlisted null) to one for all segments, counted by nflag, for refine_kernel (which may leave the fp32 decision).
  // LDS: 32 * ceil(k_s / 32) padded rows, then the workgroup's near-ties
  extern __shared__ __attribute__((aligned(16))) char cent[];
  __shared__ int nleft;

  const int wg = xcd_logical_block(blockIdx.x, gridDim.x);
  const int sg = wg / pieces_per_seg, piece = wg - sg * pieces_per_seg;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const int nfrag = (si.L_s + 31) / 32;
  const int per = ((nfrag + pieces_per_seg - 1) / pieces_per_seg + NF - 1) / NF * NF;
  const int f_lo = piece * per, f_hi = min(nfrag, f_lo + per);
  if (f_lo >= f_hi) return;
  const size_t gp0 = (size_t)si.unit * N_idx + si.seg_start;
  if (bounds) bounds += si.unit * bounds_skip;
  const bf16_t* X = xhat + gp0 * D;
  const bf16_t* Cs = chat + (size_t)sg * kk * D;
  uint16_t* left = reinterpret_cast<uint16_t*>(cent + rows_lds<D>(32 * ((si.k_s + 31) / 32), si.k_s, AT_ONCE));
  if (threadIdx.x == 0) nleft = 0;
  resident_load_centroids<D, 64 * NW>(Cs, si.k_s, cent);
  __syncthreads();
  auto settle = [&](int point, int cluster, int own, int others) {
    settle_point(assign, prev, bounds, round, gp0 + point, bounds ? assign[gp0 + point] : 0, cluster, own, others);
  };
  resident_assign_fragments<D, NF, NW>(X, cent, si.L_s, si.k_s, f_lo, f_hi, [](int) { return NoState{}; },
                                       [&](int point, int cluster, int best, int second, NoState) {
                                         const bool near = key_gap(best, second) < kAssignGuard;
                                         if (near) left[atomicAdd(&nleft, 1)] = (uint16_t)(point - 32 * f_lo);
                                         if (!near || (!AT_ONCE && !nlisted)) settle(point, cluster, best, second);
                                       });
  __syncthreads();
  if constexpr (AT_ONCE)
    settle_left<D, NW>(X, Cs, si.k_s, left, nleft, 32 * f_lo, cent, settle);
  else if (nlisted)
    publish_list(left, nleft, 32 * f_lo, listed + gp0, &nlisted[sg]);
  else
    publish_list(left, nleft, (int)gp0 + 32 * f_lo, listed, nflag);
}

// ============================================================================
// Assign, later rounds: only the centroids that the update recomputed (`changed`) are
// compared with the points; every other similarity is what it was.  With `own` and `others`
// of PointBounds and c1, c2 the two best similarities over the changed centroids:
//   own centroid unchanged   c1 below own: the point stays; c1 above own: it moves to c1's
//   own centroid changed     c1 above `others`: no unchanged centroid can beat it, c1's cluster;
//                            otherwise the point is compared with every centroid
// each by more than the guard of the fp32 similarities; what is closer is compared with every
// centroid as well (assign_listed_kernel).  (A near-tie that was decided in fp64 stays decided while no changed centroid
// comes near.)  So the partition is, in every round, the one
// that the full comparison gives.
// The share of changed centroids falls from 82 % in the third round to 3 % in the tenth on
// 8192-token segments of 512 clusters, and 1 % of the points need every centroid: a round costs
// between a full pass and reading xhat once (16 sequences x 120K tokens: 1.9 ms full, 0.8 ms
// at the streaming rate).
//
// A workgroup lists the changed centroids of a segment, copies their rows into LDS and streams
// a share of the segment's points past them as in the kernel above, two accumulator sets while
// many tiles make the matrix pipe the bound, else the next fragment's rows requested ahead.
// Points that need every centroid are listed for assign_listed_kernel, or (AT_ONCE: a few segments,
// where a launch costs more than the listed points) compared when the workgroup has streamed its points;
// its first rows are then always requested before the list of changed centroids is made (a late round of
// 32 segments of 8192 points: three launches of 4.5 + 16 + 12 us, 25 us so; 31 us without the rows requested ahead).
// Two launches share the segments by their number of changed centroids: up to
// delta_light_rows a workgroup of 8 waves needs half of a CU's LDS, so that one workgroup's start
// and end (chains of short dependent steps, 10 .. 25 us) run under another's streaming;
// segments with more take a whole CU with 16 waves.
// ============================================================================
constexpr int LIGHT_POINTS = 2048;

template <int D>
constexpr int delta_light_rows() {
  return D == 128 ? 256 : 512;  // 68 / 72 KiB of rows
}

template <int D>
inline size_t delta_lds(int kmax, int rows, int points, bool at_once) {
  const size_t padded = 32 * (size_t)((kmax + 31) / 32);
  const size_t held = padded < (size_t)rows ? padded : rows;
  return rows_lds<D>((int)held, kmax, at_once) + padded / 8 + sizeof(uint16_t) * (held + points);
}

// The segments with lo < (changed centroids) <= hi; `hi` rows (or all, if fewer) fit in LDS.
template <int D, int NW, bool AT_ONCE>
__global__ __launch_bounds__(64 * NW, 4) void assign_delta_kernel(
    const bf16_t* __restrict__ xhat, const bf16_t* __restrict__ chat, int32_t* __restrict__ assign,
    int32_t* __restrict__ prev, PointBounds* all_bounds, long long bounds_skip, const int32_t* __restrict__ changed,
    const int32_t* __restrict__ nchanged, int32_t* __restrict__ listed, int32_t* __restrict__ nlisted, int lo,
    int hi, int round, int S, int L, int kk, int N_idx,
    int pieces_per_seg, int total) {
  constexpr int NT = 64 * NW;
  extern __shared__ __attribute__((aligned(16))) char cent[];
  __shared__ int wave_n[NW], nleft;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!AT_ONCE && total <= 64 * (long long)gridDim.x) {
    // whether any segment is this launch's is seen at once, not segment by segment (usually none after a few rounds: 8 us a
    // launch of 256 workgroups with 15 segments each, 5 so)
    const long long w = xcd_logical_block(blockIdx.x, gridDim.x) + lane * (long long)gridDim.x;
    const int nch = nchanged[(w < total ? (int)w : total - 1) / pieces_per_seg];
    if (!__ballot(w < total && nch > lo && nch <= hi)) return;
  }
  for (int wg = xcd_logical_block(blockIdx.x, gridDim.x); wg < total; wg += AT_ONCE ? total : gridDim.x) {
    const int sg = wg / pieces_per_seg, piece = wg - sg * pieces_per_seg;
    const int nch = nchanged[sg];
    if (nch <= lo || nch > hi) continue;  // (the same for the whole workgroup)
    const SegInfo si = seg_info(sg, S, L, kk, N_idx);
    const int nfrag = (si.L_s + 31) / 32;
    const int per = (nfrag + pieces_per_seg - 1) / pieces_per_seg;
    const int f_lo = piece * per, f_hi = min(nfrag, f_lo + per);
    if (f_lo >= f_hi) continue;
    const int ntiles_all = (si.k_s + 31) / 32, held = min(32 * ntiles_all, hi);
    uint32_t* marks = reinterpret_cast<uint32_t*>(cent + rows_lds<D>(held, si.k_s, AT_ONCE));  // one bit per centroid
    uint16_t* list = reinterpret_cast<uint16_t*>(marks + ntiles_all);           // changed centroids
    uint16_t* left = list + held;                                               // points for the full comparison
    const size_t gp0 = (size_t)si.unit * N_idx + si.seg_start;
    PointBounds* bounds = all_bounds + si.unit * bounds_skip;
    const bf16_t* X = xhat + gp0 * D;
    const bf16_t* Cs = chat + (size_t)sg * kk * D;

    // the changed centroids, in ascending order, and their rows
    const int first_mark = tid < si.k_s ? changed[(size_t)sg * kk + tid] : 0;  // (requested before the points' rows)
    auto stage = [&]() {
      if (tid == 0) nleft = 0;
      int n = 0;
      for (int c0 = 0; c0 < si.k_s; c0 += NT) {
        const int c = c0 + tid;
        const bool on = c < si.k_s && (c0 == 0 ? first_mark : changed[(size_t)sg * kk + c]) != 0;
        const uint64_t mk = __ballot(on);
        if (lane == 0) {
          wave_n[wave] = __popcll(mk);
          if (c < 32 * ntiles_all) marks[c / 32] = (uint32_t)mk;
          if (c + 32 < 32 * ntiles_all) marks[c / 32 + 1] = (uint32_t)(mk >> 32);
        }
        __syncthreads();
        int base = n;
        for (int w = 0; w < NW; ++w) {
          base += w < wave ? wave_n[w] : 0;
          n += wave_n[w];
        }
        if (on) list[base + __popcll(mk & ((1ull << lane) - 1ull))] = (uint16_t)c;
        __syncthreads();
      }
      copy_centroids<D, NT>(Cs, (nch + 31) / 32 * 32, cent, [&](int row) { return list[min(row, nch - 1)]; });
      __syncthreads();
    };

    auto fetch = [&](int point) { return PointState{assign[gp0 + point], bounds[gp0 + point]}; };
    auto decide = [&](int point, int row, int c1, int c2, const PointState& ps) {
      const size_t gp = gp0 + point;
      const int own_c = ps.cluster;
      const PointBounds pb = ps.bounds;
      const bool own_changed = (marks[own_c / 32] >> (own_c & 31)) & 1u;
      if (!own_changed && key_gap(pb.own, c1) > kAssignGuard) {
        if (c1 > pb.others) bounds[gp].others = c1;
        return;
      }
      const int rest = max(own_changed ? pb.others : max(pb.own, pb.others), c2);
      if (key_gap(c1, rest) > kAssignGuard)
        settle_point(assign, prev, bounds, round, gp, own_c, list[row], c1, rest);
      else
        left[atomicAdd(&nleft, 1)] = (uint16_t)(point - 32 * f_lo);
    };
    if (AT_ONCE || nch <= 64) {
      lean_assign_fragments<D, NW>(X, cent, si.L_s, nch, f_lo, f_hi, fetch, decide, stage);
    } else {
      stage();
      resident_assign_fragments<D, 1, NW>(X, cent, si.L_s, nch, f_lo, f_hi, fetch, decide);
    }
    __syncthreads();
    if constexpr (AT_ONCE) {
      settle_left<D, NW>(X, Cs, si.k_s, left, nleft, 32 * f_lo, cent, [&](int point, int cluster, int own, int others) {
        settle_point(assign, prev, bounds, round, gp0 + point, assign[gp0 + point], cluster, own, others);
      });
    } else {
      publish_list(left, nleft, 32 * f_lo, listed + gp0, &nlisted[sg]);
      __syncthreads();
    }
  }
}

// ============================================================================
// Assign, the points that the kernels above list, where they are not decided at once.
// A workgroup of four waves takes LIST_POINTS at a time; a segment's list is shared by LIST_SPLIT
// workgroups (the lists are uneven: a large cluster whose centroid moved can put a thousand points on
// one), the first shares of all segments before the second ones, most of which are empty.
// (A chain of short dependent steps.  At the end of each listing workgroup, in the LDS that it
// holds, the same steps added 270 .. 400 us to a round of a large batch that streams its points in 700 us.)
// ============================================================================
constexpr int LIST_SPLIT = 16;

template <int D>
__global__ __launch_bounds__(256, 4) void assign_listed_kernel(
    const bf16_t* __restrict__ xhat, const bf16_t* __restrict__ chat, int32_t* __restrict__ assign,
    int32_t* __restrict__ prev, PointBounds* bounds, long long bounds_skip, const int32_t* __restrict__ listed,
    const int32_t* __restrict__ nlisted, int32_t* __restrict__ nlisted_next, int round, int segs, int S, int L,
    int kk, int N_idx) {
  extern __shared__ __attribute__((aligned(16))) char rows[];
  const int share = blockIdx.x / segs, sg = blockIdx.x - share * segs;
  if (share == 0 && threadIdx.x == 0) nlisted_next[sg] = 0;
  const int n = nlisted[sg];
  if (share * LIST_POINTS >= n) return;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const size_t gp0 = (size_t)si.unit * N_idx + si.seg_start;
  const int32_t* left = listed + gp0;
  if (bounds) bounds += si.unit * bounds_skip;
  auto settle = [&](int point, int cluster, int own, int others) {
    settle_point(assign, prev, bounds, round, gp0 + point, bounds ? assign[gp0 + point] : 0, cluster, own, others);
  };
  for (int b0 = share * LIST_POINTS; b0 < n; b0 += LIST_SPLIT * LIST_POINTS)
    assign_listed_batch<D, 4>(xhat + gp0 * D, chat + (size_t)sg * kk * D, si.k_s, n - b0, rows,
                              [&](int i) { return left[b0 + i]; }, settle);
}

// ============================================================================
// Refine: every flagged point gets its argmax from fp64 similarities (exact for
// the stored operands up to fp64 rounding), ties to the lowest centroid.
// ============================================================================
// The argmax of the k_s fp64 similarities of one point (row x) by the 256 threads of a workgroup, ties to
// the lowest centroid; thread 0 has it, 0x7fffffff where no similarity is comparable.
template <typename T, int D>
__device__ __forceinline__ int refine_point(const T* __restrict__ x, const T* __restrict__ Cs, int k_s) {
  __shared__ double xs[D];
  __shared__ double bval[4];
  __shared__ int bidx[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (threadIdx.x < D) xs[threadIdx.x] = to_f64(x[threadIdx.x]);
  __syncthreads();
  double bv = -1.0e300;
  int bi = 0x7fffffff;
  for (int c = threadIdx.x; c < k_s; c += 256) {
    const T* row = Cs + (size_t)c * D;
    double a = 0.0;
    constexpr int EPC = Elem<T>::EPC;
#pragma unroll 2
    for (int e0 = 0; e0 < D; e0 += 4 * EPC) {  // 16-byte chunks, summed in index order
      uint4 raw[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) raw[u] = load16(row + e0 + u * EPC);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float f[EPC];
        unpack<T>(raw[u], f);
#pragma unroll
        for (int e = 0; e < EPC; ++e) a = fma(xs[e0 + u * EPC + e], (double)f[e], a);
      }
    }
    if (a > bv) {  // c ascends within a thread, so strict > keeps the lowest index
      bv = a;
      bi = c;
    }
  }
  for (int off = 32; off >= 1; off >>= 1) {
    const double ov = __shfl_xor(bv, off);
    const int oi = __shfl_xor(bi, off);
    if (ov > bv || (ov == bv && oi < bi)) {
      bv = ov;
      bi = oi;
    }
  }
  if (lane == 0) {
    bval[wave] = bv;
    bidx[wave] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < 4; ++w)
      if (bval[w] > bv || (bval[w] == bv && bidx[w] < bi)) {
        bv = bval[w];
        bi = bidx[w];
      }
  return bi;
}

template <typename T, int D>
__global__ __launch_bounds__(256) void refine_kernel(const T* __restrict__ xhat, const T* __restrict__ chat,
                                                     int32_t* __restrict__ assign,
                                                     const int32_t* __restrict__ flag_list,
                                                     const int32_t* __restrict__ flag_count, int S,
                                                     int L, int kk, int N_idx) {
  const int n = *flag_count;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const int gp = flag_list[it];
    const int unit = gp / N_idx, pos = gp - unit * N_idx;
    const int s = pos / L;
    const int L_s = min(L, N_idx - s * L), k_s = min(kk, L_s);
    const int bi = refine_point<T, D>(xhat + (size_t)gp * D, chat + ((size_t)unit * S + s) * kk * D, k_s);
    if (threadIdx.x == 0 && bi < k_s) assign[gp] = bi;  // (no similarity is comparable: the point stays where it is)
  }
}

// fp64 similarities of P points with one row each lane, summed in index order.
template <int D, int P>
__device__ __forceinline__ void similarities_f64(const float* const (&x)[P], const float* row, double (&a)[P]) {
#pragma unroll P == 1 ? 4 : 2
  for (int e0 = 0; e0 < D; e0 += 8) {
    float f[8];
    unpack<float>(load16(row + e0), *reinterpret_cast<float(*)[4]>(f));
    unpack<float>(load16(row + e0 + 4), *reinterpret_cast<float(*)[4]>(f + 4));
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) a[j] = fma((double)x[j][e0 + e], (double)f[e], a[j]);
  }
}

// Near-ties of f32 builds, decided by the workgroup that finds them: the n points near_p[] of a segment (rows X, centroids
// Cs) get the argmax of their fp64 similarities, ties to the lowest centroid.  One, two or four of the four waves share out
// the centroids, by their number; the others take other points.  A wave compares up to four points with every row
// that it reads.  (A row per lane is a cache line per lane: with one point at a time the reads are the bound.  Builds of
// few segments whose points are all near-ties, six rounds, the points one after the other by the workgroup and so:
// 2 segments of 2048 points x 128 clusters x 64 channels 633 -> 358 us, 1 of 1024 x 64 x 128 938 -> 216 us.)
template <int D>
__device__ __forceinline__ void settle_near_f32(const float* __restrict__ X, const float* __restrict__ Cs, int k_s,
                                                const int* near_p, int n, int32_t* __restrict__ assign) {
  constexpr int NW = 4, MOST = 4;
  __shared__ double bval[NW][MOST];
  __shared__ int bidx[NW][MOST];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int shares = k_s > 128 ? 4 : k_s > 64 ? 2 : 1;  // waves that share out the centroids
  const int pgroups = NW / shares, share = wave % shares, pgroup = wave / shares;
  auto pass = [&](auto points, int i0) {  // the points i0 + j * pgroups + pgroup, j < P, those past the end again
    constexpr int P = decltype(points)::value;
    const float* x[P];
    double bv[P];
    int bi[P];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int p = near_p[min(i0 + j * pgroups + pgroup, n - 1)];
      x[j] = X + (size_t)__builtin_amdgcn_readfirstlane(p) * D;
      bv[j] = -1.0e300;
      bi[j] = 0x7fffffff;
    }
    for (int c0 = 64 * share; c0 < k_s; c0 += 64 * shares) {
      const int c = c0 + lane;
      const float* row = Cs + (size_t)min(c, k_s - 1) * D;
      double a[P] = {};
      similarities_f64<D, P>(x, row, a);
#pragma unroll
      for (int j = 0; j < P; ++j)
        if (c < k_s && a[j] > bv[j]) {  // c ascends within a lane, so strict > keeps the lowest index
          bv[j] = a[j];
          bi[j] = c;
        }
    }
#pragma unroll
    for (int j = 0; j < P; ++j) {
      for (int off = 32; off >= 1; off >>= 1) {
        const double ov = __shfl_xor(bv[j], off);
        const int oi = __shfl_xor(bi[j], off);
        if (ov > bv[j] || (ov == bv[j] && oi < bi[j])) {
          bv[j] = ov;
          bi[j] = oi;
        }
      }
      if (lane == 0) {
        bval[wave][j] = bv[j];
        bidx[wave][j] = bi[j];
      }
    }
    __syncthreads();
    const int t = threadIdx.x, j = t / pgroups, first = t % pgroups * shares;  // point t, its shares' waves
    if (t < P * pgroups && i0 + t < n) {
      double v = bval[first][j];
      int c = bidx[first][j];
      for (int w = first + 1; w < first + shares; ++w)
        if (bval[w][j] > v || (bval[w][j] == v && bidx[w][j] < c)) {
          v = bval[w][j];
          c = bidx[w][j];
        }
      if (c < k_s) assign[near_p[i0 + t]] = c;  // (no similarity is comparable: the point stays where it is)
    }
    __syncthreads();
  };
  int i0 = 0;
  for (; n - i0 > pgroups; i0 += MOST * pgroups) pass(std::integral_constant<int, MOST>{}, i0);
  if (i0 < n) pass(std::integral_constant<int, 1>{}, i0);
}

// ============================================================================
// Assign, f32: workgroups of four waves on v_mfma_f32_32x32x2_f32 (fp32 products and sums).  A wave keeps 32
// points in registers as B operands; the centroids are A operands
// read from the cache: a tile of 32 rows is 128 .. 256 bytes per lane for 2048 .. 4096 cycles of the
// matrix pipe, which is the bound.  Component i of the 16-byte chunks of the wave's two halves is one
// k pair; the order of k inside a dot product is free as long as both operands agree.  A lane holds
// 16 centroids of one point; the ranking is in plain floats (inputs of any length are ranked).
// SPLIT: the four waves have the same points and share out the tiles (fewer than 1024 fragments of points,
// one per SIMD, else leave SIMDs idle); else each wave has its own points and all tiles.
// Points whose two best are closer than the guard are decided here, from fp64 similarities.
// (4096 tokens x 128 clusters x 64 channels, a round: one point per thread with a chain of fp32 FMAs 60 us; one
// wave per 32 points with all tiles and the near-ties in a launch of their own 11.4 + 3; 4.9 us so.  Split
// with 8192 fragments, 64 clusters x 128 channels: 92 us, not split 67.  Builds around the line, split and not: 768
// fragments x 512 clusters 410 and 525 us, x 64 557 and 568; 896 x 128 209 and 205, 1024 x 128 211 and 203, 1024 x 512
// 469 and 520.)  Four waves a SIMD at 128 channels, without accumulation registers: 128 segments of 4096 points x 256
// clusters 2.57 -> 2.31 ms; at 64 channels (two segments, 4096 clusters) that loses 3 %.
// ============================================================================
template <int D, bool SPLIT>
__global__ __launch_bounds__(256, D == 128 ? 4 : 1) void assign_f32_kernel(
    const float* __restrict__ xhat, const float* __restrict__ chat, int32_t* __restrict__ assign, int S, int L, int kk,
    int N_idx, int wgs_per_seg) {
  constexpr int KS = D / 8, NW = 4;  // pairs of 16-byte chunks, one per half of the wave
  constexpr int FRAGS = SPLIT ? 1 : NW;
  __shared__ float part_best[SPLIT ? NW : 1][32], part_second[SPLIT ? NW : 1][32];
  __shared__ int part_row[SPLIT ? NW : 1][32];
  __shared__ int near_p[32 * FRAGS], near_n;
  const int wg = xcd_logical_block(blockIdx.x, gridDim.x);
  const int sg = wg / wgs_per_seg, wg_frag = (wg - sg * wgs_per_seg) * FRAGS;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  if (32 * wg_frag >= si.L_s) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, col = lane & 31;
  const int frag = wg_frag + (SPLIT ? 0 : wave);
  const size_t gp0 = (size_t)si.unit * N_idx + si.seg_start;
  const float* xr = xhat + (gp0 + min(32 * frag + col, si.L_s - 1)) * D + half * 4;
  const float* Cs = chat + (size_t)sg * kk * D;
  if (threadIdx.x == 0) near_n = 0;
  uint4 b[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) b[s] = load16(xr + 8 * s);
  float best = kNegHuge, second = kNegHuge;
  int bidx = 0;
#pragma unroll 1
  for (int t = SPLIT ? wave : 0; 32 * t < si.k_s; t += SPLIT ? NW : 1) {
    const float* cr = Cs + (size_t)min(32 * t + col, si.k_s - 1) * D + half * 4;
    floatx16 acc = {};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const uint4 a = load16(cr + 8 * s);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b[s].x), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b[s].y), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b[s].z), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b[s].w), acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = 32 * t + 8 * (v / 4) + (v % 4) + 4 * half;
      const float sim = row < si.k_s ? acc[v] : kNegHuge;
      const bool up = sim > best;
      second = up ? best : fmaxf(second, sim);
      best = up ? sim : best;
      bidx = up ? row : bidx;
    }
  }
  auto merge = [&](float ob, float os, int oi) {
    second = fmaxf(fminf(best, ob), fmaxf(second, os));
    const bool other = ob > best || (ob == best && oi < bidx);
    bidx = other ? oi : bidx;
    best = fmaxf(best, ob);
  };
  // lanes l and l ^ 32 hold the same point over disjoint centroid rows, and so do the waves of SPLIT
  merge(__shfl_xor(best, 32), __shfl_xor(second, 32), __shfl_xor(bidx, 32));
  if constexpr (SPLIT) {
    if (half == 0) {
      part_best[wave][col] = best;
      part_second[wave][col] = second;
      part_row[wave][col] = bidx;
    }
  }
  __syncthreads();
  const int point = 32 * frag + col;
  if (half == 0 && (!SPLIT || wave == 0) && point < si.L_s) {
    if constexpr (SPLIT)
      for (int w = 1; w < NW; ++w) merge(part_best[w][col], part_second[w][col], part_row[w][col]);
    assign[gp0 + point] = bidx;  // (stands where nothing is comparable)
    if (best - second < kAssignGuard) near_p[atomicAdd(&near_n, 1)] = point;
  }
  __syncthreads();
  if (near_n == 1) {  // (the usual number: the point's row in LDS; 2 segments of 2046 points x 128 clusters 208 -> 204 us)
    const int p = near_p[0];
    const int bi = refine_point<float, D>(xhat + (gp0 + p) * D, Cs, si.k_s);
    if (threadIdx.x == 0 && bi < si.k_s) assign[gp0 + p] = bi;
  } else {
    settle_near_f32<D>(xhat + gp0 * D, Cs, si.k_s, near_p, near_n, assign + gp0);
  }
}

// ============================================================================
// Stable counting sort of one segment's points by cluster.  Wave w owns the
// w-th contiguous stripe of the segment and a private row of counters, so the
// scatter keeps positions ascending inside every cluster.
// ============================================================================
constexpr int SORT_HIST_INTS = 11264;  // LDS budget for the per-wave counters

// One segment's points a[0, L_s) sorted into ord[] by the calling workgroup of W waves;
// per-cluster counts and first positions to cnt[] / first[] (kk entries each).
// prev (may be null): the clusters of the round before, replaced by this round's on the way; when
// a point's cluster differs from it (and `compare` is set: not in the first round), both clusters
// are marked in changed[] (plain stores of 1: who wins does not matter).  The update step
// recomputes only marked clusters: a cluster nobody entered or left keeps its member sum and with
// it, bit for bit, its centroid.
__device__ __forceinline__ void sort_segment(const int32_t* a, int32_t* ord, int32_t* cnt, int32_t* first,
                                             int L_s, int kk, int key_bits, int* hist, int32_t* prev = nullptr,
                                             int32_t* changed = nullptr, bool compare = false) {
  const int W = blockDim.x >> 6;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int* tot = hist + W * kk;
  for (int i = tid; i < W * kk; i += blockDim.x) hist[i] = 0;
  __syncthreads();
  const int stripe = (L_s + W - 1) / W;
  const int s0 = min(L_s, wave * stripe), s1 = min(L_s, s0 + stripe);
  for (int i = s0 + lane; i < s1; i += 64) {
    const int c = a[i];
    atomicAdd(&hist[wave * kk + c], 1);
    if (prev) {
      const int before = prev[i];
      if (compare && before != c) {
        changed[before] = 1;
        changed[c] = 1;
      }
      prev[i] = c;
    }
  }
  __syncthreads();
  // per cluster: exclusive scan over the waves, total into tot[]
  for (int c = tid; c < kk; c += blockDim.x) {
    int run = 0;
    for (int w = 0; w < W; ++w) {
      const int t = hist[w * kk + c];
      hist[w * kk + c] = run;
      run += t;
    }
    tot[c] = run;
  }
  __syncthreads();
  // exclusive scan of the totals over clusters (one wave, chunks of 64)
  if (wave == 0) {
    int carry = 0;
    for (int c0 = 0; c0 < kk; c0 += 64) {
      const int c = c0 + lane;
      const int v = c < kk ? tot[c] : 0;
      int inc = v;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
      }
      if (c < kk) {
        cnt[c] = v;
        first[c] = carry + inc - v;
        tot[c] = carry + inc - v;
      }
      carry += __shfl(inc, 63);
    }
  }
  __syncthreads();
  for (int i = tid; i < W * kk; i += blockDim.x) hist[i] += tot[i % kk];
  __syncthreads();
  // scatter, 64 points of the stripe at a time
  for (int i0 = s0; i0 < s1; i0 += 64) {
    const int i = i0 + lane;
    const bool on = i < s1;
    const int key = on ? a[i] : -1;
    // lanes holding the same key
    uint64_t peers = __ballot(on);
    for (int bit = 0; bit < key_bits; ++bit) {
      const uint64_t bal = __ballot((key >> bit) & 1);
      peers &= ((key >> bit) & 1) ? bal : ~bal;
    }
    const uint64_t below = peers & ((1ull << lane) - 1ull);
    const int rank = __popcll(below), cnt_l = __popcll(peers);
    if (on) {
      const int base = hist[wave * kk + key];
      ord[base + rank] = i;
      __builtin_amdgcn_wave_barrier();
      if (rank == cnt_l - 1) hist[wave * kk + key] = base + cnt_l;
    }
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
  }
}

__global__ __launch_bounds__(1024) void sort_kernel(const int32_t* __restrict__ assign,
                                                    int32_t* __restrict__ order,
                                                    int32_t* __restrict__ count,
                                                    int32_t* __restrict__ start,
                                                    int32_t* __restrict__ flag_count,
                                                    int32_t* __restrict__ prev,
                                                    int32_t* __restrict__ changed, int first_round, int S,
                                                    int L, int kk, int N_idx, int key_bits) {
  extern __shared__ int hist[];  // [W][kk], then kk ints of scan space
  const int sg = blockIdx.x;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  if (sg == 0 && threadIdx.x == 0) {
    flag_count[0] = 0;  // the refine pass before this one has consumed it
    flag_count[1] = 0;  // the list of large clusters the update step of this round fills
  }
  sort_segment(assign + (size_t)si.unit * N_idx + si.seg_start, order + (size_t)si.unit * N_idx + si.seg_start,
               count + (size_t)sg * kk, start + (size_t)sg * kk, si.L_s, kk, key_bits, hist,
               prev ? prev + (size_t)si.unit * N_idx + si.seg_start : nullptr, changed + (size_t)sg * kk, !first_round);
}

// ============================================================================
// Update: one group of LPR lanes per cluster sums its members' xhat in fp64.
// ============================================================================
// The member rows ord[0, n) of the segment's points X (already offset to the lane's chunk)
// added to acc in fp64 in that order, U loads in flight.  STATS: also the exponent range of
// what was added.  (STREAM: the rows are read once per launch and should not displace other
// lines in the caches.)
template <typename T, int D, int U, bool STREAM, bool STATS>
__device__ __forceinline__ void sum_members(const T* X, const int32_t* ord, int n,
                                            double (&acc)[Elem<T>::EPC], int& emin, int& emax) {
  auto load_row = [](const T* p) { return STREAM ? load16_stream(p) : load16(p); };
  constexpr int EPC = Elem<T>::EPC;
  auto add = [&](const uint4& raw) {
    float f[EPC];
    unpack<T>(raw, f);
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] += (double)f[e];
    if (STATS) exponent_range<T>(raw, emin, emax);
  };
  int i = 0;
  for (; i + U <= n; i += U) {
    uint4 raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u] = load_row(X + (size_t)ord[i + u] * D);
#pragma unroll
    for (int u = 0; u < U; ++u) add(raw[u]);
  }
  if (U > 4 && i + 4 <= n) {
    uint4 raw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) raw[u] = load_row(X + (size_t)ord[i + u] * D);
#pragma unroll
    for (int u = 0; u < 4; ++u) add(raw[u]);
    i += 4;
  }
  for (; i < n; ++i) add(load16(X + (size_t)ord[i] * D));
}

// The member sum of a cluster, normalised and rounded, to dst (the lane's 16-byte chunk of the
// centroid row); members that cancel keep the centroid.
template <int EPC>
__device__ __forceinline__ void store_sums(double* sums, const double (&acc)[EPC]) {
#pragma unroll
  for (int e = 0; e < EPC; ++e) sums[e] = acc[e];
}

template <typename T, int D>
__device__ __forceinline__ void finish_centroid(const double (&acc)[Elem<T>::EPC], T* dst) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC;
  double n2 = 0.0;
#pragma unroll
  for (int e = 0; e < EPC; ++e) n2 = fma(acc[e], acc[e], n2);
  n2 = group_sum_f64<LPR>(n2);
  const double nrm = sqrt(n2);
  if (!(nrm > 0.0)) return;
  T o[EPC];
  const double rn = 1.0 / nrm;
#pragma unroll
  for (int e = 0; e < EPC; ++e) o[e] = quant_store<T>(div_shared(acc[e], nrm, rn));
  store16(dst, *reinterpret_cast<uint4*>(o));
}

// One cluster's update by the calling group of LPR lanes (lane `sub` of it): the n member
// rows ord[0, n) of the segment's points X are summed in fp64 in that order, U loads in
// flight, and the normalised sum goes to dst (the sum itself to `sums`, unless null).
template <typename T, int D, int U, bool STREAM>
__device__ __forceinline__ void update_cluster(const T* X, const int32_t* ord, int n, T* dst, int sub,
                                               double* sums = nullptr) {
  constexpr int EPC = Elem<T>::EPC;
  if (n == 0 && !sums) return;  // an empty cluster keeps its centroid
  double acc[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) acc[e] = 0.0;
  int emin = 0, emax = 0;
  sum_members<T, D, U, STREAM, false>(X + sub * EPC, ord, n, acc, emin, emax);
  if (sums) store_sums<EPC>(sums, acc);
  finish_centroid<T, D>(acc, dst);  // (a sum of nothing is zero)
}

// Clusters of more than UPD_BIG members (heavy-tailed data: a thousand tokens in one cluster)
// are summed by all groups of the workgroup, a contiguous run of members each, and the
// partial sums are added in run order.  The reference sum adds the members one by one, and
// the two agree bit for bit when no addition rounds, in either order.  That is certain when
// every partial sum of any subset of the addends is representable: all addends are multiples of
// 2^q, q the unit in the last place of the smallest exponent present, and n of them below
// 2^(emax + 1) in magnitude sum to less than n 2^(emax + 1); fp64 holds every multiple of 2^q
// below 2^(q + 53), so  emax - emin + ceil(log2 n) <= 52 - (mantissa bits of the storage type)
// suffices.  The exponent range is gathered on the way; a cluster that fails the test (a
// component spread over more than 2^34 at bf16) is summed again one by one by one group.
constexpr int UPD_BIG = 128;

// One such cluster by the NT threads of a workgroup: the n member rows ord[0, n) of the segment's points X
// to the centroid row dst (sums: also the sum itself, or null; used where the test holds).
template <typename T, int D, int NT>
__device__ __forceinline__ void update_cluster_by_workgroup(const T* X, const int32_t* ord, int n, T* dst, double* sums) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = NT / LPR;
  __shared__ double part[GROUPS * D];
  __shared__ int erange[2 * GROUPS];
  const int sub = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  const int per = (n + GROUPS - 1) / GROUPS;
  const int i0 = min(n, grp * per), i1 = min(n, i0 + per);
  double acc[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) acc[e] = 0.0;
  int emin = 255, emax = 0;
  sum_members<T, D, 4, true, true>(X + sub * EPC, ord + i0, i1 - i0, acc, emin, emax);
#pragma unroll
  for (int off = 1; off < LPR; off <<= 1) {
    emin = min(emin, __shfl_xor(emin, off));
    emax = max(emax, __shfl_xor(emax, off));
  }
#pragma unroll
  for (int e = 0; e < EPC; ++e) part[grp * D + sub * EPC + e] = acc[e];
  if (sub == 0) {
    erange[2 * grp] = emin;
    erange[2 * grp + 1] = emax;
  }
  __syncthreads();
  if (grp == 0) {
    double tot[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) tot[e] = part[sub * EPC + e];
    int lo = erange[0], hi = erange[1];
#pragma unroll 1
    for (int g = 1; g < GROUPS; ++g) {
#pragma unroll
      for (int e = 0; e < EPC; ++e) tot[e] += part[g * D + sub * EPC + e];
      lo = min(lo, erange[2 * g]);
      hi = max(hi, erange[2 * g + 1]);
    }
    const int lg = 32 - __clz(n - 1);  // ceil(log2 n), n > UPD_BIG
    if (sums) store_sums<EPC>(sums + sub * EPC, tot);
    if (hi < lo || hi - lo + lg <= 52 - MantissaBits<T>::value)  // (hi < lo: every addend is zero)
      finish_centroid<T, D>(tot, dst + sub * EPC);
    else
      update_cluster<T, D, 4, true>(X, ord, n, dst + sub * EPC, sub);
  }
  __syncthreads();
}

template <typename T, int D>
__global__ __launch_bounds__(256) void update_big_kernel(const T* __restrict__ xhat, T* __restrict__ chat,
                                                         const int32_t* __restrict__ order,
                                                         const int32_t* __restrict__ count,
                                                         const int32_t* __restrict__ start,
                                                         const int32_t* __restrict__ big_list,
                                                         const int32_t* __restrict__ big_count,
                                                         double* sums, long long sums_skip, int S, int L,
                                                         int kk, int N_idx) {
  const int nbig = *big_count;
#pragma unroll 1
  for (int b = blockIdx.x; b < nbig; b += gridDim.x) {  // (the same for every thread of the workgroup)
    const int gc = big_list[b];
    const SegInfo si = seg_info(gc / kk, S, L, kk, N_idx);
    const size_t p0 = (size_t)si.unit * N_idx + si.seg_start;
    update_cluster_by_workgroup<T, D, 256>(xhat + p0 * D, order + p0 + start[gc], count[gc], chat + (size_t)gc * D,
                                           sums ? sums + si.unit * sums_skip + (size_t)gc * D : nullptr);
  }
}

// First round: every cluster is summed (changed: cleared; sums: see update_moves_kernel, or null).
template <typename T, int D>
__global__ __launch_bounds__(256) void update_kernel(const T* __restrict__ xhat, T* __restrict__ chat,
                                                     const int32_t* __restrict__ order,
                                                     const int32_t* __restrict__ count,
                                                     const int32_t* __restrict__ start,
                                                     int32_t* __restrict__ changed,
                                                     int32_t* __restrict__ big_list,
                                                     int32_t* __restrict__ big_count, double* sums,
                                                     long long sums_skip, int S, int L, int kk, int N_idx, int nclusters) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = 256 / LPR;
  const int sub = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  const int gc = blockIdx.x * GROUPS + grp;  // sg * kk + c
  if (gc >= nclusters) return;
  const int sg = gc / kk, c = gc - sg * kk;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  if (c >= si.k_s) return;
  if (sub == 0) changed[gc] = 0;
  const int n = count[gc];
  if (n > UPD_BIG) {  // left to update_big_kernel
    if (sub == 0) big_list[atomicAdd(big_count, 1)] = gc;
    return;
  }
  const size_t p0 = (size_t)si.unit * N_idx + si.seg_start;
  update_cluster<T, D, 4, true>(xhat + p0 * D, order + p0 + start[gc], n, chat + (size_t)gc * D + sub * EPC, sub,
                                sums ? sums + si.unit * sums_skip + (size_t)gc * D + sub * EPC : nullptr);
}

// The update of the later rounds: only clusters that a point entered or left in this round
// (marked by the sort step) are summed again.  Most are untouched: a workgroup reads the marks
// of `span` (256 at most) consecutive clusters at once, lists the marked ones in LDS and its 16-lane groups take
// them from the list (one mark per group and workgroup, as in update_kernel, is a round trip and
// a workgroup launch per 16 clusters even when none of them changed).
template <typename T, int D>
__global__ __launch_bounds__(256) void update_touched_kernel(const T* __restrict__ xhat, T* __restrict__ chat,
                                                             const int32_t* __restrict__ order,
                                                             const int32_t* __restrict__ count,
                                                             const int32_t* __restrict__ start,
                                                             int32_t* __restrict__ changed,
                                                             int32_t* __restrict__ big_list,
                                                             int32_t* __restrict__ big_count, int S, int L,
                                                             int kk, int N_idx, int nclusters, int span) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = 256 / LPR;
  __shared__ int list[256];
  __shared__ int wave_n[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int gc_mine = blockIdx.x * span + tid;
  const bool on = tid < span && gc_mine < nclusters && changed[gc_mine] != 0;
  if (on) changed[gc_mine] = 0;
  const uint64_t mk = __ballot(on);
  if (lane == 0) wave_n[wave] = __popcll(mk);
  __syncthreads();
  int base = 0, n = 0;
  for (int w = 0; w < 4; ++w) {
    base += w < wave ? wave_n[w] : 0;
    n += wave_n[w];
  }
  if (on) list[base + __popcll(mk & ((1ull << lane) - 1ull))] = gc_mine;
  __syncthreads();
  const int sub = tid % LPR;
  for (int j = tid / LPR; j < n; j += GROUPS) {
    const int gc = list[j];
    const int sg = gc / kk, c = gc - sg * kk;
    const SegInfo si = seg_info(sg, S, L, kk, N_idx);
    if (c >= si.k_s) continue;
    const int members = count[gc];
    if (members > UPD_BIG) {  // left to update_big_kernel
      if (sub == 0) big_list[atomicAdd(big_count, 1)] = gc;
      continue;
    }
    const size_t p0 = (size_t)si.unit * N_idx + si.seg_start;
    update_cluster<T, D, 4, true>(xhat + p0 * D, order + p0 + start[gc], members,
                                  chat + (size_t)gc * D + sub * EPC, sub);
  }
}

// ============================================================================
// The f32 builds' update, with the sort in it (and the first and last one of bf16 builds of a few segments; sums:
// see update_moves_kernel): a workgroup owns the clusters [c_lo, c_hi) of a segment, reads
// this round's and the last round's cluster of every point of the segment, and sorts the points of its
// changed clusters (in the first round and where `all` is set: of all its clusters) into their place of order[],
// positions ascending; their counts and first places go to count[] and start[].  Then a group of lanes
// per changed cluster sums its members in that order (fp32 sums may round in fp64, so the order is kept),
// the whole workgroup one of more than UPD_BIG.  `all`: the last round; nothing is summed.
// (One workgroup per segment sorting all points, update_touched_kernel and update_big_kernel: three launches
// and 6.2 + 2 .. 12 + 1.3 us a round for 2 segments of 2048 points x 128 clusters, 4.2 .. 15 us so; a whole
// build of them 285 -> 155 us, of 100 segments of 4096 points x 256 clusters 2.03 -> 1.99 ms.)
// ============================================================================
constexpr int SCAN_NT = 512, SCAN_CLUSTERS = 64;  // threads; most clusters of a workgroup

template <typename T, int D>
__global__ __launch_bounds__(SCAN_NT) void update_scan_kernel(
    const T* __restrict__ xhat, T* __restrict__ chat, const int32_t* __restrict__ assign,
    const int32_t* __restrict__ before, int32_t* order, int32_t* __restrict__ count, int32_t* __restrict__ start,
    double* sums, long long sums_skip, int first_round, int all, int S, int L, int kk, int N_idx, int span, int pieces) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = SCAN_NT / LPR, NW = SCAN_NT / 64, U = 4;
  __shared__ int hist[NW * SCAN_CLUSTERS];   // members per (wave's stripe of points, cluster); then places
  __shared__ int lower[NW];                  // points in clusters before c_lo, per stripe
  __shared__ int changed[SCAN_CLUSTERS], cnt[SCAN_CLUSTERS], first[SCAN_CLUSTERS];
  const int wg = xcd_logical_block(blockIdx.x, gridDim.x);
  const int sg = wg / pieces, piece = wg - sg * pieces;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const int c_lo = piece * span, c_n = min(si.k_s - c_lo, span);
  if (c_n <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = tid % LPR;
  const size_t p0 = (size_t)si.unit * N_idx + si.seg_start;
  const int32_t* as = assign + p0;
  const int32_t* pv = before + p0;
  const bool every = first_round || all;
  for (int i = tid; i < NW * SCAN_CLUSTERS; i += SCAN_NT) hist[i] = 0;
  if (tid < SCAN_CLUSTERS) changed[tid] = every ? 1 : 0;
  __syncthreads();
  const int stripe = (si.L_s + NW - 1) / NW;
  const int s0 = min(si.L_s, wave * stripe), s1 = min(si.L_s, s0 + stripe);
  int below = 0;
  for (int i0 = s0; i0 < s1; i0 += 64 * U) {
    int a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + 64 * u + lane, s1 - 1);
      a[u] = as[i] - c_lo;
      b[u] = every ? a[u] : pv[i] - c_lo;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool on = i0 + 64 * u + lane < s1;
      below += __popcll(__ballot(on && a[u] < 0));
      const bool in = on && a[u] >= 0 && a[u] < c_n;
      if (in) atomicAdd(&hist[wave * SCAN_CLUSTERS + a[u]], 1);
      if (on && a[u] != b[u]) {
        if (in) changed[a[u]] = 1;
        if (b[u] >= 0 && b[u] < c_n) changed[b[u]] = 1;
      }
    }
  }
  if (lane == 0) lower[wave] = below;
  __syncthreads();
  if (!__ballot(lane < c_n && changed[min(lane, c_n - 1)])) return;  // (the same for every wave)
  if (wave == 0) {  // places: clusters in order, each cluster's stripes in order
    int n = 0, base = 0;
    for (int w = 0; w < NW; ++w) {
      const int t = lane < c_n ? hist[w * SCAN_CLUSTERS + lane] : 0;
      hist[w * SCAN_CLUSTERS + lane] = n;
      n += t;
      base += lower[w];
    }
    const int at = base + wave_incl_scan(n) - n;
    for (int w = 0; w < NW; ++w) hist[w * SCAN_CLUSTERS + lane] += at;
    cnt[lane] = n;
    first[lane] = at;
    if (lane < c_n && changed[lane]) {
      count[(size_t)sg * kk + c_lo + lane] = n;
      start[(size_t)sg * kk + c_lo + lane] = at;
    }
  }
  __syncthreads();
  for (int i1 = s0; i1 < s1; i1 += 64 * U) {
    int a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = as[min(i1 + 64 * u + lane, s1 - 1)] - c_lo;
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
      const int i = i1 + 64 * u + lane;
      const int key = u == 0 ? a[0] : u == 1 ? a[1] : u == 2 ? a[2] : a[3];
      const bool on = i < s1 && key >= 0 && key < c_n && changed[min(max(key, 0), c_n - 1)];
      uint64_t peers = __ballot(on);
      if (!peers) continue;
#pragma unroll
      for (int bit = 0; bit < 6; ++bit) {
        const uint64_t bal = __ballot((key >> bit) & 1);
        peers &= ((key >> bit) & 1) ? bal : ~bal;
      }
      const int rank = __popcll(peers & ((1ull << lane) - 1ull)), same = __popcll(peers);
      if (on) {
        const int place = hist[wave * SCAN_CLUSTERS + key];
        order[p0 + place + rank] = i;
        __builtin_amdgcn_wave_barrier();
        if (rank == same - 1) hist[wave * SCAN_CLUSTERS + key] = place + same;
      }
      __threadfence_block();
      __builtin_amdgcn_wave_barrier();
    }
  }
  if (all) return;
  __syncthreads();
  const T* X = xhat + p0 * D;
  T* Cs = chat + ((size_t)sg * kk + c_lo) * D;
  double* own = sums ? sums + si.unit * sums_skip + ((size_t)sg * kk + c_lo) * D : nullptr;
  for (int c = tid / LPR; c < c_n; c += GROUPS)
    if (changed[c] && cnt[c] <= UPD_BIG)
      update_cluster<T, D, 8, false>(X, order + p0 + first[c], cnt[c], Cs + (size_t)c * D + sub * EPC, sub,
                                     own ? own + (size_t)c * D + sub * EPC : nullptr);
  for (int c = 0; c < c_n; ++c)
    if (changed[c] && cnt[c] > UPD_BIG)
      update_cluster_by_workgroup<T, D, SCAN_NT>(X, order + p0 + first[c], cnt[c], Cs + (size_t)c * D,
                                                 own ? own + (size_t)c * D : nullptr);
}
static_assert(SCAN_CLUSTERS == 64, "a cluster per lane, six key bits");

// ============================================================================
// Update from the points that moved (later rounds of the resident bf16 path): the fp64 member
// sums are kept from round to round and only the rows of the points that changed cluster in
// this round are subtracted from one sum and added to another.  The result is the sum of the
// members bit for bit, whatever the order, when no addition rounds; that is certain when
// every sum of a subset of the segment's points is representable, the condition above with
// the exponent range of the whole segment (gathered by normalise_kernel) and n = L_s.  A segment
// that fails it (nonzero components further apart than 2^(45 - ceil(log2 L_s)), 2^32 at 8192 points;
// the benchmark's keys spread over 2^19 .. 2^28) is sorted and its changed clusters are summed again
// by the first workgroup.
// No sort and no pass over the members: a round costs the scan of the marks in prev[], 2 KiB per
// changed cluster and 512 B per moved point.
// Also leaves in changed[] and nchanged[] which centroids the next round's assign step compares.
//
// A workgroup owns the clusters [c_lo, c_hi) of a segment: it counts the arrivals and departures
// of each (MOVE_CAP at once, of MOVED_CAP points; more are taken in ranges of the points, the centroids after the last
// one), lists them by cluster in LDS, and one group of lanes per changed cluster works through its list.
// ============================================================================
constexpr int MOVE_NT = 512, MOVE_CAP = 4096, MOVED_CAP = MOVE_CAP / 2;

inline size_t update_moves_lds(int kk) {
  const size_t list = MOVE_CAP, hist = (size_t)(MOVE_NT / 64 + 1) * kk;
  return sizeof(int) * (3 * (size_t)kk + (list > hist ? list : hist)) + sizeof(int2) * MOVED_CAP;
}

template <int D>
__global__ __launch_bounds__(MOVE_NT) void update_moves_kernel(
    const bf16_t* __restrict__ xhat, bf16_t* __restrict__ chat, double* sums, long long sums_skip,
    const int32_t* __restrict__ assign, const int32_t* __restrict__ prev, int32_t* __restrict__ changed,
    int32_t* __restrict__ nchanged, int32_t* __restrict__ nchanged_next, const int32_t* __restrict__ range, int32_t* order, int32_t* count, int32_t* start, int round, int S, int L,
    int kk, int N_idx, int pieces, int key_bits) {
  constexpr int EPC = 8, LPR = D / EPC, GROUPS = MOVE_NT / LPR, U = 4;
  extern __shared__ __attribute__((aligned(16))) int moves_lds[];
  int2* moved = reinterpret_cast<int2*>(moves_lds);  // the points that moved: place, cluster before | now << 16
  int* cnt = moves_lds + 2 * MOVED_CAP;              // entries per cluster
  int* end = cnt + kk;          // behind its last entry
  int* touched = end + kk;      // the clusters with entries
  int* entry = touched + kk;    // point * 2 + (1: leaves); the sort's counters
  __shared__ int totals[2];     // entries, touched clusters
  __shared__ int nmoved;
  const int wg = xcd_logical_block(blockIdx.x, gridDim.x);
  const int sg = wg / pieces, piece = wg - sg * pieces;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = tid % LPR;
  const size_t p0 = (size_t)si.unit * N_idx + si.seg_start;
  const int32_t* as = assign + p0;
  const int32_t* pv = prev + p0;
  const bf16_t* X = xhat + p0 * D;
  const int emin = range[2 * sg], emax = range[2 * sg + 1];
  const int lg = si.L_s > 1 ? 32 - __clz(si.L_s - 1) : 0;  // ceil(log2 L_s)
  const bool exact = emax < emin || emax - emin + lg <= 52 - MantissaBits<bf16_t>::value;
  const int per = exact ? (si.k_s + pieces - 1) / pieces : si.k_s;
  const int c_lo = min(si.k_s, piece * per), c_hi = min(si.k_s, c_lo + per);
  if (piece == 0 && tid == 0) nchanged_next[sg] = 0;
  if (c_lo >= c_hi) return;

  // The points that moved, listed once: their tags are requested together, then their new clusters.  (With both visits
  // below reading tags and, one by one, clusters from memory: 105 us over the eight launches of a build of 32 segments of
  // 8192 points, 86 so, of 1920 segments 2005 and 1775, of 2048 over eighteen 4260 and 3920.  Up to 2048 points four tags a
  // thread cover a segment: 4096 segments of 1024 points 961 us with sixteen, 928 so.)
  if (tid == 0) nmoved = 0;
  __syncthreads();
  auto list = [&](auto batch) {  // tags in flight
    constexpr int TAGS = decltype(batch)::value;
    for (int i0 = tid; i0 - tid < si.L_s; i0 += TAGS * MOVE_NT) {
      int tag[TAGS], n = 0;
#pragma unroll
      for (int u = 0; u < TAGS; ++u) tag[u] = pv[min(i0 + u * MOVE_NT, si.L_s - 1)];
      uint32_t mine = 0;
#pragma unroll
      for (int u = 0; u < TAGS; ++u) {
        const bool on = i0 + u * MOVE_NT < si.L_s && tag[u] >> PREV_CLUSTER_BITS == round;
        mine |= on ? 1u << u : 0u;
        n += on ? 1 : 0;
      }
      if (!__ballot(n > 0)) continue;
      const int inc = wave_incl_scan(n), all = __builtin_amdgcn_readlane(inc, 63);
      int at = 0;
      if (lane == 0) at = atomicAdd(&nmoved, all);
      at = __builtin_amdgcn_readfirstlane(at) + inc - n;
#pragma unroll
      for (int u = 0; u < TAGS; ++u)
        if (mine >> u & 1u) {
          if (at < MOVED_CAP) moved[at] = make_int2(i0 + u * MOVE_NT, tag[u] & ((1 << PREV_CLUSTER_BITS) - 1));
          ++at;
        }
    }
  };
  if (si.L_s > 4 * MOVE_NT) list(std::integral_constant<int, 16>{});
  else list(std::integral_constant<int, 4>{});
  __syncthreads();
  const bool in_lds = nmoved <= MOVED_CAP;
  if (in_lds && nmoved > 0) {  // (the same for the whole workgroup)
    constexpr int PER = MOVED_CAP / MOVE_NT;
    const int last = nmoved - 1;
    int to[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) to[u] = as[moved[min(tid + u * MOVE_NT, last)].x];
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (tid + u * MOVE_NT <= last) moved[tid + u * MOVE_NT].y |= to[u] << 16;
    __syncthreads();
  }
  auto visit = [&](int lo, int hi, auto&& f) {  // f(cluster, entry) for the round's entries of points [lo, hi)
    auto point = [&](int i, int from, int to) {
      if (from >= c_lo && from < c_hi) f(from, 2 * i + 1);
      if (to >= c_lo && to < c_hi) f(to, 2 * i);
    };
    if (in_lds) {  // (all points)
      for (int j = tid; j < nmoved; j += MOVE_NT) point(moved[j].x, moved[j].y & 0xffff, moved[j].y >> 16);
      return;
    }
    for (int i0 = lo + tid; i0 < hi; i0 += U * MOVE_NT) {
      int tag[U];
#pragma unroll
      for (int u = 0; u < U; ++u) tag[u] = pv[min(i0 + u * MOVE_NT, hi - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * MOVE_NT;
        if (i < hi && tag[u] >> PREV_CLUSTER_BITS == round) point(i, tag[u] & ((1 << PREV_CLUSTER_BITS) - 1), as[i]);
      }
    }
  };
  auto count_entries = [&](int lo, int hi) {
    for (int c = c_lo + tid; c < c_hi; c += MOVE_NT) cnt[c] = 0;
    __syncthreads();
    visit(lo, hi, [&](int c, int) { atomicAdd(&cnt[c], 1); });
    __syncthreads();
    if (wave == 0) {  // first places and the list of touched clusters
      int at = 0, n = 0;
      for (int c0 = c_lo; c0 < c_hi; c0 += 64) {
        const int c = c0 + lane;
        const int v = c < c_hi ? cnt[c] : 0;
        int inc = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int t = __shfl_up(inc, off);
          if (lane >= off) inc += t;
        }
        const uint64_t mk = __ballot(v > 0);
        if (c < c_hi) end[c] = at + inc - v;
        if (v > 0) touched[n + __popcll(mk & ((1ull << lane) - 1ull))] = c;
        at += __shfl(inc, 63);
        n += __popcll(mk);
      }
      if (lane == 0) {
        totals[0] = at;
        totals[1] = n;
      }
    }
    __syncthreads();
  };
  count_entries(0, si.L_s);
  for (int c = c_lo + tid; c < c_hi; c += MOVE_NT) changed[(size_t)sg * kk + c] = cnt[c] > 0 ? 1 : 0;
  if (tid == 0 && totals[1] > 0) atomicAdd(&nchanged[sg], totals[1]);
  if (!exact) {
    const int n = totals[1];
    sort_segment(as, order + p0, count + (size_t)sg * kk, start + (size_t)sg * kk, si.L_s, kk, key_bits, entry);
    __syncthreads();
    for (int j = tid / LPR; j < n; j += GROUPS) {
      const size_t gc = (size_t)sg * kk + touched[j];
      update_cluster<bf16_t, D, 4, false>(X, order + p0 + start[gc], count[gc], chat + gc * D + sub * EPC, sub);
    }
    return;
  }
  const int span = totals[0] <= MOVE_CAP ? si.L_s : MOVE_CAP / 2;  // (in_lds: never more)
  for (int lo = 0; lo < si.L_s; lo += span) {
    const int hi = min(si.L_s, lo + span);
    if (span < si.L_s) {
      __syncthreads();
      count_entries(lo, hi);
    }
    visit(lo, hi, [&](int c, int e) { entry[atomicAdd(&end[c], 1)] = e; });
    __syncthreads();
    const int n = totals[1];
    for (int j = tid / LPR; j < n; j += GROUPS) {
      const int c = touched[j];
      const int ne = cnt[c], e0 = end[c] - ne;
      const size_t gc = (size_t)sg * kk + c;
      double* own = sums + si.unit * sums_skip + gc * D + sub * EPC;
      double acc[EPC];
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[e] = own[e];
      for (int i = 0; i < ne; i += U) {
        int en[U];
        uint4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) en[u] = entry[e0 + min(i + u, ne - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) raw[u] = load16(X + (size_t)(en[u] >> 1) * D + sub * EPC);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float f[EPC];
          unpack<bf16_t>(raw[u], f);
          const double sign = i + u >= ne ? 0.0 : (en[u] & 1) ? -1.0 : 1.0;
#pragma unroll
          for (int e = 0; e < EPC; ++e) acc[e] = fma(sign, (double)f[e], acc[e]);
        }
      }
      store_sums<EPC>(own, acc);
      if (span == si.L_s) finish_centroid<bf16_t, D>(acc, chat + gc * D + sub * EPC);
    }
  }
  if (span == si.L_s) return;
  // Taken in ranges: a centroid comes from the round's last sum alone.  (A sum of some of the moves may
  // not be one of any round, and where the last one is zero the centroid of the round before stays.)
  __syncthreads();
  for (int c = c_lo + tid / LPR; c < c_hi; c += GROUPS) {
    const size_t gc = (size_t)sg * kk + c;
    if (!changed[gc]) continue;
    const double* own = sums + si.unit * sums_skip + gc * D + sub * EPC;
    double acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = own[e];
    finish_centroid<bf16_t, D>(acc, chat + gc * D + sub * EPC);
  }
}

// ============================================================================
// Short segments (an index update's 1K tokens into 64 clusters; small builds): all T
// iterations of one segment in ONE workgroup, with the centroids, the
// assignments, the sorted order and the cluster counts in LDS from the first
// iteration to the last.  Per iteration: assign (the resident MFMA form), near-ties
// re-decided with fp64 similarities by one wave each, and the update of the clusters that a
// point entered or left, straight into the LDS centroid rows; a round in which no point
// moves ends the rounds.  Launches per build: 5 instead of 4 T + 3.
//
// KEEP > 0 (up to 1024 points at d = 128, 2048 at d = 64): every wave holds KEEP fragments of points in
// registers from the first round to the last; else they are read again in every round (256 KiB
// per workgroup and round at 1024 points).
// SUMS (the member sums fit in 64 KiB of LDS): later rounds add the points that moved to one sum and
// take them out of another, wherever that is exact; they need no sort and no pass over members.
// Else a round sorts the points and sums the members of the changed clusters.
// 128 segments of 1024 points x 64 clusters, ten rounds: 200 us with every member summed again and the
// points read again in each round, 165 with the changed clusters summed, 105 us so (about 3.5 us assign, where the
// matrix instructions take 1.7, and 4 us update a round).  120K tokens x 16 in such segments: build
// 17.4 -> 11.6 ms; in segments of 2048 points x 128 clusters (neither KEEP nor SUMS) 17.9 -> 15.1 ms.  Whole builds of
// 32 segments, ten rounds: 1024 points x 128 clusters (KEEP alone) 301 -> 215 us, 2048 x 64 (SUMS alone) 393 -> 318.
// ============================================================================
constexpr int SMALL_L_MAX = 2048;   // points per segment
constexpr int SMALL_K_MAX = 128;    // clusters per segment
constexpr int SMALL_NW = 16;        // most waves
// With the points in registers half as many waves of twice the registers.  (The others keep 16: the
// gathers of the update are chains of round trips; 8 waves took 494 instead of 442 us for 16 segments of
// 2048 points x 128 clusters x 8 KV heads.)
template <int KEEP>
constexpr int small_waves() { return KEEP > 0 ? SMALL_NW / 2 : SMALL_NW; }

template <int D>
inline size_t small_kmeans_lds(int kk, bool keep_sums) {
  return (size_t)32 * ((kk + 31) / 32) * ResidentTile<D>::ROWB +
         sizeof(int) * ((size_t)SMALL_NW * kk + kk + 3 * SMALL_L_MAX + 4 * (size_t)kk) +
         (keep_sums ? sizeof(double) * D * (size_t)kk : 0);
}

template <int D, int KEEP, bool SUMS>
__global__ __launch_bounds__(64 * small_waves<KEEP>()) void kmeans_small_kernel(
    const bf16_t* __restrict__ xhat, const bf16_t* __restrict__ chat, int32_t* __restrict__ order,
    int32_t* __restrict__ count, int32_t* __restrict__ start, WindowRoute window, int segs, int S, int L, int kk,
    int N_idx, int iters, int key_bits) {
  using RT = ResidentTile<D>;
  constexpr int NW = small_waves<KEEP>(), NT = 64 * NW, LPR = D / 8, GROUPS = NT / LPR;
  if ((int)blockIdx.x >= segs) {  // the workgroups behind the segments' route an update's window
    route_window<8>(window, (size_t)(blockIdx.x - segs) * NT + threadIdx.x, (size_t)(gridDim.x - segs) * NT);
    return;
  }
  extern __shared__ __attribute__((aligned(16))) char small_lds[];
  char* cent = small_lds;
  int* hist = reinterpret_cast<int*>(small_lds + (size_t)32 * ((kk + 31) / 32) * RT::ROWB);  // sort_segment's
  int* a_s = hist + NW * kk + kk;   // cluster of every point
  int* ord_s = a_s + SMALL_L_MAX;         // points by cluster; before the sort: the near-tie list
  int* cnt_s = ord_s + SMALL_L_MAX;
  int* first_s = cnt_s + kk;
  int* changed_s = first_s + kk;
  int* prev_s = changed_s + kk;           // every point's cluster of the round before
  double* sums = reinterpret_cast<double*>(prev_s + SMALL_L_MAX);  // (SUMS) member sums
  int* flags = ord_s;
  __shared__ int nflag, nmoved;
  __shared__ int seg_emin, seg_emax;
  const int sg = blockIdx.x;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t p0 = (size_t)si.unit * N_idx + si.seg_start;
  const bf16_t* X = xhat + p0 * D;
  [[maybe_unused]] const int nfrag = (si.L_s + 31) / 32;
  uint4 kept[KEEP > 0 ? KEEP : 1][RT::KS];
  if constexpr (KEEP > 0) load_kept_fragments<D, KEEP, NW>(X, si.L_s, kept);
  resident_load_centroids<D, NT>(chat + (size_t)sg * kk * D, si.k_s, cent);
#ifdef WAVE_TRACE  // phase times of workgroup 0 (100 MHz clock), printed at the end
  unsigned long long tp[5] = {0, 0, 0, 0, 0}, tl = wall_clock64();
  int nf_total = 0;
#define WAVE_PHASE(k) do { const unsigned long long now_ = wall_clock64(); tp[k] += now_ - tl; tl = now_; } while (0)
#else
#define WAVE_PHASE(k) do { } while (0)
#endif
  // SUMS: where no fp64 addition of the segment's points rounds (see update_moves_kernel), the member
  // sums stay from round to round and the points that moved are taken out of one and added to another
  bool moves = false;
  if constexpr (SUMS) {
    if (tid == 0) {
      seg_emin = 255;
      seg_emax = 0;
    }
    __syncthreads();
    // (from the registers, or eight chunks in flight.  Chunk by chunk from memory and element by element: 20 us of a
    // workgroup's start at 1024 points; ten rounds of 128 segments beside an update's window 118 us, 105 so; whole builds of
    // 128 x 1024 x 64 169 and 159 us, of 1024 such segments 790 and 732)
    ExponentRange seen;
    if constexpr (KEEP > 0) {
#pragma unroll
      for (int f = 0; f < KEEP; ++f)  // (rows beyond the segment repeat its last one)
#pragma unroll
        for (int s = 0; s < RT::KS; ++s) seen.add(kept[f][s]);
    } else {
      constexpr int U = 8;
      const int chunks = si.L_s * RT::CPR;
      for (int i0 = tid; i0 < chunks; i0 += U * NT) {
        uint4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) raw[u] = load16(X + (size_t)min(i0 + u * NT, chunks - 1) * 8);
#pragma unroll
        for (int u = 0; u < U; ++u) seen.add(raw[u]);
      }
    }
    int emin, emax;
    seen.range(emin, emax);
    for (int off = 32; off >= 1; off >>= 1) {
      emin = min(emin, __shfl_xor(emin, off));
      emax = max(emax, __shfl_xor(emax, off));
    }
    if (lane == 0) {
      atomicMin(&seg_emin, emin);
      atomicMax(&seg_emax, emax);
    }
    __syncthreads();
    const int lg = si.L_s > 1 ? 32 - __clz(si.L_s - 1) : 0;  // ceil(log2 L_s)
    moves = seg_emax < seg_emin || seg_emax - seg_emin + lg <= 52 - MantissaBits<bf16_t>::value;
  }
  for (int t = 0; t < iters; ++t) {
    if (tid == 0) nflag = nmoved = 0;
    __syncthreads();
    WAVE_PHASE(0);
    auto emit = [&](int point, int cluster, int best, int second, NoState) {
      a_s[point] = cluster;
      if (key_gap(best, second) < kAssignGuard) flags[atomicAdd(&nflag, 1)] = point;
    };
    if constexpr (KEEP > 0)
      assign_kept_fragments<D, KEEP, NW>(kept, cent, si.L_s, si.k_s, emit);
    else
      lean_assign_fragments<D, NW>(X, cent, si.L_s, si.k_s, 0, nfrag, [](int) { return NoState{}; }, emit, [] {});
    __syncthreads();
    WAVE_PHASE(1);
    for (int c = tid; c < kk; c += NT) changed_s[c] = 0;  // (every wave is done with the last round's)
    // near-ties: fp64 similarities in index order against the LDS copy of the centroids,
    // ties to the lowest centroid (the arithmetic of refine_kernel)
    const int nf = nflag;
#ifdef WAVE_TRACE
    nf_total += nf;
#endif
    for (int it = wave; it < nf; it += NW) {
      const int point = flags[it];
      const bf16_t* xr = X + (size_t)point * D;
      double bv = -1.0e300;
      int bi = 0x7fffffff;
      for (int c = lane; c < si.k_s; c += 64) {
        const char* row = cent + (size_t)c * RT::ROWB;
        double acc = 0.0;
#pragma unroll 4
        for (int e0 = 0; e0 < D; e0 += 8) {
          float xf[8], cf[8];
          unpack<bf16_t>(load16(xr + e0), xf);
          unpack<bf16_t>(load16(row + e0 * 2), cf);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc = fma((double)xf[e], (double)cf[e], acc);
        }
        if (acc > bv) {  // c ascends within a lane, so strict > keeps the lowest index
          bv = acc;
          bi = c;
        }
      }
      for (int off = 32; off >= 1; off >>= 1) {
        const double ov = __shfl_xor(bv, off);
        const int oi = __shfl_xor(bi, off);
        if (ov > bv || (ov == bv && oi < bi)) {
          bv = ov;
          bi = oi;
        }
      }
      if (lane == 0 && bi < si.k_s) a_s[point] = bi;  // (nothing comparable: the fp32 decision stands)
    }
    __syncthreads();
    WAVE_PHASE(2);
    if (SUMS && moves && t > 0) {
      for (int i = tid; i < si.L_s; i += NT) {
        const int to = a_s[i], from = prev_s[i];
        if (to != from) {
          changed_s[to] = changed_s[from] = 1;
          ord_s[atomicAdd(&nmoved, 1)] = i;
        }
      }
      __syncthreads();
      const int n = nmoved;
      if (n == 0 || t + 1 == iters) break;  // (nothing moved: all later rounds would repeat this one)
      constexpr int PER = D / 64, U = 4;
      for (int e = wave; e < n; e += U * NW) {
        int point[U];
        float x[U][PER];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          point[u] = ord_s[min(e + u * NW, n - 1)];
#pragma unroll
          for (int j = 0; j < PER; ++j) x[u][j] = to_f32(X[(size_t)point[u] * D + 64 * j + lane]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (e + u * NW < n) {
            const int to = a_s[point[u]], from = prev_s[point[u]];
#pragma unroll
            for (int j = 0; j < PER; ++j) {
              atomicAdd(&sums[to * D + 64 * j + lane], (double)x[u][j]);
              atomicAdd(&sums[from * D + 64 * j + lane], -(double)x[u][j]);
            }
            prev_s[point[u]] = to;  // (every lane the same; no other wave has this point)
          }
      }
      __syncthreads();
      WAVE_PHASE(3);
      for (int c = tid / LPR; c < si.k_s; c += GROUPS)
        if (changed_s[c]) {
          double acc[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = sums[c * D + (tid % LPR) * 8 + e];
          finish_centroid<bf16_t, D>(acc, reinterpret_cast<bf16_t*>(cent + (size_t)c * RT::ROWB) + (tid % LPR) * 8);
        }
      WAVE_PHASE(4);
      continue;
    }
    sort_segment(a_s, ord_s, cnt_s, first_s, si.L_s, kk, key_bits, hist, prev_s, changed_s, t > 0);
    __syncthreads();
    WAVE_PHASE(3);
    if (t > 0) {
      bool any = false;
      for (int c = lane; c < si.k_s; c += 64) any |= changed_s[c] != 0;
      if (!__ballot(any)) break;  // (the same for every wave)
    }
    if (t + 1 < iters)
      for (int c = tid / LPR; c < si.k_s; c += GROUPS)
        if (t == 0 || changed_s[c])  // (a cluster that no point entered or left keeps its sum)
          update_cluster<bf16_t, D, 8, false>(
              X, ord_s + first_s[c], cnt_s[c], reinterpret_cast<bf16_t*>(cent + (size_t)c * RT::ROWB) + (tid % LPR) * 8,
              tid % LPR, SUMS ? sums + c * D + (tid % LPR) * 8 : nullptr);
    WAVE_PHASE(4);
  }
#ifdef WAVE_TRACE
  if (blockIdx.x == 0 && (tid == 0 || tid == 1023))
    printf("kmeans_small tid %d (x10 ns): top %llu assign %llu refine %llu sort %llu update %llu; near-ties %d\n", tid,
           tp[0], tp[1], tp[2], tp[3], tp[4], nf_total);
#endif
#undef WAVE_PHASE
  if (SUMS && moves && iters > 1) {  // (the last rounds did not sort)
    __syncthreads();
    sort_segment(a_s, ord_s, cnt_s, first_s, si.L_s, kk, key_bits, hist);
    __syncthreads();
  }
  for (int i = tid; i < si.L_s; i += NT) order[p0 + i] = ord_s[i];
  for (int c = tid; c < kk; c += NT) {
    count[(size_t)sg * kk + c] = cnt_s[c];
    start[(size_t)sg * kk + c] = first_s[c];
  }
}

// ============================================================================
// Finalize: sizes, offsets, mean of raw keys, value sums, permuted rows.  A group of lanes per cluster, R of its members
// in flight: the rows lie anywhere in the segment, and where the clusters do not fill the CUs what the launch takes is
// one cluster's chain of round trips.  In us, two, four, eight and sixteen in flight (6, 4, 3 and 2 waves a SIMD): 1024
// flushed rows of 128 units 37.5, 33.2, 32.3, 33.8; 2 fp32 segments of 2048 points 13.3, 11.4, 10.6, 11.2; 8 units
// of 32768 tokens 54, 51, 53, 55; 16 x 122880 3280, 3260, 3220, 3105; 64 x 65536 3725, 3715, 3670, 3860.
// Two where a cluster has fewer than four members on average and the workgroups are not all resident at once: most of
// eight rows would be repeats of the last.  Two and eight: 1024 segments of 1024 points x 700 clusters 281 and 406 us, x 512
// 246 and 308, x 360 221 and 230, x 300 213 and 214, x 256 216 and 211; 32 of them x 700 15.3 and 16.8, x 360 (resident)
// 13.7 and 12.9.
// ============================================================================
template <typename T, int D, int R>
__global__ __launch_bounds__(256) void finalize_kernel(
    const T* __restrict__ K, const T* __restrict__ V, const int32_t* __restrict__ order,
    const int32_t* __restrict__ count, const int32_t* __restrict__ start, T* __restrict__ centroids,
    T* __restrict__ vsum, int32_t* __restrict__ sizes, int32_t* __restrict__ offsets,
    int32_t* __restrict__ perm, T* __restrict__ k_perm, T* __restrict__ v_perm, int S, int L, int kk,
    int N, int N_idx, int n_sink, int m, int mc, int nclusters, int row_stride, int row_base, int pos_base) {
  // row_base, pos_base: added to the offsets and to the positions (an update's clusters continue
  // the rows and the token positions of the index they are written behind)
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = 256 / LPR;
  const int sub = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  const int gc = blockIdx.x * GROUPS + grp;
  if (gc >= nclusters) return;
  const int sg = gc / kk, c = gc - sg * kk;
  const SegInfo si = seg_info(sg, S, L, kk, N_idx);
  if (c >= si.k_s) return;
  const int n = count[gc], st = start[gc];
  const int cid = si.s * kk + c;  // only the last segment can have fewer than kk clusters
  const size_t urow = (size_t)si.unit * N_idx;
  const size_t orow = (size_t)si.unit * row_stride;  // rows per unit in perm / k_perm / v_perm
  const int row0 = si.seg_start + st;
  if (sub == 0) {
    sizes[(size_t)si.unit * mc + cid] = n;  // mc: clusters per unit in the meta-index arrays
    offsets[(size_t)si.unit * (mc + 1) + cid] = row0 + row_base;
    if (cid == m - 1) offsets[(size_t)si.unit * (mc + 1) + m] = N_idx + row_base;
  }
  const int32_t* ord = order + urow + si.seg_start + st;
  const T* Ku = K + ((size_t)si.unit * N + n_sink + si.seg_start) * D + sub * EPC;
  const T* Vu = V + ((size_t)si.unit * N + n_sink + si.seg_start) * D + sub * EPC;
  double ka[EPC], va[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) ka[e] = va[e] = 0.0;
  for (int i = 0; i < n; i += R) {
    int p[R];
    uint4 k[R], v[R];
#pragma unroll
    for (int u = 0; u < R; ++u) p[u] = ord[min(i + u, n - 1)];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      k[u] = load16(Ku + (size_t)p[u] * D);
      v[u] = load16(Vu + (size_t)p[u] * D);
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
      if (u > 0 && i + u >= n) continue;
      const size_t row = orow + row0 + i + u;
      float f[EPC];
      store16(k_perm + row * D + sub * EPC, k[u]);
      store16(v_perm + row * D + sub * EPC, v[u]);
      if (sub == 0) perm[row] = n_sink + si.seg_start + p[u] + pos_base;
      unpack<T>(k[u], f);
#pragma unroll
      for (int e = 0; e < EPC; ++e) ka[e] += (double)f[e];
      unpack<T>(v[u], f);
#pragma unroll
      for (int e = 0; e < EPC; ++e) va[e] += (double)f[e];
    }
  }
  T oc[EPC], ov[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) {
    oc[e] = quant_store<T>(n > 0 ? ka[e] / (double)n : 0.0);
    ov[e] = quant_store<T>(va[e]);
  }
  store16(centroids + ((size_t)si.unit * mc + cid) * D + sub * EPC, *reinterpret_cast<uint4*>(oc));
  store16(vsum + ((size_t)si.unit * mc + cid) * D + sub * EPC, *reinterpret_cast<uint4*>(ov));
}

// Steady rows: the first ns and the last (N - local_start) tokens of every unit.
template <typename T, int D>
__global__ __launch_bounds__(256) void steady_copy_kernel(const T* __restrict__ K, const T* __restrict__ V,
                                                          T* __restrict__ ks, T* __restrict__ vs, int N,
                                                          int ns, int local_start, int p,
                                                          int p_stride, int rows_total) {
  constexpr int EPC = Elem<T>::EPC, LPR = D / EPC, GROUPS = 256 / LPR;
  const int sub = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  for (int row = blockIdx.x * GROUPS + grp; row < rows_total; row += gridDim.x * GROUPS) {
    const int unit = row / p, i = row - unit * p;
    const int src = i < ns ? i : local_start + (i - ns);
    const size_t dst = (size_t)unit * p_stride + i;  // p_stride: rows per unit in the steady buffers
    store16(ks + dst * D + sub * EPC, load16(K + ((size_t)unit * N + src) * D + sub * EPC));
    store16(vs + dst * D + sub * EPC, load16(V + ((size_t)unit * N + src) * D + sub * EPC));
  }
}

__global__ void zero_int_kernel(int32_t* p) { *p = 0; }
// p[i * stride] = v for i < n
__global__ void fill_int_kernel(int32_t* p, int n, size_t stride, int32_t v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[(size_t)i * stride] = v;
}

// ============================================================================
// Host
// ============================================================================
static int min_kL(const wave_index& ix) {
  return ix.clusters_per_segment < ix.segment_len ? ix.clusters_per_segment : ix.segment_len;
}

// A segment's centroid rows fit in LDS beside the lists of assign_delta_kernel (k = 512 at
// d = 128 is 136 KiB of the 160 KiB).
static bool centroids_resident(int dtype, int d, int kmax) {
  return dtype == WAVE_BF16 && (size_t)32 * ((kmax + 31) / 32) * (d * 2 + 16) <= 144 * 1024;
}

// Builds whose rounds are all full passes (fewer than four points per cluster) keep the centroids in LDS
// only for many segments of many points at d = 128; elsewhere the centroids staged tile by tile are
// the faster form, whether they fit or not: to copy a segment's rows first costs more than it saves
// on its few points, and one workgroup per CU leaves a last round of them.  Builds in ms, staged
// and resident: 528 segments of 2000 points x 512 centroids 2.46 and 2.70, 2112 of them 8.86 and 8.60,
// 4224 of them 17.3 and 16.5; 4096 of 1024 x 512 18.6 and 18.7, of 512 x 256 14.0 and 15.8; at d = 64
// 4224 of 2000 x 512 10.7 and 11.2.
static bool resident_full_passes(int dtype, int d, int kmax, int Lmax, int segs) {
  return centroids_resident(dtype, d, kmax) && d == 128 && Lmax >= 1536 && segs >= 2048;
}

// Segments that one workgroup clusters by itself (kmeans_small_kernel).
static bool small_segments(const wave_index& ix) {
  return ix.dtype == WAVE_BF16 && (ix.segment_len < ix.N_idx ? ix.segment_len : ix.N_idx) <= SMALL_L_MAX &&
         min_kL(ix) <= SMALL_K_MAX;
}

// Builds whose later rounds compare the points with the changed centroids only.  What these rounds
// keep (bounds per point, member sums per cluster, a few counters per segment) lies in the index's
// own k_perm and v_perm rows (of an update: the new ones), which only the last step writes: 8 bytes
// per point in k_perm, then 6 counters per segment in the first unit's; 8 d bytes per cluster in
// v_perm.  That fits with four points per cluster or more.
static bool delta_rounds(const wave_index& ix) {
  if (!centroids_resident(ix.dtype, ix.d, min_kL(ix))) return false;
  const long long segs = (long long)ix.B * ix.Hkv * ix.S, points = ix.N_idx;
  return 4ll * ix.S * min_kL(ix) <= points && 8 * points + 24 * segs + 16 <= 2ll * ix.d * points &&
         segs * LIST_SPLIT * 256 < (1ll << 32);  // (a launch has fewer than 2^32 threads)
}

BuildGeom build_geometry(const wave_index& ix) {
  BuildGeom g{};
  g.units = ix.B * ix.Hkv;
  g.segs = g.units * ix.S;
  if (ix.m == 0) {
    g.total = 0;
    return g;
  }
  const size_t es = ix.dtype == WAVE_BF16 ? 2 : 4;
  const size_t pts = (size_t)g.units * ix.N_idx;
  const size_t ncl = (size_t)g.segs * min_kL(ix);
  size_t o = 0;
  g.off_xhat = o;   o = align_up(o + pts * ix.d * es);
  g.off_chat = o;   o = align_up(o + ncl * ix.d * es);
  g.off_assign = o; o = align_up(o + pts * sizeof(int32_t));
  g.off_order = o;  o = align_up(o + pts * sizeof(int32_t));
  g.off_prev = o;   o = align_up(o + pts * sizeof(int32_t));
  g.off_count = o;  o = align_up(o + 3 * ncl * sizeof(int32_t));   // count, start, changed marks
  g.off_flag = o;   o = align_up(o + pts * sizeof(int32_t));
  g.off_nflag = o;  o = align_up(o + 256);
  g.off_init = o;   o = align_up(o + (size_t)g.segs * ix.d * sizeof(double));  // segment means
  g.total = o;
  return g;
}

// WAVE_NO_SMALL_KMEANS=1 in the environment keeps short segments on the one-launch-per-step
// kernels (the tests run both forms against the oracle).
static bool no_small_kmeans() {
  const char* e = getenv("WAVE_NO_SMALL_KMEANS");
  return e && e[0] == '1';
}

// Whether launch_build takes an update's window: its segments go to kmeans_small_kernel, a workgroup and a CU each, and
// what the idle CUs take longer for the window than a launch of the whole chip is no more than the clustering.  A CU
// moves 36 GB/s (64 of them 2.33 TB/s, 104 3.3, 128 4.3), the whole chip 5.3 TB/s; the clustering takes about 10 us and
// 9 a round of 1024 points (1, 3, 10 rounds: 30, 58, 105), under 340 points 3 a round; after ten few points move.  A
// quarter of the CUs is the least that was measured.
// An update of segments of 1024 tokens, ten rounds, d = 128, window routed first and beside, in us: 128 segments, window
// 1024 212 and 163; 192, window 1024 267 and 256, window 8192 521 and 804; of 512 tokens, 176, window 1024 152 and 148,
// window 4096 263 and 332; of 1024 tokens, three rounds, 152, window 1024 193 and 169, 176 211 and 214.
bool build_routes_window(const wave_index& ix, const WindowRoute& window, int iters) {
  const long long segs = (long long)ix.B * ix.Hkv * ix.S;
  if (ix.m == 0 || !small_segments(ix) || no_small_kmeans() || segs > 192) return false;
  const double bytes = 64.0 * (double)window.total();  // a chunk of a key and of a value, read and written
  const double rounds = iters < 10 ? iters : 10, points = ix.segment_len < 340 ? 340 : ix.segment_len;
  return bytes / (36e3 * (double)(256 - segs)) <= bytes / 5.3e6 + 10.0 + rounds * 9.0 / 1024 * points;  // us
}

static int key_bits_for(int kk) {
  int b = 1;
  while ((1 << b) < kk) ++b;
  return b;
}

// What an incremental round of a bf16 build needs beside the points and centroids; all null elsewhere.
// bounds, changed: null in a round that compares every point with every centroid; with `bounds` alone
// such a round leaves what the next one needs to compare with the changed centroids only, and in prev
// which points moved.  nlisted: points listed per segment (all zero; nlisted_next is cleared), or null:
// near-ties of all segments go to one list, for refine_kernel.
struct AssignRound {
  int32_t* prev;
  PointBounds* bounds;
  long long bounds_skip;
  const int32_t *changed, *nchanged;
  int32_t *nlisted, *nlisted_next;
};

// One assign step of round `round`.
template <typename T, int D>
static void launch_assign(const T* xhat, const T* chat, int32_t* assign, const AssignRound& ar, int round, int32_t* flag,
                          int32_t* nflag, int S, int L, int kk, int N_idx, int segs, int refine_wgs, hipStream_t st) {
  const auto [prev, bounds, bounds_skip, changed, nchanged, nlisted, nlisted_next] = ar;
  const int Lmax = L < N_idx ? L : N_idx, kmax = kk < Lmax ? kk : Lmax;
  if constexpr (sizeof(T) == 2) {
    if (nlisted || resident_full_passes(WAVE_BF16, D, kmax, Lmax, segs)) {
      // At least two workgroups per long segment keep the last round of workgroups short; a few
      // segments are cut finer, down to a fragment per wave, until every CU has its share (32 segments
      // of 8192 points x 512 centroids: 104 us a full pass with 2 each, 37 us so).
      auto cut = [&](int points, int wgs_wanted, int least_points) {
        int pieces = (Lmax + points - 1) / points;
        const int want = wgs_wanted / segs, most = (Lmax + least_points - 1) / least_points;
        return want > pieces ? (want < most ? want : (most > pieces ? most : pieces)) : pieces;
      };
      int pieces = cut(ASSIGN_POINTS, 256, 512);
      if (pieces < 2 && Lmax > 2048) pieces = 2;
      // One workgroup per CU or fewer: each decides the points of its list itself, and a later round is one
      // launch for segments of all numbers of changed centroids instead of three (builds of 32 segments of 8192
      // points 704 and 621 us, of 80 1956 and 1818, of 128 1743 and 1646; 512 waiting workgroups hide the chain
      // at a list's end better).  Not where a workgroup takes a whole segment and CUs stay idle: the three
      // launches cut it finer (136 segments of 2048 points 457, at once 464 us).
      const bool at_once = nlisted && segs * pieces <= 256 && (pieces > 1 || Lmax <= 512);
      if (at_once && changed) {
        WAVE_LAUNCH("assign_delta", (assign_delta_kernel<D, 16, true>), segs * pieces, 1024,
                    delta_lds<D>(kmax, 1 << 20, ASSIGN_POINTS, true), st, xhat, chat, assign, prev, bounds, bounds_skip,
                    changed, nchanged, flag, nlisted, 0, 1 << 20, round, S, L, kk, N_idx, pieces, segs * pieces);
      } else if (at_once) {
        WAVE_LAUNCH("assign_mfma", (assign_resident_kernel<D, 1, 16, true>), segs * pieces, 1024,
                    resident_lds<D>(kmax, true), st, xhat, chat, assign, prev, bounds, bounds_skip, flag, nlisted, nflag,
                    round, S, L, kk, N_idx, pieces);
      } else if (changed) {
        constexpr int light = delta_light_rows<D>();
        const int light_pieces = cut(LIGHT_POINTS, 512, 256);
        if (kmax > light) {  // (usually none after a few rounds: no more workgroups than a CU each)
          const int total = segs * pieces;
          WAVE_LAUNCH("assign_delta", (assign_delta_kernel<D, 16, false>), total < 256 ? total : 256, 1024,
                      delta_lds<D>(kmax, 1 << 20, ASSIGN_POINTS, false), st, xhat, chat, assign, prev, bounds, bounds_skip, changed,
                      nchanged, flag, nlisted, light, 1 << 20, round, S, L, kk, N_idx, pieces, total);
        }
        WAVE_LAUNCH("assign_delta", (assign_delta_kernel<D, 8, false>), segs * light_pieces, 512,
                    delta_lds<D>(kmax, light, LIGHT_POINTS, false), st, xhat, chat, assign, prev, bounds, bounds_skip, changed,
                    nchanged, flag, nlisted, 0, light, round, S, L, kk, N_idx, light_pieces, segs * light_pieces);
      } else
        WAVE_LAUNCH("assign_mfma", (assign_resident_kernel<D, 1, 16, false>), segs * pieces, 1024, resident_lds<D>(kmax, false),
                    st, xhat, chat, assign, prev, bounds, bounds_skip, flag, nlisted, nflag, round, S, L, kk, N_idx, pieces);
      if (at_once) return;
      if (nlisted) {
        WAVE_LAUNCH("assign_listed", (assign_listed_kernel<D>), segs * LIST_SPLIT, 256, listed_lds<D>(kmax), st, xhat,
                    chat, assign, prev, bounds, bounds_skip, flag, nlisted, nlisted_next, round, segs, S, L, kk, N_idx);
        return;
      }
    } else {  // the centroids are staged through LDS tile by tile
      constexpr int PWG = 8 * 32;
      const int wps = (Lmax + PWG - 1) / PWG;
      WAVE_LAUNCH("assign_mfma", (assign_mfma_kernel<D, 1, 8>), segs * wps, 64 * 8, 0, st, xhat, chat,
                  assign, flag, nflag, S, L, kk, N_idx, wps);
    }
    WAVE_LAUNCH("refine", (refine_kernel<T, D>), refine_wgs, 256, 0, st, xhat, chat, assign, flag, nflag, S,
                L, kk, N_idx);
  } else {
    const int frags = (Lmax + 31) / 32;
    if (segs * frags < 1024)
      WAVE_LAUNCH("assign_f32", (assign_f32_kernel<D, true>), segs * frags, 256, 0, st, xhat, chat, assign, S, L, kk,
                  N_idx, frags);
    else
      WAVE_LAUNCH("assign_f32", (assign_f32_kernel<D, false>), segs * ((frags + 3) / 4), 256, 0, st, xhat, chat, assign,
                  S, L, kk, N_idx, (frags + 3) / 4);
  }
}

template <typename T, int D>
static wave_status build_td(const void* K_, const void* V_, const wave_index& ix, int iters,
                            uint64_t seed, void* ws, hipStream_t st, int seg_id_base, int row_base,
                            int pos_base, const WindowRoute* window) {
  const T* K = static_cast<const T*>(K_);
  const T* V = static_cast<const T*>(V_);
  const int units = ix.B * ix.Hkv;
  const int ns = ix.n_sink < ix.N ? ix.n_sink : ix.N;
  const int local_start = ns + ix.N_idx;
  if (ix.p > 0) {
    const int rows = units * ix.p;
    const int grid = (rows + 15) / 16 < 65536 ? (rows + 15) / 16 : 65536;
    WAVE_LAUNCH("steady_copy", (steady_copy_kernel<T, D>), grid, 256, 0, st, K, V,
                static_cast<T*>(ix.k_steady), static_cast<T*>(ix.v_steady), ix.N, ns, local_start, ix.p,
                steady_stride(ix), rows);
  }
  if (ix.m == 0) {
    // nothing to cluster: offsets[0] = 0 in every unit (units are cluster_stride + 1 entries apart)
    if (ix.offsets)
      WAVE_LAUNCH("fill", fill_int_kernel, (units + 255) / 256, 256, 0, st, ix.offsets, units,
                  (size_t)cluster_stride(ix) + 1, 0);
    return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_ERR_HIP;
  }

  const BuildGeom g = build_geometry(ix);
  char* w = static_cast<char*>(ws);
  T* xhat = reinterpret_cast<T*>(w + g.off_xhat);
  T* chat = reinterpret_cast<T*>(w + g.off_chat);
  int32_t* assign = reinterpret_cast<int32_t*>(w + g.off_assign);
  int32_t* order = reinterpret_cast<int32_t*>(w + g.off_order);
  const int kk = min_kL(ix);
  const int ncl = g.segs * kk;
  int32_t* count = reinterpret_cast<int32_t*>(w + g.off_count);
  int32_t* start = count + ncl;
  const int S = ix.S, L = ix.segment_len, N_idx = ix.N_idx;
  const bool small = window || (small_segments(ix) && !no_small_kmeans());
  const bool delta = !small && iters <= PREV_ROUNDS && delta_rounds(ix);
  int32_t* changed = start + ncl;  // per cluster: a point entered or left it in the current round
  int32_t* prev = reinterpret_cast<int32_t*>(w + g.off_prev);  // every point's cluster of the round before
  // (see delta_rounds)
  PointBounds* bounds = delta ? reinterpret_cast<PointBounds*>(ix.k_perm) : nullptr;
  double* sums = delta ? reinterpret_cast<double*>(ix.v_perm) : nullptr;
  const long long unit8 = (long long)row_stride(ix) * D * (long long)sizeof(T) / 8;  // 8-byte words per unit there
  const long long bounds_skip = unit8 - N_idx, sums_skip = unit8 - (long long)S * kk * D;
  int32_t* per_seg = delta ? reinterpret_cast<int32_t*>(bounds + N_idx) : nullptr;
  int32_t* range = per_seg;  // smallest and largest exponent of a segment's normalised keys
  // changed centroids, and points listed by the assign step (of even and of odd rounds: each round
  // clears the other one)
  int32_t *nchanged[2] = {}, *nlisted[2] = {};
  for (int i = 0; i < 2 && delta; ++i) {
    nchanged[i] = per_seg + (2 + i) * (size_t)g.segs;
    nlisted[i] = per_seg + (4 + i) * (size_t)g.segs;
  }
  int32_t* flag = reinterpret_cast<int32_t*>(w + g.off_flag);
  int32_t* nflag = reinterpret_cast<int32_t*>(w + g.off_nflag);
  double* mean = reinterpret_cast<double*>(w + g.off_init);
  constexpr int GROUPS = 256 / (D / Elem<T>::EPC);
  // what the first steps read: K, or the window's rows where they lie
  const T* K_in = window ? reinterpret_cast<const T*>(window->k_old) + (size_t)window->ns * D : K;
  const int N_in = window ? window->p_old : ix.N;

  {
    // A few segments: pieces of at least 256 rows until every CU has two workgroups.  Their sums go where the order of
    // the points comes later (4 bytes a point).
    int pieces = 1;
    const int Lmax = L < N_idx ? L : N_idx;
    while (g.segs * pieces < 512 && pieces < 16 && Lmax / (2 * pieces) >= 256 &&
           (size_t)g.segs * 2 * pieces * D * sizeof(double) <= (size_t)units * N_idx * sizeof(int32_t))
      pieces *= 2;
    double* sums_of = pieces > 1 ? reinterpret_cast<double*>(order) : mean;
    WAVE_LAUNCH("seg_mean", (seg_mean_kernel<T, D>), g.segs * pieces, 256, 0, st, K_in, sums_of, nflag, range, nchanged[1],
                nlisted[0], S, L, kk, N_in, N_idx, ns, pieces);
    const int half = NORM_ROWS / 2;
    const bool halves = range ? 4 * GROUPS <= half && g.segs * ((Lmax + half - 1) / half) <= 256
                              : g.segs * ((Lmax + NORM_ROWS - 1) / NORM_ROWS) < 256;
    int row_step = halves ? half : NORM_ROWS, chunks = (Lmax + row_step - 1) / row_step;
    if (g.segs * chunks > NORM_RESIDENT && g.segs * ((chunks + 1) / 2) <= NORM_RESIDENT) {
      row_step *= 2;
      chunks = (chunks + 1) / 2;
    }
    WAVE_LAUNCH("normalise", (normalise_kernel<T, D>), g.segs * chunks, 256, 0, st, K_in, sums_of, mean, xhat, range, S, L, kk,
                N_in, N_idx, ns, chunks, row_step, pieces);
  }
  {
    int pieces = 1;  // a workgroup for every CU, of at least 32 draws
    while (g.segs * pieces < 256 && kk / pieces >= 64) pieces *= 2;
    int buckets = 64;
    while (buckets < kk) buckets *= 2;
    WAVE_LAUNCH("init", (init_kernel<T, D>), g.segs * pieces, 256, sizeof(int) * (3 * (size_t)kk + buckets), st, xhat, chat,
                S, L, kk, N_idx, ix.Hkv, seed, seg_id_base, pieces, buckets);
  }

  const int cl_grid = (ncl + GROUPS - 1) / GROUPS;
  // update_scan_kernel: at least as many clusters a workgroup as it has groups of lanes, more where that leaves
  // a workgroup for every CU: each reads a segment's assignments (100 fp32 segments of 4096 points, 8 workgroups a
  // segment 2.06 ms a build, 4 1.99).
  int scan_span = SCAN_NT / (D / Elem<T>::EPC);
  while (2 * scan_span <= SCAN_CLUSTERS && (long long)g.segs * ((kk + 2 * scan_span - 1) / (2 * scan_span)) >= 256)
    scan_span *= 2;
  const int scan_pieces = (kk + scan_span - 1) / scan_span;
  if constexpr (sizeof(T) == 4) {
    // Two launches a round.  The assignments of even and of odd rounds have an array each.
    for (int t = 0; t < iters; ++t) {
      int32_t* now = t & 1 ? prev : assign;
      launch_assign<T, D>(xhat, chat, now, AssignRound{}, t, flag, nflag, S, L, kk, N_idx, g.segs, 0, st);
      WAVE_LAUNCH("update", (update_scan_kernel<T, D>), g.segs * scan_pieces, SCAN_NT, 0, st, xhat, chat, now,
                  t & 1 ? assign : prev, order, count, start, nullptr, 0, t == 0 ? 1 : 0, t + 1 == iters ? 1 : 0, S, L, kk,
                  N_idx, scan_span, scan_pieces);
    }
  } else {
    int W = SORT_HIST_INTS / kk;
    if (W > 16) W = 16;
    if (W < 1) W = 1;
    const size_t sort_lds = ((size_t)W * kk + kk) * sizeof(int);
    const int kb = key_bits_for(kk);
    if (small) {
      auto run = [&](auto kernel, int waves, bool keep_sums) {
        // (a workgroup takes a CU at these sizes: the window goes to the others, as far as it has a chunk for each thread)
        const size_t wanted = window ? (window->total() + 64 * waves - 1) / (64 * waves) : 0;
        const int movers = (int)(wanted < (size_t)(256 - g.segs) ? wanted : (size_t)(256 - g.segs));
        WAVE_LAUNCH("kmeans_small", kernel, g.segs + movers, 64 * waves, small_kmeans_lds<D>(kk, keep_sums), st, xhat, chat,
                    order, count, start, window ? *window : WindowRoute{}, g.segs, S, L, kk, N_idx, iters, kb);
      };
      constexpr int KEEP = 512 / D, KW = small_waves<KEEP>();  // (128 registers a lane)
      const bool keep = (L < N_idx ? L : N_idx) <= 32 * KEEP * KW;
      const bool keep_sums = (size_t)kk * D <= 8192;  // 64 KiB
      if (keep && keep_sums) run(kmeans_small_kernel<D, KEEP, true>, KW, true);
      else if (keep) run(kmeans_small_kernel<D, KEEP, false>, KW, false);
      else if (keep_sums) run(kmeans_small_kernel<D, 0, true>, SMALL_NW, true);
      else run(kmeans_small_kernel<D, 0, false>, SMALL_NW, false);
    }
    auto sort = [&](int32_t* prev_or_null, int t) {
      WAVE_LAUNCH("sort", sort_kernel, g.segs, 64 * W, sort_lds, st, assign, order, count, start, nflag,
                  prev_or_null, changed, t == 0 ? 1 : 0, S, L, kk, N_idx, kb);
    };
    // clusters whose marks a workgroup of the later updates reads: 256 in a large batch; few enough to
    // give 1024 workgroups, down to one per group of lanes (2 segments of 128 clusters in one workgroup:
    // 125 us a round, 12 us so)
    int span = (ncl + 1023) / 1024;
    span = span < GROUPS ? GROUPS : (span > 256 ? 256 : span);
    auto update = [&](int t) {
      // (first round: nothing to compare with, every cluster is updated and every mark cleared.
      // Large clusters go onto a list, which the second kernel takes: nflag[1] counts them and
      // the flagged-point list, consumed by refine, is free to hold them)
      if (t == 0)
        WAVE_LAUNCH("update", (update_kernel<T, D>), cl_grid, 256, 0, st, xhat, chat, order, count,
                    start, changed, flag, nflag + 1, sums, sums_skip, S, L, kk, N_idx, ncl);
      else
        WAVE_LAUNCH("update", (update_touched_kernel<T, D>), (ncl + span - 1) / span, 256, 0, st, xhat, chat,
                    order, count, start, changed, flag, nflag + 1, S, L, kk, N_idx, ncl, span);
      const int big_grid = ncl / UPD_BIG + 1 < 2048 ? ncl / UPD_BIG + 1 : 2048;
      WAVE_LAUNCH("update", (update_big_kernel<T, D>), big_grid, 256, 0, st, xhat, chat, order, count,
                  start, flag, nflag + 1, sums, sums_skip, S, L, kk, N_idx);
    };
    // The first and the last round of a few segments: several workgroups sort and sum a segment, not one (32
    // segments of 8192 points x 512 clusters: sort, update and large clusters 42 us, 36 us so, a build of 6 segments
    // of 4096 x 256 495 and 483 us); 224 segments pay for reading their assignments eight times (3.01 and 3.13 ms).  Of
    // 8192 x 512, eight workgroups each, 64 segments are level (1106 and 1109), 96 and 127 lose 1.4 and 2.4 %; of 4096 x
    // 256, four each, 96 are level (567) and 127 gain 1 %, 144 would lose 2 % (849 and 866 us).
    const bool scan = delta && g.segs < 128;
    for (int t = 0; t < iters && !small; ++t) {
      // Rounds 0 and 1 meet all new centroids; from round 2 on only the changed ones are compared.
      const AssignRound ar{prev, t >= 1 ? bounds : nullptr, bounds_skip, delta && t >= 2 ? changed : nullptr,
                           nchanged[(t + 1) & 1], nlisted[t & 1], nlisted[(t + 1) & 1]};
      launch_assign<T, D>(xhat, chat, assign, ar, t, flag, nflag, S, L, kk, N_idx, g.segs, 1024, st);
      const bool last = t + 1 == iters;
      if (scan && (t == 0 || last)) {
        WAVE_LAUNCH("update", (update_scan_kernel<T, D>), g.segs * scan_pieces, SCAN_NT, 0, st, xhat, chat, assign, assign,
                    order, count, start, sums, sums_skip, t == 0 ? 1 : 0, last ? 1 : 0, S, L, kk, N_idx, scan_span,
                    scan_pieces);
        continue;
      }
      if (!delta || t == 0 || last) sort(delta ? nullptr : prev, t);
      if (last) break;
      if (delta && t >= 1) {
        // a few segments are shared by several workgroups each, of at least 64 clusters
        int pieces = 1;
        while (g.segs * pieces < 512 && kk / pieces >= 128) pieces *= 2;
        WAVE_LAUNCH("update", (update_moves_kernel<D>), g.segs * pieces, MOVE_NT, update_moves_lds(kk), st, xhat,
                    chat, sums, sums_skip, assign, prev, changed, nchanged[t & 1], nchanged[(t + 1) & 1], range, order, count, start, t, S, L, kk, N_idx, pieces, kb);
        continue;
      }
      update(t);
    }
  }
  const bool many_rows = cl_grid <= 3 * 256 || (long long)S * kk * 4 <= N_idx;  // (eight in flight: 3 workgroups a CU)
  auto finalize = [&](auto kernel) {
    WAVE_LAUNCH("finalize", kernel, cl_grid, 256, 0, st, K, V, order, count, start,
                static_cast<T*>(ix.centroids), static_cast<T*>(ix.vsum), ix.sizes, ix.offsets, ix.perm,
                static_cast<T*>(ix.k_perm), static_cast<T*>(ix.v_perm), S, L, kk, ix.N, N_idx, ns, ix.m,
                cluster_stride(ix), ncl, row_stride(ix), row_base, pos_base);
  };
  if (many_rows) finalize(finalize_kernel<T, D, 8>);
  else finalize(finalize_kernel<T, D, 2>);
  return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_ERR_HIP;
}

wave_status launch_build(const void* K, const void* V, const wave_index& ix, int iters, uint64_t seed,
                         void* ws, hipStream_t st, int seg_id_base, int row_base, int pos_base,
                         const WindowRoute* window) {
  if (ix.dtype == WAVE_BF16) {
    if (ix.d == 128) return build_td<bf16_t, 128>(K, V, ix, iters, seed, ws, st, seg_id_base, row_base, pos_base, window);
    if (ix.d == 64) return build_td<bf16_t, 64>(K, V, ix, iters, seed, ws, st, seg_id_base, row_base, pos_base, window);
  } else {
    if (ix.d == 128) return build_td<float, 128>(K, V, ix, iters, seed, ws, st, seg_id_base, row_base, pos_base, window);
    if (ix.d == 64) return build_td<float, 64>(K, V, ix, iters, seed, ws, st, seg_id_base, row_base, pos_base, window);
  }
  return WAVE_ERR_SHAPE;
}

template <typename T, int D>
static wave_status assign_step_td(const void* xhat, const void* chat, int L_s, int k_s, int32_t* assign,
                                  void* ws, hipStream_t st) {
  int32_t* nflag = static_cast<int32_t*>(ws);
  int32_t* flag = nflag + 64;
  hipLaunchKernelGGL(zero_int_kernel, dim3(1), dim3(1), 0, st, nflag);
  // one unit, one segment: S = 1, L = N_idx = L_s, kk = k_s
  AssignRound ar{};
  if (centroids_resident(sizeof(T) == 2 ? WAVE_BF16 : WAVE_F32, D, k_s)) {
    ar.nlisted = nflag;
    ar.nlisted_next = nflag + 1;
  }
  launch_assign<T, D>(static_cast<const T*>(xhat), static_cast<const T*>(chat), assign, ar, 0, flag, nflag, 1, L_s, k_s, L_s,
                      1, 256, st);
  return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_ERR_HIP;
}

wave_status launch_assign_step(const void* xhat, const void* chat, int dtype, int L_s, int k_s, int d,
                               int32_t* assign, void* ws, hipStream_t st) {
  if (dtype == WAVE_BF16) {
    if (d == 128) return assign_step_td<bf16_t, 128>(xhat, chat, L_s, k_s, assign, ws, st);
    if (d == 64) return assign_step_td<bf16_t, 64>(xhat, chat, L_s, k_s, assign, ws, st);
  } else {
    if (d == 128) return assign_step_td<float, 128>(xhat, chat, L_s, k_s, assign, ws, st);
    if (d == 64) return assign_step_td<float, 64>(xhat, chat, L_s, k_s, assign, ws, st);
  }
  return WAVE_ERR_SHAPE;
}

}  // namespace wave
