// Message build (difference, linear quantisation, cache commit) and message recovery
// (dequantise, receiver-side cache update) - Sec. 5 and Alg. 2.
//
// Both kernels give one message row to a group of G = 2^glog lanes (a whole wavefront,
// looping, for rows of more than 64 vectors). A row is held in registers between the
// min/max pass and the coding pass, so it is read from HBM exactly once; the commit
// reuses the same registers. The number of rows comes from device memory (*n_sent);
// the grid is sized for max_sent and surplus groups leave at once.
//
// fp32 sequence (must match on every implementation for bit-equal codes):
//   inv = Lv / (hi - lo)            one correctly rounded division per row
//   q   = floor(fma(m - lo, inv, 0.5)) clamped to [0, Lv]
//   back: scale = (hi - lo) / Lv,   m~ = fma(q, scale, lo)
#include <algorithm>

#include "cdf_common.h"

namespace cdf {

constexpr int kQuantThreads = 256;
// The number of message rows is only known on the device, so grids are sized for the capacity -
// but never beyond this many blocks: the kernels walk the rows in strides, so a call that sends
// nothing costs 0.03 ms instead of up to 0.9 ms of empty blocks (5 M rows), while a call that sends
// everything still runs within a few per cent of a grid with one block per group of rows (smaller
// caps measured up to 25 % slower there).
constexpr int64_t kMessageGridCap = 131072;

// Statistics, codes, meta and cache commit of one message row held in registers: x = current row,
// z = cached row, m = what is sent. Every lane of the group must call it (the row statistics use
// cross-lane exchanges); `live` gates all stores. out / meta_row / pz point at this row's codes,
// its two meta floats and its cached row.
template <typename T, int EPV, int NIT, int BITS, int QS>
__device__ __forceinline__ void encode_row(bool live, int lg, int G, int nvec, const float (&x)[NIT][EPV],
                                           const float (&z)[NIT][EPV], const float (&m)[NIT][EPV], int commit,
                                           int delta, uint8_t* out, float* meta_row, T* pz) {
  // row statistics
  float lo = __builtin_inff(), hi = -__builtin_inff(), amax = 0.0f;
#pragma unroll
  for (int i = 0; i < NIT; ++i) {
    if (lg + i * G < nvec) {
#pragma unroll
      for (int c = 0; c < EPV; ++c) {
        lo = fminf(lo, m[i][c]);
        hi = fmaxf(hi, m[i][c]);
        amax = fmaxf(amax, fabsf(m[i][c]));
      }
    }
  }
  float m0 = 0.0f, m1 = 0.0f, inv = 0.0f, scale = 0.0f, sub = 0.0f;
  int qlo = 0, qhi = 0;
  if (QS == CDF_Q_MINMAX) {
    lo = group_min(lo, G);
    hi = group_max(hi, G);
    const float Lv = static_cast<float>((1 << BITS) - 1);
    const float range = hi - lo;
    inv = range > 0.0f ? Lv / range : 0.0f;
    scale = range / Lv;
    sub = lo;
    m0 = lo;
    m1 = hi;
    qlo = 0;
    qhi = (1 << BITS) - 1;
  } else if (QS == CDF_Q_SYMMETRIC) {
    amax = group_max(amax, G);
    const float Qm = static_cast<float>((1 << (BITS - 1)) - 1);
    inv = amax > 0.0f ? Qm / amax : 0.0f;
    scale = amax / Qm;
    sub = 0.0f;
    m0 = scale;
    m1 = 0.0f;
    qhi = (1 << (BITS - 1)) - 1;
    qlo = -qhi;
  }
  if (live && lg == 0) {
    meta_row[0] = m0;
    meta_row[1] = m1;
  }

#pragma unroll
  for (int i = 0; i < NIT; ++i) {
    const int v = lg + i * G;
    const bool on = live && v < nvec;
    float dq[EPV];
    if (QS == CDF_Q_NONE) {
      if (on) VecIO<float, EPV>::store(reinterpret_cast<float*>(out) + static_cast<int64_t>(v) * EPV, m[i]);
#pragma unroll
      for (int c = 0; c < EPV; ++c) dq[c] = m[i][c];
    } else {
      int q[EPV];
#pragma unroll
      for (int c = 0; c < EPV; ++c) {
        float t = floorf(__fmaf_rn(m[i][c] - sub, inv, 0.5f));
        t = fminf(fmaxf(t, static_cast<float>(qlo)), static_cast<float>(qhi));  // clamp, then convert
        const int qi = static_cast<int>(t);
        q[c] = on ? qi : 0;
        dq[c] = QS == CDF_Q_MINMAX ? __fmaf_rn(static_cast<float>(qi), scale, m0) : static_cast<float>(qi) * scale;
      }
      constexpr unsigned CM = (1u << BITS) - 1u;
      if (EPV == 1 && BITS == 4) {
        // two lanes share a byte: the even element's lane stores both nibbles
        const int partner = __shfl_xor(q[0], 1, kWave);
        if (on && (v & 1) == 0)
          out[v >> 1] = static_cast<uint8_t>((q[0] & CM) | ((partner & CM) << 4));
      } else {
        unsigned word = 0;
#pragma unroll
        for (int c = 0; c < EPV; ++c) word |= (static_cast<unsigned>(q[c]) & CM) << (BITS * c);
        if (on) {
          constexpr int NB = EPV * BITS / 8;  // bytes per lane-vector: 4, 2 or 1
          uint8_t* dstp = out + static_cast<int64_t>(v) * NB;
          if (NB == 4) *reinterpret_cast<uint32_t*>(dstp) = word;
          else if (NB == 2) *reinterpret_cast<uint16_t*>(dstp) = static_cast<uint16_t>(word);
          else *dstp = static_cast<uint8_t>(word);
        }
      }
    }
    if (on) {
      if (commit == CDF_COMMIT_CUR) {
        VecIO<T, EPV>::store(pz + static_cast<int64_t>(v) * EPV, x[i]);
      } else if (commit == CDF_COMMIT_DEQ) {
        float nv[EPV];
#pragma unroll
        for (int c = 0; c < EPV; ++c) nv[c] = delta ? z[i][c] + dq[c] : dq[c];
        VecIO<T, EPV>::store(pz + static_cast<int64_t>(v) * EPV, nv);
      }
    }
  }
}

// `NIT` vectors of EPV elements per lane: covers rows of up to 64*NIT vectors.
template <typename T, int EPV, int NIT, int BITS, int QS>
__global__ __launch_bounds__(kQuantThreads) void quantize_kernel(
    const T* __restrict__ cur, T* cached, const int* __restrict__ idx, const int* __restrict__ n_sent_p, int max_sent,
    int dim, int64_t ld, int glog, int commit, int delta, uint8_t* __restrict__ codes,
    float* __restrict__ meta) {
  const int n_sent = min(*n_sent_p, max_sent);   // never past the capacity of idx / codes / meta
  const int lane = threadIdx.x & 63;
  const int G = 1 << glog;
  const int lg = lane & (G - 1);
  const int rows_per_wave = 64 >> glog;
  const int gwave = blockIdx.x * (kQuantThreads / 64) + (threadIdx.x >> 6);
  const int nvec = dim / EPV;
  const int64_t rb = QS == CDF_Q_NONE ? static_cast<int64_t>(dim) * 4 : (static_cast<int64_t>(dim) * BITS + 7) / 8;
  // the grid is capped; a wavefront walks its share of the rows (the bound is the same for all its lanes)
  const int wave_stride = gridDim.x * (kQuantThreads / 64) * rows_per_wave;
  for (int kb = gwave * rows_per_wave; kb < n_sent; kb += wave_stride) {
  const int k = kb + (lane >> glog);
  const bool live = k < n_sent;

  float x[NIT][EPV], z[NIT][EPV], m[NIT][EPV];
  int64_t r = 0;
  if (live) r = idx[k];
  const T* pc = cur + r * ld;
  T* pz = cached + r * ld;
#pragma unroll
  for (int i = 0; i < NIT; ++i) {
    const int v = lg + i * G;
#pragma unroll
    for (int c = 0; c < EPV; ++c) x[i][c] = z[i][c] = 0.0f;
    if (live && v < nvec) {
      VecIO<T, EPV>::load(pc + static_cast<int64_t>(v) * EPV, x[i]);
      if (delta || commit == CDF_COMMIT_DEQ) VecIO<T, EPV>::load(pz + static_cast<int64_t>(v) * EPV, z[i]);
    }
#pragma unroll
    for (int c = 0; c < EPV; ++c) m[i][c] = delta ? x[i][c] - z[i][c] : x[i][c];
  }

  encode_row<T, EPV, NIT, BITS, QS>(live, lg, G, nvec, x, z, m, commit, delta,
                                    codes + static_cast<int64_t>(live ? k : 0) * rb,
                                    meta + 2 * static_cast<int64_t>(live ? k : 0), pz);
  }
}

// Cache test and message build in one pass over the rows (the two steps of Alg. 2's mirror loop
// back to back): every row is read once, tested (either norm), and - if it fails the test -
// coded and committed from the same registers. The position of a row's message in the output is
// only known after the count of sent rows before it, so codes and meta go to a row-indexed
// scratch area first and place_messages_kernel moves them to their final place (one byte per
// element instead of re-reading the rows at eight). Blocks of kTestRows rows, one count per block,
// as the cache test writes them; 4 or 16 wavefronts share a block's rows (small inputs take 16: a wavefront
// walks its rows one memory round trip after another, and 64 rows by four of them leave the chip idle: with 4 / 16
// 757 rows of 128 in 17.6 / 8.2 us, 20 000 of 256 in 41 / 24, 55 978 of 41 in 39 / 31; with more than eight elements a lane
// the registers of 16 wavefronts cost more than they bring: 55 978 rows of 602 in 68 / 75 us, 214 000 of 1024 bf16 in 347 /
// 431). A form of this kernel in which a workgroup waited for the counts of those before it and wrote every message
// straight to its place saved the second kernel and took longer at every size (18.1, 32, 33 us on the first three).
constexpr int kTestRows = kRowsPerBlock;
constexpr int kTestThreadsMax = 1024;
constexpr int kTestWideBlocks = 4096;   // blocks up to which they take 16 wavefronts
__host__ __device__ constexpr int test_threads(int per_lane) { return per_lane > 8 ? kQuantThreads : kTestThreadsMax; }

template <typename T, int EPV, int NIT, int BITS, int QS>
__global__ __launch_bounds__(test_threads(NIT * EPV)) void test_encode_kernel(
    const T* __restrict__ cur, T* cached, int n_rows, int dim, int64_t ld, float eps, int norm, int glog, int commit,
    int delta, uint8_t* __restrict__ mask, int* __restrict__ block_counts, uint8_t* __restrict__ codes_scratch,
    float* __restrict__ meta_scratch) {
  constexpr int NACC = 4 / EPV;  // L2 norm: accumulators per lane-component, as in the cache test
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int G = 1 << glog;
  const int lg = lane & (G - 1), sub = lane >> glog;
  const int rows_per_step = 64 >> glog;
  const int nvec = dim / EPV;
  const int64_t rb = (static_cast<int64_t>(dim) * BITS + 7) / 8;
  const int waves = blockDim.x >> 6, rows_per_wave = kTestRows / waves;
  const int row0 = blockIdx.x * kTestRows + wave * rows_per_wave;
  int sent_here = 0;
  for (int s = 0; s < rows_per_wave; s += rows_per_step) {
    const int row = row0 + s + sub;
    const bool live = row < n_rows && s + sub < rows_per_wave;
    const int64_t r = live ? row : 0;
    const T* pc = cur + r * ld;
    T* pz = cached + r * ld;
    float x[NIT][EPV], z[NIT][EPV], m[NIT][EPV];
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int v = lg + i * G;
#pragma unroll
      for (int c = 0; c < EPV; ++c) x[i][c] = z[i][c] = 0.0f;
      if (live && v < nvec) {
        VecIO<T, EPV>::load(pc + static_cast<int64_t>(v) * EPV, x[i]);
        VecIO<T, EPV>::load(pz + static_cast<int64_t>(v) * EPV, z[i]);
      }
#pragma unroll
      for (int c = 0; c < EPV; ++c) m[i][c] = delta ? x[i][c] - z[i][c] : x[i][c];
    }
    // the test, in the cache test's own order of operations (masks must agree bit for bit)
    float D, C, thr;
    if (norm == CDF_NORM_LINF) {
      D = 0.0f;
      C = 0.0f;
#pragma unroll
      for (int i = 0; i < NIT; ++i)
#pragma unroll
        for (int c = 0; c < EPV; ++c) {
          D = fmaxf(D, fabsf(x[i][c] - z[i][c]));
          C = fmaxf(C, fabsf(z[i][c]));
        }
      D = group_max(D, G);
      C = group_max(C, G);
      thr = eps * C;
    } else {
      // vector i of a lane feeds accumulator i mod NACC; lanes past the row end add exact zeros
      float ad[NACC][EPV], ac[NACC][EPV];
#pragma unroll
      for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int c = 0; c < EPV; ++c) ad[a][c] = ac[a][c] = 0.0f;
#pragma unroll
      for (int i = 0; i < NIT; ++i)
#pragma unroll
        for (int c = 0; c < EPV; ++c) {
          const float d = x[i][c] - z[i][c];
          ad[i % NACC][c] = __fmaf_rn(d, d, ad[i % NACC][c]);
          ac[i % NACC][c] = __fmaf_rn(z[i][c], z[i][c], ac[i % NACC][c]);
        }
      float Da[NACC], Ca[NACC];
#pragma unroll
      for (int a = 0; a < NACC; ++a) {
        float d, c;
        if (EPV == 4) {
          d = (ad[a][0] + ad[a][1 % EPV]) + (ad[a][2 % EPV] + ad[a][3 % EPV]);
          c = (ac[a][0] + ac[a][1 % EPV]) + (ac[a][2 % EPV] + ac[a][3 % EPV]);
        } else if (EPV == 2) {
          d = ad[a][0] + ad[a][1 % EPV];
          c = ac[a][0] + ac[a][1 % EPV];
        } else {
          d = ad[a][0];
          c = ac[a][0];
        }
        Da[a] = group_sum(d, G);
        Ca[a] = group_sum(c, G);
      }
      if (NACC == 4) {
        D = (Da[0] + Da[1 % NACC]) + (Da[2 % NACC] + Da[3 % NACC]);
        C = (Ca[0] + Ca[1 % NACC]) + (Ca[2 % NACC] + Ca[3 % NACC]);
      } else if (NACC == 2) {
        D = Da[0] + Da[1 % NACC];
        C = Ca[0] + Ca[1 % NACC];
      } else {
        D = Da[0];
        C = Ca[0];
      }
      const float e2 = eps * eps;
      thr = e2 * C;
    }
    const bool send = live && D > thr;
    const bool head = live && lg == 0;
    if (head) mask[row] = send ? 1 : 0;
    sent_here += __popcll(__ballot(head && send));
    encode_row<T, EPV, NIT, BITS, QS>(send, lg, G, nvec, x, z, m, commit, delta, codes_scratch + r * rb,
                                      meta_scratch + 2 * r, pz);
  }
  __shared__ int wave_cnt[kTestThreadsMax / 64];
  if (lane == 0) wave_cnt[wave] = sent_here;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < waves; ++w) t += wave_cnt[w];
    block_counts[blockIdx.x] = t;
  }
}

// The messages of a block's sent rows, moved from the row-indexed scratch to their places: row list, codes and
// meta of rank k go to entries k of the outputs. offsets[b] = sent rows before block b; without it (inputs of at most
// kCountedBlocks blocks) every block adds up the counts before its own - a few kilobytes from L2 in place of a launch
// and of one block's work on the whole list: 20 us for 55 978 rows. Rows are moved in 16-byte pieces from and to any
// alignment, the last piece of a row ending with it (a byte at a time before: 602-byte rows, 16 + 23 -> 13 us for both
// parts at 37 % sent; 4.98 M rows of 64 bytes, all sent, 346 + 22 -> 152 us).
constexpr int kCountedBlocks = 2048;

__global__ __launch_bounds__(256) void place_messages_kernel(const uint8_t* __restrict__ mask, int n_rows,
                                                             const int* __restrict__ counts,
                                                             const int* __restrict__ offsets,
                                                             const uint8_t* __restrict__ scratch,
                                                             const float* __restrict__ meta_scratch, int rb,
                                                             int* __restrict__ idx, int* __restrict__ n_sent,
                                                             uint8_t* __restrict__ codes, float* __restrict__ meta) {
  static_assert(kTestRows == 64, "one wavefront ranks a block's rows");
  __shared__ int rows[kTestRows];
  __shared__ int wave_sum[4];
  __shared__ int sent;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.x * kTestRows;
  if (wave == 0) {
    const bool on = row0 + lane < n_rows && mask[row0 + lane] != 0;
    const unsigned long long b = __ballot(on);
    if (on) rows[__popcll(b & ((1ull << lane) - 1ull))] = row0 + lane;
    if (lane == 0) sent = __popcll(b);
  }
  int before = 0;
  if (!offsets) {
    for (int i = tid; i < static_cast<int>(blockIdx.x); i += 256) before += counts[i];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) before += __shfl_xor(before, off, kWave);
    if (lane == 0) wave_sum[wave] = before;
  }
  __syncthreads();
  before = offsets ? offsets[blockIdx.x] : (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
  const int cnt = sent;
  if (tid == 0 && blockIdx.x == gridDim.x - 1) *n_sent = before + cnt;
  if (tid < cnt) idx[before + tid] = rows[tid];
  if (tid < 2 * cnt) meta[2 * static_cast<int64_t>(before) + tid] = meta_scratch[2 * static_cast<int64_t>(rows[tid >> 1]) + (tid & 1)];
  typedef uint32_t u4u __attribute__((ext_vector_type(4), aligned(1)));
  uint8_t* out = codes + static_cast<int64_t>(before) * rb;
  const int piece = rb >= 16 ? 16 : 1, pieces = rb >= 16 ? (rb + 15) / 16 : rb;
  int lpr = 1;                                   // lanes per row: a power of two
  while (lpr < pieces && lpr < 64) lpr <<= 1;
  const int l = tid & (lpr - 1);
  for (int k = tid / lpr; k < cnt; k += 256 / lpr) {
    const uint8_t* src = scratch + static_cast<int64_t>(rows[k]) * rb;
    uint8_t* dst = out + static_cast<int64_t>(k) * rb;
    for (int i = l; i < pieces; i += lpr) {
      if (piece == 16) {
        const int at = min(i * 16, rb - 16);
        *reinterpret_cast<u4u*>(dst + at) = *reinterpret_cast<const u4u*>(src + at);
      } else {
        dst[i] = src[i];
      }
    }
  }
}

template <typename T, int EPV, int NIT, int BITS, int QS>
__global__ __launch_bounds__(kQuantThreads) void dequantize_kernel(
    const uint8_t* __restrict__ codes, const float* __restrict__ meta, const int* __restrict__ idx,
    const int* __restrict__ n_sent_p, int max_sent, int dim, int glog, T* dst, int64_t ld, int accumulate) {
  const int n_sent = min(*n_sent_p, max_sent);
  const int lane = threadIdx.x & 63;
  const int G = 1 << glog;
  const int lg = lane & (G - 1);
  const int rows_per_wave = 64 >> glog;
  const int gwave = blockIdx.x * (kQuantThreads / 64) + (threadIdx.x >> 6);
  const int nvec = dim / EPV;
  const int64_t rb = QS == CDF_Q_NONE ? static_cast<int64_t>(dim) * 4 : (static_cast<int64_t>(dim) * BITS + 7) / 8;
  const int wave_stride = gridDim.x * (kQuantThreads / 64) * rows_per_wave;
  for (int kb = gwave * rows_per_wave; kb < n_sent; kb += wave_stride) {
  const int k = kb + (lane >> glog);
  if (k >= n_sent) continue;
  const int64_t r = idx[k];
  const uint8_t* in = codes + static_cast<int64_t>(k) * rb;
  T* pd = dst + r * ld;
  const float m0 = meta[2 * static_cast<int64_t>(k)], m1 = meta[2 * static_cast<int64_t>(k) + 1];
  float scale = 0.0f;
  if (QS == CDF_Q_MINMAX) scale = (m1 - m0) / static_cast<float>((1 << BITS) - 1);
  if (QS == CDF_Q_SYMMETRIC) scale = m0;
#pragma unroll
  for (int i = 0; i < NIT; ++i) {
    const int v = lg + i * G;
    if (v >= nvec) continue;
    float val[EPV];
    if (QS == CDF_Q_NONE) {
      VecIO<float, EPV>::load(reinterpret_cast<const float*>(in) + static_cast<int64_t>(v) * EPV, val);
    } else {
      unsigned word;
      constexpr unsigned CM = (1u << BITS) - 1u;
      if (EPV == 1 && BITS == 4) {
        word = (in[v >> 1] >> (4 * (v & 1))) & CM;
      } else {
        constexpr int NB = EPV * BITS / 8 > 0 ? EPV * BITS / 8 : 1;
        const uint8_t* sp = in + static_cast<int64_t>(v) * NB;
        if (NB == 4) word = *reinterpret_cast<const uint32_t*>(sp);
        else if (NB == 2) word = *reinterpret_cast<const uint16_t*>(sp);
        else word = *sp;
      }
#pragma unroll
      for (int c = 0; c < EPV; ++c) {
        int q = static_cast<int>((word >> (BITS * c)) & CM);
        if (QS == CDF_Q_MINMAX) {
          val[c] = __fmaf_rn(static_cast<float>(q), scale, m0);
        } else {
          constexpr int SGN = 1 << (BITS - 1);
          q = (q ^ SGN) - SGN;
          val[c] = static_cast<float>(q) * scale;
        }
      }
    }
    if (accumulate) {
      float old[EPV];
      VecIO<T, EPV>::load(pd + static_cast<int64_t>(v) * EPV, old);
#pragma unroll
      for (int c = 0; c < EPV; ++c) val[c] = old[c] + val[c];
    }
    VecIO<T, EPV>::store(pd + static_cast<int64_t>(v) * EPV, val);
  }
  }
}

struct RowShape {
  int epv, nit, glog;
};

// Lane-vector width, vectors per lane and lanes per row for rows of `dim` elements.
static bool row_shape(int32_t dim, int epv, RowShape* s) {
  const int nvec = dim / epv;
  int nit = 1;
  s->epv = epv;
  while (nit * 64 < nvec) nit <<= 1;
  if (nit > 8) return false;
  s->nit = nit;
  s->glog = nvec >= 64 ? 6 : log2_ceil(nvec);
  if (epv == 1 && s->glog == 0) s->glog = 1;  // nibble pairs need two lanes
  return true;
}

#define CDF_DISPATCH_NIT(K, T, E, B, Q, nit, ...)          \
  switch (nit) {                                            \
    case 1: K<T, E, 1, B, Q> __VA_ARGS__; break;            \
    case 2: K<T, E, 2, B, Q> __VA_ARGS__; break;            \
    case 4: K<T, E, 4, B, Q> __VA_ARGS__; break;            \
    default: K<T, E, 8, B, Q> __VA_ARGS__; break;           \
  }
#define CDF_DISPATCH_EPV(K, T, B, Q, epv, nit, ...)                            \
  switch (epv) {                                                                \
    case 4: CDF_DISPATCH_NIT(K, T, 4, B, Q, nit, __VA_ARGS__) break;            \
    case 2: CDF_DISPATCH_NIT(K, T, 2, B, Q, nit, __VA_ARGS__) break;            \
    default: CDF_DISPATCH_NIT(K, T, 1, B, Q, nit, __VA_ARGS__) break;           \
  }
#define CDF_DISPATCH_Q(K, T, bits, qs, epv, nit, ...)                                              \
  if (qs == CDF_Q_NONE) { CDF_DISPATCH_EPV(K, T, 8, CDF_Q_NONE, epv, nit, __VA_ARGS__) }           \
  else if (qs == CDF_Q_MINMAX && bits == 8) { CDF_DISPATCH_EPV(K, T, 8, CDF_Q_MINMAX, epv, nit, __VA_ARGS__) } \
  else if (qs == CDF_Q_MINMAX) { CDF_DISPATCH_EPV(K, T, 4, CDF_Q_MINMAX, epv, nit, __VA_ARGS__) }  \
  else if (bits == 8) { CDF_DISPATCH_EPV(K, T, 8, CDF_Q_SYMMETRIC, epv, nit, __VA_ARGS__) }        \
  else { CDF_DISPATCH_EPV(K, T, 4, CDF_Q_SYMMETRIC, epv, nit, __VA_ARGS__) }

size_t filter_workspace_bytes(int64_t n_rows);
int scan_counts(const int* counts, int nblocks, int* offsets, int32_t* n_sent, hipStream_t st);

// Workspace of the one-pass test + message build: block counts and offsets, then row-indexed codes
// and meta. Sized for 8-bit codes of `dim` elements (the largest quantised row).
size_t test_encode_workspace_bytes(int64_t n_rows, int32_t dim) {
  const size_t rows = static_cast<size_t>(n_rows > 0 ? n_rows : 0);
  return filter_workspace_bytes(n_rows) + align_up(rows * static_cast<size_t>(dim), 256) + align_up(rows * 8, 256);
}

}  // namespace cdf

using namespace cdf;

extern "C" size_t cdf_code_row_bytes(int32_t dim, int bits, cdf_qscheme qs) {
  if (dim <= 0) return 0;
  if (qs == CDF_Q_NONE) return static_cast<size_t>(dim) * 4;
  return (static_cast<size_t>(dim) * bits + 7) / 8;
}

// Widest row the message kernels take for this width / pitch / type, assuming 16-byte aligned base
// pointers: 512 lane-vectors of the widest vector both allow.
extern "C" int32_t cdf_max_message_dim(int32_t dim, int64_t ld, cdf_dtype dt) {
  if (dim <= 0 || ld < dim || (dt != CDF_F32 && dt != CDF_BF16)) return 0;
  return 512 * pick_epv(dim, ld, elem_bytes(dt), nullptr);
}

static int check_scheme(const char* fn, int bits, cdf_qscheme qs, cdf_dtype dt) {
  if (dt != CDF_F32 && dt != CDF_BF16) CDF_FAIL(CDF_ERR_UNSUPPORTED, "%s: dtype %d", fn, (int)dt);
  if (qs != CDF_Q_MINMAX && qs != CDF_Q_SYMMETRIC && qs != CDF_Q_NONE)
    CDF_FAIL(CDF_ERR_UNSUPPORTED, "%s: scheme %d", fn, (int)qs);
  if (qs != CDF_Q_NONE && bits != 8 && bits != 4) CDF_FAIL(CDF_ERR_UNSUPPORTED, "%s: bits %d", fn, bits);
  return CDF_OK;
}

extern "C" int cdf_quantize(const void* cur, void* cached, const int32_t* idx, const int32_t* n_sent,
                            int32_t max_sent, int32_t dim, int64_t ld, cdf_dtype dt, int bits, cdf_qscheme qs,
                            cdf_commit commit, int delta, uint8_t* codes, float* meta, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  CDF_REQUIRE(max_sent >= 0 && dim > 0 && ld >= dim, "cdf_quantize: bad shape max_sent=%d dim=%d ld=%lld",
              max_sent, dim, (long long)ld);
  int rc = check_scheme("cdf_quantize", bits, qs, dt);
  if (rc != CDF_OK) return rc;
  CDF_REQUIRE(commit == CDF_COMMIT_NONE || commit == CDF_COMMIT_CUR || commit == CDF_COMMIT_DEQ,
              "cdf_quantize: commit %d", (int)commit);
  if (max_sent == 0) return CDF_OK;
  CDF_REQUIRE(cur && idx && n_sent && codes && meta, "cdf_quantize: null pointer");
  CDF_REQUIRE(cached || (!delta && commit == CDF_COMMIT_NONE),
              "cdf_quantize: cached is null but delta/commit need it");
  const size_t esz = elem_bytes(dt);
  CDF_REQUIRE(aligned(cur, esz) && (!cached || aligned(cached, esz)) && aligned(idx, 4) && aligned(n_sent, 4) &&
                  aligned(meta, 8) && aligned(codes, 16),
              "cdf_quantize: misaligned pointer (codes needs 16 bytes, meta 8)");
  RowShape s;
  if (!row_shape(dim, pick_epv(dim, ld, esz, cur, cached), &s))
    CDF_FAIL(CDF_ERR_UNSUPPORTED, "cdf_quantize: dim %d too wide for its alignment (max %d)", dim, 512 * s.epv);
  const int rows_per_block = (kQuantThreads / 64) * (64 >> s.glog);
  const int nblocks = static_cast<int>(std::min<int64_t>(ceil_div(max_sent, rows_per_block), kMessageGridCap));
#define ARGS_F32 <<<nblocks, kQuantThreads, 0, st>>>(static_cast<const float*>(cur), static_cast<float*>(cached), \
                 idx, n_sent, max_sent, dim, ld, s.glog, (int)commit, delta ? 1 : 0, codes, meta)
#define ARGS_BF16 <<<nblocks, kQuantThreads, 0, st>>>(static_cast<const bf16_t*>(cur), static_cast<bf16_t*>(cached), \
                 idx, n_sent, max_sent, dim, ld, s.glog, (int)commit, delta ? 1 : 0, codes, meta)
  prof_begin(K_QUANTIZE, st);
  if (dt == CDF_F32) { CDF_DISPATCH_Q(quantize_kernel, float, bits, qs, s.epv, s.nit, ARGS_F32) }
  else { CDF_DISPATCH_Q(quantize_kernel, bf16_t, bits, qs, s.epv, s.nit, ARGS_BF16) }
  prof_end(K_QUANTIZE, st);
#undef ARGS_F32
#undef ARGS_BF16
  CDF_LAUNCH_CHECK("cdf_quantize");
  return CDF_OK;
}

extern "C" int cdf_dequantize(const uint8_t* codes, const float* meta, const int32_t* idx, const int32_t* n_sent,
                              int32_t max_sent, int32_t dim, int bits, cdf_qscheme qs, void* dst, int64_t ld,
                              cdf_dtype dt, int accumulate, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  CDF_REQUIRE(max_sent >= 0 && dim > 0 && ld >= dim, "cdf_dequantize: bad shape max_sent=%d dim=%d ld=%lld",
              max_sent, dim, (long long)ld);
  int rc = check_scheme("cdf_dequantize", bits, qs, dt);
  if (rc != CDF_OK) return rc;
  if (max_sent == 0) return CDF_OK;
  CDF_REQUIRE(codes && meta && idx && n_sent && dst, "cdf_dequantize: null pointer");
  const size_t esz = elem_bytes(dt);
  CDF_REQUIRE(aligned(dst, esz) && aligned(idx, 4) && aligned(n_sent, 4) && aligned(meta, 8) && aligned(codes, 16),
              "cdf_dequantize: misaligned pointer (codes needs 16 bytes, meta 8)");
  RowShape s;
  if (!row_shape(dim, pick_epv(dim, ld, esz, dst), &s))
    CDF_FAIL(CDF_ERR_UNSUPPORTED, "cdf_dequantize: dim %d too wide for its alignment (max %d)", dim, 512 * s.epv);
  const int rows_per_block = (kQuantThreads / 64) * (64 >> s.glog);
  const int nblocks = static_cast<int>(std::min<int64_t>(ceil_div(max_sent, rows_per_block), kMessageGridCap));
#define ARGS_F32 <<<nblocks, kQuantThreads, 0, st>>>(codes, meta, idx, n_sent, max_sent, dim, s.glog, static_cast<float*>(dst), \
                 ld, accumulate ? 1 : 0)
#define ARGS_BF16 <<<nblocks, kQuantThreads, 0, st>>>(codes, meta, idx, n_sent, max_sent, dim, s.glog, static_cast<bf16_t*>(dst), \
                 ld, accumulate ? 1 : 0)
  prof_begin(K_DEQUANTIZE, st);
  if (dt == CDF_F32) { CDF_DISPATCH_Q(dequantize_kernel, float, bits, qs, s.epv, s.nit, ARGS_F32) }
  else { CDF_DISPATCH_Q(dequantize_kernel, bf16_t, bits, qs, s.epv, s.nit, ARGS_BF16) }
  prof_end(K_DEQUANTIZE, st);
#undef ARGS_F32
#undef ARGS_BF16
  CDF_LAUNCH_CHECK("cdf_dequantize");
  return CDF_OK;
}

namespace cdf {

// Cache test followed by the message build, as the layer steps need them. One pass over the rows
// when the messages are quantised and the workspace is large
// enough (test_encode_workspace_bytes); otherwise cdf_cache_filter then cdf_quantize. Both routes
// compute every row with the same instruction sequence: mask, idx, codes, meta and the committed
// cache are bit-identical.
int test_and_encode(const void* cur, void* cached, int32_t n_rows, int32_t dim, int64_t ld, cdf_dtype dt, float eps,
                    cdf_norm norm, int bits, cdf_qscheme qs, cdf_commit commit, int delta, uint8_t* mask, int32_t* idx,
                    int32_t* n_sent, uint8_t* codes, float* meta, void* ws, size_t ws_bytes, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  RowShape s = {};
  const size_t esz = elem_bytes(dt);
  const bool types_ok = (dt == CDF_F32 || dt == CDF_BF16) && (qs == CDF_Q_MINMAX || qs == CDF_Q_SYMMETRIC) &&
                        (bits == 8 || bits == 4) && (norm == CDF_NORM_LINF || norm == CDF_NORM_L2) && n_rows > 0 && dim > 0 && ld >= dim &&
                        cur && cached && mask && idx && n_sent && codes && meta && eps >= 0.0f && eps <= 3.0e38f &&
                        (commit == CDF_COMMIT_NONE || commit == CDF_COMMIT_CUR || commit == CDF_COMMIT_DEQ);
  const bool one_pass = types_ok && ws && aligned(ws, 256) && ws_bytes >= test_encode_workspace_bytes(n_rows, dim) &&
                        aligned(cur, esz) && aligned(cached, esz) && aligned(meta, 8) && aligned(codes, 16) &&
                        aligned(idx, 4) && aligned(n_sent, 4) && row_shape(dim, pick_epv(dim, ld, esz, cur, cached), &s);
  if (!one_pass) {
    const int rc = cdf_cache_filter(cur, cached, n_rows, dim, ld, dt, eps, norm, mask, idx, n_sent, ws, ws_bytes, stream);
    if (rc != CDF_OK) return rc;
    return cdf_quantize(cur, cached, idx, n_sent, n_rows, dim, ld, dt, bits, qs, commit, delta, codes, meta, stream);
  }
  const int nblocks = static_cast<int>(ceil_div(n_rows, kTestRows));
  char* w = static_cast<char*>(ws);
  int* counts = reinterpret_cast<int*>(w);
  int* offsets = counts + scan_stride(nblocks);
  uint8_t* cs = reinterpret_cast<uint8_t*>(w + filter_workspace_bytes(n_rows));
  float* ms = reinterpret_cast<float*>(w + filter_workspace_bytes(n_rows) +
                                       align_up(static_cast<size_t>(n_rows) * static_cast<size_t>(dim), 256));
  const int64_t rb = (static_cast<int64_t>(dim) * bits + 7) / 8;
  const int threads = nblocks <= kTestWideBlocks ? test_threads(s.nit * s.epv) : kQuantThreads;
#define ARGS_F32 <<<nblocks, threads, 0, st>>>(static_cast<const float*>(cur), static_cast<float*>(cached), n_rows, \
                 dim, ld, eps, (int)norm, s.glog, (int)commit, delta ? 1 : 0, mask, counts, cs, ms)
#define ARGS_BF16 <<<nblocks, threads, 0, st>>>(static_cast<const bf16_t*>(cur), static_cast<bf16_t*>(cached), n_rows, \
                 dim, ld, eps, (int)norm, s.glog, (int)commit, delta ? 1 : 0, mask, counts, cs, ms)
#define CDF_DISPATCH_QQ(K, T, ...)                                                                         \
  if (qs == CDF_Q_MINMAX && bits == 8) { CDF_DISPATCH_EPV(K, T, 8, CDF_Q_MINMAX, s.epv, s.nit, __VA_ARGS__) } \
  else if (qs == CDF_Q_MINMAX) { CDF_DISPATCH_EPV(K, T, 4, CDF_Q_MINMAX, s.epv, s.nit, __VA_ARGS__) }      \
  else if (bits == 8) { CDF_DISPATCH_EPV(K, T, 8, CDF_Q_SYMMETRIC, s.epv, s.nit, __VA_ARGS__) }            \
  else { CDF_DISPATCH_EPV(K, T, 4, CDF_Q_SYMMETRIC, s.epv, s.nit, __VA_ARGS__) }
  prof_begin(K_TEST_ENCODE, st);
  if (dt == CDF_F32) { CDF_DISPATCH_QQ(test_encode_kernel, float, ARGS_F32) }
  else { CDF_DISPATCH_QQ(test_encode_kernel, bf16_t, ARGS_BF16) }
  prof_end(K_TEST_ENCODE, st);
#undef ARGS_F32
#undef ARGS_BF16
#undef CDF_DISPATCH_QQ
  CDF_LAUNCH_CHECK("test_and_encode/encode");
  const bool counted = nblocks <= kCountedBlocks;
  if (!counted) {
    const int rc = scan_counts(counts, nblocks, offsets, n_sent, st);
    if (rc != CDF_OK) return rc;
  }
  {
    ProfScope ps(K_PLACE, st);
    place_messages_kernel<<<nblocks, 256, 0, st>>>(mask, n_rows, counts, counted ? nullptr : offsets, cs, ms,
                                                   static_cast<int>(rb), idx, n_sent, codes, meta);
  }
  CDF_LAUNCH_CHECK("test_and_encode/place");
  return CDF_OK;
}

}  // namespace cdf

extern "C" int cdf_set_message_wait_limit(int polls) {
  (void)polls;   // no route waits for another workgroup any more
  return CDF_OK;
}

extern "C" int cdf_cache_filter_quantize(const void* cur, void* cached, int32_t n_rows, int32_t dim, int64_t ld,
                                         cdf_dtype dt, float eps, cdf_norm norm, int bits, cdf_qscheme qs,
                                         cdf_commit commit, int delta, uint8_t* mask, int32_t* idx, int32_t* n_sent,
                                         uint8_t* codes, float* meta, void* ws, size_t ws_bytes, void* stream) {
  return cdf::test_and_encode(cur, cached, n_rows, dim, ld, dt, eps, norm, bits, qs, commit, delta, mask, idx, n_sent,
                              codes, meta, ws, ws_bytes, stream);
}
