// CSR aggregation Y = A X over the normalised adjacency (Sec. 3.1) and its transposed
// counterpart for back-propagation (the same kernel on the CSR of A^T).
//
// Work split: the stored entries are cut into chunks of 64 to 1024 consecutive entries and
// each wavefront takes one chunk, whatever rows it covers - a power-law degree
// distribution (rows of 1 to several 10^5 entries) therefore loads every wavefront
// equally. Inside a chunk the wavefront's lane groups walk one run of consecutive entries each
// (spmm_walk_kernel); several gather instructions are in flight at a time and the sums are kept
// in fp32 registers.
//
// Rows that straddle chunk borders: the piece at the start of a chunk that continues an
// earlier row goes to phead[chunk], the piece at the end of a chunk that continues into
// the next goes to ptail[chunk] (both fp32); a second kernel adds a row's pieces in
// chunk order and writes the row once. No atomics on results: they are bit-reproducible.
//
// spmm_transform_kernel is the aggregation with the dense transform in its row epilogue: the
// whole wavefront takes one entry at a time (lane l reads elements [l*EPV, l*EPV+EPV) of each
// 64*EPV-wide pass; column ids and values reach all lanes through v_readlane), so that a finished
// row is whole in one wavefront.
#include <type_traits>

#include "cdf_common.h"

namespace cdf {

constexpr int kChunk = 256;        // stored entries per wavefront on matrices of 1 M entries or more (smallest there)
constexpr int kSpmmThreads = 256;  // 4 wavefronts per block
constexpr int kSpmmWaves = kSpmmThreads / 64;

// chunk_row[c] = row that holds stored entry c*chunk (c >= 1; entry 0 is handled as row 0).
__global__ void chunk_rows_kernel(const int64_t* __restrict__ rowptr, int n_rows, int* __restrict__ chunk_row,
                                  int kChunk) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rows) return;
  const int64_t a = rowptr[r], b = rowptr[r + 1];
  for (int64_t c = (a + kChunk - 1) / kChunk; c * kChunk < b; ++c) chunk_row[c] = r;
}

// The dense transform of the layer applied to every finished row (Sec. 3.1, first equation as one
// kernel): z = m W for the aggregated row m, W [dim x G] with G <= 64, kept in LDS.
struct XformArgs {
  const float* W;  // dim x G, row-major
  float* Z;        // nullable, rows x G
  float* H;        // nullable, rows x G: relu ? max(z, 0) : z
  int G;
  int relu;
};

// z[lane] = sum_f row[f] * W[f][lane] for lane < G, f ascending, one fused multiply-add each; `row` is
// in LDS (every lane reads the same address: a broadcast), W in LDS or global memory.
__device__ __forceinline__ void transform_row(const float* row, const float* W, int dim, const XformArgs& xf,
                                              int64_t out_row, int lane) {
  if (lane >= xf.G) return;
  float z = 0.0f;
  int f = 0;
  for (; f + 4 <= dim; f += 4) {
    const float4 m = *reinterpret_cast<const float4*>(row + f);
    z = __fmaf_rn(m.x, W[(f + 0) * xf.G + lane], z);
    z = __fmaf_rn(m.y, W[(f + 1) * xf.G + lane], z);
    z = __fmaf_rn(m.z, W[(f + 2) * xf.G + lane], z);
    z = __fmaf_rn(m.w, W[(f + 3) * xf.G + lane], z);
  }
  for (; f < dim; ++f) z = __fmaf_rn(row[f], W[f * xf.G + lane], z);
  const int64_t at = out_row * xf.G + lane;
  if (xf.Z) xf.Z[at] = z;
  if (xf.H) xf.H[at] = xf.relu ? (z > 0.0f ? z : 0.0f) : z;
}

// LDS of the transforming variants: W, then one row buffer per wavefront (rows padded to 4 floats)
__host__ __device__ inline int xf_row_floats(int dim) { return (dim + 3) / 4 * 4; }

template <typename T, int EPV, int NP>
__global__ __launch_bounds__(kSpmmThreads) void spmm_transform_kernel(
    const int64_t* __restrict__ rowptr, const int* __restrict__ colidx, const float* __restrict__ vals,
    int n_rows, int64_t nnz, const T* __restrict__ X, int64_t ldx, T* __restrict__ Y,
    int64_t ldy, int dim, const int* __restrict__ chunk_row, int64_t nchunks, float* __restrict__ phead, float* __restrict__ ptail,
    int* __restrict__ tail_row, int kChunk, XformArgs xf) {
  constexpr int U = (8 / NP) > 0 ? (8 / NP) : 1;  // feature rows in flight per wavefront
  extern __shared__ __align__(16) float xf_lds[];
  const int lane = threadIdx.x & 63;
  // the wavefront index is the same in all lanes: say so, and everything derived from it
  // (chunk bounds, row cursor, loop counters) lives in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < dim * xf.G; i += kSpmmThreads) xf_lds[i] = xf.W[i];
  __syncthreads();
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kSpmmWaves + wave;
  if (chunk >= nchunks) return;
  const int64_t s = chunk * kChunk;
  const int L = static_cast<int>(nnz - s < kChunk ? nnz - s : kChunk);
  int my_col = 0, krel = 0;
  float my_val = 0.0f;

  int r = chunk == 0 ? 0 : chunk_row[chunk];
  bool head = chunk > 0 && rowptr[r] < s;

  // window of 64 row ends, relative to s and clipped, one per lane
  auto load_rel = [&](int rbase) -> int {
    const int rr = rbase + lane;
    if (rr < n_rows) {
      const int64_t d = rowptr[rr + 1] - s;
      return d > kChunk ? kChunk + 1 : static_cast<int>(d);
    }
    return kChunk + 2;  // past the last row: matches nothing
  };
  int r_base = r;
  int rel = load_rel(r_base);
  int cur_end = __builtin_amdgcn_readlane(rel, 0);

  bool col_on[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) col_on[p] = (p * 64 + lane) * EPV < dim;

  float acc[NP][EPV];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int c = 0; c < EPV; ++c) acc[p][c] = 0.0f;

  auto next_row = [&]() {
    ++r;
    if (r - r_base == 64) {
      r_base = r;
      rel = load_rel(r_base);
    }
    cur_end = __builtin_amdgcn_readlane(rel, r - r_base);
  };
  // a finished row: stored, then transformed
  auto store_y = [&](int row) {
    T* py = Y + static_cast<int64_t>(row) * ldy;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (col_on[p]) VecIO<T, EPV>::store(py + (p * 64 + lane) * EPV, acc[p]);
    // the row goes to this wavefront's LDS buffer, then every lane < G forms one output
    float* rb = xf_lds + xf_row_floats(dim * xf.G) + wave * xf_row_floats(dim);
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (col_on[p]) {
#pragma unroll
        for (int c = 0; c < EPV; ++c) rb[(p * 64 + lane) * EPV + c] = acc[p][c];
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    transform_row(rb, xf_lds, dim, xf, row, lane);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the next row is written only after every lane has read this one
  };
  auto store_partial = [&](float* buf) {
    float* pp = buf + chunk * static_cast<int64_t>(dim);
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (col_on[p]) {
#pragma unroll
        for (int c = 0; c < EPV; ++c) pp[(p * 64 + lane) * EPV + c] = acc[p][c];
      }
  };
  auto clear_acc = [&]() {
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int c = 0; c < EPV; ++c) acc[p][c] = 0.0f;
  };
  // the row that just ended inside this chunk
  auto flush_row = [&]() {
    if (head) store_partial(phead);
    else store_y(r);
    head = false;
    clear_acc();
  };

  // one entry: gather is already in x, add it to the open row (closing rows that ended before it)
  auto consume = [&](const float (&xr)[NP][EPV], int j) {
    while (krel == cur_end) {
      flush_row();
      next_row();
    }
    const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_val), j));
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (col_on[p]) {
#pragma unroll
        for (int c = 0; c < EPV; ++c) acc[p][c] = __fmaf_rn(v, xr[p][c], acc[p][c]);
      }
    ++krel;
  };
  auto gather = [&](float (&xr)[NP][EPV], int j) {
    const int c = __builtin_amdgcn_readlane(my_col, j);
    const T* px = X + static_cast<int64_t>(c) * ldx;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (col_on[p]) VecIO<T, EPV>::load(px + (p * 64 + lane) * EPV, xr[p]);
  };

  for (int base = 0; base < L; base += 64) {
    const int cnt = L - base < 64 ? L - base : 64;
    my_col = 0;
    my_val = 0.0f;
    if (lane < cnt) {
      my_col = colidx[s + base + lane];
      my_val = vals[s + base + lane];
    }
    int j = 0;
    for (; j + U <= cnt; j += U) {  // U gathers in flight, no guards
      float x[U][NP][EPV];
#pragma unroll
      for (int u = 0; u < U; ++u) gather(x[u], j + u);
#pragma unroll
      for (int u = 0; u < U; ++u) consume(x[u], j + u);
    }
    for (; j < cnt; ++j) {
      float x[NP][EPV];
      gather(x, j);
      consume(x, j);
    }
  }

  // end of the chunk (krel == L): the open row either ends here or runs on
  int tr = -1;
  if (cur_end > L) {
    if (head) {
      store_partial(phead);  // the whole chunk lies inside one row
    } else {
      store_partial(ptail);
      tr = r;
    }
  } else {
    flush_row();
    next_row();
    // empty rows between this chunk's last entry and the next chunk's first
    while (r < n_rows && cur_end == L) {
      store_y(r);  // acc is zero
      next_row();
    }
  }
  if (lane == 0) tail_row[chunk] = tr;
}

// ---- the aggregation kernel ------------------------------------------------------------------------
// A lane group of LPR lanes walks its own run of consecutive stored entries: one gather instruction then
// serves 64 / LPR entries of 64 / LPR runs, each lane holding EPV columns of its run's open row. grid.y
// cuts the feature matrix into vertical slices of LPR * EPV columns.
//
// What bounds it: the gathered lines - the L2 <-> fabric interface where the table exceeds the caches, the
// instruction stream where it does not. A group owns its run, so an entry costs a gather, EPV multiply-adds
// and one test of a bit: no masks and no exchange between groups at a row end (a row that ends in the middle
// of a run is stored by its group alone; what crosses runs is combined once per chunk). With groups sharing a
// window of 64 entries and exchanging partial sums at every row end, the kernel before this one took 185 / 200
// us at 256 floats a row on 1.8 M entries (matrix / transpose), 539 / 353 us at 602, 74 / 76 us at 41, and 4.6 ms on
// 49 M entries that hit the caches; this one takes 100 / 89, 373 / 224, 33 / 31 us and 3.2 ms. On matrices far
// larger than the caches (144 M entries, 256 floats) both take 21 ms.
// A lane fetches four (column, value) pairs at a time, a group therefore whole lines of the CSR arrays: fetched
// eight entries at a time those lines were requested four times over (23.0 against 21.7 ms on that matrix).
// EPV elements of T from any element-aligned address (global memory takes 16-byte accesses there).
template <typename T, int EPV>
struct RawVec;
template <>
struct RawVec<float, 4> {
  typedef float v_t __attribute__((ext_vector_type(4), aligned(4)));
  v_t v;
  __device__ __forceinline__ void load(const float* p) { v = *reinterpret_cast<const v_t*>(p); }
  __device__ __forceinline__ void fma_into(float w, float (&acc)[4]) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = __fmaf_rn(w, v[c], acc[c]);
  }
  template <bool STREAM = false>
  static __device__ __forceinline__ void store(float* p, const float (&a)[4]) {
    const v_t t = {a[0], a[1], a[2], a[3]};
    if (STREAM) __builtin_nontemporal_store(t, reinterpret_cast<v_t*>(p));
    else *reinterpret_cast<v_t*>(p) = t;
  }
};
template <>
struct RawVec<bf16_t, 8> {
  typedef uint32_t v_t __attribute__((ext_vector_type(4), aligned(2)));
  v_t v;
  __device__ __forceinline__ void load(const bf16_t* p) { v = *reinterpret_cast<const v_t*>(p); }
  __device__ __forceinline__ void fma_into(float w, float (&acc)[8]) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      acc[2 * c] = __fmaf_rn(w, __uint_as_float(v[c] << 16), acc[2 * c]);
      acc[2 * c + 1] = __fmaf_rn(w, __uint_as_float(v[c] & 0xffff0000u), acc[2 * c + 1]);
    }
  }
  template <bool STREAM = false>
  static __device__ __forceinline__ void store(bf16_t* p, const float (&a)[8]) {
    v_t t;
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] = f2bf(a[2 * c]) | (static_cast<uint32_t>(f2bf(a[2 * c + 1])) << 16);
    if (STREAM) __builtin_nontemporal_store(t, reinterpret_cast<v_t*>(p));
    else *reinterpret_cast<v_t*>(p) = t;
  }
};
template <typename T>
struct RawVec<T, 1> {
  T v;
  __device__ __forceinline__ void load(const T* p) { v = *p; }
  __device__ __forceinline__ void fma_into(float w, float (&acc)[1]) const {
    float x[1];
    VecIO<T, 1>::load(&v, x);
    acc[0] = __fmaf_rn(w, x[0], acc[0]);
  }
  template <bool STREAM = false>
  static __device__ __forceinline__ void store(T* p, const float (&a)[1]) { VecIO<T, 1>::store(p, a); }
};

constexpr int kWalkBlock = 8;   // entries of a run fetched together (8 gathers in flight per lane)

// LDS ints per wavefront: a bit per entry of the chunk (last of its row), and that row's number
__host__ __device__ constexpr int walk_lds_ints(int chunk) { return chunk / 32 + chunk; }

template <typename T, int EPV, int LPR, bool QUAD>
__global__ __launch_bounds__(kSpmmThreads) void spmm_walk_kernel(
    const int64_t* __restrict__ rowptr, const int* __restrict__ colidx, const float* __restrict__ vals,
    int n_rows, int64_t nnz, const T* __restrict__ X, uint64_t ldx, T* __restrict__ Y, T* __restrict__ Y2,
    int64_t ldy, int dim, const int* __restrict__ chunk_row, int plan_step, int64_t nchunks, float* __restrict__ phead,
    float* __restrict__ ptail, int* __restrict__ tail_row, int kChunk, int stream_csr) {
  constexpr int NG = 64 / LPR;
  constexpr int KB = kWalkBlock;
  // (column, value) pairs a lane fetches at a time, and entries of its run that its group then holds
  constexpr int NLD = QUAD ? 4 : LPR >= KB ? 1 : KB / LPR;
  constexpr int HOLD = QUAD ? 4 * LPR : KB;
  constexpr bool kAnyPitch = EPV == 1;            // the other instances multiply 32-bit factors
  extern __shared__ int walk_lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kSpmmWaves + wave;
  if (chunk >= nchunks) return;
  const int g = lane / LPR, lg = lane % LPR;
  // this lane's columns; lanes past the row end take the row's last EPV columns once more (same sums, same stores)
  const int col0 = min(static_cast<int>(blockIdx.y) * (LPR * EPV) + lg * EPV, dim - EPV);
  const int64_t s = chunk * kChunk;
  const int L = static_cast<int>(nnz - s < kChunk ? nnz - s : kChunk);
  unsigned* ends = reinterpret_cast<unsigned*>(walk_lds + wave * walk_lds_ints(kChunk));
  int* row_of = reinterpret_cast<int*>(ends) + kChunk / 32;

  auto store_row = [&](int row, const float (&a)[EPV]) {
    const uint64_t at = (kAnyPitch ? static_cast<uint64_t>(row) * static_cast<uint64_t>(ldy)
                                   : static_cast<uint64_t>(static_cast<uint32_t>(row)) * static_cast<uint32_t>(ldy)) + col0;
    // finished rows are not read again here: streamed past the caches that hold the gathered rows
    if (Y) RawVec<T, EPV>::template store<true>(Y + at, a);
    if (Y2) {
      float pos[EPV];
#pragma unroll
      for (int c = 0; c < EPV; ++c) pos[c] = a[c] > 0.0f ? a[c] : 0.0f;
      RawVec<T, EPV>::template store<true>(Y2 + at, pos);
    }
  };
  auto store_piece = [&](float* buf, const float (&a)[EPV]) {
    float* p = buf + chunk * static_cast<int64_t>(dim) + col0;
    if constexpr (EPV == 1) {
      *p = a[0];
    } else {
#pragma unroll
      for (int h = 0; h < EPV; h += 4) {
        const float q[4] = {a[h], a[h + 1], a[h + 2], a[h + 3]};
        RawVec<float, 4>::store(p + h, q);
      }
    }
  };

  // ---- where rows end inside the chunk ----
  for (int w = lane; w < kChunk / 32; w += 64) ends[w] = 0u;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int r0 = chunk == 0 ? 0 : chunk_row[chunk * plan_step];
  bool head = false;   // the chunk's first row began in an earlier chunk
  int tr = -1;         // row that runs on past the chunk
  for (int base = r0;; base += 64) {
    const int rr = base + lane;
    const bool in = rr < n_rows;
    const int64_t d0 = in ? rowptr[rr] - s : kChunk + 1, d1 = in ? rowptr[rr + 1] - s : kChunk + 1;
    const int e0 = d0 < 0 ? -1 : d0 > kChunk ? kChunk + 1 : static_cast<int>(d0);
    const int e1 = d1 > kChunk ? kChunk + 1 : static_cast<int>(d1);
    if (base == r0) head = __builtin_amdgcn_readfirstlane(e0) < 0;
    if (in && e1 > e0 && e1 <= L) {
      atomicOr(&ends[(e1 - 1) >> 5], 1u << ((e1 - 1) & 31));
      row_of[e1 - 1] = rr;
    }
    const unsigned long long on = __ballot(in && e0 < L && e1 > L);
    if (on != 0ull) tr = base + __builtin_ctzll(on);
    // rows without entries: the chunk that holds the entry before them writes their zeros
    unsigned long long empty = __ballot(in && e0 == e1 && e0 <= L && (e0 > 0 || chunk == 0));
    while (empty != 0ull) {
      unsigned long long m = empty;   // group g takes the g-th of the next NG empty rows
      int mine = -1;
#pragma unroll 1
      for (int q = 0; q < NG && m != 0ull; ++q) {
        if (q == g) mine = base + __builtin_ctzll(m);
        m &= m - 1;
      }
      empty = m;
      float zero[EPV];
#pragma unroll
      for (int c = 0; c < EPV; ++c) zero[c] = 0.0f;
      if (mine >= 0) store_row(mine, zero);
    }
    if (__ballot(!in || e1 > L) != 0ull) break;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  // ---- every lane group walks its run of the chunk ----
  const int run = kChunk / NG;      // a multiple of KB
  const int beg = g * run;
  bool open = g == 0 ? head : ((ends[(beg - 1) >> 5] >> ((beg - 1) & 31)) & 1u) == 0u;   // run starts inside a row
  bool ended = false;               // a row ended inside this run
  int first_row = 0;                // the first one, if it began before the run: its part is kept aside
  float acc[EPV], first[EPV];
#pragma unroll
  for (int c = 0; c < EPV; ++c) acc[c] = first[c] = 0.0f;

  const T* xs = X + col0;
  const int* cp = colidx + s + beg;
  const float* vp = vals + s + beg;
  // entries k .. k + HOLD - 1 of the run: lane lg holds NLD consecutive ones (or, where a group is wider than a
  // block, lane lg % KB holds one)
  int col[NLD];
  float val[NLD];
  auto fetch = [&](int k0, auto full) {
    const int k = k0 + (NLD > 1 ? lg * NLD : lg % KB);
    if constexpr (decltype(full)::value && NLD == 4) {
      typedef int i4u __attribute__((ext_vector_type(4), aligned(4)));
      typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
      i4u c;
      f4u v;
      if (stream_csr) {
        c = __builtin_nontemporal_load(reinterpret_cast<const i4u*>(cp + k));
        v = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(vp + k));
      } else {
        c = *reinterpret_cast<const i4u*>(cp + k);
        v = *reinterpret_cast<const f4u*>(vp + k);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        col[q] = c[q];
        val[q] = v[q];
      }
    } else {
#pragma unroll
      for (int q = 0; q < NLD; ++q) {
        const bool ok = decltype(full)::value || beg + k + q < L;
        col[q] = ok ? cp[k + q] : 0;
        val[q] = ok ? vp[k + q] : 0.0f;
      }
    }
  };
  auto walk = [&](auto full) {
    constexpr bool FULL = decltype(full)::value;
    fetch(0, full);
    for (int kb = 0; kb < run; kb += KB) {
      if (!FULL && kb >= L) break;   // no group has entries left (uniform)
      const int e = beg + kb;
      const unsigned bits = (ends[e >> 5] >> (e & 31)) & ((1u << KB) - 1u);
      RawVec<T, EPV> x[KB];
      float v[KB];
      const int src0 = g * LPR + (kb % HOLD) / NLD;
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const unsigned c = static_cast<unsigned>(__shfl(col[u % NLD], src0 + u / NLD, kWave));
        v[u] = __shfl(val[u % NLD], src0 + u / NLD, kWave);
        if (FULL || e + u < L) {
          if (kAnyPitch) x[u].load(xs + c * ldx);
          else x[u].load(reinterpret_cast<const T*>(reinterpret_cast<const char*>(xs) +
                                                    static_cast<uint64_t>(c) * static_cast<uint32_t>(ldx * sizeof(T))));
        }
      }
      if ((kb + KB) % HOLD == 0 && kb + KB < run) fetch(kb + KB, full);
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        if (FULL || e + u < L) x[u].fma_into(v[u], acc);
        if (bits & (1u << u)) {
          const int row = row_of[e + u];
          if (open) {
            first_row = row;
#pragma unroll
            for (int c = 0; c < EPV; ++c) first[c] = acc[c];
          } else {
            store_row(row, acc);
          }
          open = false;   // every later row begins inside the run
          ended = true;
#pragma unroll
          for (int c = 0; c < EPV; ++c) acc[c] = 0.0f;
        }
      }
    }
  };
  const bool began_open = open;
  if (L == kChunk) walk(std::true_type{});
  else walk(std::false_type{});

  // ---- rows that cross runs: what is left open is carried over the groups, in group order ----
  bool any = ended;   // a row ended in this group or in the scanned ones before it
#pragma unroll
  for (int d = LPR; d < 64; d <<= 1) {
    float up[EPV];
#pragma unroll
    for (int c = 0; c < EPV; ++c) up[c] = __shfl_up(acc[c], d, kWave);
    const bool up_any = __shfl_up(any ? 1 : 0, d, kWave) != 0;
    if (lane >= d) {
      if (!any) {
#pragma unroll
        for (int c = 0; c < EPV; ++c) acc[c] = up[c] + acc[c];
      }
      any = any || up_any;
    }
  }
  // what the groups before this one left open
  float carry[EPV];
#pragma unroll
  for (int c = 0; c < EPV; ++c) {
    carry[c] = __shfl_up(acc[c], LPR % 64, kWave);
    if (g == 0 || LPR == 64) carry[c] = 0.0f;
  }
  const int up_any = __shfl_up(any ? 1 : 0, LPR % 64, kWave);
  const bool before = LPR < 64 && g > 0 && up_any != 0;
  if (ended && began_open) {
#pragma unroll
    for (int c = 0; c < EPV; ++c) first[c] = carry[c] + first[c];
    if (head && !before) store_piece(phead, first);
    else store_row(first_row, first);
  }
  if (g == NG - 1) {
    if (head && !any) store_piece(phead, acc);   // the whole chunk lies inside one row
    else if (tr >= 0) store_piece(ptail, acc);
  }
  const bool none = __shfl(any ? 1 : 0, 63, kWave) == 0;
  if (lane == 0 && blockIdx.y == 0) tail_row[chunk] = head && none ? -1 : tr;
}

// Adds the pieces of every row that straddles chunk borders, in chunk order. grid.y cuts the columns, so that
// the longest rows (hundreds of pieces, one after another) are summed by several wavefronts.
template <typename T, int EPV>
__global__ __launch_bounds__(kSpmmThreads) void spmm_fixup_kernel(
    const int64_t* __restrict__ rowptr, const int* __restrict__ tail_row, int64_t nchunks,
    const float* __restrict__ phead, const float* __restrict__ ptail, T* __restrict__ Y, T* __restrict__ Y2,
    int64_t ldy, int dim, int n_rows, int kChunk) {
  constexpr int NF = EPV == 1 ? 1 : 4;   // floats per piece vector
  constexpr int NV = EPV / NF;
  constexpr int U = 8 / NV;              // pieces in flight
  const int lane = threadIdx.x & 63;
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kSpmmWaves + (threadIdx.x >> 6);
  if (chunk >= nchunks) return;
  const int r = tail_row[chunk];
  if (r < 0 || r >= n_rows) return;
  if ((static_cast<int>(blockIdx.y) * 64 + lane) * EPV >= dim) return;
  const int col = min((static_cast<int>(blockIdx.y) * 64 + lane) * EPV, dim - EPV);
  // last chunk that starts inside row r: the one that holds the row's last entry (the row runs past
  // this chunk, so it has one). Computed, not walked: the longest rows span hundreds of chunks.
  const int64_t last = (rowptr[r + 1] - 1) / kChunk;
  float acc[EPV];
  RawVec<float, NF> t[U][NV];
  auto load = [&](const float* buf, int64_t c, RawVec<float, NF> (&v)[NV]) {
#pragma unroll
    for (int h = 0; h < NV; ++h) v[h].load(buf + c * static_cast<int64_t>(dim) + col + h * NF);
  };
  auto add = [&](const RawVec<float, NF> (&v)[NV]) {
#pragma unroll
    for (int h = 0; h < NV; ++h) {
      float a[NF];
#pragma unroll
      for (int c = 0; c < NF; ++c) a[c] = acc[h * NF + c];
      v[h].fma_into(1.0f, a);
#pragma unroll
      for (int c = 0; c < NF; ++c) acc[h * NF + c] = a[c];
    }
  };
#pragma unroll
  for (int c = 0; c < EPV; ++c) acc[c] = 0.0f;
  load(ptail, chunk, t[0]);
  add(t[0]);
  int64_t c2 = chunk + 1;
  for (; c2 + U - 1 <= last; c2 += U) {
#pragma unroll
    for (int q = 0; q < U; ++q) load(phead, c2 + q, t[q]);
#pragma unroll
    for (int q = 0; q < U; ++q) add(t[q]);
  }
  for (; c2 <= last; ++c2) {
    load(phead, c2, t[0]);
    add(t[0]);
  }
  if (Y) RawVec<T, EPV>::store(Y + static_cast<int64_t>(r) * ldy + col, acc);
  if (Y2) {
#pragma unroll
    for (int c = 0; c < EPV; ++c) acc[c] = acc[c] > 0.0f ? acc[c] : 0.0f;
    RawVec<T, EPV>::store(Y2 + static_cast<int64_t>(r) * ldy + col, acc);
  }
}

// Entries per wavefront: 64 or 128 on small matrices (so that even a few thousand entries spread over
// all compute units and a wavefront's serial walk stays short), 256 from 1 M entries, up to 1024 for
// large ones (fewer straddling-row pieces). Always a multiple of 64; a function of nnz alone.
int spmm_chunk(int64_t nnz) {
  int c = 64;
  while (c < kChunk && nnz / (2 * c) >= 4096) c *= 2;
  while (c >= kChunk && c < 1024 && nnz / (2 * c) >= 65536) c *= 2;
  return c;
}

// The same for the transforming variant (fp32): the summed row is stored and then transformed (W from
// global memory: only rows that straddle chunk borders come here).
template <int EPV>
__global__ __launch_bounds__(kSpmmThreads) void spmm_fixup_transform_kernel(
    const int64_t* __restrict__ rowptr, const int* __restrict__ tail_row, int64_t nchunks,
    const float* __restrict__ phead, const float* __restrict__ ptail, float* __restrict__ Y, int64_t ldy, int dim,
    int n_rows, int kChunk, XformArgs xf) {
  extern __shared__ __align__(16) float xf_lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kSpmmWaves + wave;
  if (chunk >= nchunks) return;
  const int r = tail_row[chunk];
  if (r < 0 || r >= n_rows) return;
  const int64_t last = (rowptr[r + 1] - 1) / kChunk;
  float* rb = xf_lds + wave * xf_row_floats(dim);
  for (int col = lane * EPV; col < dim; col += 64 * EPV) {
    float acc[EPV];
#pragma unroll
    for (int c = 0; c < EPV; ++c) acc[c] = ptail[chunk * static_cast<int64_t>(dim) + col + c];
    for (int64_t c2 = chunk + 1; c2 <= last; ++c2)
#pragma unroll
      for (int c = 0; c < EPV; ++c) acc[c] = acc[c] + phead[c2 * static_cast<int64_t>(dim) + col + c];
    if (Y) VecIO<float, EPV>::store(Y + static_cast<int64_t>(r) * ldy + col, acc);
#pragma unroll
    for (int c = 0; c < EPV; ++c) rb[col + c] = acc[c];
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  transform_row(rb, xf.W, dim, xf, r, lane);
}

int64_t spmm_chunks(int64_t nnz) { return nnz <= 0 ? 1 : ceil_div(nnz, spmm_chunk(nnz)); }

// Upper bound of spmm_chunks over every matrix of at most nnz entries (the chunk size steps up with nnz,
// so the count itself is not monotone).
static int64_t spmm_chunks_bound(int64_t nnz) {
  if (nnz <= 0) return 1;
  const int64_t small = ceil_div(nnz, 64) < 8192 ? ceil_div(nnz, 64) : 8192;
  const int64_t large = ceil_div(nnz, kChunk);
  return small > large ? small : large;
}

size_t spmm_workspace_bytes(int64_t nnz, int32_t dim) {
  const int64_t nc = spmm_chunks_bound(nnz);
  return align_up(static_cast<size_t>(nc) * 2 * sizeof(int), 256) +
         2 * align_up(static_cast<size_t>(nc) * dim * sizeof(float), 256);
}

// Lanes per entry: a slice of the feature matrix is lpr lane-vectors (16 bytes each) wide.
//  - Rows of whole 128-byte lines: slices of one line (8 lanes) keep the gathered table small, slices of two
//    lines (16) halve what is spent per entry and slice. Two lines as long as such a slice of the matrix fits
//    the 256 MB memory-side cache. Measured, 8 / 16 lanes at 256 floats a row: 68 k gathered rows (18 MB a
//    slice) 97 / 89 us, 300 k (77 MB) 3.39 / 3.16 ms; 2.1 M (537 MB) 20.5 / 23.9 ms, 7.1 M (1.8 GB) 21.7 /
//    23.0 ms; 476 k rows of 1024 bf16 (122 MB) 647 / 601 us.
//  - Other rows of at most 32 vectors: one slice, the group just wide enough (rows start anywhere in a line,
//    so every extra slice fetches a line twice: 100 floats, 32 / 16 / 8 lanes 2.97 / 3.54 / 4.66 ms).
//  - Longer ones: 16 (602 floats, 8 / 16 / 32 lanes: 399 / 373 / 400 us).
static int pick_lanes(int dim, int epv, int64_t n_cols) {
  const int nvec = static_cast<int>(ceil_div(dim, epv));
  int lpr = 2;
  if (nvec > 8 && dim % (8 * epv) == 0) return nvec % 16 == 0 && n_cols * 256 <= (int64_t(256) << 20) ? 16 : 8;
  if (nvec > 32) return 16;
  while (lpr < nvec) lpr <<= 1;
  return lpr;
}

template <typename T, int EPV>
static int launch_spmm(const cdf_csr* A, const T* X, int64_t ldx, T* Y, T* Y2, int64_t ldy, int dim, void* ws,
                       hipStream_t st) {
  const int plan_chunk = spmm_chunk(A->nnz);
  const int64_t plan_chunks = spmm_chunks(A->nnz);
  const int nvec = static_cast<int>(ceil_div(dim, EPV));
  const int lpr = EPV == 1 ? 8 : pick_lanes(dim, EPV, A->n_cols);
  const int slices = static_cast<int>(ceil_div(nvec, lpr));
  // the plan's chunks, several at a time where the lane groups are many: a run has at least one block of entries
  int chunk = plan_chunk, step = 1;
  while (chunk < kWalkBlock * (64 / lpr)) {
    chunk *= 2;
    step *= 2;
  }
  const int64_t nc = A->nnz <= 0 ? 1 : ceil_div(A->nnz, chunk);
  char* w = static_cast<char*>(ws);
  int* own_chunk_row = reinterpret_cast<int*>(w);
  int* tail_row = own_chunk_row + plan_chunks;
  w += align_up(static_cast<size_t>(plan_chunks) * 2 * sizeof(int), 256);
  float* phead = reinterpret_cast<float*>(w);
  w += align_up(static_cast<size_t>(nc) * dim * sizeof(float), 256);
  float* ptail = reinterpret_cast<float*>(w);

  // chunk -> row table: the caller's plan (built once per matrix by cdf_spmm_plan), else rebuilt here
  const int* chunk_row = A->plan;
  if (!chunk_row) {
    {
      ProfScope ps(K_SPMM_PLAN, st);
      chunk_rows_kernel<<<static_cast<unsigned>(ceil_div(A->n_rows, 256)), 256, 0, st>>>(A->rowptr, A->n_rows,
                                                                                         own_chunk_row, plan_chunk);
    }
    CDF_LAUNCH_CHECK("cdf_spmm/chunk_rows");
    chunk_row = own_chunk_row;
  }
  const unsigned nblocks = static_cast<unsigned>(ceil_div(nc, kSpmmWaves));
  const dim3 grid(nblocks, static_cast<unsigned>(slices));
  // the CSR arrays are streamed past the caches where they exceed the memory-side cache and cannot be found
  // there by the next slice (144 M entries: 21.6 -> 21.3 ms; 1.8 M entries: 90 -> 99 us, hence the line)
  const int stream_csr = A->nnz * 8 > (int64_t(256) << 20) ? 1 : 0;
  const size_t lds = static_cast<size_t>(kSpmmWaves) * walk_lds_ints(chunk) * sizeof(int);
#define CDF_SPMM_ARGS                                                                                            \
  (A->rowptr, A->colidx, A->vals, A->n_rows, A->nnz, X, static_cast<uint64_t>(ldx), Y, Y2, ldy, dim, chunk_row, step, \
   nc, phead, ptail, tail_row, chunk, stream_csr)
  prof_begin(K_SPMM_WALK, st);
#define CDF_WALK(LPRV)                                                                             \
  if (chunk >= 256) spmm_walk_kernel<T, EPV, LPRV, true><<<grid, kSpmmThreads, lds, st>>> CDF_SPMM_ARGS; \
  else spmm_walk_kernel<T, EPV, LPRV, false><<<grid, kSpmmThreads, lds, st>>> CDF_SPMM_ARGS
  if constexpr (EPV == 1) {
    CDF_WALK(8);
  } else {
    switch (lpr) {
      case 2: CDF_WALK(2); break;
      case 4: CDF_WALK(4); break;
      case 8: CDF_WALK(8); break;
      case 16: CDF_WALK(16); break;
      default: CDF_WALK(32); break;
    }
  }
#undef CDF_WALK
  prof_end(K_SPMM_WALK, st);
#undef CDF_SPMM_ARGS
  CDF_LAUNCH_CHECK("cdf_spmm/walk");
  {
    ProfScope ps(K_SPMM_FIXUP, st);
    const dim3 fgrid(nblocks, static_cast<unsigned>(ceil_div(nvec, 64)));
    spmm_fixup_kernel<T, EPV><<<fgrid, kSpmmThreads, 0, st>>>(A->rowptr, tail_row, nc, phead, ptail, Y, Y2, ldy, dim,
                                                              A->n_rows, chunk);
  }
  CDF_LAUNCH_CHECK("cdf_spmm/fixup");
  return CDF_OK;
}

// Y = A X and/or Y2 = max(A X, 0); either output may be null, both share ldy.
int spmm_run(const char* fn, const cdf_csr* A, const void* X, int64_t ldx, void* Y, void* Y2, int64_t ldy,
             int32_t dim, cdf_dtype dt, void* ws, size_t ws_bytes, hipStream_t st) {
  CDF_REQUIRE(A != nullptr, "%s: matrix is null", fn);
  CDF_REQUIRE(A->n_rows >= 0 && A->n_cols >= 0 && A->nnz >= 0 && dim > 0 && ldx >= dim && ldy >= dim,
              "%s: bad shape rows=%d cols=%d nnz=%lld dim=%d ldx=%lld ldy=%lld", fn, A->n_rows, A->n_cols,
              (long long)A->nnz, dim, (long long)ldx, (long long)ldy);
  if (dt != CDF_F32 && dt != CDF_BF16) CDF_FAIL(CDF_ERR_UNSUPPORTED, "%s: dtype %d", fn, (int)dt);
  if (A->n_rows == 0) return CDF_OK;
  CDF_REQUIRE(A->rowptr && (Y || Y2) && (A->nnz == 0 || (A->colidx && A->vals && X)), "%s: null pointer", fn);
  const size_t esz = elem_bytes(dt);
  CDF_REQUIRE(aligned(A->rowptr, 8) && aligned(A->colidx, 4) && aligned(A->vals, 4) && aligned(X, esz) &&
                  aligned(Y, esz) && aligned(Y2, esz),
              "%s: misaligned pointer", fn);
  if (!ws || !aligned(ws, 256) || ws_bytes < spmm_workspace_bytes(A->nnz, dim))
    CDF_FAIL(CDF_ERR_WORKSPACE, "%s: workspace too small or unaligned (%zu < %zu)", fn, ws_bytes,
             spmm_workspace_bytes(A->nnz, dim));
  // 16-byte lane vectors at any alignment; rows narrower than one (and pitches of 4 GiB and more) go element-wise
  const int full = dt == CDF_BF16 ? 8 : 4;
  const bool vec = dim >= full && static_cast<uint64_t>(ldx) * esz <= 0xffffffffu && static_cast<uint64_t>(ldy) * esz <= 0xffffffffu;
  constexpr int kMaxCols = 1 << 18;   // per launch (grid.y)
  for (int col0 = 0; col0 < dim; col0 += kMaxCols) {
    const int d = dim - col0 < kMaxCols ? dim - col0 : kMaxCols;
    const bool v = vec && d >= full;
    int rc;
    if (dt == CDF_F32) {
      const float* x = static_cast<const float*>(X) + col0;
      float* y = Y ? static_cast<float*>(Y) + col0 : nullptr;
      float* y2 = Y2 ? static_cast<float*>(Y2) + col0 : nullptr;
      rc = v ? launch_spmm<float, 4>(A, x, ldx, y, y2, ldy, d, ws, st) : launch_spmm<float, 1>(A, x, ldx, y, y2, ldy, d, ws, st);
    } else {
      const bf16_t* x = static_cast<const bf16_t*>(X) + col0;
      bf16_t* y = Y ? static_cast<bf16_t*>(Y) + col0 : nullptr;
      bf16_t* y2 = Y2 ? static_cast<bf16_t*>(Y2) + col0 : nullptr;
      rc = v ? launch_spmm<bf16_t, 8>(A, x, ldx, y, y2, ldy, d, ws, st) : launch_spmm<bf16_t, 1>(A, x, ldx, y, y2, ldy, d, ws, st);
    }
    if (rc != CDF_OK) return rc;
  }
  return CDF_OK;
}

int dense_fwd_ws(const void* M, int64_t ldm, cdf_dtype dt, const float* W, int32_t n, int32_t f_in, int32_t f_out,
                 int relu, float* Z, float* H, void* ws, size_t ws_bytes, void* stream);

// Can the aggregation carry the dense transform in its row epilogue? fp32 rows read as 16-byte lane
// vectors, at most 64 output columns, W and four row buffers within 64 KB of LDS.
bool spmm_transform_ok(const void* X, int64_t ldx, const void* M, int64_t ldm, int32_t dim, int32_t g, cdf_dtype dt) {
  if (dt != CDF_F32 || dim % 4 != 0 || ldx % 4 != 0 || ldm % 4 != 0 || !aligned(X, 16) || !aligned(M, 16)) return false;
  if (g < 1 || g > 64 || dim > 1024) return false;
  const size_t lds = (static_cast<size_t>(xf_row_floats(dim * g)) + kSpmmWaves * xf_row_floats(dim)) * sizeof(float);
  return lds <= 65536;
}

// M = A X, Z = M W, H = sigma(Z) in one pass over the matrix (plus the fix-up of straddling rows).
int spmm_transform_run(const char* fn, const cdf_csr* A, const float* X, int64_t ldx, const float* W, int32_t dim,
                       int32_t g, int relu, float* M, int64_t ldm, float* Z, float* H, void* ws, size_t ws_bytes,
                       hipStream_t st) {
  CDF_REQUIRE(A != nullptr && A->n_rows >= 0 && A->nnz >= 0, "%s: bad matrix", fn);
  if (A->n_rows == 0) return CDF_OK;
  CDF_REQUIRE(A->rowptr && M && W && (Z || H) && (A->nnz == 0 || (A->colidx && A->vals && X)), "%s: null pointer", fn);
  CDF_REQUIRE(aligned(A->rowptr, 8) && aligned(W, 4) && aligned(Z, 4) && aligned(H, 4), "%s: misaligned pointer", fn);
  if (!ws || !aligned(ws, 256) || ws_bytes < spmm_workspace_bytes(A->nnz, dim))
    CDF_FAIL(CDF_ERR_WORKSPACE, "%s: workspace too small or unaligned (%zu < %zu)", fn, ws_bytes,
             spmm_workspace_bytes(A->nnz, dim));
  const int chunk = spmm_chunk(A->nnz);
  const int64_t nc = spmm_chunks(A->nnz);
  char* w = static_cast<char*>(ws);
  int* own_chunk_row = reinterpret_cast<int*>(w);
  int* tail_row = own_chunk_row + nc;
  w += align_up(static_cast<size_t>(nc) * 2 * sizeof(int), 256);
  float* phead = reinterpret_cast<float*>(w);
  w += align_up(static_cast<size_t>(nc) * dim * sizeof(float), 256);
  float* ptail = reinterpret_cast<float*>(w);
  const int* chunk_row = A->plan;
  if (!chunk_row) {
    {
      ProfScope ps(K_SPMM_PLAN, st);
      chunk_rows_kernel<<<static_cast<unsigned>(ceil_div(A->n_rows, 256)), 256, 0, st>>>(A->rowptr, A->n_rows,
                                                                                         own_chunk_row, chunk);
    }
    CDF_LAUNCH_CHECK("spmm + transform/chunk_rows");
    chunk_row = own_chunk_row;
  }
  const unsigned nblocks = static_cast<unsigned>(ceil_div(nc, kSpmmWaves));
  const XformArgs xf = {W, Z, H, g, relu ? 1 : 0};
  const size_t lds_main = (static_cast<size_t>(xf_row_floats(dim * g)) + kSpmmWaves * xf_row_floats(dim)) * sizeof(float);
  const size_t lds_fix = static_cast<size_t>(kSpmmWaves) * xf_row_floats(dim) * sizeof(float);
  const int np = static_cast<int>(ceil_div(dim, 256));
#define CDF_XF_ARGS                                                                                              \
  (A->rowptr, A->colidx, A->vals, A->n_rows, A->nnz, X, ldx, M, ldm, dim, chunk_row, nc, phead, ptail, tail_row, \
   chunk, xf)
  prof_begin(K_SPMM_XFORM, st);
  if (np <= 1) spmm_transform_kernel<float, 4, 1><<<nblocks, kSpmmThreads, lds_main, st>>> CDF_XF_ARGS;
  else if (np <= 2) spmm_transform_kernel<float, 4, 2><<<nblocks, kSpmmThreads, lds_main, st>>> CDF_XF_ARGS;
  else spmm_transform_kernel<float, 4, 4><<<nblocks, kSpmmThreads, lds_main, st>>> CDF_XF_ARGS;
  prof_end(K_SPMM_XFORM, st);
#undef CDF_XF_ARGS
  CDF_LAUNCH_CHECK("spmm + transform/main");
  {
    ProfScope ps(K_SPMM_FIXUP, st);
    spmm_fixup_transform_kernel<4><<<nblocks, kSpmmThreads, lds_fix, st>>>(A->rowptr, tail_row, nc, phead, ptail, M, ldm,
                                                                           dim, A->n_rows, chunk, xf);
  }
  CDF_LAUNCH_CHECK("spmm + transform/fixup");
  return CDF_OK;
}

}  // namespace cdf

using namespace cdf;

extern "C" int cdf_spmm_dense_fwd(const cdf_csr* A, const void* X, int64_t ldx, cdf_dtype dt, const float* W,
                                  int32_t f_in, int32_t f_out, int relu, void* M, int64_t ldm, float* Z, float* H,
                                  void* ws, size_t ws_bytes, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  CDF_REQUIRE(A != nullptr && f_in > 0 && f_out > 0 && ldx >= f_in && ldm >= f_in,
              "cdf_spmm_dense_fwd: bad shape f_in=%d f_out=%d ldx=%lld ldm=%lld", f_in, f_out, (long long)ldx,
              (long long)ldm);
  if (spmm_transform_ok(X, ldx, M, ldm, f_in, f_out, dt))
    return spmm_transform_run("cdf_spmm_dense_fwd", A, static_cast<const float*>(X), ldx, W, f_in, f_out, relu,
                              static_cast<float*>(M), ldm, Z, H, ws, ws_bytes, st);
  const int rc = spmm_run("cdf_spmm_dense_fwd", A, X, ldx, M, nullptr, ldm, f_in, dt, ws, ws_bytes, st);
  if (rc != CDF_OK) return rc;
  return dense_fwd_ws(M, ldm, dt, W, A->n_rows, f_in, f_out, relu, Z, H, ws, ws_bytes, stream);
}

extern "C" int cdf_spmm_fwd(const cdf_csr* A, const void* X, int64_t ldx, void* Y, int64_t ldy, int32_t dim,
                            cdf_dtype dt, void* ws, size_t ws_bytes, void* stream) {
  return spmm_run("cdf_spmm_fwd", A, X, ldx, Y, nullptr, ldy, dim, dt, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

extern "C" int cdf_spmm_bwd(const cdf_csr* At, const void* dY, int64_t ldy, void* dX, int64_t ldx, int32_t dim,
                            cdf_dtype dt, void* ws, size_t ws_bytes, void* stream) {
  return spmm_run("cdf_spmm_bwd", At, dY, ldy, dX, nullptr, ldx, dim, dt, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

extern "C" size_t cdf_spmm_plan_bytes(int64_t nnz) {
  return nnz < 0 ? 0 : align_up(static_cast<size_t>(spmm_chunks(nnz)) * sizeof(int), 256);
}

extern "C" int cdf_spmm_plan(const cdf_csr* A, int32_t* plan, size_t plan_bytes, void* stream) {
  CDF_REQUIRE(A != nullptr, "cdf_spmm_plan: matrix is null");
  CDF_REQUIRE(A->n_rows >= 0 && A->nnz >= 0, "cdf_spmm_plan: bad shape rows=%d nnz=%lld", A->n_rows, (long long)A->nnz);
  if (!plan || !aligned(plan, 4) || plan_bytes < cdf_spmm_plan_bytes(A->nnz))
    CDF_FAIL(CDF_ERR_WORKSPACE, "cdf_spmm_plan: plan buffer too small (%zu < %zu)", plan_bytes,
             cdf_spmm_plan_bytes(A->nnz));
  if (A->n_rows == 0) return CDF_OK;
  CDF_REQUIRE(A->rowptr && aligned(A->rowptr, 8), "cdf_spmm_plan: row pointers null or misaligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  {
    ProfScope ps(K_SPMM_PLAN, st);
    chunk_rows_kernel<<<static_cast<unsigned>(ceil_div(A->n_rows, 256)), 256, 0, st>>>(A->rowptr, A->n_rows, plan,
                                                                                       spmm_chunk(A->nnz));
  }
  CDF_LAUNCH_CHECK("cdf_spmm_plan");
  return CDF_OK;
}
