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

// A matrix as the walk reads it. chunk_row: the row in which every plan_step-th chunk of the table's size starts.
struct WalkMatrix {
  const int64_t* rowptr;
  const int* colidx;
  const float* vals;
  const int* chunk_row;
  int n_rows;
  int64_t nnz;
  const int* row_map;   // row of the result for every row of the matrix; null: the same
};
// The same, as far as only the device knows it (the parts of a split matrix, see below).
struct WalkDims {
  int n_rows;
  int whole;        // the matrix was not split: read it instead of this part
  int64_t nnz;
  int64_t first;    // where the part's entries begin in colidx / vals
};
__device__ __forceinline__ void apply_dims(WalkMatrix& m, const WalkMatrix& whole, const WalkDims* dims) {
  if (!dims) return;
  if (dims->whole) {
    m = whole;
    return;
  }
  m.n_rows = dims->n_rows;
  m.nnz = dims->nnz;
  m.colidx += dims->first;
  m.vals += dims->first;
}
__host__ __device__ inline int64_t walk_chunks(int64_t nnz, int chunk) { return nnz <= 0 ? 1 : (nnz + chunk - 1) / chunk; }

// XCD_RANGES: contiguous eighths of the chunks on one XCD each (workgroup b runs on XCD b mod 8)
template <typename T, int EPV, int LPR, bool QUAD, bool XCD_RANGES = false>
__global__ __launch_bounds__(kSpmmThreads) void spmm_walk_kernel(
    WalkMatrix m, WalkMatrix whole, const WalkDims* __restrict__ dims, const T* __restrict__ X, uint64_t ldx,
    T* __restrict__ Y, T* __restrict__ Y2, int64_t ldy, int dim, int plan_step, float* __restrict__ phead,
    float* __restrict__ ptail, int* __restrict__ tail_row, int kChunk, int stream_csr) {
  apply_dims(m, whole, dims);
  if (m.n_rows == 0) return;
  const int64_t* __restrict__ rowptr = m.rowptr;
  const int* __restrict__ colidx = m.colidx;
  const float* __restrict__ vals = m.vals;
  const int n_rows = m.n_rows;
  const int64_t nnz = m.nnz, nchunks = walk_chunks(nnz, kChunk);
  constexpr int NG = 64 / LPR;
  constexpr int KB = kWalkBlock;
  // (column, value) pairs a lane fetches at a time, and entries of its run that its group then holds
  constexpr int NLD = QUAD ? 4 : LPR >= KB ? 1 : KB / LPR;
  constexpr int HOLD = QUAD ? 4 * LPR : KB;
  constexpr bool kAnyPitch = EPV == 1;            // the other instances multiply 32-bit factors
  extern __shared__ int walk_lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t block = blockIdx.x;
  if (XCD_RANGES) {
    const int64_t per = (nchunks + 8 * kSpmmWaves - 1) / (8 * kSpmmWaves);
    if (block >> 3 >= per) return;
    block = (block & 7) * per + (block >> 3);
  }
  const int64_t chunk = block * kSpmmWaves + wave;
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
  const int r0 = chunk == 0 ? 0 : m.chunk_row[chunk * plan_step];
  bool head = false;   // the chunk's first row began in an earlier chunk
  int tr = -1;         // row that runs on past the chunk
  for (int base = r0;; base += 64) {
    const int rr = base + lane;
    const bool in = rr < n_rows;
    const int64_t d0 = in ? rowptr[rr] - s : kChunk + 1, d1 = in ? rowptr[rr + 1] - s : kChunk + 1;
    const int e0 = d0 < 0 ? -1 : d0 > kChunk ? kChunk + 1 : static_cast<int>(d0);
    const int e1 = d1 > kChunk ? kChunk + 1 : static_cast<int>(d1);
    if (base == r0) head = __builtin_amdgcn_readfirstlane(e0) < 0;
    const int out = in ? (m.row_map ? m.row_map[rr] : rr) : 0;
    if (in && e1 > e0 && e1 <= L) {
      atomicOr(&ends[(e1 - 1) >> 5], 1u << ((e1 - 1) & 31));
      row_of[e1 - 1] = out;
    }
    const unsigned long long on = __ballot(in && e0 < L && e1 > L);
    if (on != 0ull) tr = base + __builtin_ctzll(on);
    // rows without entries: the chunk that holds the entry before them writes their zeros
    unsigned long long empty = __ballot(in && e0 == e1 && e0 <= L && (e0 > 0 || chunk == 0));
    while (empty != 0ull) {
      int mine = -1;   // group g takes the g-th of the next NG empty rows
#pragma unroll 1
      for (int q = 0; q < NG && empty != 0ull; ++q) {
        if (q == g) mine = __builtin_ctzll(empty);
        empty &= empty - 1;
      }
      const int zero_row = __shfl(out, mine < 0 ? 0 : mine, kWave);
      float zero[EPV];
#pragma unroll
      for (int c = 0; c < EPV; ++c) zero[c] = 0.0f;
      if (mine >= 0) store_row(zero_row, zero);
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
    WalkMatrix m, WalkMatrix whole, const WalkDims* __restrict__ dims, const int* __restrict__ tail_row,
    const float* __restrict__ phead, const float* __restrict__ ptail, T* __restrict__ Y, T* __restrict__ Y2,
    int64_t ldy, int dim, int kChunk) {
  apply_dims(m, whole, dims);
  if (m.n_rows == 0) return;
  const int64_t* __restrict__ rowptr = m.rowptr;
  const int n_rows = m.n_rows;
  const int64_t nchunks = walk_chunks(m.nnz, kChunk);
  constexpr int NF = EPV == 1 ? 1 : 4;   // floats per piece vector
  constexpr int NV = EPV / NF;
  constexpr int U = 8 / NV;              // pieces in flight
  const int lane = threadIdx.x & 63;
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kSpmmWaves + (threadIdx.x >> 6);
  if (chunk >= nchunks) return;
  const int r = tail_row[chunk];
  if (r < 0 || r >= n_rows) return;
  const int out = m.row_map ? m.row_map[r] : r;
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
  if (Y) RawVec<T, EPV>::store(Y + static_cast<int64_t>(out) * ldy + col, acc);
  if (Y2) {
#pragma unroll
    for (int c = 0; c < EPV; ++c) acc[c] = acc[c] > 0.0f ? acc[c] : 0.0f;
    RawVec<T, EPV>::store(Y2 + static_cast<int64_t>(out) * ldy + col, acc);
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

// what every call needs: chunk tables and the pieces of straddling rows
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

// Chunk of a launch: the plan's, several at a time where the lane groups are many (a run has at least one block of
// entries); *step = plan chunks in one.
static int walk_chunk(int64_t nnz, int lpr, int* step) {
  int chunk = spmm_chunk(nnz);
  *step = 1;
  while (chunk < kWalkBlock * (64 / lpr)) {
    chunk *= 2;
    *step *= 2;
  }
  return chunk;
}

// One walk over a matrix and the sums of its straddling rows. dims != null: sizes on the device, m.nnz and m.n_rows are
// what the grid is made for.
template <typename T, int EPV, bool XCD_RANGES>
static int launch_walk(const WalkMatrix& m, const WalkMatrix& whole, const WalkDims* dims, const T* X, int64_t ldx, T* Y,
                       T* Y2, int64_t ldy, int dim, int lpr, int chunk, int step, int stream_csr, float* phead,
                       float* ptail, int* tail_row, hipStream_t st) {
  const int nvec = static_cast<int>(ceil_div(dim, EPV));
  const int64_t nc = walk_chunks(m.nnz, chunk);
  const int64_t nblocks = XCD_RANGES ? 8 * ceil_div(nc, 8 * kSpmmWaves) : ceil_div(nc, kSpmmWaves);
  const dim3 grid(static_cast<unsigned>(nblocks), static_cast<unsigned>(ceil_div(nvec, lpr)));
  const size_t lds = static_cast<size_t>(kSpmmWaves) * walk_lds_ints(chunk) * sizeof(int);
#define CDF_WALK(LPRV, QUADV)                                                                                     \
  spmm_walk_kernel<T, EPV, LPRV, QUADV, XCD_RANGES><<<grid, kSpmmThreads, lds, st>>>(                             \
      m, whole, dims, X, static_cast<uint64_t>(ldx), Y, Y2, ldy, dim, step, phead, ptail, tail_row, chunk, stream_csr)
#define CDF_WALK_Q(LPRV)                                                                                          \
  do {                                                                                                            \
    if constexpr (XCD_RANGES) CDF_WALK(LPRV, true);                                                               \
    else if (chunk >= 256) CDF_WALK(LPRV, true);                                                                  \
    else CDF_WALK(LPRV, false);                                                                                   \
  } while (0)
  prof_begin(K_SPMM_WALK, st);
  if constexpr (EPV == 1) {
    CDF_WALK_Q(8);
  } else {
    switch (lpr) {
      case 2: CDF_WALK_Q(2); break;
      case 4: CDF_WALK_Q(4); break;
      case 8: CDF_WALK_Q(8); break;
      case 16: CDF_WALK_Q(16); break;
      default: CDF_WALK_Q(32); break;
    }
  }
  prof_end(K_SPMM_WALK, st);
#undef CDF_WALK_Q
#undef CDF_WALK
  CDF_LAUNCH_CHECK("cdf_spmm/walk");
  {
    ProfScope ps(K_SPMM_FIXUP, st);
    const dim3 fgrid(static_cast<unsigned>(ceil_div(nc, kSpmmWaves)), static_cast<unsigned>(ceil_div(nvec, 64)));
    spmm_fixup_kernel<T, EPV><<<fgrid, kSpmmThreads, 0, st>>>(m, whole, dims, tail_row, phead, ptail, Y, Y2, ldy, dim, chunk);
  }
  CDF_LAUNCH_CHECK("cdf_spmm/fixup");
  return CDF_OK;
}

// ---- large matrices: column classes on XCDs -----------------------------------------------------------
// Where the gathered table is far larger than the caches, every XCD's L2 holds the same hottest rows of X, because
// every XCD sees every column. Splitting the columns into eight classes (a hash of the column) and giving each XCD the
// entries of one class lets the eight L2s hold eight times as many different rows: on the 144 M entries of an R-MAT
// partition (7.1 M columns, 256 floats) the rows of 128 and more entries, 87 % of all, took 18.5 ms in one walk and 11.7 ms
// split (its transpose 12.2 -> 6.5 for 63 %; 49 M Chung-Lu entries 5.3 -> 3.9 for 89 %). Classes by column range instead of
// by hash, which would need no copy of the entries: 12.4, 7.1 and 4.9 ms.
// A row's entries then give eight partial rows, added up at the end: that pays for long rows only. Rows of at least T
// entries ("long", T a power of two from 128 on, the smallest for which the partial rows fit the workspace) are cut into
// units of at most kUnit entries (so that no wavefront partitions a row of 10^5 alone), each unit's entries are copied
// class by class, and the virtual matrix of 8 x units rows is walked with a contiguous eighth of it on each XCD. The
// short rows' entries are copied together and walked as before. If the long rows hold less than half of the entries the
// matrix is walked whole, as it is where no column is read much more often than another. All counts stay on the device: grids are made for the largest, surplus workgroups leave.
constexpr int kUnit = 16384;
constexpr int kLongRow = 128;
constexpr int kBuckets = 16;
constexpr int kSplitRows = 1024;      // rows per block of the row passes
constexpr int kSplitCounts = 8192;    // counts per block of the virtual row pointers' scan

struct SplitState {
  unsigned long long entries[kBuckets];   // of rows of 128 << b .. entries
  int units[kBuckets], rows[kBuckets];
  int empty, threshold, n_units;
  int totals[4];   // written by the scans, not used
  WalkDims long_part, short_part;
};

__device__ __forceinline__ int row_bucket(int64_t len) {
  return len < kLongRow ? -1 : min(63 - __builtin_clzll(static_cast<unsigned long long>(len)) - 7, kBuckets - 1);
}
__device__ __forceinline__ int row_units(int64_t len) { return static_cast<int>((len + kUnit - 1) / kUnit); }
__device__ __forceinline__ int column_class(int col) { return (static_cast<unsigned>(col) * 2654435761u >> 13) & 7; }

__global__ __launch_bounds__(64) void split_clear_kernel(SplitState* st) {
  if (threadIdx.x < kBuckets) {
    st->entries[threadIdx.x] = 0ull;
    st->units[threadIdx.x] = st->rows[threadIdx.x] = 0;
    st->empty = 0;
  }
}

__global__ __launch_bounds__(256) void split_count_rows_kernel(const int64_t* __restrict__ rowptr, int n_rows, SplitState* st) {
  __shared__ unsigned long long ent[kBuckets];
  __shared__ int uni[kBuckets], num[kBuckets], none;
  if (threadIdx.x == 0) none = 0;
  if (threadIdx.x < kBuckets) {
    ent[threadIdx.x] = 0ull;
    uni[threadIdx.x] = num[threadIdx.x] = 0;
  }
  __syncthreads();
  for (int64_t r = blockIdx.x * 256ll + threadIdx.x; r < n_rows; r += gridDim.x * 256ll) {
    const int64_t len = rowptr[r + 1] - rowptr[r];
    const int b = row_bucket(len);
    if (b >= 0) {
      atomicAdd(&ent[b], static_cast<unsigned long long>(len));
      atomicAdd(&uni[b], row_units(len));
      atomicAdd(&num[b], 1);
    }
    if (len == 0) atomicAdd(&none, 1);
  }
  __syncthreads();
  if (threadIdx.x == 0 && none > 0) atomicAdd(&st->empty, none);
  if (threadIdx.x < kBuckets && uni[threadIdx.x] > 0) {
    atomicAdd(&st->entries[threadIdx.x], ent[threadIdx.x]);
    atomicAdd(&st->units[threadIdx.x], uni[threadIdx.x]);
    atomicAdd(&st->rows[threadIdx.x], num[threadIdx.x]);
  }
}

// Threshold, sizes of the two parts, or "whole". Classes gain only where some columns come up far more often than
// others: of 16384 sampled entries at least one in 16 has to repeat a column (a hash of it) seen before. Columns drawn
// evenly repeat by 3 % and lose 1 to 11 % by the split (64 M entries in 1 and 4 M columns); the R-MAT partition repeats by
// 9 %, its transpose by 19, the Chung-Lu one by 13.
constexpr int kSamples = 16384, kSampleBits = 18, kSampleThreads = 1024;
__global__ __launch_bounds__(kSampleThreads) void split_decide_kernel(SplitState* st, const int* __restrict__ colidx, int n_rows,
                                                                      int64_t nnz, int unit_cap) {
  __shared__ unsigned seen[(1 << kSampleBits) / 32];
  __shared__ int distinct;
  for (int i = threadIdx.x; i < (1 << kSampleBits) / 32; i += kSampleThreads) seen[i] = 0u;
  if (threadIdx.x == 0) distinct = 0;
  constexpr int PER = kSamples / kSampleThreads;
  const int64_t step = nnz / kSamples;   // the caller's nnz is 2^24 or more
  int col[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const unsigned i = q * kSampleThreads + threadIdx.x;
    col[q] = colidx[i * step + (i * 2654435761u >> 7) % step];
  }
  __syncthreads();
  int fresh = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const unsigned h = static_cast<unsigned>(col[q]) * 2654435761u >> (32 - kSampleBits);
    fresh += (atomicOr(&seen[h >> 5], 1u << (h & 31)) >> (h & 31) & 1u) ^ 1u;
  }
  atomicAdd(&distinct, fresh);
  __syncthreads();
  if (threadIdx.x != 0) return;
  const bool skewed = (kSamples - distinct) * 16 >= kSamples;
  int units = 0, rows = 0, best = kBuckets;
  unsigned long long entries = 0, taken = 0;
  int n_units = 0, n_long = 0;
  for (int b = kBuckets - 1; b >= 0; --b) {
    units += st->units[b];
    rows += st->rows[b];
    entries += st->entries[b];
    if (units > unit_cap) break;
    best = b;
    taken = entries;
    n_units = units;
    n_long = rows;
  }
  const bool split = skewed && best < kBuckets && n_units > 0 && taken * 2 >= static_cast<unsigned long long>(nnz);
  if (!split) {
    taken = 0;
    n_units = n_long = 0;
  }
  st->threshold = split ? kLongRow << best : 0x7fffffff;
  st->n_units = n_units;
  st->short_part = {n_rows - n_long - st->empty, split ? 0 : 1, nnz - static_cast<int64_t>(taken), 0};
  st->long_part = {8 * n_units, 0, static_cast<int64_t>(taken), nnz - static_cast<int64_t>(taken)};
}

// exclusive start of v within the block of 256 threads, total in *all
__device__ __forceinline__ int block_scan_256(int v, int* all) {
  __shared__ int wsum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += t;
  }
  __syncthreads();
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int base = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) base += wsum[w];
    sum += wsum[w];
  }
  *all = sum;
  return base + incl - v;
}

// Per block of kSplitRows rows: units of the long rows, entries and number of the short ones (of those that have
// any) -> sums[0 .. 2][block].
// ASSIGN: with the blocks' offsets in their place, the short part's row pointers and rows and the list of units.
template <bool ASSIGN>
__global__ __launch_bounds__(256) void split_rows_kernel(const int64_t* __restrict__ rowptr, int n_rows, const SplitState* st,
                                                         int* __restrict__ sums, int64_t sum_stride,
                                                         int64_t* __restrict__ short_ptr, int* __restrict__ short_row,
                                                         int* __restrict__ unit_row, int64_t* __restrict__ unit_beg) {
  int* at_block = sums + blockIdx.x;
  if (st->short_part.whole) {   // nothing to split; the scans that follow read these
    if (!ASSIGN && threadIdx.x < 3) at_block[threadIdx.x * sum_stride] = 0;
    return;
  }
  const int threshold = st->threshold;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kSplitRows + threadIdx.x * 4;
  int64_t at[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) at[q] = rowptr[min(r0 + q, static_cast<int64_t>(n_rows))];
  int units = 0, entries = 0, rows = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t len = at[q + 1] - at[q];
    if (r0 + q >= n_rows) break;
    if (len >= threshold) {
      units += row_units(len);
    } else if (len > 0) {
      entries += static_cast<int>(len);
      ++rows;
    }
  }
  int all[3];
  int u = block_scan_256(units, &all[0]);
  int e = block_scan_256(entries, &all[1]);
  int j = block_scan_256(rows, &all[2]);
  if (!ASSIGN) {
    if (threadIdx.x == 0) {
#pragma unroll
      for (int q = 0; q < 3; ++q) at_block[q * sum_stride] = all[q];
    }
    return;
  }
  u += at_block[0];
  e += at_block[sum_stride];
  j += at_block[2 * sum_stride];
  const int n_units = st->n_units;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t r = r0 + q;
    if (r >= n_rows) break;
    const int64_t len = at[q + 1] - at[q];
    if (len >= threshold) {
      for (int64_t b = at[q]; b < at[q + 1] && u < n_units; b += kUnit, ++u) {
        unit_row[u] = static_cast<int>(r);
        unit_beg[u] = b;
      }
    } else if (len > 0) {
      short_ptr[j] = e;
      short_row[j] = static_cast<int>(r);
      e += static_cast<int>(len);
      ++j;
    }
    if (r == n_rows - 1) short_ptr[j] = e;
  }
}

constexpr unsigned long long kEven = 0x00ff00ff00ff00ffull;   // every second byte

// One wavefront per unit: entries per class -> counts[class * units + unit]. A lane counts in bytes of one 64-bit word.
__global__ __launch_bounds__(256) void split_count_kernel(const int64_t* __restrict__ rowptr, const int* __restrict__ colidx,
                                                          const SplitState* st, const int* __restrict__ unit_row,
                                                          const int64_t* __restrict__ unit_beg, int* __restrict__ counts) {
  const int n_units = st->n_units;
  const int lane = threadIdx.x & 63;
  const int u = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (u >= n_units) return;
  const int64_t beg = unit_beg[u], row_end = rowptr[unit_row[u] + 1];
  const int len = static_cast<int>(row_end - beg < kUnit ? row_end - beg : kUnit);
  const int* cp = colidx + beg;
  constexpr int U = 8;
  unsigned long long even = 0, odd = 0;   // four 16-bit counts each
  for (int k = 0; k < len;) {
    unsigned long long bytes = 0;
    const int stop = min(len, k + 128 * 64);   // at most 128 counts in a byte
    for (; k + U * 64 <= stop; k += U * 64) {
      int col[U];
#pragma unroll
      for (int q = 0; q < U; ++q) col[q] = cp[k + q * 64 + lane];
#pragma unroll
      for (int q = 0; q < U; ++q) bytes += 1ull << (8 * column_class(col[q]));
    }
    for (; k < stop; k += 64)
      if (k + lane < stop) bytes += 1ull << (8 * column_class(cp[k + lane]));
    even += bytes & kEven;
    odd += (bytes >> 8) & kEven;
  }
  // 64 lanes of up to 256: 16384 at most
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    even += __shfl_xor(even, off, kWave);
    odd += __shfl_xor(odd, off, kWave);
  }
  if (lane < 8)
    counts[static_cast<int64_t>(lane) * n_units + u] = static_cast<int>(((lane & 1 ? odd : even) >> (16 * (lane >> 1))) & 0xffff);
}

// One wavefront per unit: its entries copied to their classes' runs, in a fixed order. kPlace entries at a time are sorted
// by class in LDS, so that a run is written in pieces of about 64 entries (8 at a time,
// as they come: 957 us on 109 M entries, so 546 us).
constexpr int kPlace = 512;
__global__ __launch_bounds__(256) void split_place_kernel(const int64_t* __restrict__ rowptr, const int* __restrict__ colidx,
                                                          const float* __restrict__ vals, const SplitState* st,
                                                          const int* __restrict__ unit_row, const int64_t* __restrict__ unit_beg,
                                                          const int64_t* __restrict__ vptr, int* __restrict__ out_col,
                                                          float* __restrict__ out_val) {
  __shared__ int lds_col[4][kPlace];
  __shared__ float lds_val[4][kPlace];
  const int n_units = st->n_units;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int u = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave);
  if (u >= n_units) return;
  int* sc = lds_col[wave];
  float* sv = lds_val[wave];
  const int64_t beg = unit_beg[u], row_end = rowptr[unit_row[u] + 1];
  const int len = static_cast<int>(row_end - beg < kUnit ? row_end - beg : kUnit);
  const int* cp = colidx + beg;
  const float* vp = vals + beg;
  constexpr int U = kPlace / 64;
  int64_t next = 0;   // lane x < 8: class x's next place
  if (lane < 8) next = vptr[static_cast<int64_t>(lane) * n_units + u] + st->long_part.first;
  for (int k0 = 0; k0 < len; k0 += kPlace) {
    int col[U];
    float val[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const bool on = k0 + q * 64 + lane < len;
      col[q] = on ? cp[k0 + q * 64 + lane] : 0;
      val[q] = on ? vp[k0 + q * 64 + lane] : 0.0f;
    }
    // counts per class in 16-bit fields (even and odd classes in a word each): this lane's, then those of the lanes
    // before it, on top of where the class begins in LDS
    unsigned long long bytes = 0;
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (k0 + q * 64 + lane < len) bytes += 1ull << (8 * column_class(col[q]));
    unsigned long long at2[2] = {bytes & kEven, (bytes >> 8) & kEven};
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned long long t0 = __shfl_up(at2[0], off, kWave), t1 = __shfl_up(at2[1], off, kWave);
      if (lane >= off) {
        at2[0] += t0;
        at2[1] += t1;
      }
    }
    const unsigned long long all0 = __shfl(at2[0], 63, kWave), all1 = __shfl(at2[1], 63, kWave);
    unsigned long long start0 = 0, start1 = 0;
    int run = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      start0 |= static_cast<unsigned long long>(run) << (16 * x);
      run += static_cast<int>(all0 >> (16 * x)) & 0xffff;
      start1 |= static_cast<unsigned long long>(run) << (16 * x);
      run += static_cast<int>(all1 >> (16 * x)) & 0xffff;
    }
    at2[0] += start0 - (bytes & kEven);
    at2[1] += start1 - ((bytes >> 8) & kEven);
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int cls = column_class(col[q]), sh = 16 * (cls >> 1);
      const int at = static_cast<int>((cls & 1 ? at2[1] : at2[0]) >> sh) & 0xffff;
      if (k0 + q * 64 + lane < len) {
        at2[0] += static_cast<unsigned long long>(cls & 1 ? 0 : 1) << sh;
        at2[1] += static_cast<unsigned long long>(cls & 1) << sh;
        sc[at] = col[q];
        sv[at] = val[q];
      }
    }
    const int field = 16 * ((lane & 7) >> 1);
    const int start = static_cast<int>((lane & 1 ? start1 : start0) >> field) & 0xffff;
    const int mine = static_cast<int>((lane & 1 ? all1 : all0) >> field) & 0xffff;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int64_t shift = next - start;   // place in the runs less place in LDS
    const int n = min(len - k0, kPlace);
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int i = q * 64 + lane;
      const int c = i < n ? sc[i] : 0;
      const int64_t to = __shfl(shift, column_class(c), kWave) + i;
      if (i < n) {
        out_col[to] = c;
        out_val[to] = sv[i];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    next += mine;
  }
}

// Virtual row pointers: exclusive sums of 8 x units counts, kSplitCounts to a block. APPLY false: the blocks' sums.
template <bool APPLY>
__global__ __launch_bounds__(256) void split_vptr_kernel(const int* __restrict__ counts, const SplitState* st,
                                                         int* __restrict__ block_sum, int64_t* __restrict__ vptr) {
  const int64_t n = 8ll * st->n_units;
  constexpr int PER = kSplitCounts / 256;
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kSplitCounts + threadIdx.x * PER;
  int v[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    v[q] = i0 + q < n ? counts[i0 + q] : 0;
    sum += v[q];
  }
  int all;
  int run = block_scan_256(sum, &all);
  if (!APPLY) {
    if (threadIdx.x == 0) block_sum[blockIdx.x] = all;
    return;
  }
  run += block_sum[blockIdx.x];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (i0 + q <= n) vptr[i0 + q] = run;   // entry n too: the total
    run += v[q];
  }
}

// entries of the short rows, 16 lanes to a row; zeros for the rows that have none (left in the short part, a long
// run of them would fall to one wavefront)
__global__ __launch_bounds__(256) void split_short_kernel(const int64_t* __restrict__ rowptr, const int* __restrict__ colidx,
                                                          const float* __restrict__ vals, const SplitState* st,
                                                          const int64_t* __restrict__ short_ptr,
                                                          const int* __restrict__ short_row, int* __restrict__ out_col,
                                                          float* __restrict__ out_val, int n_rows, float* __restrict__ Y,
                                                          float* __restrict__ Y2, int64_t ldy, int dim) {
  if (st->short_part.whole) return;
  const int n = st->short_part.n_rows;
  const int l = threadIdx.x & 15;
  constexpr int U = 4;   // rows in flight: each is a chain of three loads (one row: 191 and 597 us on 1.9 and 6.9 M rows)
  for (int64_t j = ((blockIdx.x * 256ll + threadIdx.x) >> 4) * U; j < n; j += gridDim.x * 16ll * U) {
    int64_t a[U], to[U + 1];
#pragma unroll
    for (int q = 0; q <= U; ++q) to[q] = short_ptr[min(j + q, static_cast<int64_t>(n))];
#pragma unroll
    for (int q = 0; q < U; ++q) a[q] = rowptr[short_row[min(j + q, static_cast<int64_t>(n) - 1)]];
    int col[U];
    float val[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const bool on = l < to[q + 1] - to[q];
      col[q] = on ? colidx[a[q] + l] : 0;
      val[q] = on ? vals[a[q] + l] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int64_t len = to[q + 1] - to[q];
      if (l < len) {
        out_col[to[q] + l] = col[q];
        out_val[to[q] + l] = val[q];
      }
      for (int64_t k = l + 16; k < len; k += 16) {
        out_col[to[q] + k] = colidx[a[q] + k];
        out_val[to[q] + k] = vals[a[q] + k];
      }
    }
  }
  if (st->empty == 0) return;
  for (int64_t r = (blockIdx.x * 256ll + threadIdx.x) >> 4; r < n_rows; r += gridDim.x * 16ll) {
    if (rowptr[r] != rowptr[r + 1]) continue;
    for (int c = l; c < dim; c += 16) {
      if (Y) Y[r * ldy + c] = 0.0f;
      if (Y2) Y2[r * ldy + c] = 0.0f;
    }
  }
}

__global__ __launch_bounds__(256) void split_chunk_rows_kernel(const int64_t* __restrict__ ptr, const WalkDims* dims,
                                                               int* __restrict__ chunk_row, int chunk) {
  if (dims->whole) return;
  for (int64_t r = blockIdx.x * 256ll + threadIdx.x; r < dims->n_rows; r += gridDim.x * 256ll) {
    const int64_t a = ptr[r], b = ptr[r + 1];
    for (int64_t c = (a + chunk - 1) / chunk; c * chunk < b; ++c) chunk_row[c] = static_cast<int>(r);
  }
}

// long rows: the sum of their units' partial rows, class by class, unit by unit
__global__ __launch_bounds__(256) void split_combine_kernel(const int64_t* __restrict__ rowptr, const SplitState* st,
                                                            const int* __restrict__ unit_row, const int64_t* __restrict__ unit_beg,
                                                            const float* __restrict__ partial, float* __restrict__ Y,
                                                            float* __restrict__ Y2, int64_t ldy, int dim) {
  const int n_units = st->n_units;
  const int lane = threadIdx.x & 63;
  const int u = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (u >= n_units) return;
  const int r = unit_row[u];
  const int64_t beg = rowptr[r];
  if (unit_beg[u] != beg) return;   // the row's first unit sums them all
  const int k = row_units(rowptr[r + 1] - beg);
  for (int c0 = lane * 4; c0 < dim; c0 += 256) {
    const int col = min(c0, dim - 4);
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int j = 0; j < k; ++j) {
      RawVec<float, 4> t[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) t[x].load(partial + (static_cast<int64_t>(x) * n_units + u + j) * dim + col);
#pragma unroll
      for (int x = 0; x < 8; ++x) t[x].fma_into(1.0f, acc);
    }
    const int64_t at = static_cast<int64_t>(r) * ldy + col;
    if (Y) RawVec<float, 4>::store(Y + at, acc);
    if (Y2) {
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = acc[c] > 0.0f ? acc[c] : 0.0f;
      RawVec<float, 4>::store(Y2 + at, acc);
    }
  }
}

// fp32 rows. The copies cost by the entry (1.1 ms on 144 M entries), the gain is by the entry and column, hence the line
// at 128 columns: 144 M entries, 128 columns 11.0 -> 8.9 ms (A) and 9.7 -> 9.0 ms (its transpose), 64 columns
// 5.5 -> 5.0 and 4.0 -> 4.6 ms. The table of one line per row has to exceed what the L2s hold four times over and
// more, and a column has to be read often; smaller work does not carry the dozen small launches (60 us).
static bool split_pays(const cdf_csr* A, int dim) {
  return dim >= kSplitColumns && A->nnz >= (int64_t(1) << 24) && A->nnz < (int64_t(1) << 31) - kSplitRows && A->nnz * dim >= int64_t(4000000000) &&
         static_cast<int64_t>(A->n_cols) * 128 >= (int64_t(128) << 20) && A->nnz >= 8 * static_cast<int64_t>(A->n_cols);
}

// most units: long rows, and the cuts of the longest ones
static int64_t split_unit_bound(int64_t nnz) { return nnz / kLongRow + nnz / kUnit + 1; }
// bytes of partial rows: 12 for every entry (191 k long rows of 144 M entries need 11 at 256 columns)
static size_t split_partial_bytes(int64_t nnz) { return align_up(static_cast<size_t>(nnz) * 12, 256); }

size_t split_workspace_bytes(int64_t n_rows, int64_t nnz) {
  if (nnz < (int64_t(1) << 24) || nnz >= (int64_t(1) << 31) - kSplitRows) return 0;
  const size_t u = static_cast<size_t>(split_unit_bound(nnz)), rows = static_cast<size_t>(n_rows);
  const size_t rb = 3 * (static_cast<size_t>(ceil_div(n_rows, kSplitRows)) + 4), vb = 8 * u / kSplitCounts + 5;
  return 1024 + align_up((rows + 1) * 8, 256) + align_up(rows * 4, 256) + 2 * align_up(rb * 4, 256) +
         2 * align_up(vb * 4, 256) + align_up(u * 4, 256) +
         align_up(u * 8, 256) + align_up(8 * u * 4, 256) + align_up((8 * u + 1) * 8, 256) +
         2 * align_up(static_cast<size_t>(nnz) * 4, 256) + 2 * align_up(static_cast<size_t>(spmm_chunks_bound(nnz) + 1) * 4, 256) +
         split_partial_bytes(nnz);
}

int scan_counts(const int* counts, int nblocks, int* offsets, int32_t* n_sent, hipStream_t st);

static int launch_split(const WalkMatrix& A, const float* X, int64_t ldx, float* Y, float* Y2, int64_t ldy,
                        int dim, int lpr, int chunk, int step, int stream_csr, float* phead, float* ptail, int* tail_row,
                        char* w, hipStream_t st) {
  const int64_t nnz = A.nnz, u_bound = split_unit_bound(nnz);
  const int plan_chunk = chunk / step;
  auto take = [&](size_t bytes) {
    char* p = w;
    w += align_up(bytes, 256);
    return p;
  };
  SplitState* state = reinterpret_cast<SplitState*>(take(1024));
  static_assert(sizeof(SplitState) <= 1024, "state");
  const int row_blocks = static_cast<int>(ceil_div(A.n_rows, kSplitRows));
  int64_t* short_ptr = reinterpret_cast<int64_t*>(take((static_cast<size_t>(A.n_rows) + 1) * 8));
  int* short_row = reinterpret_cast<int*>(take(static_cast<size_t>(A.n_rows) * 4));
  const int64_t sum_stride = (row_blocks + 3) / 4 * 4;   // the scans read and write 16-byte vectors
  int* sums = reinterpret_cast<int*>(take(3 * (static_cast<size_t>(row_blocks) + 4) * 4));
  int* sums_at = reinterpret_cast<int*>(take(3 * (static_cast<size_t>(row_blocks) + 4) * 4));
  const int v_blocks = static_cast<int>(8 * u_bound / kSplitCounts + 1);
  int* vb = reinterpret_cast<int*>(take((static_cast<size_t>(v_blocks) + 4) * 4));
  int* vb_at = reinterpret_cast<int*>(take((static_cast<size_t>(v_blocks) + 4) * 4));
  int* unit_row = reinterpret_cast<int*>(take(static_cast<size_t>(u_bound) * 4));
  int64_t* unit_beg = reinterpret_cast<int64_t*>(take(static_cast<size_t>(u_bound) * 8));
  int* counts = reinterpret_cast<int*>(take(8 * static_cast<size_t>(u_bound) * 4));
  int64_t* vptr = reinterpret_cast<int64_t*>(take((8 * static_cast<size_t>(u_bound) + 1) * 8));
  int* col = reinterpret_cast<int*>(take(static_cast<size_t>(nnz) * 4));
  float* val = reinterpret_cast<float*>(take(static_cast<size_t>(nnz) * 4));
  int* long_chunk = reinterpret_cast<int*>(take(static_cast<size_t>(spmm_chunks(nnz) + 1) * 4));
  int* short_chunk = reinterpret_cast<int*>(take(static_cast<size_t>(spmm_chunks(nnz) + 1) * 4));
  float* partial = reinterpret_cast<float*>(w);
  const int64_t fit = static_cast<int64_t>(split_partial_bytes(nnz) / (static_cast<size_t>(8) * dim * sizeof(float)));
  const int unit_cap = static_cast<int>(fit < u_bound ? fit : u_bound);
  const unsigned row_grid = static_cast<unsigned>(row_blocks < 8192 ? row_blocks * 4 : 32768);
  const unsigned unit_grid = static_cast<unsigned>(ceil_div(unit_cap > 0 ? unit_cap : 1, 4));
  {
    ProfScope ps(K_SPMM_SPLIT, st);
    split_clear_kernel<<<1, 64, 0, st>>>(state);
    split_count_rows_kernel<<<row_blocks < 2048 ? row_blocks : 2048, 256, 0, st>>>(A.rowptr, A.n_rows, state);
    split_decide_kernel<<<1, kSampleThreads, 0, st>>>(state, A.colidx, A.n_rows, nnz, unit_cap);
    split_rows_kernel<false><<<row_blocks, 256, 0, st>>>(A.rowptr, A.n_rows, state, sums, sum_stride, nullptr, nullptr,
                                                         nullptr, nullptr);
  }
  CDF_LAUNCH_CHECK("cdf_spmm/split rows");
  int rc = CDF_OK;
  for (int q = 0; q < 3 && rc == CDF_OK; ++q)
    rc = scan_counts(sums + q * sum_stride, row_blocks, sums_at + q * sum_stride, &state->totals[q], st);
  if (rc != CDF_OK) return rc;
  {
    ProfScope ps(K_SPMM_SPLIT, st);
    split_rows_kernel<true><<<row_blocks, 256, 0, st>>>(A.rowptr, A.n_rows, state, sums_at, sum_stride, short_ptr, short_row,
                                                        unit_row, unit_beg);
    split_count_kernel<<<unit_grid, 256, 0, st>>>(A.rowptr, A.colidx, state, unit_row, unit_beg, counts);
    split_vptr_kernel<false><<<v_blocks, 256, 0, st>>>(counts, state, vb, nullptr);
  }
  CDF_LAUNCH_CHECK("cdf_spmm/split units");
  rc = scan_counts(vb, v_blocks, vb_at, &state->totals[3], st);
  if (rc != CDF_OK) return rc;
  {
    ProfScope ps(K_SPMM_SPLIT, st);
    split_vptr_kernel<true><<<v_blocks, 256, 0, st>>>(counts, state, vb_at, vptr);
    split_place_kernel<<<unit_grid, 256, 0, st>>>(A.rowptr, A.colidx, A.vals, state, unit_row, unit_beg, vptr, col, val);
    split_short_kernel<<<row_grid, 256, 0, st>>>(A.rowptr, A.colidx, A.vals, state, short_ptr, short_row, col, val,
                                                 A.n_rows, Y, Y2, ldy, dim);
    split_chunk_rows_kernel<<<4096, 256, 0, st>>>(vptr, &state->long_part, long_chunk, plan_chunk);
    split_chunk_rows_kernel<<<4096, 256, 0, st>>>(short_ptr, &state->short_part, short_chunk, plan_chunk);
  }
  CDF_LAUNCH_CHECK("cdf_spmm/split copy");
  // slices of one line: the classes' tables are what has to fit
  const int long_lpr = dim % 32 == 0 ? 8 : lpr;
  const WalkMatrix lm = {vptr, col, val, long_chunk, 0, nnz, nullptr}, sm = {short_ptr, col, val, short_chunk, 0, nnz, short_row};
  rc = launch_walk<float, 4, true>(lm, A, &state->long_part, X, ldx, partial, nullptr, dim, dim, long_lpr, chunk, step,
                                   stream_csr, phead, ptail, tail_row, st);
  if (rc != CDF_OK) return rc;
  rc = launch_walk<float, 4, false>(sm, A, &state->short_part, X, ldx, Y, Y2, ldy, dim, lpr, chunk, step, stream_csr, phead,
                                    ptail, tail_row, st);
  if (rc != CDF_OK) return rc;
  {
    ProfScope ps(K_SPMM_COMBINE, st);
    split_combine_kernel<<<unit_grid, 256, 0, st>>>(A.rowptr, state, unit_row, unit_beg, partial, Y, Y2, ldy, dim);
  }
  CDF_LAUNCH_CHECK("cdf_spmm/combine");
  return CDF_OK;
}

template <typename T, int EPV>
static int launch_spmm(const cdf_csr* A, const T* X, int64_t ldx, T* Y, T* Y2, int64_t ldy, int dim, void* ws,
                       size_t ws_bytes, hipStream_t st) {
  const int plan_chunk = spmm_chunk(A->nnz);
  const int64_t plan_chunks = spmm_chunks(A->nnz);
  const int lpr = EPV == 1 ? 8 : pick_lanes(dim, EPV, A->n_cols);
  int step;
  const int chunk = walk_chunk(A->nnz, lpr, &step);
  const int64_t nc = walk_chunks(A->nnz, chunk);
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
  // the CSR arrays are streamed past the caches where they exceed the memory-side cache and cannot be found
  // there by the next slice (144 M entries: 21.6 -> 21.3 ms; 1.8 M entries: 90 -> 99 us, hence the line)
  const int stream_csr = A->nnz * 8 > (int64_t(256) << 20) ? 1 : 0;
  const WalkMatrix m = {A->rowptr, A->colidx, A->vals, chunk_row, A->n_rows, A->nnz, nullptr};
  if constexpr (std::is_same<T, float>::value && EPV == 4) {
    const size_t used = spmm_workspace_bytes(A->nnz, dim);
    if (split_pays(A, dim) && ws_bytes >= used + split_workspace_bytes(A->n_rows, A->nnz))
      return launch_split(m, X, ldx, Y, Y2, ldy, dim, lpr, chunk, step, stream_csr, phead, ptail, tail_row,
                          static_cast<char*>(ws) + used, st);
  }
  return launch_walk<T, EPV, false>(m, m, nullptr, X, ldx, Y, Y2, ldy, dim, lpr, chunk, step, stream_csr, phead, ptail,
                                    tail_row, st);
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
      rc = v ? launch_spmm<float, 4>(A, x, ldx, y, y2, ldy, d, ws, ws_bytes, st) : launch_spmm<float, 1>(A, x, ldx, y, y2, ldy, d, ws, ws_bytes, st);
    } else {
      const bf16_t* x = static_cast<const bf16_t*>(X) + col0;
      bf16_t* y = Y ? static_cast<bf16_t*>(Y) + col0 : nullptr;
      bf16_t* y2 = Y2 ? static_cast<bf16_t*>(Y2) + col0 : nullptr;
      rc = v ? launch_spmm<bf16_t, 8>(A, x, ldx, y, y2, ldy, d, ws, ws_bytes, st) : launch_spmm<bf16_t, 1>(A, x, ldx, y, y2, ldy, d, ws, ws_bytes, st);
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
