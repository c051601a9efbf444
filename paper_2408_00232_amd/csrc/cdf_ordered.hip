// The transposed aggregation and dM = dZ W^T in the order of summation that a backward step with
// CDF_COMMIT_DEQ has always had. With that commit the sender's gradient cache takes the RECOVERED message, so
// a change in the last bit of a gradient that puts one element on the other side of a code's edge moves the
// committed row by a whole code step (1.7e-5 of the codes for the kernels of cdf_spmm.hip and cdf_gemm.hip): a
// run is then no longer the run it was, and what a peer or a saved cache holds from before no longer matches what
// this side would have committed. The other commits store the row itself and have no such step; they, and
// every other caller, take the faster kernels (mid 602->256, transposed aggregation 353 us here, 224 there).
//
// Aggregation: a chunk of 64 to 1024 stored entries per wavefront. ordered_row_kernel gives the whole wavefront to
// one entry at a time; ordered_sliced_kernel gives LPR lanes to an entry and combines the groups' sums at every row
// end. Rows that straddle chunk borders are finished by ordered_fixup_kernel.
#include <type_traits>

#include "cdf_common.h"

namespace cdf {

constexpr int kOrderedThreads = 256;  // 4 wavefronts per block
constexpr int kOrderedWaves = kOrderedThreads / 64;

int spmm_chunk(int64_t nnz);
int64_t spmm_chunks(int64_t nnz);
size_t spmm_workspace_bytes(int64_t nnz, int32_t dim);

// chunk_row[c] = row that holds stored entry c*chunk (c >= 1; entry 0 is handled as row 0).
__global__ void ordered_chunk_rows_kernel(const int64_t* __restrict__ rowptr, int n_rows, int* __restrict__ chunk_row,
                                  int kChunk) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rows) return;
  const int64_t a = rowptr[r], b = rowptr[r + 1];
  for (int64_t c = (a + kChunk - 1) / kChunk; c * kChunk < b; ++c) chunk_row[c] = r;
}

template <typename T, int EPV, int NP>
__global__ __launch_bounds__(kOrderedThreads) void ordered_row_kernel(
    const int64_t* __restrict__ rowptr, const int* __restrict__ colidx, const float* __restrict__ vals,
    int n_rows, int64_t nnz, const T* __restrict__ X, int64_t ldx, T* __restrict__ Y,
    int64_t ldy, int dim, const int* __restrict__ chunk_row, int64_t nchunks, float* __restrict__ phead, float* __restrict__ ptail,
    int* __restrict__ tail_row, int kChunk) {
  constexpr int U = (8 / NP) > 0 ? (8 / NP) : 1;  // feature rows in flight per wavefront
  const int lane = threadIdx.x & 63;
  // the wavefront index is the same in all lanes: say so, and everything derived from it
  // (chunk bounds, row cursor, loop counters) lives in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kOrderedWaves + wave;
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
  auto store_y = [&](int row) {
    T* py = Y + static_cast<int64_t>(row) * ldy;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (col_on[p]) VecIO<T, EPV>::store(py + (p * 64 + lane) * EPV, acc[p]);
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

// Column-sliced variant for rows that are several cache lines wide. The feature matrix is
// processed in vertical slices of SW = LPR * EPV elements (grid.y = slice); within a slice a
// gather instruction serves 64 / LPR stored entries at once, LPR lanes each. Narrow slices shrink
// the table the gathers hit by dim / SW, so far more of its rows stay in the 4 MB L2 of an XCD
// and in the memory-side cache; the CSR arrays are re-read once per slice (8 bytes per entry
// against SW * 4 of features). Entries of a row are spread round-robin over the lane groups and
// the groups' partial sums are combined when the row ends - a fixed order, no atomics.
template <typename T, int EPV, int LPR, int UREQ>
__global__ __launch_bounds__(kOrderedThreads) void ordered_sliced_kernel(
    const int64_t* __restrict__ rowptr, const int* __restrict__ colidx, const float* __restrict__ vals,
    int n_rows, int64_t nnz, const T* __restrict__ X, int64_t ldx, T* __restrict__ Y,
    int64_t ldy, int dim, const int* __restrict__ chunk_row, int64_t nchunks, float* __restrict__ phead,
    float* __restrict__ ptail, int* __restrict__ tail_row, int kChunk) {
  constexpr int EPI = 64 / LPR;  // stored entries per gather instruction
  constexpr int SW = LPR * EPV;  // slice width in elements
  constexpr int U = UREQ * EPI > 64 ? 64 / EPI : UREQ;  // gather instructions in flight (a window holds 64 entries)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kOrderedWaves + wave;
  if (chunk >= nchunks) return;
  const int g = lane / LPR, lg = lane % LPR;
  const int col0 = blockIdx.y * SW + lg * EPV;  // this lane's columns: [col0, col0 + EPV)
  const bool lane_on = col0 < dim;              // false on the lanes past the row end in a partial last slice
  const int64_t s = chunk * kChunk;
  const int L = static_cast<int>(nnz - s < kChunk ? nnz - s : kChunk);
  int my_col = 0, krel = 0;
  float my_val = 0.0f;

  int r = chunk == 0 ? 0 : chunk_row[chunk];
  bool head = chunk > 0 && rowptr[r] < s;
  auto load_rel = [&](int rbase) -> int {
    const int rr = rbase + lane;
    if (rr < n_rows) {
      const int64_t d = rowptr[rr + 1] - s;
      return d > kChunk ? kChunk + 1 : static_cast<int>(d);
    }
    return kChunk + 2;
  };
  int r_base = r;
  int rel = load_rel(r_base);
  int cur_end = __builtin_amdgcn_readlane(rel, 0);
  auto next_row = [&]() {
    ++r;
    if (r - r_base == 64) {
      r_base = r;
      rel = load_rel(r_base);
    }
    cur_end = __builtin_amdgcn_readlane(rel, r - r_base);
  };

  float acc[EPV];
#pragma unroll
  for (int c = 0; c < EPV; ++c) acc[c] = 0.0f;

  // Combine the lane groups' sums with a halving exchange: at stride 32, 16, ..., LPR each lane
  // passes one half of its components to its partner and adds the partner's other half, so the
  // row slice ends up spread over the lanes (FIN components each, starting at component cbase)
  // with a quarter of the shuffles of a full butterfly. Once a lane is down to one component the
  // remaining strides are plain sums and only the lanes with the stride bit clear keep the result.
  constexpr int FIN = EPV / EPI > 0 ? EPV / EPI : 1;
  int cbase = 0;       // first component (within this lane's EPV) that the lane owns after the exchange
  bool owner = true;   // false on lanes that hold a duplicate
  {
    int cnt = EPV;
#pragma unroll
    for (int off = 32; off >= LPR; off >>= 1) {
      const bool up = (lane & off) != 0;
      if (cnt > 1) {
        cnt >>= 1;
        if (up) cbase += cnt;
      } else if (up) {
        owner = false;
      }
    }
  }
  auto reduce_groups = [&](float (&fin)[FIN]) {
    float a[EPV];
#pragma unroll
    for (int c = 0; c < EPV; ++c) a[c] = acc[c];
    int cnt = EPV;
#pragma unroll
    for (int off = 32; off >= LPR; off >>= 1) {
      const bool up = (lane & off) != 0;
      if (cnt > 1) {
        const int half = cnt >> 1;
#pragma unroll
        for (int i = 0; i < EPV / 2; ++i) {
          if (i < half) {
            const float send = up ? a[i] : a[half + i];
            const float keep = up ? a[half + i] : a[i];
            a[i] = keep + __shfl_xor(send, off, kWave);
          }
        }
        cnt = half;
      } else {
        a[0] = a[0] + __shfl_xor(a[0], off, kWave);
      }
    }
#pragma unroll
    for (int c = 0; c < FIN; ++c) fin[c] = a[c];
  };
  auto store_y = [&](int row, const float (&fin)[FIN]) {
    if (!owner || !lane_on) return;
    const int64_t at = static_cast<int64_t>(row) * ldy + col0 + cbase;
    VecIO<T, FIN>::store(Y + at, fin);
  };
  auto store_partial = [&](float* buf, const float (&fin)[FIN]) {
    if (!owner || !lane_on) return;
    float* pp = buf + chunk * static_cast<int64_t>(dim) + col0 + cbase;
#pragma unroll
    for (int c = 0; c < FIN; ++c) pp[c] = fin[c];
  };
  auto flush_row = [&]() {
    float fin[FIN];
    reduce_groups(fin);
    if (head) store_partial(phead, fin);
    else store_y(r, fin);
    head = false;
#pragma unroll
    for (int c = 0; c < EPV; ++c) acc[c] = 0.0f;
  };

  const T* xs = X + col0;
  for (int base = 0; base < L; base += 64) {
    const int cnt = L - base < 64 ? L - base : 64;
    my_col = 0;
    my_val = 0.0f;
    if (lane < cnt) {
      my_col = colidx[s + base + lane];
      my_val = vals[s + base + lane];
    }
    for (int j = 0; j < cnt; j += EPI * U) {
      float x[U][EPV];
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = j + u * EPI + g;  // this group's entry of instruction u
        const int c = __shfl(my_col, e, kWave);
        v[u] = __shfl(my_val, e, kWave);
#pragma unroll
        for (int q = 0; q < EPV; ++q) x[u][q] = 0.0f;
        if (e < cnt && lane_on) VecIO<T, EPV>::load(xs + static_cast<int64_t>(c) * ldx, x[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int first = j + u * EPI;
        if (first < cnt) {
          const int avail = cnt - first < EPI ? cnt - first : EPI;
          int done = 0;
          while (done < avail) {
            while (krel == cur_end) {
              flush_row();
              next_row();
            }
            const int room = cur_end - krel;
            const int take = avail - done < room ? avail - done : room;
            if (g >= done && g < done + take) {
#pragma unroll
              for (int q = 0; q < EPV; ++q) acc[q] = __fmaf_rn(v[u], x[u][q], acc[q]);
            }
            done += take;
            krel += take;
          }
        }
      }
    }
  }

  int tr = -1;
  if (cur_end > L) {
    float fin[FIN];
    reduce_groups(fin);
    if (head) {
      store_partial(phead, fin);
    } else {
      store_partial(ptail, fin);
      tr = r;
    }
  } else {
    flush_row();
    next_row();
    float zero[FIN];
#pragma unroll
    for (int c = 0; c < FIN; ++c) zero[c] = 0.0f;
    while (r < n_rows && cur_end == L) {
      store_y(r, zero);
      next_row();
    }
  }
  if (lane == 0 && blockIdx.y == 0) tail_row[chunk] = tr;
}

// Adds the pieces of every row that straddles chunk borders, in chunk order.
template <typename T, int EPV>
__global__ __launch_bounds__(kOrderedThreads) void ordered_fixup_kernel(
    const int64_t* __restrict__ rowptr, const int* __restrict__ tail_row, int64_t nchunks,
    const float* __restrict__ phead, const float* __restrict__ ptail, T* __restrict__ Y,
    int64_t ldy, int dim, int n_rows, int kChunk) {
  const int lane = threadIdx.x & 63;
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kOrderedWaves + (threadIdx.x >> 6);
  if (chunk >= nchunks) return;
  const int r = tail_row[chunk];
  if (r < 0 || r >= n_rows) return;
  // last chunk that starts inside row r: the one that holds the row's last entry (the row runs past
  // this chunk, so it has one). Computed, not walked: the longest rows span hundreds of chunks.
  const int64_t last = (rowptr[r + 1] - 1) / kChunk;
  for (int col = lane * EPV; col < dim; col += 64 * EPV) {
    float acc[EPV];
#pragma unroll
    for (int c = 0; c < EPV; ++c) acc[c] = ptail[chunk * static_cast<int64_t>(dim) + col + c];
    int64_t c2 = chunk + 1;
    for (; c2 + 3 <= last; c2 += 4) {
      float t[4][EPV];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < EPV; ++c) t[q][c] = phead[(c2 + q) * static_cast<int64_t>(dim) + col + c];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < EPV; ++c) acc[c] = acc[c] + t[q][c];
    }
    for (; c2 <= last; ++c2)
#pragma unroll
      for (int c = 0; c < EPV; ++c) acc[c] = acc[c] + phead[c2 * static_cast<int64_t>(dim) + col + c];
    VecIO<T, EPV>::store(Y + static_cast<int64_t>(r) * ldy + col, acc);
  }
}

template <typename T, int EPV>
static int launch_ordered(const cdf_csr* A, const T* X, int64_t ldx, T* Y, int64_t ldy, int dim, void* ws,
                       hipStream_t st) {
  const int chunk = spmm_chunk(A->nnz);
  const int64_t nc = spmm_chunks(A->nnz);
  char* w = static_cast<char*>(ws);
  int* own_chunk_row = reinterpret_cast<int*>(w);
  int* tail_row = own_chunk_row + nc;
  w += align_up(static_cast<size_t>(nc) * 2 * sizeof(int), 256);
  float* phead = reinterpret_cast<float*>(w);
  w += align_up(static_cast<size_t>(nc) * dim * sizeof(float), 256);
  float* ptail = reinterpret_cast<float*>(w);

  // chunk -> row table: the caller's plan (built once per matrix by cdf_spmm_plan), else rebuilt here
  const int* chunk_row = A->plan;
  if (!chunk_row) {
    {
      ProfScope ps(K_SPMM_PLAN, st);
      ordered_chunk_rows_kernel<<<static_cast<unsigned>(ceil_div(A->n_rows, 256)), 256, 0, st>>>(A->rowptr, A->n_rows,
                                                                                         own_chunk_row, chunk);
    }
    CDF_LAUNCH_CHECK("ordered spmm/chunk_rows");
    chunk_row = own_chunk_row;
  }
  const unsigned nblocks = static_cast<unsigned>(ceil_div(nc, kOrderedWaves));
  const int per_pass = 64 * EPV;
  const int np = static_cast<int>(ceil_div(dim, per_pass));
  const int nvec = dim / EPV;
  constexpr bool lane16 = EPV * static_cast<int>(sizeof(T)) == 16;   // 16-byte lane vectors
#define CDF_SPMM_ARGS                                                                                      \
  (A->rowptr, A->colidx, A->vals, A->n_rows, A->nnz, X, ldx, Y, ldy, dim, chunk_row, nc, phead, ptail, \
   tail_row, chunk)
  // Lanes per entry. Rows of whole 128-byte lines with eight or more entries on average: one line per
  // row and slice (8 lanes of 16 bytes); it pays when the per-row, per-slice reduction and store are
  // amortised. Rows of at most 32 lane-vectors: one slice, the lane group just wide enough for the row.
  // Everything else: the whole wavefront per entry.
  constexpr int min_avg = 8;
  int lpr = 0, slices = 1;
  if (lane16 && dim % (8 * EPV) == 0 && A->nnz >= static_cast<int64_t>(min_avg) * A->n_rows) {
    lpr = 8;
    slices = dim / (8 * EPV);
  } else if (lane16 && nvec <= 32) {
    lpr = 2;
    while (lpr < nvec) lpr <<= 1;
  }
  if (lpr > 0) {
    if constexpr (lane16) {
      const dim3 grid(nblocks, static_cast<unsigned>(slices));
      prof_begin(K_SPMM_ORDERED, st);
      // gather instructions in flight per wavefront: long rows (the forward matrix of a power-law
      // partition averages ~70 entries) run 2-3 % faster with eight, short rows (its transpose, ~20)
      // with four - measured both ways
      const bool deep = A->nnz >= static_cast<int64_t>(40) * A->n_rows;
      switch (lpr) {
        case 2: ordered_sliced_kernel<T, EPV, 2, 4><<<grid, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS; break;
        case 4: ordered_sliced_kernel<T, EPV, 4, 4><<<grid, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS; break;
        case 8:
          if (deep) ordered_sliced_kernel<T, EPV, 8, 8><<<grid, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS;
          else ordered_sliced_kernel<T, EPV, 8, 4><<<grid, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS;
          break;
        case 16: ordered_sliced_kernel<T, EPV, 16, 4><<<grid, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS; break;
        default: ordered_sliced_kernel<T, EPV, 32, 4><<<grid, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS; break;
      }
      prof_end(K_SPMM_ORDERED, st);
      CDF_LAUNCH_CHECK("ordered spmm/sliced");
    }
  } else {
    prof_begin(K_SPMM_ORDERED, st);
    if (np <= 1) ordered_row_kernel<T, EPV, 1><<<nblocks, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS;
    else if (np <= 2) ordered_row_kernel<T, EPV, 2><<<nblocks, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS;
    else if (np <= 4) ordered_row_kernel<T, EPV, 4><<<nblocks, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS;
    else ordered_row_kernel<T, EPV, 8><<<nblocks, kOrderedThreads, 0, st>>> CDF_SPMM_ARGS;
    prof_end(K_SPMM_ORDERED, st);
    CDF_LAUNCH_CHECK("ordered spmm/main");
  }
#undef CDF_SPMM_ARGS
  {
    ProfScope ps(K_SPMM_FIXUP, st);
    ordered_fixup_kernel<T, EPV><<<nblocks, kOrderedThreads, 0, st>>>(A->rowptr, tail_row, nc, phead, ptail, Y, ldy, dim,
                                                                 A->n_rows, chunk);
  }
  CDF_LAUNCH_CHECK("ordered spmm/fixup");
  return CDF_OK;
}

// Y = A X; the checks are those of spmm_run.
int spmm_ordered_run(const char* fn, const cdf_csr* A, const void* X, int64_t ldx, void* Y, int64_t ldy,
             int32_t dim, cdf_dtype dt, void* ws, size_t ws_bytes, hipStream_t st) {
  CDF_REQUIRE(A != nullptr, "%s: matrix is null", fn);
  CDF_REQUIRE(A->n_rows >= 0 && A->n_cols >= 0 && A->nnz >= 0 && dim > 0 && ldx >= dim && ldy >= dim,
              "%s: bad shape rows=%d cols=%d nnz=%lld dim=%d ldx=%lld ldy=%lld", fn, A->n_rows, A->n_cols,
              (long long)A->nnz, dim, (long long)ldx, (long long)ldy);
  if (dt != CDF_F32 && dt != CDF_BF16) CDF_FAIL(CDF_ERR_UNSUPPORTED, "%s: dtype %d", fn, (int)dt);
  if (A->n_rows == 0) return CDF_OK;
  CDF_REQUIRE(A->rowptr && Y && (A->nnz == 0 || (A->colidx && A->vals && X)), "%s: null pointer", fn);
  const size_t esz = elem_bytes(dt);
  CDF_REQUIRE(aligned(A->rowptr, 8) && aligned(A->colidx, 4) && aligned(A->vals, 4) && aligned(X, esz) &&
                  aligned(Y, esz),
              "%s: misaligned pointer", fn);
  if (!ws || !aligned(ws, 256) || ws_bytes < spmm_workspace_bytes(A->nnz, dim))
    CDF_FAIL(CDF_ERR_WORKSPACE, "%s: workspace too small or unaligned (%zu < %zu)", fn, ws_bytes,
             spmm_workspace_bytes(A->nnz, dim));
  // widest lane-vector that both operands allow; at most 8 passes of 64 lanes per launch
  int epv = dt == CDF_BF16 ? 8 : 4;
  for (; epv > 1; epv >>= 1) {
    const size_t vb = esz * epv;
    if (dim % epv == 0 && ldx % epv == 0 && ldy % epv == 0 && aligned(X, vb) && aligned(Y, vb)) break;
  }
  const int max_cols = 64 * epv * 8;
  for (int col0 = 0; col0 < dim; col0 += max_cols) {
    const int d = dim - col0 < max_cols ? dim - col0 : max_cols;
    int rc;
    if (dt == CDF_F32) {
      const float* x = static_cast<const float*>(X) + col0;
      float* y = static_cast<float*>(Y) + col0;
      rc = epv == 4 ? launch_ordered<float, 4>(A, x, ldx, y, ldy, d, ws, st)
           : epv == 2 ? launch_ordered<float, 2>(A, x, ldx, y, ldy, d, ws, st)
                      : launch_ordered<float, 1>(A, x, ldx, y, ldy, d, ws, st);
    } else {
      const bf16_t* x = static_cast<const bf16_t*>(X) + col0;
      bf16_t* y = static_cast<bf16_t*>(Y) + col0;
      rc = epv == 8   ? launch_ordered<bf16_t, 8>(A, x, ldx, y, ldy, d, ws, st)
           : epv == 4 ? launch_ordered<bf16_t, 4>(A, x, ldx, y, ldy, d, ws, st)
           : epv == 2 ? launch_ordered<bf16_t, 2>(A, x, ldx, y, ldy, d, ws, st)
                      : launch_ordered<bf16_t, 1>(A, x, ldx, y, ldy, d, ws, st);
    }
    if (rc != CDF_OK) return rc;
  }
  return CDF_OK;
}

// ---- dM = dZ W^T, dZ = dH * [Zs > 0], on the fp32 matrix instructions ------------------------------------
// A 128 x BN tile per block of four wavefronts, MFMA 32x32x2, operands in LDS as [k][row] and [k][column].
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr int kOrderedBM = 128;
constexpr int kOrderedBK = 32;

struct OrderedDmArgs {
  const float* dH;
  const float* Zs;   // null: no mask
  const float* W;
  void* dM;
  int64_t ldo;
  int n, f, g;
};

// VEC: 16-byte aligned rows of a multiple of four elements; else element by element
template <bool VEC>
__device__ __forceinline__ void ordered_quad(const float* row, int k, int len, float (&v)[4]) {
  if (VEC) {
    VecIO<float, 4>::load(row + min(k, len - 4), v);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = k < len ? v[c] : 0.0f;
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float x = row[min(k + c, len - 1)];
      v[c] = k + c < len ? x : 0.0f;
    }
  }
}

template <typename T, int BN, bool VEC>
__global__ __launch_bounds__(kOrderedThreads, 2) void ordered_dm_kernel(OrderedDmArgs a) {
  constexpr int SA = kOrderedBM + 2, SB = BN + 2;   // strides 2 mod 8: the transposed stores use all banks
  constexpr int TM = 2, TN = BN / 64, BQ = BN / 32;
  __shared__ float As[kOrderedBK][SA];
  __shared__ float Bs[kOrderedBK][SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, lh = lane >> 5;
  const int m0 = blockIdx.x * kOrderedBM, n0 = blockIdx.y * BN;
  float ra[4][4], rz[4][4], rb[BQ][4];
  auto fetch = [&](int k0) {
    const int k = k0 + (tid & 7) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t off = static_cast<int64_t>(min(m0 + (tid >> 3) + 32 * i, a.n - 1)) * a.g;
      ordered_quad<VEC>(a.dH + off, k, a.g, ra[i]);
      if (a.Zs) ordered_quad<VEC>(a.Zs + off, k, a.g, rz[i]);
    }
#pragma unroll
    for (int i = 0; i < BQ; ++i)
      ordered_quad<VEC>(a.W + static_cast<int64_t>(min(n0 + (tid >> 3) + 32 * i, a.f - 1)) * a.g, k, a.g, rb[i]);
  };
  auto stage = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        As[(tid & 7) * 4 + c][(tid >> 3) + 32 * i] = !a.Zs || rz[i][c] > 0.0f ? ra[i][c] : 0.0f;
#pragma unroll
    for (int i = 0; i < BQ; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) Bs[(tid & 7) * 4 + c][(tid >> 3) + 32 * i] = rb[i][c];
  };
  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  fetch(0);
  for (int k0 = 0; k0 < a.g; k0 += kOrderedBK) {
    stage();
    __syncthreads();
    if (k0 + kOrderedBK < a.g) fetch(k0 + kOrderedBK);
    float fa[2][TM], fb[2][TN];   // operands of step kk + 2 are read while the products of step kk run
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[0][i] = As[lh][wm * 64 + i * 32 + l32];
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = Bs[lh][wn * (BN / 2) + j * 32 + l32];
#pragma unroll
    for (int kk = 0; kk < kOrderedBK; kk += 2) {
      const int cur = (kk >> 1) & 1, nxt = cur ^ 1;
      if (kk + 2 < kOrderedBK) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[nxt][i] = As[kk + 2 + lh][wm * 64 + i * 32 + l32];
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[nxt][j] = Bs[kk + 2 + lh][wn * (BN / 2) + j * 32 + l32];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn * (BN / 2) + j * 32 + l32;
      if (col >= a.f) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + wm * 64 + i * 32 + (e >> 2) * 8 + lh * 4 + (e & 3);
        if (row >= a.n) continue;
        const float one[1] = {acc[i][j][e]};
        VecIO<T, 1>::store(static_cast<T*>(a.dM) + static_cast<int64_t>(row) * a.ldo + col, one);
      }
    }
}

template <typename T>
static void launch_ordered_dm(const OrderedDmArgs& a, bool vec, hipStream_t st) {
  const int bn = a.f > 128 ? 256 : a.f > 64 ? 128 : 64;
  const dim3 grid(static_cast<unsigned>(ceil_div(a.n, kOrderedBM)), static_cast<unsigned>(ceil_div(a.f, bn)));
#define CDF_ORDERED_DM(BNV)                                                     \
  do {                                                                          \
    if (vec) ordered_dm_kernel<T, BNV, true><<<grid, kOrderedThreads, 0, st>>>(a); \
    else ordered_dm_kernel<T, BNV, false><<<grid, kOrderedThreads, 0, st>>>(a);    \
  } while (0)
  if (bn == 256) CDF_ORDERED_DM(256);
  else if (bn == 128) CDF_ORDERED_DM(128);
  else CDF_ORDERED_DM(64);
#undef CDF_ORDERED_DM
}

// dM [n x f] (type dt, pitch lddm) = (dH * [Zs > 0]) W^T; Zs null: no mask. Arguments checked by the caller.
void dense_dm_ordered(const float* dH, const float* Zs, const float* W, int32_t n, int32_t f, int32_t g, cdf_dtype dt,
                      void* dM, int64_t lddm, hipStream_t st) {
  ProfScope ps(K_GEMM_DM, st);
  const OrderedDmArgs a = {dH, Zs, W, dM, lddm, n, f, g};
  const bool vec = f % 4 == 0 && g % 4 == 0 && aligned(dH, 16) && aligned(Zs, 16) && aligned(W, 16);
  if (dt == CDF_F32) launch_ordered_dm<float>(a, vec, st);
  else launch_ordered_dm<bf16_t>(a, vec, st);
}

}  // namespace cdf
