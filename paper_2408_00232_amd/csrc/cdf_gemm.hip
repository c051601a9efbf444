// Dense transform of the layer and its gradients on the matrix cores (Sec. 3.1):
//   FWD : Z = M W,  H = relu(Z)                 [n x f] [f x g]
//   DM  : dM = dZ W^T,  dZ = dH * [Zs > 0]      [n x g] [g x f]
//   DW  : dW = M^T dZ                           [f x n] [n x g]   (n split into slabs)
//
// fp32 products on the bf16 matrix instructions. An fp32 value is the sum of three bf16 values exactly (each
// the rounding of what the ones before it leave: 8 + 8 + 8 significand bits), so a product of two is nine
// bf16 products; the six of them that reach 2^-24 of the result are taken (high x high, high x middle, middle
// x high, middle x middle, high x low, low x high), every one exact and accumulated in fp32. Errors against
// 64 bits are a half to a third of those of the fp32 matrix instructions this replaces, because a 32x32x16 instruction
// rounds its sum once for 16 terms (relative, 2-norm, 256x256 on 2 M rows: forward 0.9e-7 after 2.9e-7, dM 0.7e-7
// after 2.0e-7, dW 3.4e-7 after 8.3e-7).
// What bounds it: six instructions of 16 x the fp32 rate make 2.7 x the fp32 matrix rate, and the matrix pipes are
// half busy at the 1.75 GHz they then run at; the rest is memory (4.3 GB a product) and the splitting of operands in
// the vector pipe. 256x256 on 2 M rows, with fp32 instructions and now: forward 2.57 -> 1.85 ms, dM 2.66 -> 1.92, dW 2.46
// -> 1.70; 128x256 1.59 -> 1.23, 1.44 -> 1.07, 1.33 -> 1.02; 602x256 on 12 500 rows 119 -> 46 us, 98 -> 42, 86 -> 55;
// 256x41 there 22 -> 13, 23 -> 11, 30 -> 17.
//
// Tile: BM x BN outputs per block of four wavefronts (2 x 2), reduction in steps of 32. Operands are split once,
// on the way into LDS. An operand whose reduction index is contiguous in memory (M and dZ of FWD / DM, W of DM)
// is kept in blocks of eight reduction elements, a lane reads its eight with one 16-byte access; one whose reduction
// index is strided (W of FWD, M and dZ of DW) keeps its order in memory and is read with the transposing LDS
// load of gfx950 (ds_read_b64_tr_b16: the 16 lanes of a group each name 8 bytes - lane p the four columns
// 4 (p % 4) .. + 3 of row p / 4 - and lane j gets back element j % 4 of the blocks of lanes j / 4, 4 + j / 4,
// 8 + j / 4, 12 + j / 4: column j of four consecutive rows). The next k-tile is fetched into registers while
// the current one is multiplied. The ReLU mask is applied while dZ is staged, so dZ never exists in memory. dW
// partial tiles of each row slab go to the workspace and are summed in slab order by a second kernel: no
// atomics, reproducible.
//
// Infinities: a product inf x 0 of two split parts is a NaN that fp32 arithmetic would not have produced, and
// values above the largest bf16 round to one. A wavefront that finds a result that is not finite computes its
// outputs again with fp32 multiply-adds.
#include <type_traits>

#include "cdf_common.h"

namespace cdf {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));

constexpr int kGK = 32;             // reduction elements per LDS tile
constexpr int kBM = 128;            // output rows per block on large inputs (64 on small ones)

enum GemmMode { GEMM_FWD = 0, GEMM_DM = 1, GEMM_DW = 2 };

// Wavefronts along n (two along m) and, per SIMD, the wavefronts to leave registers for. FWD and DM at 128 columns: four,
// so that eight wavefronts of 64 x 32 outputs hide each other's LDS reads (256x256 on 2 M rows 1.81 ms against 1.99 with
// four of 64 x 64); dW holds two strided operands and the mask and spills at that, its wavefronts take 64 x 64 (1.66 ms).
constexpr int gemm_waves_n(int mode, int bn) { return mode == GEMM_DW ? 2 : bn / 32; }
constexpr int gemm_threads(int mode, int bn) { return 128 * gemm_waves_n(mode, bn); }
constexpr int gemm_occupancy(int mode, int bm, int bn) { return bm == 64 || (mode != GEMM_DW && bn == 128) ? 4 : 2; }

struct GemmArgs {
  // FWD: A = M (type T, ld lda), B = W           ; out0 = Z, out1 = H
  // DM : A = dH, mask = Zs (fp32, ld = g)        ; B = W ; outT = dM (type T, ld ldo)
  // DW : A = M (type T), B = dH, mask = Zs       ; out0 = partial slabs
  const void* A;
  int64_t lda;
  const float* B;
  const float* mask;  // Zs; null: no mask (FWD, or no ReLU)
  float* out0;
  float* out1;
  void* outT;
  int64_t ldo;
  int n, f, g;        // problem: n rows, f_in, f_out
  int relu;
  int slab_rows;      // DW: rows of M / dZ per slab
  int slabs;
};

// eight consecutive elements from an element-aligned address
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  const f4u a = *reinterpret_cast<const f4u*>(p), b = *reinterpret_cast<const f4u*>(p + 4);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = a[j];
    v[4 + j] = b[j];
  }
}
__device__ __forceinline__ void load8(const bf16_t* p, float (&v)[8]) {
  typedef uint32_t u4u __attribute__((ext_vector_type(4), aligned(2)));
  const u4u a = *reinterpret_cast<const u4u*>(p);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[2 * j] = __uint_as_float(a[j] << 16);
    v[2 * j + 1] = __uint_as_float(a[j] & 0xffff0000u);
  }
}
__device__ __forceinline__ float load1(const float* p) { return *p; }
__device__ __forceinline__ float load1(const bf16_t* p) { return bf2f(*p); }

// v = part[0] + part[1] + part[2] (P = 3) or part[0] (P = 1, v a bf16 value), packed in pairs
template <int P>
__device__ __forceinline__ void split8(const float (&v)[8], u32x4_t (&part)[P]) {
  float r[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = v[j];
#pragma unroll
  for (int p = 0; p < P; ++p) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{r[2 * q], r[2 * q + 1]}), bf16x2));
      part[p][q] = w;
      if (p + 1 < P) {
        r[2 * q] -= __uint_as_float(w << 16);
        r[2 * q + 1] -= __uint_as_float(w & 0xffff0000u);
      }
    }
  }
}

// LDS tile of an operand, P parts. Contiguous reduction index: [part][k / 8][row][k % 8], so that the 16-byte reads of
// consecutive lanes are consecutive (with 16 reduction elements a row half of them met in a bank: 2.5e8
// conflict cycles in dM 256x256 on 2 M rows, now 1.0e8; 602x256 on 12 500 rows 54 -> 42 us), the k-blocks 64 bytes further apart than their size so that a store of four rows' k-blocks
// uses all banks. Strided: [part][k][column], rows 16 banks apart modulo 64, so that the four rows a transposing load
// touches use disjoint banks.
template <int N, int P, bool STRIDED, int NT>
struct OperandTile {
  static constexpr int kRow = N + 32;
  static constexpr int kBlock = N * 8 + 32;
  static constexpr int kPart = STRIDED ? kGK * kRow : kGK / 8 * kBlock;
  static constexpr int kItems = N * (kGK / 8) / NT;   // eight-element items per thread
  uint16_t data[P * kPart];

  // item i of a thread: (row of the operand, first k) or (k, first column)
  static __device__ __forceinline__ int item_major(int i, int tid) {
    const int c = tid + NT * i;
    return STRIDED ? c / (N / 8) : c / (kGK / 8);
  }
  static __device__ __forceinline__ int item_minor(int i, int tid) {
    const int c = tid + NT * i;
    return (STRIDED ? c % (N / 8) : c % (kGK / 8)) * 8;
  }
  __device__ __forceinline__ void put(int i, int tid, const float (&v)[8]) {
    u32x4_t part[P];
    split8<P>(v, part);
    const int major = item_major(i, tid), minor = item_minor(i, tid);
    const int at = STRIDED ? major * kRow + minor : (minor >> 3) * kBlock + major * 8;
#pragma unroll
    for (int p = 0; p < P; ++p) *reinterpret_cast<u32x4_t*>(&data[p * kPart + at]) = part[p];
  }
  // operand of a 32x32x16 product, rows / columns base .. base + 31, reduction elements ks .. ks + 15: lane (l32, lh)
  // supplies row / column base + l32, k = ks + 8 lh .. + 7
  __device__ __forceinline__ bf16x8 get(int p, int ks, int base, int lane) const {
    if (STRIDED) {
      const int grp = lane >> 4, q = lane & 15;
      const uint16_t* at = &data[p * kPart + (ks + (grp >> 1) * 8 + (q >> 2)) * kRow + base + (grp & 1) * 16 + (q & 3) * 4];
      typedef __attribute__((address_space(3))) short4v* lds_ptr;
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at));
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + 4 * kRow));
      const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, v);
    }
    return *reinterpret_cast<const bf16x8*>(&data[p * kPart + ((ks >> 3) + (lane >> 5)) * kBlock + (base + (lane & 31)) * 8]);
  }
};

template <typename T, int MODE, int BM, int BN, bool MASK>
__global__ __launch_bounds__(gemm_threads(MODE, BN), gemm_occupancy(MODE, BM, BN)) void gemm_kernel(GemmArgs a) {
  constexpr int NT = gemm_threads(MODE, BN), WN = gemm_waves_n(MODE, BN);
  constexpr int TM = BM / 64, TN = BN / 32 / WN;   // 32 x 32 tiles per wavefront
  constexpr int PA = std::is_same<T, bf16_t>::value && MODE != GEMM_DM ? 1 : 3;
  constexpr int PB = 3;
  constexpr bool SA = MODE == GEMM_DW, SB = MODE != GEMM_DM;
  constexpr bool kMaskA = MASK && MODE == GEMM_DM, kMaskB = MASK && MODE == GEMM_DW;
  using TA = typename std::conditional<MODE == GEMM_DM, float, T>::type;
  using TileA = OperandTile<BM, PA, SA, NT>;
  using TileB = OperandTile<BN, PB, SB, NT>;
  constexpr int AI = TileA::kItems, BI = TileB::kItems;
  __shared__ __attribute__((aligned(16))) TileA As;
  __shared__ __attribute__((aligned(16))) TileB Bs;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, lh = lane >> 5;

  // Output tile and reduction range. Workgroup b runs on XCD b mod 8 (each with an L2 of its own): the column blocks
  // of one row tile (FWD, DM) and the tiles of one row slab (DW), which read the same rows, get consecutive slots
  // of one XCD.
  const int Mdim = MODE == GEMM_DW ? a.f : a.n, Ndim = MODE == GEMM_DM ? a.f : a.g;
  const int tiles_m = (Mdim + BM - 1) / BM, tiles_n = (Ndim + BN - 1) / BN;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  int tile_m, tile_n, slab = 0, Kbeg = 0, Kend = MODE == GEMM_FWD ? a.f : a.g;
  if (MODE == GEMM_DW) {
    const int t = slot % (tiles_m * tiles_n);
    slab = slot / (tiles_m * tiles_n) * 8 + xcd;
    if (slab >= a.slabs) return;
    tile_m = t % tiles_m;
    tile_n = t / tiles_m;
    Kbeg = slab * a.slab_rows;
    Kend = min(a.n, Kbeg + a.slab_rows);
  } else {
    tile_n = slot % tiles_n;
    tile_m = slot / tiles_n * 8 + xcd;
    if (tile_m >= tiles_m) return;
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const TA* Ap = static_cast<const TA*>(a.A);

  // Whole steps of the reduction are loaded from an address that is the same for the block plus an offset per item
  // that never changes; what lies past the output's edge is clamped (it feeds outputs that are never stored): rows to
  // the last one, columns of a strided operand to the last item with a column inside, which then reads up to seven
  // elements into the operand's next row. The last, partial step - and, at such an edge, the step that holds the
  // operand's last row - goes element by element, with zeros past the reduction's end. The branches are the same for
  // the block, and nothing waits for a load of a whole step before the products of the current tile have been issued
  // (the ReLU mask is applied at staging).
  float ra[AI][8], rb[BI][8], rz[kMaskA ? AI : kMaskB ? BI : 1][8];
  const int64_t lda = MODE == GEMM_DM ? a.g : a.lda;
  constexpr int kOffsetPitch = 1 << 22;   // rows up to this pitch: 32-bit offsets inside a tile
  const bool edge_a = SA && m0 + BM > Mdim, edge_b = SB && n0 + BN > Ndim;
  const bool near = lda < kOffsetPitch && a.g < kOffsetPitch && !(edge_a && lda < 8) && !(edge_b && a.g < 8);
  uint32_t offa[AI], offb[BI];   // bytes
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int major = TileA::item_major(i, tid), minor = TileA::item_minor(i, tid);
    offa[i] = static_cast<uint32_t>((SA ? major : min(major, Mdim - 1 - m0)) * static_cast<int>(near ? lda : 0) +
                                    (SA ? min(minor, (Mdim - 1 - m0) & ~7) : minor)) * sizeof(TA);
  }
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int major = TileB::item_major(i, tid), minor = TileB::item_minor(i, tid);
    offb[i] = static_cast<uint32_t>((SB ? major : min(major, Ndim - 1 - n0)) * (near ? a.g : 0) +
                                    (SB ? min(minor, (Ndim - 1 - n0) & ~7) : minor)) * 4u;
  }
  auto at = [](const auto* p, uint32_t bytes) {
    return reinterpret_cast<decltype(p)>(reinterpret_cast<const char*>(p) + bytes);
  };
  // element j of an item: (row, k + j) of a contiguous operand, (k, col + j) of a strided one
  auto load_checked = [&](const auto* base, int64_t ld, bool strided, int major, int minor, int lines, float (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = strided ? major : minor + j, line = min(strided ? minor + j : major, lines - 1);
      const int kc = min(k, Kend - 1);
      const float x = load1(base + (strided ? static_cast<int64_t>(kc) * ld + line : static_cast<int64_t>(line) * ld + kc));
      v[j] = k < Kend ? x : 0.0f;
    }
  };
  auto fetch = [&](int k0) {
    const int64_t ua = SA ? k0 * lda + m0 : m0 * lda + k0;
    const int64_t ub = SB ? static_cast<int64_t>(k0) * a.g + n0 : static_cast<int64_t>(n0) * a.g + k0;
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      load8(at(Ap + ua, offa[i]), ra[i]);
      if (kMaskA) load8(at(a.mask + ua, offa[i]), rz[kMaskA ? i : 0]);
    }
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      load8(at(a.B + ub, offb[i]), rb[i]);
      if (kMaskB) load8(at(a.mask + ub, offb[i]), rz[kMaskB ? i : 0]);
    }
  };
  auto fetch_checked = [&](int k0) {
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      const int major = (SA ? k0 : m0) + TileA::item_major(i, tid), minor = (SA ? m0 : k0) + TileA::item_minor(i, tid);
      load_checked(Ap, lda, SA, major, minor, Mdim, ra[i]);
      if (kMaskA) load_checked(a.mask, lda, SA, major, minor, Mdim, rz[kMaskA ? i : 0]);
    }
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      const int major = (SB ? k0 : n0) + TileB::item_major(i, tid), minor = (SB ? n0 : k0) + TileB::item_minor(i, tid);
      load_checked(a.B, a.g, SB, major, minor, Ndim, rb[i]);
      if (kMaskB) load_checked(a.mask, a.g, SB, major, minor, Ndim, rz[kMaskB ? i : 0]);
    }
  };
  auto stage = [&]() {
    auto masked = [](float (&v)[8], const float (&z)[8]) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = z[j] > 0.0f ? v[j] : 0.0f;
    };
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      if (kMaskA) masked(ra[i], rz[kMaskA ? i : 0]);
      As.put(i, tid, ra[i]);
    }
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      if (kMaskB) masked(rb[i], rz[kMaskB ? i : 0]);
      Bs.put(i, tid, rb[i]);
    }
  };

  // the high x high products and the rest in sums of their own: added to one sum, the small products lose their last
  // bits to its size (256x256: error 2.4e-7 instead of 0.9e-7, and 4e-6 instead of 4e-7 over the rows of a dW slab)
  f32x16 acc[TM][TN], low[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.0f;

  auto products = [&]() {
#pragma unroll
    for (int ks = 0; ks < kGK; ks += 16) {
      bf16x8 fb[PB][TN];
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[p][j] = Bs.get(p, ks, (wn * TN + j) * 32, lane);
#pragma unroll
      for (int p = 0; p < PA; ++p) {
        bf16x8 fa[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = As.get(p, ks, wm * (BM / 2) + i * 32, lane);
#pragma unroll
        for (int q = 0; q < PB - (PA == 1 ? 0 : p); ++q)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) {
              f32x16& sum = p + q > 0 ? low[i][j] : acc[i][j];
              sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[q][j], sum, 0, 0, 0);
            }
      }
    }
  };
  // whole steps first, then checked ones (an edge's items end in the next row, so the operand's last row is not theirs)
  const int Kall = MODE == GEMM_DW ? a.n : Kend;
  const int Kedge = edge_a || edge_b ? min(Kend, Kall - 1) : Kend;
  const int Kfast = near && Kedge > Kbeg ? Kbeg + (Kedge - Kbeg) / kGK * kGK : Kbeg;
  if (Kbeg < Kfast) fetch(Kbeg);
  for (int k0 = Kbeg; k0 < Kfast; k0 += kGK) {
    stage();
    __syncthreads();
    if (k0 + kGK < Kfast) fetch(k0 + kGK);
    products();
    __syncthreads();
  }
  if (Kfast < Kend) fetch_checked(Kfast);
  for (int k0 = Kfast; k0 < Kend; k0 += kGK) {
    stage();
    __syncthreads();
    if (k0 + kGK < Kend) fetch_checked(k0 + kGK);
    products();
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] += low[i][j][e];

  auto store = [&](int row, int col, float v) {
    if (MODE == GEMM_FWD) {
      const int64_t off = static_cast<int64_t>(row) * a.g + col;
      if (a.out0) a.out0[off] = v;
      if (a.out1) a.out1[off] = a.relu ? (v > 0.0f ? v : 0.0f) : v;
    } else if (MODE == GEMM_DM) {
      const float one[1] = {v};
      VecIO<T, 1>::store(static_cast<T*>(a.outT) + static_cast<int64_t>(row) * a.ldo + col, one);
    } else {
      a.out0[(static_cast<int64_t>(slab) * a.f + row) * a.g + col] = v;
    }
  };

  // ---- epilogue: lane holds column l32 and rows (e/4)*8 + lh*4 + e%4 of each 32x32 tile ----
  // A workgroup whose tile lies inside the output stores without per-element checks (one uniform branch).
  float odd = 0.0f;   // becomes a NaN if a result is infinite or NaN
  auto store_tile = [&](auto checked) {
    constexpr bool CHECK = decltype(checked)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + (wn * TN + j) * 32 + l32;
        if (CHECK && col >= Ndim) continue;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = m0 + wm * (BM / 2) + i * 32 + (e >> 2) * 8 + lh * 4 + (e & 3);
          if (CHECK && row >= Mdim) continue;
          odd = __fmaf_rn(acc[i][j][e], 0.0f, odd);
          store(row, col, acc[i][j][e]);
        }
      }
  };
  if (m0 + BM <= Mdim && n0 + BN <= Ndim) store_tile(std::false_type{});
  else store_tile(std::true_type{});

  if (__ballot(odd != odd) != 0ull) {   // this wavefront's outputs again, in fp32 arithmetic
#pragma unroll 1
    for (int t = lane; t < (BM / 2) * (TN * 32); t += 64) {
      const int row = m0 + wm * (BM / 2) + t / (TN * 32), col = n0 + wn * (TN * 32) + t % (TN * 32);
      if (row >= Mdim || col >= Ndim) continue;
      float v = 0.0f;
#pragma unroll 1
      for (int k = Kbeg; k < Kend; ++k) {
        float x, y;
        if (MODE == GEMM_FWD) {
          x = load1(Ap + static_cast<int64_t>(row) * a.lda + k);
          y = a.B[static_cast<int64_t>(k) * a.g + col];
        } else if (MODE == GEMM_DM) {
          const int64_t off = static_cast<int64_t>(row) * a.g + k;
          x = load1(Ap + off);
          if (kMaskA) x = a.mask[off] > 0.0f ? x : 0.0f;
          y = a.B[static_cast<int64_t>(col) * a.g + k];
        } else {
          const int64_t off = static_cast<int64_t>(k) * a.g + col;
          x = load1(Ap + static_cast<int64_t>(k) * a.lda + row);
          y = a.B[off];
          if (kMaskB) y = a.mask[off] > 0.0f ? y : 0.0f;
        }
        v = __fmaf_rn(x, y, v);
      }
      store(row, col, v);
    }
  }
}

// dW[i] = sum over slabs in a fixed order: 16 interleaved running sums (slab k goes to sum k mod 16), combined by
// halving. 64 outputs per block of 16 wavefronts, eight loads in flight each: bound by the partials' bytes (586 slabs
// of 100 x 256 in 26 us; four wavefronts, one load after another, took 115 us).
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(kReduceWaves * 64) void reduce_slabs_kernel(const float* __restrict__ part, int slabs,
                                                                         int64_t count, float* __restrict__ out) {
  __shared__ float sh[kReduceWaves][64];
  const int e = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 64 + e;
  const float* p = part + (i < count ? i : count - 1);
  float s = 0.0f;
  int k = g;
  for (; k + 7 * kReduceWaves < slabs; k += 8 * kReduceWaves) {
    float t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = p[(k + u * kReduceWaves) * count];
#pragma unroll
    for (int u = 0; u < 8; ++u) s = s + t[u];
  }
  for (; k < slabs; k += kReduceWaves) s = s + p[k * count];
  sh[g][e] = s;
  __syncthreads();
#pragma unroll
  for (int h = kReduceWaves / 2; h > 0; h >>= 1) {
    if (g < h) sh[g][e] = sh[g][e] + sh[g + h][e];
    __syncthreads();
  }
  if (g == 0 && i < count) out[i] = sh[0][e];
}

constexpr size_t kDwPartialCap = size_t(512) << 20;  // bytes of slab partials at most

constexpr int kDwSlab = 256;     // rows per slab at least, where the slabs fill the chip that way
constexpr int kDwMinSlab = 64;   // and otherwise (a multiple of the k-tile)

// `fine`: slabs shorter than kDwSlab where a block could otherwise not be had for every CU. A slab is a serial loop over
// its rows, 0.5 us and more per 32 of them (512 rows,
// 128x16: 15.6 -> 10.3 us in slabs of 64 rows; 12500 rows, 256x41: 17 -> 12.9 us in slabs of 128); where the chip is full, the
// partials' bytes cost more than shorter slabs save, hence the line at 256 blocks.
static void dw_split(int n, int f, int g, bool fine, int* slab_rows, int* slabs) {
  int64_t rows = kDwSlab;
  const size_t per = static_cast<size_t>(f) * g * sizeof(float);
  // enough blocks to fill the chip a few times over (tiles x slabs >= ~1500), not more
  const int64_t tiles = ceil_div(f, kBM) * ceil_div(g, g > 64 ? 128 : 64);
  // (both loops stop at one slab at the latest: rows >= n)
  while (rows < n && ceil_div(n, rows * 2) * tiles >= 1536) rows *= 2;
  while (rows < n && static_cast<size_t>(ceil_div(n, rows)) * per > kDwPartialCap) rows *= 2;
  while (fine && rows > kDwMinSlab && ceil_div(n, rows / 2) * tiles <= 256) rows /= 2;
  *slab_rows = static_cast<int>(rows);
  *slabs = static_cast<int>(ceil_div(n > 0 ? n : 1, rows));
}

// Upper bound of the slab partials for any n' <= n, f' <= f, g' <= g (so that a workspace sized
// for the largest layer serves every layer): the split keeps slabs * tiles below about 3072 and
// a tile's partial is at most 128 x 256 floats; never more than one slab per kDwMinSlab rows.
size_t dense_workspace_bytes(int64_t n, int32_t f, int32_t g) {
  const size_t tiles = static_cast<size_t>(ceil_div(f, kBM)) * static_cast<size_t>(ceil_div(g, 64));
  const size_t by_grid = (3072 + tiles) * static_cast<size_t>(kBM) * 256 * sizeof(float);
  const size_t by_rows = static_cast<size_t>(ceil_div(n > 0 ? n : 1, kDwMinSlab)) * f * g * sizeof(float);
  return align_up(by_grid < by_rows ? by_grid : by_rows, 256);
}

// Tile of the output per block. The widest columns the output fills read the row operand once (dW, whose row slabs
// make enough blocks and whose tiles split both operands, is better at 128); inputs too small to give two blocks
// to every compute unit take narrower ones, then half the rows.
template <typename T, int MODE>
static void launch_gemm(const GemmArgs& a, hipStream_t st) {
  ProfScope ps(MODE == GEMM_FWD ? K_GEMM_FWD : MODE == GEMM_DW ? K_GEMM_DW : K_GEMM_DM, st);
  const int Mdim = MODE == GEMM_DW ? a.f : a.n, Ndim = MODE == GEMM_DM ? a.f : a.g;
  int bm = kBM, bn = Ndim > 64 ? 128 : 64;
  if (std::is_same<T, bf16_t>::value) bn = 64;   // (layouts the bf16 kernels do not take)
  if (MODE != GEMM_DW) {
    while (bn > 64 && ceil_div(Mdim, bm) * ceil_div(Ndim, bn) < 512) bn /= 2;
    if (bn == 64 && ceil_div(Mdim, bm) * ceil_div(Ndim, bn) < 512 && std::is_same<T, float>::value) bm = 64;
  }
  const int64_t tiles_m = ceil_div(Mdim, bm), tiles_n = ceil_div(Ndim, bn);
  const int64_t blocks = MODE == GEMM_DW ? ceil_div(a.slabs, 8) * 8 * tiles_m * tiles_n : ceil_div(tiles_m, 8) * 8 * tiles_n;
  const unsigned grid = static_cast<unsigned>(blocks);
#define CDF_GEMM(BMV, BNV)                                                                       \
  do {                                                                                           \
    if (MODE != GEMM_FWD && a.mask) gemm_kernel<T, MODE, BMV, BNV, MODE != GEMM_FWD><<<grid, gemm_threads(MODE, BNV), 0, st>>>(a); \
    else gemm_kernel<T, MODE, BMV, BNV, false><<<grid, gemm_threads(MODE, BNV), 0, st>>>(a);                \
  } while (0)
  if constexpr (std::is_same<T, bf16_t>::value) {
    CDF_GEMM(128, 64);
  } else {
    if (bn == 128) CDF_GEMM(128, 128);
    else if (bm == 128) CDF_GEMM(128, 64);
    else CDF_GEMM(64, 64);
  }
#undef CDF_GEMM
}

// bf16 matrix-core kernels for bf16-stored activations
bool dense_fwd_bf16_ok(const void* M, int64_t ldm, int32_t f_in);
int launch_dense_fwd_bf16(const void* M, int64_t ldm, const float* W, int32_t n, int32_t f_in, int32_t f_out, int relu,
                          float* Z, float* H, void* ws, size_t ws_bytes, hipStream_t st);
bool dense_bwd_bf16_ok(const void* M, const float* W, const float* Zs, const float* dH, int32_t f_out);
int launch_dense_dm_bf16(const float* dH, const float* Zs, const float* W, int32_t n, int32_t f_in, int32_t f_out,
                         int relu, void* dM, int64_t lddm, void* ws, size_t ws_bytes, hipStream_t st);
bool dense_dw_bf16_ok(const void* M, int64_t ldm, const float* Zs, const float* dH, int32_t f_in, int32_t f_out);
int launch_dense_dw_bf16(const void* M, int64_t ldm, const float* dH, const float* Zs, int32_t n, int32_t f_in,
                         int32_t f_out, int relu, int slab_rows, int slabs, float* part, hipStream_t st);

}  // namespace cdf

using namespace cdf;

namespace cdf {
// The dense forward product with an optional workspace (the layer steps have one): with it the bf16
// path splits the weight once per call instead of once per block.
int dense_fwd_ws(const void* M, int64_t ldm, cdf_dtype dt, const float* W, int32_t n, int32_t f_in, int32_t f_out,
                 int relu, float* Z, float* H, void* ws, size_t ws_bytes, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  CDF_REQUIRE(n >= 0 && f_in > 0 && f_out > 0 && ldm >= f_in, "cdf_dense_fwd: bad shape n=%d f_in=%d f_out=%d ldm=%lld",
              n, f_in, f_out, (long long)ldm);
  if (dt != CDF_F32 && dt != CDF_BF16) CDF_FAIL(CDF_ERR_UNSUPPORTED, "cdf_dense_fwd: dtype %d", (int)dt);
  if (n == 0) return CDF_OK;
  CDF_REQUIRE(M && W && (Z || H), "cdf_dense_fwd: null pointer");
  const size_t esz = elem_bytes(dt);
  CDF_REQUIRE(aligned(M, esz) && aligned(W, 4) && aligned(Z, 4) && aligned(H, 4), "cdf_dense_fwd: misaligned pointer");
  GemmArgs a = {};
  a.A = M; a.lda = ldm; a.B = W; a.out0 = Z; a.out1 = H; a.n = n; a.f = f_in; a.g = f_out; a.relu = relu ? 1 : 0;
  if (dt == CDF_F32) launch_gemm<float, GEMM_FWD>(a, st);
  else if (dense_fwd_bf16_ok(M, ldm, f_in)) launch_dense_fwd_bf16(M, ldm, W, n, f_in, f_out, relu ? 1 : 0, Z, H, ws, ws_bytes, st);
  else launch_gemm<bf16_t, GEMM_FWD>(a, st);
  CDF_LAUNCH_CHECK("cdf_dense_fwd");
  return CDF_OK;
}
}  // namespace cdf

extern "C" int cdf_dense_fwd(const void* M, int64_t ldm, cdf_dtype dt, const float* W, int32_t n, int32_t f_in,
                             int32_t f_out, int relu, float* Z, float* H, void* stream) {
  return dense_fwd_ws(M, ldm, dt, W, n, f_in, f_out, relu, Z, H, nullptr, 0, stream);
}

namespace cdf {
void dense_dm_ordered(const float* dH, const float* Zs, const float* W, int32_t n, int32_t f, int32_t g, cdf_dtype dt,
                      void* dM, int64_t lddm, hipStream_t st);

// The body of cdf_dense_bwd; ordered_dm: fp32-instruction dM with the order of summation of cdf_ordered.hip (where
// the bf16 kernels do not take the product).
int dense_bwd_ws(const void* M, int64_t ldm, cdf_dtype dt, const float* W, const float* Zs, const float* dH, int32_t n,
                 int32_t f_in, int32_t f_out, int relu, float* dW, void* dM, int64_t lddm, bool ordered_dm, void* ws,
                 size_t ws_bytes, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  CDF_REQUIRE(n >= 0 && f_in > 0 && f_out > 0 && ldm >= f_in && (!dM || lddm >= f_in),
              "cdf_dense_bwd: bad shape n=%d f_in=%d f_out=%d ldm=%lld lddm=%lld", n, f_in, f_out, (long long)ldm,
              (long long)lddm);
  if (dt != CDF_F32 && dt != CDF_BF16) CDF_FAIL(CDF_ERR_UNSUPPORTED, "cdf_dense_bwd: dtype %d", (int)dt);
  CDF_REQUIRE(dW != nullptr, "cdf_dense_bwd: dW is null");
  CDF_REQUIRE(n == 0 || (M && W && dH && (!relu || Zs)), "cdf_dense_bwd: null pointer");
  const size_t esz = elem_bytes(dt);
  CDF_REQUIRE(aligned(M, esz) && aligned(W, 4) && aligned(Zs, 4) && aligned(dH, 4) && aligned(dW, 4) &&
                  aligned(dM, esz),
              "cdf_dense_bwd: misaligned pointer");
  int slab_rows, slabs;
  size_t need = 0;
  // a workspace for slabs of kDwSlab rows is accepted too (and bf16 activations keep those: their results are the same
  // bits whatever the workspace)
  for (int fine = dt == CDF_F32 ? 1 : 0; fine >= 0; --fine) {
    dw_split(n, f_in, f_out, fine != 0, &slab_rows, &slabs);
    need = align_up(static_cast<size_t>(slabs) * f_in * f_out * sizeof(float), 256);
    if (ws_bytes >= need) break;
  }
  if (!ws || !aligned(ws, 16) || ws_bytes < need)
    CDF_FAIL(CDF_ERR_WORKSPACE, "cdf_dense_bwd: workspace too small (%zu < %zu)", ws_bytes, need);
  float* part = static_cast<float*>(ws);
  const int64_t count = static_cast<int64_t>(f_in) * f_out;
  // bf16-stored activations: dM and (for whole 128 x 64 tiles) dW on the bf16 matrix cores, fp32 operands
  // split into a bf16 high and low part
  const bool bf16_cores = dt == CDF_BF16 && n > 0 && dense_bwd_bf16_ok(M, W, relu ? Zs : nullptr, dH, f_out);
  // dW = M^T dZ
  {
    GemmArgs a = {};
    a.A = M; a.lda = ldm; a.B = dH; a.mask = relu ? Zs : nullptr; a.out0 = part; a.n = n; a.f = f_in; a.g = f_out;
    a.relu = relu ? 1 : 0; a.slab_rows = slab_rows; a.slabs = slabs;
    if (dt == CDF_F32) launch_gemm<float, GEMM_DW>(a, st);
    else if (n > 0 && dense_dw_bf16_ok(M, ldm, relu ? Zs : nullptr, dH, f_in, f_out))
      launch_dense_dw_bf16(M, ldm, dH, relu ? Zs : nullptr, n, f_in, f_out, relu ? 1 : 0, slab_rows, slabs, part, st);
    else launch_gemm<bf16_t, GEMM_DW>(a, st);
    CDF_LAUNCH_CHECK("cdf_dense_bwd/dW");
    {
      ProfScope ps(K_GEMM_DW_REDUCE, st);
      reduce_slabs_kernel<<<static_cast<unsigned>(ceil_div(count, 64)), kReduceWaves * 64, 0, st>>>(part, slabs, count, dW);
    }
    CDF_LAUNCH_CHECK("cdf_dense_bwd/reduce");
  }
  // dM = dZ W^T
  if (dM && n > 0) {
    GemmArgs a = {};
    a.A = dH; a.lda = f_out; a.B = W; a.mask = relu ? Zs : nullptr; a.outT = dM; a.ldo = lddm; a.n = n; a.f = f_in; a.g = f_out;
    a.relu = relu ? 1 : 0;
    if (ordered_dm && !bf16_cores) dense_dm_ordered(dH, relu ? Zs : nullptr, W, n, f_in, f_out, dt, dM, lddm, st);
    else if (dt == CDF_F32) launch_gemm<float, GEMM_DM>(a, st);
    // (the workspace is free again: the slab partials of dW have been reduced on this stream)
    else if (bf16_cores) launch_dense_dm_bf16(dH, Zs, W, n, f_in, f_out, relu ? 1 : 0, dM, lddm, ws, ws_bytes, st);
    else launch_gemm<bf16_t, GEMM_DM>(a, st);
    CDF_LAUNCH_CHECK("cdf_dense_bwd/dM");
  }
  return CDF_OK;
}
}  // namespace cdf

extern "C" int cdf_dense_bwd(const void* M, int64_t ldm, cdf_dtype dt, const float* W, const float* Zs,
                             const float* dH, int32_t n, int32_t f_in, int32_t f_out, int relu, float* dW, void* dM,
                             int64_t lddm, void* ws, size_t ws_bytes, void* stream) {
  return dense_bwd_ws(M, ldm, dt, W, Zs, dH, n, f_in, f_out, relu, dW, dM, lddm, false, ws, ws_bytes, stream);
}
