// gfx950 kernels of the DID engine.
//
// One DID iteration (Alg. 3 of Gao & Chu, AAAI-18) is carried out as
//   colpass  column pass over X: E = X - B C (MFMA), f partials = sum E^2 (float64),
//            H = B^T E (MFMA), by shares of the rows where X is narrow,
//   sweep    the coordinate sweep over the rows of C (float64 MFMA chain), and C's E order,
//   packv    C's W order, V = tril(C C^T) partials of the updated C (MFMA, float64 sums); the
//            last block sums the f partials,
//   rowpass  row pass over X: E' = X - B C' (MFMA) and W = E' C'^T per column range (MFMA),
//   reduce   fixed-order sums of the W and V partials (the paper's one Allreduce),
//   bupdate  incremental update of the columns of B (the sweep's chain, a wave per 16 rows),
//            B's E order, partials of G = B^T B,
//   finish   the sum of G's partials, and B's H order.
// Every MFMA product is float32-accurate: each float32 operand is split into two fp16
// pieces under a power-of-two scale and each product is formed from three fp16 MFMAs
// (split2 and mfma_x3 below).
//
// The coordinate sweep over c_j is written in inner-product form.  With the residual
// e_j of the column at the start of the sweep and h = B^T e_j, the running inner product
// b_i^T e_j after coordinates k < i moved by delta c_k is h_i - sum_{k<i} (b_i^T b_k)
// delta c_k, so eq. up:c becomes c_ij := [c_ij + (h_i - sum_{k<i} G_ik delta c_kj) / G_ii]_+
// with G = B^T B.  This is the same identity Section 4 uses for the columns of B (the
// v_ik delta b_k term); it turns the K dependent length-M reductions of the sweep into
// one MFMA contraction plus O(K^2) float64 work per column.
//
// MFMA lane layouts used (v_mfma_f32_32x32x16_f16): lane l supplies A[l%32][8(l/32) + t]
// and B[8(l/32) + t][l%32], t = 0..7; accumulator register i of lane l holds
// D[row32(i, l/32)][l%32] with row32(i, h) = 8*(i/4) + 4*h + i%4.  Because the
// accumulator's row index pairs with l/32, accumulator registers 8q..8q+7 can be fed back
// directly (after the split) as the B operand of a second MFMA that reduces over those
// sixteen rows; no lane shuffles are needed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "did_kernels.h"

namespace didk {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int row32(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

// 16-byte unit counts of the packed operand buffers (layouts at the packing code below),
// the single definition every kernel takes its offsets and strides from.
template <int KP>
struct CqL {  // one 32-column tile of packed C
  static constexpr int E0 = (KP / 16) * 2 * 64;  // E-order units
  static constexpr int E = E0 + 8;               // ... and the tile's 32 inverse column scales
  static constexpr int W = (KP / 32) * 2 * 2 * 64;  // W-order units
  static constexpr int T = E + W;
};
template <int KP>
struct BqL {  // one 32-row chunk of packed B
  static constexpr int E = (KP / 16) * 2 * 64;      // E-order units
  static constexpr int H = (KP / 32) * 2 * 2 * 64;  // H-order units
  static constexpr int S = E + H;                   // the chunk's 32 row scales start here
  static constexpr int C = S + 8;
};
static_assert(CqL<32>::T == cq_units(32) && CqL<64>::T == cq_units(64), "packed C layout");
static_assert(CqL<32>::E == cq_units_e(32) && CqL<64>::E == cq_units_e(64), "packed C layout");
static_assert(BqL<32>::C == bq_units_chunk(32) && BqL<64>::C == bq_units_chunk(64), "packed B layout");
static_assert(BqL<32>::E == bq_units_e(32) && BqL<64>::E == bq_units_e(64), "packed B layout");

// Scaled two-way fp16 split, used for the products whose operands carry a power-of-two
// scale per row, column or tile.  For a value y whose scale group has its largest magnitude
// in [2^14, 2^15), hi = fp16(y) and lo = fp16(y - hi) (both rounded to nearest even; y - hi
// is exact in float32).  For |y| >= 2^-3 both pieces are normal fp16 numbers and
// |y - hi - lo| <= 2^-22 |y|; smaller values keep an absolute error below 2^-25 (the fp16
// subnormal spacing), 2^-40 of the group's largest magnitude.  A float32 product a*b is
// then formed from the three piece products hi*hi, hi*lo, lo*hi (each exact in float32,
// accumulated in float32 by the MFMA); the dropped lo*lo is below 2^-22 |a b|.  (A
// three-way bf16 split by truncation reaches the same accuracy with six MFMAs per product:
// bf16 keeps the float32 exponent range, but its 8-bit significand needs a third piece.)
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
struct Split2 {
  f16x8 p[2];
};

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// y - hi for the low (SEL = 0) or high (SEL = 1) fp16 half of hp, in one mixed-precision
// fma (v_fma_mix_f32 widens the fp16 operand inside the instruction).  Exact: y - hi is a
// float32 number, so this is the same value as y - (float)hi.
template <int SEL>
__device__ __forceinline__ float sub_f16(float y, f16x2 hp) {
  float r;
  const unsigned u = __builtin_bit_cast(unsigned, hp);
  if constexpr (SEL == 0)
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(u), "v"(y));
  else
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(u), "v"(y));
  return r;
}

// hi: two values per packed conversion; lo = fp16(y - hi) with y - hi formed from the
// packed hi directly, so a value costs two instructions (rather than a scalar conversion
// and its inverse, a subtraction and a share of two packings).
__device__ __forceinline__ Split2 split2(const float (&v)[8]) {
  Split2 r;
#pragma unroll
  for (int t = 0; t < 8; t += 2) {
    f16x2 hp;
    hp.x = (_Float16)v[t];
    hp.y = (_Float16)v[t + 1];
    const float l0 = sub_f16<0>(v[t], hp);
    const float l1 = sub_f16<1>(v[t + 1], hp);
    r.p[0][t] = hp.x;
    r.p[0][t + 1] = hp.y;
    r.p[1][t] = (_Float16)l0;
    r.p[1][t + 1] = (_Float16)l1;
  }
  return r;
}

// v_mfma_f32_32x32x16_f16: D(32x32, fp32) += A(32x16) B(16x32); lane l supplies
// A[l%32][8(l/32) + t] and B[8(l/32) + t][l%32] for t = 0..7 (the layout at the top).
__device__ __forceinline__ f32x16 mfma16h(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// acc += a * b as three fp16 MFMAs, smallest terms first.
__device__ __forceinline__ f32x16 mfma_x3(const f16x8 (&a)[2], const f16x8 (&b)[2], f32x16 acc) {
  acc = mfma16h(a[1], b[0], acc);
  acc = mfma16h(a[0], b[1], acc);
  acc = mfma16h(a[0], b[0], acc);
  return acc;
}

__device__ __forceinline__ f16x8 as_f16x8(f32x4 v) { return __builtin_bit_cast(f16x8, v); }
__device__ __forceinline__ f32x4 f16_as_f32x4(f16x8 v) { return __builtin_bit_cast(f32x4, v); }

// Scale exponent of a group whose largest magnitude is x: the s with x 2^s in [2^14, 2^15)
// (x = m 2^e with m in [0.5, 1), so s = 15 - e), kept within [-113, 126] so that 2^s and
// 2^-s are normal float32 numbers; 0 for an all-zero group.
__device__ __forceinline__ int scale_exp(float x) {
  if (!(x > 0.0f)) return 0;
  int e;
  (void)frexpf(x, &e);
  const int s = 15 - e;
  return s < -113 ? -113 : (s > 126 ? 126 : s);
}
__device__ __forceinline__ float pow2f(int s) { return ldexpf(1.0f, s); }

// Largest spread of scale exponents at which a group of rows of B (a 32-row chunk) or of
// columns of C (a 32-column tile) shares one scale, that of its largest member.
constexpr int kUniformSpread = 2;

// Element types of X as the passes read it: float (column-major, as given), or one of the
// two tiled storages (layout in did_kernels.h), bf16 or float32 (xtf32, a distinct type so
// that the tiled loads are selected at compile time).
struct xtf32 {
  float v;
};
// Four floats at any float's address: 16-byte loads of global memory need no more alignment than
// 4 bytes.  As-given X with M no multiple of 4 (or not aligned to 16) took 4-byte loads that touch
// 32 columns each; us per column pass, 3809 x 2248, K = 49: 32, now 25.8; one batch of 14 jobs,
// K > 32 and K <= 32: 1929, 904, now 1000, 387.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
template <typename XT>
struct x_is_tiled {
  static constexpr bool value = std::is_same<XT, __bf16>::value || std::is_same<XT, xtf32>::value;
};

// Packed C (Cq), per 32-column tile T, in 16-byte units of eight fp16 values
// (UE = KP/16 * 2 * 64 + 8):
//   E order, unit (s*2 + p)*64 + l, element t: piece p of
//       C[16s + 8(l/32) + t][j] * 2^t_j,  j = 32T + l%32
//       (B operand of E = X - BC in the column pass; A operand of E'^T in the row pass),
//       with t_j = scale_exp(max_k C[k][j]) per column;
//   units KP/16 * 2 * 64 + u, u < 8: the inverse scales 2^-t_j of the tile's 32 columns
//       (float32, column 32T + 4u + e in element e);
//   W order, unit UE + ((b*2 + q)*2 + p)*64 + l, element t: piece p of
//       C[kk][32T + row32(8q + t, l/32)] * 2^w_kk,  kk = 32b + l%32,
//       with w_kk = scale_exp(max_j C[kk][j]) per row, over all N columns
//       (A operand of W^T in the row pass; both operands of C C^T).
// Entries with kk >= K or column >= N are zero.  The E order depends only on the column, so
// it is written by the kernel that changes C (the sweep, or k_packc).  The sweep also gathers
// the row maxima into Csc[0, KP) with atomic maxima (exact, so the result does not depend on
// the order; the column pass before it clears them), and k_packv writes the W order
// afterwards, storing 2^-w_kk into Csc[KP + kk].
//
// dst[e] = src[e] for e = threadIdx.x, threadIdx.x + 256, ... < n (a block of 256 threads
// copying between global memory and LDS): each thread issues G loads before their stores,
// so that it waits for one memory round trip per G elements (a plain strided loop is
// compiled as load, wait, store).
template <int G = 16>
__device__ __forceinline__ void block_copy(float* dst, const float* src, int n) {
  int e = threadIdx.x;
  for (; e + (G - 1) * 256 < n; e += G * 256) {
    float v[G];
#pragma unroll
    for (int u = 0; u < G; ++u) v[u] = src[e + u * 256];
#pragma unroll
    for (int u = 0; u < G; ++u) dst[e + u * 256] = v[u];
  }
  for (; e < n; e += 256) dst[e] = src[e];
}

// pack_block takes the (up to) kPackTiles tiles of columns j0 .. j0 + nv - 1, whose values sit
// in LDS as Ct[j * K + kk] (j relative to j0); every thread builds whole 16-byte units, so
// the global stores are coalesced.  All threads of the block call it, after Ct is
// complete; it takes 256 ints of LDS scratch (cs) from the caller.  Two tiles a block: with
// eight, 600 x 9000 had 36 blocks (K = 40: 13.1 us, now 8.0; at 10^6 columns 85 and 105).
constexpr int kPackTiles = 2;
template <int KP>
__device__ __forceinline__ void pack_block(f32x4* __restrict__ Cq, int64_t j0, int nv, const float* Ct, int K,
                                           int64_t ntiles, int* cs) {
  constexpr int KS = KP / 16;
  constexpr int UE0 = CqL<KP>::E0;
  constexpr int UT = CqL<KP>::T;  // units per tile of the target buffer
  constexpr int GE = kPackTiles * KS * 64;  // E groups per block: (tile, s, half, jj)
  const int tid = threadIdx.x;     // cs[j]: scale exponent of column j0 + j
  const int64_t T0 = j0 >> 5;
  {
    float mx = 0.0f;
    if (tid < nv)
      for (int kk = 0; kk < K; ++kk) mx = fmaxf(mx, Ct[tid * K + kk]);
    int sc = scale_exp(mx);
    // a tile's 32 columns are 32 consecutive lanes: when the scales of its nonzero columns
    // lie within kUniformSpread of each other, every column takes the smallest, so that
    // the passes scale the tile's products with one multiplier (the tile is then flagged
    // by the sign of its first inverse scale, below)
    const bool has = tid < nv && mx > 0.0f;
    int smin = has ? sc : INT_MAX, smax = has ? sc : INT_MIN;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
      smin = min(smin, __shfl_xor(smin, off, 64));
      smax = max(smax, __shfl_xor(smax, off, 64));
    }
    if (smin <= smax && smax - smin <= kUniformSpread) sc = smin;
    cs[tid] = sc;
  }
  __syncthreads();
  for (int g = tid; g < GE; g += 256) {
    const int tb = g / (KS * 64), rem = g % (KS * 64), sh = rem >> 5, jj = rem & 31;
    const int s = sh >> 1, h = sh & 1;
    if (T0 + tb >= ntiles) continue;
    const int j = 32 * tb + jj;
    const float sc = pow2f(cs[j]);
    float v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int kk = 16 * s + 8 * h + t;
      v[t] = (j < nv && kk < K) ? Ct[j * K + kk] * sc : 0.0f;
    }
    const Split2 sp = split2(v);
    f32x4* tile = Cq + (T0 + tb) * UT;
#pragma unroll
    for (int p = 0; p < 2; ++p) tile[(s * 2 + p) * 64 + jj + 32 * h] = f16_as_f32x4(sp.p[p]);
  }
  if (tid < 8 * kPackTiles) {  // inverse scales: tile tid / 8, unit tid % 8
    const int tb = tid >> 3, u = tid & 7;
    if (T0 + tb < ntiles) {
      f32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = pow2f(-cs[32 * tb + 4 * u + e]);
      if (u == 0) {  // all 32 columns on one scale: the sign of the first flags it
        bool same = true;
        for (int j = 1; j < 32; ++j) same = same && cs[32 * tb + j] == cs[32 * tb];
        if (same) w[0] = -w[0];
      }
      Cq[(T0 + tb) * UT + UE0 + u] = w;
    }
  }
}

// Pair index q -> (a, b) with a >= b, q = a(a+1)/2 + b.
__device__ __forceinline__ void pair_of(int q, int& a, int& b) {
  int r = (int)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);
  while ((r + 1) * (r + 2) / 2 <= q) ++r;
  while (r * (r + 1) / 2 > q) --r;
  a = r;
  b = q - r * (r + 1) / 2;
}

// ------------------------------------------------------------------ initial draws
__global__ void k_fill_uniform(float* out, int64_t n, uint64_t key) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint64_t z = mix64(key + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull);
    out[i] = (float)(z >> 40) * 0x1.0p-24f;  // 24 random bits: exact in float32, [0, 1)
  }
}

hipError_t fill_uniform(float* out, int64_t n, uint64_t key, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  k_fill_uniform<<<(unsigned)blocks, 256, 0, st>>>(out, n, key);
  return hipGetLastError();
}

__global__ void k_scale(float* p, int64_t n, float a) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] *= a;
}

hipError_t scale(float* p, int64_t n, float a, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  k_scale<<<(unsigned)blocks, 256, 0, st>>>(p, n, a);
  return hipGetLastError();
}

// Keeps the loads before it ahead of those after it (X is not __restrict__ in the passes: the
// loads of memory known not to change would move across).
__device__ __forceinline__ void load_order() { asm volatile("" ::: "memory"); }

// threadIdx.x, anew for each item of a grouped kernel: what follows from it (lane addresses in
// LDS and the like) would otherwise be computed ahead of the loop over the items and held in
// registers beside the item's own (grouped column pass, K > 32: 240 VGPRs, now 160; W-order
// packing 256 and spills, now 220; us in one batch of 24 jobs 479, 462, and, K <= 32, 33.9, 24.5).
__device__ __forceinline__ int item_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// ------------------------------------------------------------------ tiled storage of X
// Both tiled copies of X (layout in did_kernels.h), elements of type ET (bf16 rounded to
// nearest even, or float32), zero outside M x N; and the check of its entries: flag |= 1 if
// any is negative, NaN or infinite.
//
// Bound by memory: X is read once and two copies written.  A wave takes a 32 x 32 tile, its
// lanes consecutive rows, which gives the row-pass copy's units as they are; the column-pass
// copy's come from the transpose through LDS, whose rows are 40 floats apart (16-byte aligned,
// and without bank conflicts both ways).  A block's waves take neighbouring chunks of one column
// tile, 512 bytes of each column.  Times: 5000 x 10^6 12.2 ms (4.9 TB/s read and written), bf16
// 5000 x 62500 0.58 ms, the 12 jobs of a serving run (2.5 GB of X, most of odd M) 1.63 ms; with a
// thread per output unit, whose row-pass half gathered 4 bytes at a time, and the check in a pass
// of its own 28.5, 1.75, 3.63 ms; with lanes along the columns, 16 bytes each where M and the
// alignment allow, 12.9, 0.61 ms, and 2.48 ms where they do not.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bool x_entry_ok(float v) { return v >= 0.0f && v <= 3.4028234663852886e38f; }

template <typename ET>
__global__ __launch_bounds__(256) void k_tile_x(const float* __restrict__ src, int64_t M, int64_t N, int64_t nchunks,
                                                int64_t ntiles, ET* __restrict__ xc, ET* __restrict__ xr, int* flag) {
  constexpr int E = 16 / (int)sizeof(ET);  // values per unit
  constexpr int Q = 16 / E;               // units per lane
  constexpr int P = 40;                   // row pitch of the transpose
  __shared__ __align__(16) float sh[4][32 * P];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, h = l >> 5, r = l & 31;
  float* const tr = sh[wave];
  auto put = [&](ET* tile, const float (&v)[16]) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      ET o[E];
#pragma unroll
      for (int t = 0; t < E; ++t) o[t] = (ET)v[E * q + t];
      *reinterpret_cast<u32x4*>(tile + (q * 64 + l) * E) = __builtin_bit_cast(u32x4, o);
    }
  };
  bool ok = true;
  for (int64_t T = blockIdx.x; T < ntiles; T += gridDim.x) {
    for (int64_t c = (int64_t)blockIdx.y * 4 + wave; c < nchunks; c += 4 * (int64_t)gridDim.y) {
      const int64_t m = c * 32 + r, j = T * 32 + 4 * h;
      float v[16];  // v[4 q + e]: row m of column j + 8 q + e
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int64_t ji = j + 8 * (i >> 2) + (i & 3);
        v[i] = (ji < N && m < M) ? src[ji * M + m] : 0.0f;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) ok = ok && x_entry_ok(v[i]);
      put(xr + (c * ntiles + T) * 1024, v);
#pragma unroll
      for (int i = 0; i < 16; ++i) tr[(8 * (i >> 2) + 4 * h + (i & 3)) * P + r] = v[i];
      load_order();  // the wave's own LDS rows: its accesses run in order, the compiler keeps them so
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(tr + r * P + 8 * q + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * q + e] = x[e];
      }
      load_order();
      __builtin_amdgcn_wave_barrier();
      put(xc + (T * nchunks + c) * 1024, v);
    }
  }
  if (!ok) atomicOr(flag, 1);
}

// A block per column tile, and several where those are fewer than the GPU holds (8 a CU).
hipError_t tile_x(const Shape& s, const float* src, void* xc, void* xr, int* flag, hipStream_t st) {
  const int64_t nt = n_tiles(s), gx = std::min<int64_t>(nt, 1 << 20);
  const int64_t gy = std::max<int64_t>(1, std::min<int64_t>((s.nchunks + 3) / 4, 4096 / gx));
  const dim3 g((unsigned)gx, (unsigned)gy);
  if (s.xbf16)
    k_tile_x<__bf16><<<g, 256, 0, st>>>(src, s.M, s.N, s.nchunks, nt, static_cast<__bf16*>(xc),
                                        static_cast<__bf16*>(xr), flag);
  else
    k_tile_x<float><<<g, 256, 0, st>>>(src, s.M, s.N, s.nchunks, nt, static_cast<float*>(xc), static_cast<float*>(xr),
                                       flag);
  return hipGetLastError();
}

// The 16 values of one lane's accumulator tile from a tiled copy of X.
__device__ __forceinline__ f32x16 ld_tile(const __bf16* tile, int l) {
  f32x16 v;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(tile + (q * 64 + l) * 8);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[8 * q + 2 * k] = __builtin_bit_cast(float, w[k] << 16);
      v[8 * q + 2 * k + 1] = __builtin_bit_cast(float, w[k] & 0xffff0000u);
    }
  }
  return v;
}
__device__ __forceinline__ f32x16 ld_tile(const xtf32* tile, int l) {
  f32x16 v;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 w = *reinterpret_cast<const f32x4*>(tile + (q * 64 + l) * 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[4 * q + k] = w[k];
  }
  return v;
}

// ------------------------------------------------------------------ validation
// flag |= 1 if any entry is negative, NaN or infinite (X must lie in R_+^{M x N}).
__global__ void k_validate(const float* p, int64_t n, int vec4, int* flag) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  if (vec4) {
    const int64_t n4 = n / 4;
    const f32x4* p4 = reinterpret_cast<const f32x4*>(p);
    for (int64_t i = t0; i < n4; i += stride) {
      const f32x4 v = p4[i];
      for (int u = 0; u < 4; ++u) bad |= !x_entry_ok(v[u]);
    }
    for (int64_t i = 4 * n4 + t0; i < n; i += stride) bad |= !x_entry_ok(p[i]);
  } else {
    for (int64_t i = t0; i < n; i += stride) bad |= !x_entry_ok(p[i]);
  }
  if (bad) atomicOr(flag, 1);
}

hipError_t validate(const float* p, int64_t n, int vec4, int* flag, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n / (vec4 ? 4 : 1) + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 16384) blocks = 16384;
  k_validate<<<(unsigned)blocks, 256, 0, st>>>(p, n, vec4, flag);
  return hipGetLastError();
}

// ------------------------------------------------------------------ B update + packing
// Packed operand buffer of B (rows >= M and columns >= K stay zero from allocation).  A
// 16-byte unit holds the eight fp16 values lane l feeds to one MFMA; chunk c's units form
// one contiguous run of UC = 2 * UE + 8 units (UE = KP/16 * 2 * 64):
//   unit c*UC + (s*2 + p)*64 + l, element t: piece p of -B[m][16s + 8(l/32) + t] * 2^s_m,
//       m = 32c + l%32, with s_m = scale_exp(max_k B[m][k])  (A operand of E = X - B C in
//       the column pass; B operand of E'^T in the row pass);
//   unit c*UC + UE + ((b*2 + q)*2 + p)*64 + l, element t: piece p of
//       B[32c + row32(8q + t, l/32)][kk] * 2^u_kk, kk = 32b + l%32, with
//       u_kk = scale_exp(max_m B[m][kk])   (A operand of H = B^T E);
//   units c*UC + 2*UE + u, u < 8: 2^-s_m of rows m = 32c + 4u + e (float32, element e).
// The per-row part is written by the B update; the per-column part
// needs the column maxima over all rows, which the B update gathers into Bsc[0, KP) with
// atomic maxima (exact, so the result does not depend on the order), and is written by
// k_finish_b afterwards, which also stores 2^-u_kk into Bsc[KP + kk].
constexpr int kBupRows = 64;  // rows of B per block of the update

// H-order units of the two chunks 2*bid, 2*bid + 1 from B and the column maxima in
// Bsc[0, KP); block 0 also stores 2^-u_kk into Bsc[KP + kk].  256 threads.
template <int KP>
__device__ __forceinline__ void packh_body(const float* __restrict__ B, int64_t M, int K, int64_t nchunks,
                                           _Float16* __restrict__ Bq, float* __restrict__ Bsc, int64_t bid) {
  constexpr int NB = KP / 32;
  constexpr int UE = BqL<KP>::E;
  constexpr int64_t UC = BqL<KP>::C;
  constexpr int GC = NB * 2 * 64;  // groups (b, q, lane) per chunk
  __shared__ float us[KP];
  const int tid = threadIdx.x;
  if (tid < KP) {
    const int u = tid < K ? scale_exp(Bsc[tid]) : 0;
    us[tid] = pow2f(u);
    if (bid == 0) Bsc[KP + tid] = pow2f(-u);
  }
  __syncthreads();
  for (int g = tid; g < 2 * GC; g += 256) {
    const int64_t c = 2 * bid + g / GC;
    if (c >= nchunks) continue;
    const int rem = g % GC, bq = rem >> 6, l = rem & 63;
    const int b = bq >> 1, q = bq & 1, h = l >> 5;
    const int kk = 32 * b + (l & 31);
    const float sc = us[kk];
    float v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int64_t m = 32 * c + row32(8 * q + t, h);
      v[t] = (m < M && kk < K) ? B[(int64_t)kk * M + m] * sc : 0.0f;
    }
    const Split2 sp = split2(v);
    f32x4* u = reinterpret_cast<f32x4*>(Bq) + c * UC + UE + (int64_t)(bq * 2) * 64 + l;
    u[0] = f16_as_f32x4(sp.p[0]);
    u[64] = f16_as_f32x4(sp.p[1]);
  }
}

// The buffers that an allocation-free call finds as the last one left them: the packed
// operands, scales, V and W are cleared, the column ranges written and the iteration counter
// reset, by fill kernels' stores (no memset node, so that the call can be captured).  One launch
// instead of eight, each bound by its own latency (600 x 9000, K = 40: 19 us and 7 gaps, now
// 6.7); the last block's one thread writes the ranges beside the others' fills.
struct ZeroSpans {
  f32x4* p[6];
  int64_t n[6];  // 16-byte units
};

__global__ __launch_bounds__(256) void k_static_setup(ZeroSpans z, int64_t* tb, int64_t T, int64_t P, int64_t S,
                                                      int64_t* tdev) {
  if (blockIdx.x == gridDim.x - 1) {
    if (threadIdx.x == 0) {
      (void)range_bounds(T, P, S, tb);
      *tdev = 0;
    }
    return;
  }
  const int64_t stride = (int64_t)(gridDim.x - 1) * 256;
#pragma unroll
  for (int q = 0; q < 6; ++q)
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < z.n[q]; i += stride) z.p[q][i] = f32x4{0, 0, 0, 0};
}

hipError_t static_setup(const Shape& s, void* Bq, void* Cq, float* Bsc, float* Csc, double* V, double* W, int64_t* tb,
                        int64_t T, int64_t P, int64_t S, int64_t* tdev, hipStream_t st) {
  const int64_t bytes[6] = {packed_b_elems(s) * 2,        cq_bytes(s), bsc_floats(s.KP) * 4, bsc_floats(s.KP) * 4,
                            (int64_t)s.KP * s.KP * 8, (int64_t)s.KP * s.Mpad * 8};
  void* const p[6] = {Bq, Cq, Bsc, Csc, V, W};
  ZeroSpans z;
  int64_t most = 0;
  for (int q = 0; q < 6; ++q) {
    z.p[q] = static_cast<f32x4*>(p[q]);
    z.n[q] = bytes[q] / 16;
    most = std::max(most, z.n[q]);
  }
  const int64_t blocks = std::min<int64_t>((most + 255) / 256, 2048);
  k_static_setup<<<(unsigned)(blocks + 1), 256, 0, st>>>(z, tb, T, P, S, tdev);
  return hipGetLastError();
}

__global__ void k_zero_f32(float* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0.0f;
}

// ------------------------------------------------------------------ column pass
// Block = WPB waves (4 or 8) = 32 WPB consecutive columns, a 32-column tile each, and one of
// csplit shares of the rows, which every wave walks in 32-row chunks:
//   P    = (-B[chunk, :] 2^s) (C[:, cols] 2^t)     (KP/16 scaled fp16 steps)
//   acc  = X[chunk, cols] + P 2^-(s_m + t_j)        (one fma per entry) -> E = X - B C
//   fsum += sum acc^2                               (float64)
//   H   += (B[chunk, :] 2^u)^T (acc 2^v)            (2 scaled fp16 steps per 32 rows of H)
// Every float32 product is formed by three fp16 MFMAs over scaled two-way splits (split2).
// The operands of P carry one power-of-two scale per row of B and per column of C, fixed
// when they are packed; those of H one per column of B (packed) and one per column of E,
// v_j, chosen per chunk from the chunk's largest |E| in the column and never raised: when
// it drops, the running H of the column is rescaled (exactly, by a power of two) before the
// chunk is added.  Powers of two commute with rounding, so the scales change no result
// beyond the splits themselves.  The packed B run of chunk c+1 is staged into LDS (double
// buffer shared by the four waves) and the X tile of chunk c+1 is loaded into registers
// while chunk c is computed.  H is written per 32-column tile, K rounded up to a multiple
// of 4 rows of 32 floats each (what a wave of the sweep reads is then contiguous).
//
// RW (the carried-residual form): the E-order operand and the row scales of each chunk
// come from BqE (delta B in a carried iteration, B in a refresh iteration) while the
// H-order operand comes from Bq, and E is stored to the column-major float32 residual
// Rout (rvec4: 16-byte stores are aligned), so that the row pass can carry it on.  The
// source X is then either the data (refresh) or Rout itself (carry: E = R - delta B C).
//
// The B run goes from global memory straight into LDS (16 bytes a lane, no staging registers).
// The chunk's closing barrier must wait for it, but not for the X tile of the next chunk, whose
// loads are issued after it: stage_barrier leaves the last NX loads (those of the X tile) in
// flight (X in tile order; X as given, whose edge tiles issue other numbers of loads, is waited
// for).  With __syncthreads, which waits for every load, each chunk waited
// out the X tile's latency.
// us per column pass before and after: 5000 x 10^6, K = 50, tiled float32: 4922, 4474 (and three
// waves per SIMD, the staging registers gone); bf16 5000 x 62500: 286, 271; 24 jobs in a batch, K
// <= 32: 398, 356.
//
// What bounds it now: large float32 X in tile order, memory (5000 x 10^6, K = 50: 22 GB counted
// at 4.9 to 5.0 TB/s, 12 jobs of a serving run, K <= 32, 4.75 TB/s of X; a large copy reaches 4.75);
// K > 32 with X in bf16, the matrix units and the clock they leave (24 MFMAs per chunk and wave:
// busy 46 % of the cycles at 1.9 GHz; at 5000 x 10^6 58 % at 1.43 GHz); small X, latency.
template <typename XT>
struct x_loads {  // loads of one X tile per lane where their number is fixed, else 0
  static constexpr int value = std::is_same<XT, xtf32>::value ? 4 : (std::is_same<XT, __bf16>::value ? 2 : 0);
};
// s_waitcnt with vmcnt(NX) and lgkmcnt(0) (the builtin, so that the compiler's own waits count
// it), then the barrier.  tests/test_stage_waits.py and tests/test_stage_waits_all.py check the
// generated code: NX loads, and no others, lie between the staging and each of these waits.
template <int NX>
__device__ __forceinline__ void stage_barrier() {
  load_order();
  __builtin_amdgcn_s_waitcnt(NX | 0x70);
  __builtin_amdgcn_s_barrier();
  load_order();
}

// U units (16 bytes each) to LDS at dst by a block of 64 WPB threads, 64 units per load; src(u)
// is the address of unit u.  RUNS: the 64 units of a load are one contiguous run, which a
// buffer load takes from its (wave-uniform) first unit.  Otherwise (the carried form, whose
// units come from two buffers) each lane gives its own address to a global_load_lds, which the
// compiler takes for a flat access, after which it waits for all loads at every use of one.
template <int U, int WPB, bool RUNS, class Src>
__device__ __forceinline__ void stage_units(f32x4* dst, int wave, int l, Src src) {
  auto put = [&](int u0, int n) {
    const auto to = (__attribute__((address_space(3))) void*)&dst[u0];
    if constexpr (RUNS)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          __builtin_amdgcn_make_buffer_rsrc((void*)src(u0), 0, 16 * n, 0x00020000), to, 16, 16 * l, 0, 0, 0);
    else
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src(u0 + l), to, 16, 0, 0);
  };
  constexpr int FULL = U / (64 * WPB);
#pragma unroll
  for (int v = 0; v < FULL; ++v) put(64 * (WPB * v + wave), 64);
  constexpr int REST = U - FULL * 64 * WPB;  // by the first waves
  if (64 * wave < REST) {
    const int n = REST - 64 * wave < 64 ? REST - 64 * wave : 64;
    if (l < n) put(FULL * 64 * WPB + 64 * wave, n);
  }
}

template <int KP, bool WITH_H, typename XT, bool RW = false, int WPB = 4>
__device__ __forceinline__ void colpass_body(const XT* X, int64_t M, int64_t N, int K,
                                             const f32x4* __restrict__ Cq, const _Float16* __restrict__ Bq,
                                             float* Bsc, float* __restrict__ Csc, float* __restrict__ Hout,
                                             double* __restrict__ fpart, int64_t nchunks, int csplit,
                                             int64_t bid, const _Float16* __restrict__ BqE = nullptr,
                                             float* Rout = nullptr, int rvec4 = 0) {
  constexpr int NB = KP / 32;
  constexpr int KS = KP / 16;
  constexpr int UE = BqL<KP>::E;      // 16-byte units of the E operand per chunk
  constexpr int US = BqL<KP>::S;      // the chunk's 32 row scales
  constexpr int U = BqL<KP>::C;       // the chunk's whole run
  constexpr int UCT = CqL<KP>::T;     // units per packed C tile
  constexpr int UCE0 = CqL<KP>::E0;   // the tile's inverse column scales
  __shared__ f32x4 sb0[U], sb1[U];  // the two stages of B
  __shared__ double fw[WPB];
  // the wave index is uniform: from a scalar register, so that wave-based addresses stay scalar
  const int tid = KP > 32 ? item_tid() : threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, half = l >> 5,
            lc = l & 31;
  // block bid: share bid / ncb of the rows (chunks c0 .. c1 - 1) of column block bid % ncb
  const int64_t ncb = (N + 32 * WPB - 1) / (32 * WPB), share = bid / ncb;
  const int64_t c0 = nchunks * share / csplit, c1 = nchunks * (share + 1) / csplit;
  const int64_t T = (bid - share * ncb) * WPB + wave;  // this wave's 32-column tile
  const int64_t j0 = T * 32;
  const int64_t col = j0 + lc;
  const bool colok = col < N;
  const bool tileok = j0 < N;
  // X of this tile from a wave-uniform base plus a 32-bit lane offset
  const XT* xtile = X + (tileok ? j0 : 0) * M;
  const uint32_t loff = (uint32_t)(lc * M + 4 * half);

  // the maxima that this iteration's sweep and B update gather start from zero
  if (WITH_H && bid == 0 && tid < KP) Csc[tid] = Bsc[tid] = 0.0f;
  f16x8 cP[KS][2];  // pieces of C[16s + 8*half + t][col] 2^t_col, from the packed tile
  float ct = 1.0f;  // 2^-t_col
  if (tileok) {
    const f32x4* ctile = Cq + T * UCT;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int p = 0; p < 2; ++p) cP[s][p] = as_f16x8(ctile[(s * 2 + p) * 64 + l]);
    ct = fabsf(reinterpret_cast<const float*>(ctile + UCE0)[lc]);  // column 0's may carry the tile's flag
  } else {
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int p = 0; p < 2; ++p) cP[s][p] = as_f16x8(f32x4{0, 0, 0, 0});
  }
  f32x16 H[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) H[b][i] = 0.0f;
  int vcur = 126;  // current scale exponent of this column's E operand (never raised)
  double fs0 = 0.0, fs1 = 0.0;

  constexpr int NX = RW ? 0 : x_loads<XT>::value;
  auto cdma = [&](int64_t c, int buf) {
    stage_units<U, WPB, !RW>(buf ? sb1 : sb0, wave, l, [&](int u) {
      const _Float16* base = Bq;
      if constexpr (RW) base = (u < UE || u >= US) ? BqE : Bq;
      return reinterpret_cast<const f32x4*>(base) + c * U + u;
    });
    load_order();
  };
  // the residual store of the carried form: the accumulator layout of E, column-major
  float* const rtile = RW ? Rout + (tileok ? j0 : 0) * M : nullptr;
  const uint32_t roff = (uint32_t)(lc * M + 4 * half);
  const bool rfull = RW && rvec4 && tileok && (j0 + 32 <= N);  // wave-uniform
  auto rstore = [&](int64_t c, const f32x16& e) {
    const int64_t m0 = c * 32;
    if (rfull && m0 + 32 <= M) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(rtile + m0 + 8 * q + roff) = f32x4{e[4 * q], e[4 * q + 1], e[4 * q + 2], e[4 * q + 3]};
    } else if (tileok) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int64_t r = m0 + 8 * q + 4 * half + t;
          if (colok && r < M) rtile[(int64_t)lc * M + r] = e[4 * q + t];
        }
    }
  };
  const bool tilefull = j0 + 32 <= N;  // wave-uniform
  auto xload = [&](int64_t c) {
    f32x16 v;
    if constexpr (x_is_tiled<XT>::value) {  // tiled copy XC
      // A wave past the last tile reads tile 0, in bounds (no branch in the chunk loop);
      // its f partial is dropped and it stores no H.
      return ld_tile(X + ((tileok ? T : 0) * nchunks + c) * 1024, l);
    } else {  // column-major float32 X
      const int64_t m0 = c * 32;
      if (tilefull && m0 + 32 <= M) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float* xb = xtile + m0 + 8 * q;  // wave-uniform base, 32-bit lane offset
          const f32x4_any t = *reinterpret_cast<const f32x4_any*>(xb + loff);
          v[4 * q + 0] = t[0];
          v[4 * q + 1] = t[1];
          v[4 * q + 2] = t[2];
          v[4 * q + 3] = t[3];
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int64_t r = m0 + 8 * q + 4 * half + e;
            v[4 * q + e] = (colok && r < M) ? xtile[(int64_t)lc * M + r] : 0.0f;
          }
      }
      return v;
    }
  };

  // One chunk: compute chunk c from the X tile in xc (loaded one chunk earlier) and the
  // staged B operands in LDS buffer buf (a constant where step is called); meanwhile stage chunk c+1's B operands and load
  // its X tile into xn (the two tiles alternate roles from one chunk to the next, so
  // nothing is copied).
  auto step = [&](int64_t c, int buf, const f32x16& xc, f32x16& xn) {
    const int64_t cn = c + 1 < c1 ? c + 1 : c;
    cdma(cn, buf ^ 1);
    xn = xload(cn);
    load_order();
    // E of the chunk, a value of its own (not written over the X tile, which would make the
    // two alternating tiles cost a copy per chunk)
    f32x16 acc;
    {  // E = X - B C: KS steps of three MFMAs, operands of step s+1 read from LDS during step s
      const f32x4* ue = (buf ? sb1 : sb0) + l;
      f16x8 a[2], an[2];
      f32x16 P;
#pragma unroll
      for (int i = 0; i < 16; ++i) P[i] = 0.0f;
#pragma unroll
      for (int p = 0; p < 2; ++p) a[p] = as_f16x8(ue[p * 64]);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) {
#pragma unroll
          for (int p = 0; p < 2; ++p) an[p] = as_f16x8(ue[((s + 1) * 2 + p) * 64]);
        }
        P = mfma_x3(a, cP[s], P);
        if (s + 1 < KS) {
#pragma unroll
          for (int p = 0; p < 2; ++p) a[p] = an[p];
        }
      }
      // rows row32(4q + e, half) = 8q + 4 half + e: their inverse scales are unit 2q + half.
      // A negative first scale flags a chunk whose rows share one scale (the B update):
      // one multiplier for the whole tile.
      const f32x4* rs = (buf ? sb1 : sb0) + US;
      const float s0 =
          __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, rs[0][0])));
      if (s0 < 0.0f) {
        const float mu = -s0 * ct;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = fmaf(P[i], mu, xc[i]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 r4 = rs[2 * q + half];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[4 * q + e] = fmaf(P[4 * q + e], r4[e] * ct, xc[4 * q + e]);
        }
      }
    }
    if constexpr (RW) rstore(c, acc);
    {  // sum of squares of this 32x32 tile in float32, accumulated across tiles in float64
      float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        a0 += acc[i] * acc[i];
        a1 += acc[i + 1] * acc[i + 1];
      }
      if (c & 1) fs1 += (double)(a0 + a1);
      else fs0 += (double)(a0 + a1);
    }
    if (WITH_H) {
      // scale of this chunk's E operand: the largest |E| of the column over the chunk (the
      // lane and its partner l ^ 32 hold the column's 32 rows)
      float em = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) em = fmaxf(em, fabsf(acc[i]));
      em = fmaxf(em, __shfl_xor(em, 32, 64));
      int v = scale_exp(em);
      v = (em > 0.0f && v < vcur) ? v : vcur;
      if (__ballot(v != vcur)) {  // wave-uniform: rescale only when some column's scale drops
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i) H[b][i] = ldexpf(H[b][i], v - vcur);
        vcur = v;
      }
      const f32x4* uh = (buf ? sb1 : sb0) + UE + l;
      f16x8 h[2], hn[2];
      f16x8 eP[2][2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float y[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) y[t] = ldexpf(acc[8 * q + t], v);
        const Split2 sp = split2(y);
#pragma unroll
        for (int p = 0; p < 2; ++p) eP[q][p] = sp.p[p];
      }
      // accumulators alternate: (b, q) = (0, 0), (1, 0), ..., (0, 1), (1, 1), ...; each H[b]
      // still takes q = 0 before q = 1
      auto hunit = [&](int gg) { return ((gg % NB) * 2 + gg / NB) * 2; };
#pragma unroll
      for (int p = 0; p < 2; ++p) h[p] = as_f16x8(uh[(hunit(0) + p) * 64]);
#pragma unroll
      for (int gg = 0; gg < NB * 2; ++gg) {
        if (gg + 1 < NB * 2) {
#pragma unroll
          for (int p = 0; p < 2; ++p) hn[p] = as_f16x8(uh[(hunit(gg + 1) + p) * 64]);
        }
        H[gg % NB] = mfma_x3(h, eP[gg / NB], H[gg % NB]);
        if (gg + 1 < NB * 2) {
#pragma unroll
          for (int p = 0; p < 2; ++p) h[p] = hn[p];
        }
      }
    }
    stage_barrier<NX>();
  };

  f32x16 x0 = xload(c0);
  cdma(c0, 0);
  stage_barrier<0>();
  f32x16 x1;
  for (int64_t c = c0; c < c1; c += 2) {
    step(c, 0, x0, x1);
    if (c + 1 < c1) step(c + 1, 1, x1, x0);
  }

  if (WITH_H && tileok) {  // the tile's rows of H, 32 columns each (zeros past K and N)
    const float* ku = Bsc + KP;  // 2^-u_kk
    const int K4 = (K + 3) / 4 * 4;
    float* ht = Hout + share * h_stride(N, K) + T * (K4 * 32) + lc;
    // The scales are loaded together, 16 at a time (32 cost the as-given row pass a wave per
    // SIMD): under the stores' condition each load would be waited for by itself, 16 NB round
    // trips in turn.  us per column and row pass: 600 x 9000, K = 40: 21.2, 17.7, now 20.3,
    // 16.4; 1868 x 40000, K = 60: 96.8, 82.7, now 89.8, 81.6; 24 jobs in one batch, K > 32:
    // 491, 469, now 480, 448.
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float kv[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) kv[i] = ku[32 * b + row32(i, half)];
      load_order();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int kk = 32 * b + row32(i, half);
        if (kk < K4) ht[kk * 32] = ldexpf(H[b][i], -vcur) * kv[i];
      }
    }
  }

  double fsum = fs0 + fs1;
  if (!tileok) fsum = 0.0;  // a wave past the last tile
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) fsum += __shfl_xor(fsum, off, 64);
  if (l == 0) fw[wave] = fsum;
  __syncthreads();
  if (tid == 0) {  // the block's waves in a fixed pairwise order
    double w4[2];
#pragma unroll
    for (int h = 0; h < WPB / 4; ++h) w4[h] = (fw[4 * h] + fw[4 * h + 1]) + (fw[4 * h + 2] + fw[4 * h + 3]);
    fpart[bid] = WPB == 8 ? w4[0] + w4[1] : w4[0];
  }
}

template <int KP, bool WITH_H, typename XT, int WPB>
__global__ __launch_bounds__(64 * WPB, 8 / WPB) void k_colpass(const XT* X, int64_t M, int64_t N, int K,
                                                               const f32x4* __restrict__ Cq,
                                                               const _Float16* __restrict__ Bq,
                                                               float* Bsc, float* __restrict__ Csc,
                                                               float* __restrict__ Hout, double* __restrict__ fpart,
                                                               int64_t nchunks, int csplit) {
  colpass_body<KP, WITH_H, XT, false, WPB>(X, M, N, K, Cq, Bq, Bsc, Csc, Hout, fpart, nchunks, csplit, blockIdx.x);
}

// The carried-residual form of the column pass (always forms H).
template <int KP, typename XT>
__global__ __launch_bounds__(256, 2) void k_colpass_rw(const XT* X, int64_t M, int64_t N, int K,
                                                       const f32x4* __restrict__ Cq, const _Float16* __restrict__ Bq,
                                                       const _Float16* __restrict__ BqE,
                                                       float* Bsc, float* __restrict__ Csc, float* __restrict__ Hout,
                                                       double* __restrict__ fpart, int64_t nchunks, int csplit,
                                                       float* R, int rvec4) {
  colpass_body<KP, true, XT, true>(X, M, N, K, Cq, Bq, Bsc, Csc, Hout, fpart, nchunks, csplit, blockIdx.x, BqE, R,
                                   rvec4);
}

int64_t colpass_blocks(const Shape& s) {
  const int64_t cols = 32 * (int64_t)(s.cwpb == 8 ? 8 : 4);
  return (s.N + cols - 1) / cols * s.csplit;
}

// Row shares of the column pass.  A block walks its rows chunk by chunk, so a narrow X leaves
// most of the GPU idle (N = 575: 5 blocks), and one a little past two blocks per CU pays for
// the CUs that run three (N = 70000: 547 blocks).  Each share costs a prologue and a partial of H
// (about 3 chunks' time) and its reading by the sweep; the smallest estimate over shares of at
// least 4 chunks is taken, within max_split (the caller's scratch).  us per column pass (with its
// event) at one share and as chosen: 10304 x 575, K = 25: 467, 29.7; 3809 x 2248, K = 49: 210,
// 27.2; 500 x 2000, K = 10: 26.2, 11.7; 600 x 9000, K = 40: 44.6, 21.7; as given 784 x 70000, K =
// 16: 75.4, 60.9; 1868 x 40000, K = 60: 124, 108; in tile order 56.5, 55.1 and 93, 95.
//
// `resident` counts two blocks per CU.  A CU holds three of the present kernels, or four (K <= 32
// in tile order), but a third beside two takes time, not only room: with 768 in its place 784 x
// 70000 as given is left whole (75.1), while 1868 x 40000 takes two shares for three (as given 107,
// in tile order 84); the other shapes above choose the same.
int column_split(const Shape& s, int64_t max_split) {
  const int64_t nb = (s.N + 127) / 128, resident = 512;
  const int64_t most = std::min<int64_t>(std::min<int64_t>(max_split, s.nchunks / 4), 64);
  int best = 1;
  const double share = 0.5 + (double)s.N * s.K / 1.05e6;
  double cost = 0.0;
  for (int64_t p = 1; p <= std::max<int64_t>(most, 1); ++p) {
    const double rounds = (double)((nb * p + resident - 1) / resident);
    const double t = rounds * ((double)((s.nchunks + p - 1) / p) + 3.0) + share * (double)p;
    if (p == 1 || t < cost) {
      best = (int)p;
      cost = t;
    }
  }
  return best;
}

template <typename XT, int WPB>
static void colpass_launch_w(const Shape& s, const XT* X, const f32x4* C, const _Float16* Bq, float* Bsc, float* Csc,
                             float* Hout, double* fpart, int with_h, hipStream_t st) {
  const unsigned g = (unsigned)colpass_blocks(s);
  if (s.KP == 32) {
    if (with_h)
      k_colpass<32, true, XT, WPB><<<g, 64 * WPB, 0, st>>>(X, s.M, s.N, s.K, C, Bq, Bsc, Csc, Hout, fpart, s.nchunks, s.csplit);
    else
      k_colpass<32, false, XT, WPB><<<g, 64 * WPB, 0, st>>>(X, s.M, s.N, s.K, C, Bq, Bsc, Csc, Hout, fpart, s.nchunks, s.csplit);
  } else {
    if (with_h)
      k_colpass<64, true, XT, WPB><<<g, 64 * WPB, 0, st>>>(X, s.M, s.N, s.K, C, Bq, Bsc, Csc, Hout, fpart, s.nchunks, s.csplit);
    else
      k_colpass<64, false, XT, WPB><<<g, 64 * WPB, 0, st>>>(X, s.M, s.N, s.K, C, Bq, Bsc, Csc, Hout, fpart, s.nchunks, s.csplit);
  }
}

template <typename XT>
static void colpass_launch(const Shape& s, const XT* X, const f32x4* C, const _Float16* Bq, float* Bsc, float* Csc,
                           float* Hout, double* fpart, int with_h, hipStream_t st) {
  if (s.cwpb == 8)
    colpass_launch_w<XT, 8>(s, X, C, Bq, Bsc, Csc, Hout, fpart, with_h, st);
  else
    colpass_launch_w<XT, 4>(s, X, C, Bq, Bsc, Csc, Hout, fpart, with_h, st);
}

template <typename XT>
static void colpass_rw_launch(const Shape& s, const XT* X, const f32x4* C, const _Float16* Bq,
                              const _Float16* BqE, float* Bsc, float* Csc, float* Hout, double* fpart, float* R,
                              hipStream_t st) {
  const unsigned g = (unsigned)colpass_blocks(s);
  const int rvec4 = (s.M % 4 == 0) && ((reinterpret_cast<uintptr_t>(R) & 15) == 0);
  if (s.KP == 32)
    k_colpass_rw<32, XT><<<g, 256, 0, st>>>(X, s.M, s.N, s.K, C, Bq, BqE, Bsc, Csc, Hout, fpart, s.nchunks, s.csplit, R, rvec4);
  else
    k_colpass_rw<64, XT><<<g, 256, 0, st>>>(X, s.M, s.N, s.K, C, Bq, BqE, Bsc, Csc, Hout, fpart, s.nchunks, s.csplit, R, rvec4);
}

hipError_t colpass_carry(const Shape& s, const void* X, int refresh, const void* Cqv, const _Float16* Bq,
                         const _Float16* BqD, float* Bsc, float* Csc, float* Hout, double* fpart, float* R,
                         hipStream_t st) {
  const f32x4* C = static_cast<const f32x4*>(Cqv);
  if (!refresh) {  // E = R - delta B C, in place
    colpass_rw_launch(s, static_cast<const float*>(R), C, Bq, BqD, Bsc, Csc, Hout, fpart, R, st);
  } else if (s.xbf16) {  // E = X - B C from the stored data
    colpass_rw_launch(s, static_cast<const __bf16*>(X), C, Bq, Bq, Bsc, Csc, Hout, fpart, R, st);
  } else if (s.xtiled) {
    colpass_rw_launch(s, static_cast<const xtf32*>(X), C, Bq, Bq, Bsc, Csc, Hout, fpart, R, st);
  } else {
    colpass_rw_launch(s, static_cast<const float*>(X), C, Bq, Bq, Bsc, Csc, Hout, fpart, R, st);
  }
  return hipGetLastError();
}

hipError_t colpass(const Shape& s, const void* X, const void* Cqv, const _Float16* Bq, float* Bsc, float* Csc,
                   float* Hout, double* fpart, int with_h, hipStream_t st) {
  const f32x4* C = static_cast<const f32x4*>(Cqv);
  if (s.xbf16)
    colpass_launch(s, static_cast<const __bf16*>(X), C, Bq, Bsc, Csc, Hout, fpart, with_h, st);
  else if (s.xtiled)
    colpass_launch(s, static_cast<const xtf32*>(X), C, Bq, Bsc, Csc, Hout, fpart, with_h, st);
  else
    colpass_launch(s, static_cast<const float*>(X), C, Bq, Bsc, Csc, Hout, fpart, with_h, st);
  return hipGetLastError();
}

// ------------------------------------------------------------------ coordinate sweep
// With h = B^T e_j from the column pass and G = B^T B, the coordinates of a column are
// updated in ascending order in float64:
//   c_kj := [c_kj + h_k / G_kk]_+,  then h_q -= G_qk (c_kj^new - c_kj^old) for q > k,
// which is eq. up:c with b_q^T e_j kept up to date through inner products; a coordinate
// with G_kk = 0 (zero column of B) is skipped.
//
// What bounds it: the chain of K coordinates (latency) while N is small; at large N the
// float64 work (K^2 / 2 FMAs per column: matrix and vector float64 have the same rate here
// and do not overlap) and the H, C and Cq traffic.  The running h of a wave's columns sit in
// the accumulator layout of v_mfma_f64_16x16x4 (subtile u of 16 columns: lane 16 g + n holds
// coordinates 4 r + g of column 16 u + n), so that four coordinates are updated at a time:
// permlane swaps bring a column's four sums into one lane, which forms the four updates;
// their changes, moved back, are the B operand of one float64 MFMA per subtile and 16 later
// coordinates (A operand: G, in the lane order it has in memory).
//
// A wave takes U subtiles: U = 4 (a 4 x 4 transpose, one column per lane) does a step's
// updates for 64 columns at once, the form for large N; U = 1 (every lane of a column forms
// its four updates) has a quarter of the MFMAs per step and four times the waves, the form
// while those still find idle SIMDs (sweep_u).  (One thread per column, with K running sums
// and G read by scalar loads, waited on those loads at every coordinate and read and packed
// its columns through serial LDS loops.)  us per launch
// before and after: 500 x 2000, K = 10: 19.0, 5.2; 3809 x 2248, K = 49: 60.6, 16.1 (11.6 before H
// came as 12 shares' partials); 784 x 70000, K = 16: 25.6, 11.6; 1868 x 40000, K = 60: 69.0, 28.8;
// N = 10^6, K = 50: 397, 308.
//
// Division: h / G_kk is formed from the correctly rounded reciprocal, one residual fma and
// one correction (Markstein's method: the correctly rounded quotient, so that cancellations
// the closed form makes exact stay exact), with v_div_fixup for the special operands.  A
// skipped coordinate takes G_kk = inf: its quotient is 0 (NaN where h overflowed) and its change
// is held to 0.
typedef double f64x4 __attribute__((ext_vector_type(4)));

// 4 x 4 transpose of x[0..3] across the wave's four rows of 16 lanes: x[i] of row g becomes
// x[g] of row i.
__device__ __forceinline__ void transpose4(double (&x)[4]) {
  unsigned w[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t v = __builtin_bit_cast(uint64_t, x[i]);
    w[i][0] = (unsigned)v;
    w[i][1] = (unsigned)(v >> 32);
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
#pragma unroll
    for (int i = 0; i < 4; i += 2) {  // odd rows of w[i] against even rows of w[i + 1]
      const auto t = __builtin_amdgcn_permlane16_swap(w[i][e], w[i + 1][e], false, false);
      w[i][e] = t[0];
      w[i + 1][e] = t[1];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {  // rows 2, 3 of w[i] against rows 0, 1 of w[i + 2]
      const auto t = __builtin_amdgcn_permlane32_swap(w[i][e], w[i + 2][e], false, false);
      w[i][e] = t[0];
      w[i + 2][e] = t[1];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = __builtin_bit_cast(double, ((uint64_t)w[i][1] << 32) | (uint64_t)w[i][0]);
}

// x of the four lanes of a column (rows 0..3 of the wave), in each of them.
__device__ __forceinline__ void gather4(double x, double (&o)[4]) {
  o[0] = o[1] = o[2] = o[3] = x;
  transpose4(o);
}

// Ordering of a wave's own LDS traffic between its lanes (no instruction).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Operands of the four coordinates 4 s .. 4 s + 3 of each step of the coupled updates with
// the symmetric matrix A (G for the columns of C), in LDS: gd[s][0..3] reciprocals and
// [4..7] values of A's diagonal (0 and inf for a skipped coordinate), [8..13] A(1,0), A(2,0),
// A(2,1), A(3,0), A(3,1), A(3,2).
template <int NT>
struct TriOps {
  alignas(16) double gd[4 * NT][14];
};

template <int NT>
__device__ __forceinline__ void tri_stage(TriOps<NT>& o, const double* __restrict__ A, int lda) {
  const int tid = threadIdx.x;
  if (tid < 64 * NT) {
    const int s = tid >> 4, e = tid & 15;
    if (e < 14) {
      int a, b;
      if (e < 8) {
        a = b = e & 3;
      } else {
        const int q = e - 8;  // (1,0) (2,0) (2,1) (3,0) (3,1) (3,2)
        a = q < 1 ? 1 : (q < 3 ? 2 : 3);
        b = q - a * (a - 1) / 2;
      }
      double v = A[(4 * s + a) * lda + 4 * s + b];
      if (e < 8) {
        const bool on = v > 0.0;
        v = e < 4 ? (on ? 1.0 / v : 0.0) : (on ? v : __builtin_inf());
      }
      o.gd[s][e] = v;
    }
  }
}

// The four coordinates of one step for one line: sums hv, old values co (float32); returns
// the new float32 values in cn and minus the float64 changes in d.  The change is formed as
// max(h / A_ii, -old) (what [old + h / A_ii]_+ - old is; at least 0 for a skipped coordinate),
// which keeps the dependent chain at six operations per coordinate.
__device__ __forceinline__ void tri_step(const double (&gd)[14], double (&hv)[4], const f32x4& co, f32x4& cn,
                                         double (&d)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double old = (double)co[i];
    double q = hv[i] * gd[i];
    q = fma(fma(-q, gd[4 + i], hv[i]), gd[i], q);
    q = __builtin_amdgcn_div_fixup(q, gd[4 + i], hv[i]);
    const double lo = gd[i] > 0.0 ? -old : 0.0;
    const double c = q > lo ? q : lo;
    cn[i] = (float)(old + c);
    d[i] = -c;
#pragma unroll
    for (int j = i + 1; j < 4; ++j) hv[j] -= gd[8 + j * (j - 1) / 2 + i] * c;
  }
}

// The chain of one wave's 16 U lines (columns of C, rows of B).  On entry h[u][b] holds the
// sums of subtile u (16 lines) and coordinates 16 b .. 16 b + 15 in the MFMA accumulator
// layout (values past K are not used), and ct points at the lane's line in LDS (lane l's own
// line for U = 4, line l % 16 for U = 1), which is updated in place.  Returns the line's
// largest new value; step(s, new, old) is called once per step of four coordinates.
//
// The loop over 16-coordinate blocks is rolled: the remaining blocks of h move down one
// place per turn.
template <int NT, int U, class Step>
__device__ __forceinline__ float tri_chain(const TriOps<NT>& ops, f64x4 (&h)[U][NT], const double* __restrict__ A,
                                           int lda, int K, float* ct, Step step) {
  static_assert(U == 4 || U == 1, "");
  const int l = threadIdx.x & 63, g = l >> 4;
  const double* Al = A + g * lda + (l & 15);  // A[l / 16][l % 16]
  float mx = 0.0f;
#pragma clang loop unroll(disable)
  for (int sb = 0; sb < NT; ++sb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int s = 4 * sb + r;
      if (4 * s < K) {
        double ga[NT];  // A is symmetric: 16 consecutive lanes read 16 consecutive entries of a row
#pragma unroll
        for (int b = (r == 3 ? 1 : 0); b < NT; ++b) ga[b] = Al[4 * s * lda + 16 * min(sb + b, NT - 1)];
        double gd[14], x[4], d[4];
#pragma unroll
        for (int e = 0; e < 14; ++e) gd[e] = ops.gd[s][e];
        f32x4* const cp = reinterpret_cast<f32x4*>(ct + 4 * s);
        const f32x4 co = *cp;
        if constexpr (U == 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = h[u][0][r];
          transpose4(x);
        } else {
          gather4(h[0][0][r], x);
        }
        f32x4 cn;
        tri_step(gd, x, co, cn, d);
        if (U == 4 || g == 0) *cp = cn;
        step(s, cn, co);
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, cn[i]);
        if constexpr (U == 4)
          transpose4(d);
        else  // this lane's own coordinate 4 s + g
          d[0] = g < 2 ? (g == 0 ? d[0] : d[1]) : (g == 2 ? d[2] : d[3]);
#pragma unroll
        for (int b = (r == 3 ? 1 : 0); b < NT; ++b)
          if (sb + b < NT) {
#pragma unroll
            for (int u = 0; u < U; ++u)
              h[u][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[b], d[u], h[u][b], 0, 0, 0);
          }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int b = 0; b + 1 < NT; ++b) h[u][b] = h[u][b + 1];
  }
  return mx;
}

// Scale of a column (lane) of a 32-column tile (half a wave) from the column's largest
// magnitude mx: when the scales of the tile's nonzero columns lie within kUniformSpread of
// each other, every column takes the smallest, so that the passes scale the tile's products
// with one multiplier; one: whether all 32 columns share one scale.
__device__ __forceinline__ int tile_scale(float mx, bool& one) {
  int sc = scale_exp(mx);
  int smin = mx > 0.0f ? sc : INT_MAX, smax = mx > 0.0f ? sc : INT_MIN;
#pragma unroll
  for (int off = 1; off < 32; off <<= 1) {
    smin = min(smin, __shfl_xor(smin, off, 64));
    smax = max(smax, __shfl_xor(smax, off, 64));
  }
  one = smin > smax;  // an all-zero tile: every scale is 0
  if (smin <= smax && smax - smin <= kUniformSpread) {
    sc = smin;
    one = true;
  }
  return sc;
}

// Floats per line of the lines' values in LDS: K rounded up to a multiple of 4 whose
// quarter is odd, so that 16-byte accesses of a wave's lanes to their lines are free of
// bank conflicts.
__host__ __device__ inline int line_ld(int K) {
  const int q = (K + 3) / 4;
  return 4 * (q | 1);
}

// E-order units p = p0, p0 + dp, ... of line jj of a 32-line tile, from the line in LDS
// times m.  Units whose coordinates all lie past K stay zero.
__device__ __forceinline__ void pack_e(f32x4* __restrict__ tile, const float* ct, int jj, float m, int K, int p0,
                                       int dp) {
#pragma clang loop unroll(disable)
  for (int p = p0; 8 * p < K; p += dp) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(ct + 8 * p);
    f32x4 b = f32x4{0, 0, 0, 0};
    if (8 * p + 4 < K) b = *reinterpret_cast<const f32x4*>(ct + 8 * p + 4);
    float v[8];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v[t] = a[t] * m;
      v[4 + t] = b[t] * m;
    }
    const Split2 sp = split2(v);
    f32x4* dst = tile + (p >> 1) * 128 + jj + 32 * (p & 1);
    dst[0] = f16_as_f32x4(sp.p[0]);
    dst[64] = f16_as_f32x4(sp.p[1]);
  }
}

// Subtiles per wave of an instance's sweep: one while a wave per 16 columns still finds
// idle SIMDs.  us per launch at U = 1 and U = 4: 9.8 and 14.0 at N = 9000, K = 40; 29.9 and
// 24.8 at N = 40000, K = 60; batches of mixed N, which fill the GPU together, prefer U = 4
// from N = 8192 on (39.8 us per grouped launch at a line of 32768, 33.3 at 8192).  One line for
// both, between the two, so that a batched instance equals its solo run bit for bit.
__host__ __device__ inline int sweep_u(int64_t N) { return N <= 16384 ? 1 : 4; }
inline int64_t sweep_blocks(int64_t N) { return (N + 64 * sweep_u(N) - 1) / (64 * sweep_u(N)); }

// LDS of a sweep block beside its lines (64 U columns, and as many changes in the carried form)
template <int NT>
struct SweepLds {
  TriOps<NT> ops;
  float mx[4][64];    // largest C' per coordinate, per wave
  float lmx[2][256];  // largest magnitude per line: C', and delta C in the carried form
};
inline size_t sweep_dyn_lds(int K, int u, bool rw) { return (size_t)64 * u * line_ld(K) * sizeof(float) * (rw ? 2 : 1); }

// Sweep of the 64 U columns of block bid.  H comes as csplit partials (added in float64 in
// order), each stored per 32-column tile (h_stride floats; row k of a tile is 32 consecutive
// floats; columns past N hold zeros).  The updated columns go back
// to C and, scaled and split, to the E-order units of Cq; the rows' maxima are added to
// Csc[0, KP).  With RW (the carried-residual form) delta C = C' - C (float32 difference of the
// stored values) is packed into CqD's E-order units too.
template <int KP, int NT, int U, bool RW>
__device__ __forceinline__ void sweep_body(SweepLds<NT>& S, float* lines, const float* __restrict__ Hin,
                                           int csplit, float* __restrict__ C, f32x4* __restrict__ Cq,
                                           float* __restrict__ Csc, int64_t N, int K, const double* __restrict__ G,
                                           int64_t bid, f32x4* __restrict__ CqD) {
  constexpr int NL = 64 * U;             // lines per block
  constexpr int CPI = NT <= 2 ? 2 : 1;   // lines per load of C (64 lanes over 64 / CPI coordinates)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int64_t nt = (N + 31) / 32, j0 = bid * NL, T0 = bid * (NL / 32);
  const int nv = N - j0 < NL ? (int)(N - j0) : NL;  // the block's columns
  const int K4 = (K + 3) / 4 * 4;
  const int LD = line_ld(K);
  float* const Cb = C + j0 * K;
  f64x4 h[U][NT];
  {  // lane 16 g + n: row 4 s + g, column n of the subtile (rows past K are read, not used; a
     // subtile past the last tile reads that tile again)
    float hn[U][4 * NT];
    auto hload = [&](int64_t p) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int sub = U == 4 ? 4 * wave + u : wave;
        const int64_t T = T0 + (sub >> 1) < nt ? T0 + (sub >> 1) : nt - 1;
        const float* const ht = Hin + p * h_stride(N, K) + T * (K4 * 32) + 16 * (sub & 1) + (l >> 4) * 32 + (l & 15);
#pragma unroll
        for (int s = 0; s < 4 * NT; ++s) hn[u][s] = ht[s * 128];
      }
    };
    hload(0);
    // the block's columns of C into LDS, coalesced and all in flight at once; zeros past N
    constexpr int LPW = 16 * U / CPI;
    const int kk = l & (64 / CPI - 1), c0 = wave * CPI + (CPI == 2 ? l >> 5 : 0);
    float v[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) v[i] = Cb[(uint32_t)(min(c0 + 4 * CPI * i, nv - 1) * K + min(kk, K - 1))];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const int j = c0 + 4 * CPI * i;
      if (kk < LD) lines[j * LD + kk] = (kk < K && j < nv) ? v[i] : 0.0f;
    }
    tri_stage<NT>(S.ops, G, KP);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < 4 * NT; ++s) h[u][s >> 2][s & 3] = (double)hn[u][s];
#pragma unroll U == 1 ? 4 : 1
    for (int p = 1; p < csplit; ++p) {
      hload(p);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int s = 0; s < 4 * NT; ++s) h[u][s >> 2][s & 3] += (double)hn[u][s];
    }
  }
  __syncthreads();
  {
    const int line = U == 4 ? 64 * wave + l : 16 * wave + (l & 15);
    float* const ct = lines + line * LD;
    float md = 0.0f;
    const float mx = tri_chain<NT, U>(S.ops, h, G, KP, K, ct, [&](int s, const f32x4& cn, const f32x4& co) {
      if constexpr (RW) {
        f32x4 dc;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          dc[i] = cn[i] - co[i];
          md = fmaxf(md, fabsf(dc[i]));
        }
        if (U == 4 || l < 16) *reinterpret_cast<f32x4*>(ct + NL * LD + 4 * s) = dc;
      }
    });
    if (U == 4 || l < 16) {
      S.lmx[0][line] = mx;
      if constexpr (RW) S.lmx[1][line] = md;
    }
  }
  __syncthreads();
  // scale and pack: line tid % NL, its units dealt over the threads that share it
  {
    const int j = tid % NL, jj = j & 31;
    const int64_t T = T0 + (j >> 5);
    const bool ok = j < nv;
    bool one;
    const int sc = tile_scale(ok ? S.lmx[0][j] : 0.0f, one);
    if (T < nt) {
      f32x4* const tile = Cq + T * CqL<KP>::T;
      pack_e(tile, lines + j * LD, jj, pow2f(sc), K, tid / NL, 256 / NL);
      if (tid < NL) {  // inverse scales; the sign of column 0's flags a shared scale
        const float inv = pow2f(-sc);
        reinterpret_cast<float*>(tile + CqL<KP>::E0)[jj] = (one && jj == 0) ? -inv : inv;
      }
      if constexpr (RW) {
        f32x4* const td = CqD + T * CqL<KP>::E;
        const int sd = scale_exp(ok ? S.lmx[1][j] : 0.0f);
        pack_e(td, lines + (NL + j) * LD, jj, pow2f(sd), K, tid / NL, 256 / NL);
        if (tid < NL) reinterpret_cast<float*>(td + CqL<KP>::E0)[jj] = pow2f(-sd);
      }
    }
  }
  // C' back, coalesced, and its rows' maxima (C >= 0: integer order = float order)
  {
    const int kk = l & (64 / CPI - 1), c0 = wave * CPI + (CPI == 2 ? l >> 5 : 0);
    float cmax = 0.0f;
    if (kk < K) {
#pragma unroll 8
      for (int c = c0; c < nv; c += 4 * CPI) {
        const float v = lines[c * LD + kk];
        cmax = fmaxf(cmax, v);
        Cb[(uint32_t)(c * K + kk)] = v;
      }
    }
    if constexpr (CPI == 2) cmax = fmaxf(cmax, __shfl_xor(cmax, 32, 64));
    S.mx[wave][l] = cmax;
    __syncthreads();
    if (tid < K) {
      const float m = fmaxf(fmaxf(S.mx[0][tid], S.mx[1][tid]), fmaxf(S.mx[2][tid], S.mx[3][tid]));
      if (m > 0.0f) atomicMax(reinterpret_cast<int*>(Csc) + tid, __float_as_int(m));
    }
  }
}

template <int KP, int NT, int U, bool RW>
__global__ __launch_bounds__(256, 2) void k_sweep(const float* __restrict__ Hin, int csplit,
                                                  float* __restrict__ C, f32x4* __restrict__ Cq,
                                                  float* __restrict__ Csc, int64_t N, int K,
                                                  const double* __restrict__ G, f32x4* __restrict__ CqD) {
  __shared__ SweepLds<NT> S;
  extern __shared__ __align__(16) float lines[];
  sweep_body<KP, NT, U, RW>(S, lines, Hin, csplit, C, Cq, Csc, N, K, G, blockIdx.x, CqD);
}

// ------------------------------------------------------------------ B update
// b_mi := [b_mi + (w_mi - sum_{k < i} v_ik delta b_mk) / v_ii]_+ for i ascending, row by row (V
// only couples the columns of one row): the sweep's chain with W for H and V for G, in the
// form of 16 rows per wave.  A block takes 64 rows: it updates them in LDS, writes them back
// and packs them (E order, scaled per row; with RW, the carried-residual form, also the change
// -delta B = B^t - B^{t+1} of the stored float32 values, into BqD), adds the columns' maxima
// to bmax and forms its partial of G = B^T B (float64 MFMA, products exact in float64) over
// 16-coordinate blocks.  update = 0 packs and forms G from B as it is.  Bq may be null (thin path).
//
// Bound by the chain's latency.  (One thread per row, a quarter of the block's waves, with V in
// LDS took 11.4 us at M = 500, K = 10, 47 us at M = 3809, K = 49 and 70 us at M = 5000, K = 50;
// now 7.9, 19.3 and 28.3 us.)
template <int NT>
struct BupLds {
  TriOps<NT> ops;
  float mx[4][64];           // largest value per column of B, per wave
  float lmx[2][kBupRows];    // largest magnitude per row: B, and delta B in the carried form
};
inline size_t bup_dyn_lds(int K, bool rw) { return (size_t)kBupRows * line_ld(K) * sizeof(float) * (rw ? 2 : 1); }

template <int KP, int NT, bool RW>
__device__ __forceinline__ void bupdate_body(BupLds<NT>& S, float* lines, float* __restrict__ B, int64_t M, int K,
                                             const double* __restrict__ W, int64_t Mpad, const double* __restrict__ V,
                                             _Float16* __restrict__ Bq, float* __restrict__ bmax,
                                             double* __restrict__ Gpart, int update, int64_t bid,
                                             _Float16* __restrict__ BqD) {
  constexpr int64_t UC = BqL<KP>::C;
  constexpr int US = BqL<KP>::S;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, g = l >> 4;
  const int64_t m0 = bid * kBupRows;
  const int nv = M - m0 < kBupRows ? (int)(M - m0) : kBupRows;  // the block's rows
  const int LD = line_ld(K);
  f64x4 h[1][NT];
  if (update) {  // lane 16 g + n: coordinate 4 s + g of row 16 wave + n
    const double* const wr = W + (m0 + min(16 * wave + (l & 15), nv - 1));
#pragma unroll
    for (int s = 0; s < 4 * NT; ++s) h[0][s >> 2][s & 3] = wr[(int64_t)min(4 * s + g, K - 1) * Mpad];
    if (16 * wave + (l & 15) >= nv) {  // a row past M: stays zero
#pragma unroll
      for (int b = 0; b < NT; ++b) h[0][b] = f64x4{0, 0, 0, 0};
    }
  }
  // the block's rows of B into LDS (lane = row), zeros past M and K
  for (int k0 = 4 * wave; k0 < LD; k0 += 16) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = B[(int64_t)min(k0 + i, K - 1) * M + m0 + min(l, nv - 1)];
    f32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = (l < nv && k0 + i < K) ? v[i] : 0.0f;
    *reinterpret_cast<f32x4*>(lines + l * LD + k0) = o;
  }
  if (update) tri_stage<NT>(S.ops, V, KP);
  __syncthreads();
  {
    const int line = 16 * wave + (l & 15);
    float* const ct = lines + line * LD;
    float mx = 0.0f, md = 0.0f;
    if (update) {
      mx = tri_chain<NT, 1>(S.ops, h, V, KP, K, ct, [&](int s, const f32x4& cn, const f32x4& co) {
        if constexpr (RW) {
          f32x4 dc;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            dc[i] = cn[i] - co[i];
            md = fmaxf(md, fabsf(dc[i]));
          }
          if (l < 16) *reinterpret_cast<f32x4*>(ct + kBupRows * LD + 4 * s) = dc;
        }
      });
    } else {
      for (int k = 0; k < K; ++k) mx = fmaxf(mx, ct[k]);
      if constexpr (RW)
        for (int k = g; k < LD; k += 4) ct[kBupRows * LD + k] = 0.0f;
    }
    if (l < 16) {
      S.lmx[0][line] = mx;
      if constexpr (RW) S.lmx[1][line] = md;
    }
  }
  __syncthreads();
  if (update) {  // back to B (lane = row)
    for (int k = wave; k < K; k += 4) {
      const float v = lines[l * LD + k];
      if (l < nv) B[(int64_t)k * M + m0 + l] = v;
    }
  }
  if (Bq) {  // row l: its E-order units are dealt over the four waves
    const int64_t c = (m0 >> 5) + (l >> 5);
    const int r = l & 31;
    bool one;
    const int sc = tile_scale(l < nv ? S.lmx[0][l] : 0.0f, one);
    if (l < nv) {
      f32x4* const u = reinterpret_cast<f32x4*>(Bq) + c * UC;
      pack_e(u, lines + l * LD, r, -pow2f(sc), K, wave, 4);
      if (wave == 0) {  // inverse scales; the sign of row 0's flags a scale shared by the chunk
        const float inv = pow2f(-sc);
        reinterpret_cast<float*>(u + US)[r] = (one && r == 0) ? -inv : inv;
      }
      if constexpr (RW) {
        f32x4* const ud = reinterpret_cast<f32x4*>(BqD) + c * UC;
        const int sd = scale_exp(S.lmx[1][l]);
        pack_e(ud, lines + (kBupRows + l) * LD, r, -pow2f(sd), K, wave, 4);
        if (wave == 0) reinterpret_cast<float*>(ud + US)[r] = pow2f(-sd);
      }
    }
    // column maxima (B >= 0: integer order = float order)
    float cm = 0.0f;
    if (l < K) {
#pragma unroll
      for (int i = 0; i < 16; ++i) cm = fmaxf(cm, lines[(16 * wave + i) * LD + l]);
    }
    S.mx[wave][l] = cm;
    __syncthreads();
    if (tid < K) {
      const float m = fmaxf(fmaxf(S.mx[0][tid], S.mx[1][tid]), fmaxf(S.mx[2][tid], S.mx[3][tid]));
      if (m > 0.0f) atomicMax(reinterpret_cast<int*>(bmax) + tid, __float_as_int(m));
    }
  }
  // partial of G over the block's rows, blocks (ta >= tb) of 16 x 16 coordinates dealt over the
  // waves: lane 16 g + n supplies B[4 t + g][16 ta + n] and B[4 t + g][16 tb + n], four rows a step
  constexpr int NBLK = NT * (NT + 1) / 2, NP = 16 * NT * (16 * NT + 1) / 2;
#pragma clang loop unroll(disable)
  for (int q = wave; q < NBLK; q += 4) {
    const int ta = q < 1 ? 0 : (q < 3 ? 1 : (q < 6 ? 2 : 3)), tb = q - ta * (ta + 1) / 2;
    const int ka = 16 * ta + (l & 15), kb = 16 * tb + (l & 15);
    const float* const la = lines + g * LD + min(ka, K - 1);
    const float* const lb = lines + g * LD + min(kb, K - 1);
    f64x4 acc = f64x4{0, 0, 0, 0};
#pragma unroll 4
    for (int t = 0; t < kBupRows / 4; ++t) {
      const double x = ka < K ? (double)la[4 * t * LD] : 0.0, y = kb < K ? (double)lb[4 * t * LD] : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = 16 * ta + 4 * r + g;
      if (a >= kb) Gpart[bid * NP + a * (a + 1) / 2 + kb] = acc[r];
    }
  }
}

template <int KP, int NT, bool RW>
__global__ __launch_bounds__(256, 2) void k_bupdate(float* __restrict__ B, int64_t M, int K,
                                                    const double* __restrict__ W, int64_t Mpad,
                                                    const double* __restrict__ V, _Float16* __restrict__ Bq,
                                                    float* __restrict__ bmax, double* __restrict__ Gpart, int update,
                                                    _Float16* __restrict__ BqD) {
  __shared__ BupLds<NT> S;
  extern __shared__ __align__(16) float lines[];
  bupdate_body<KP, NT, RW>(S, lines, B, M, K, W, Mpad, V, Bq, bmax, Gpart, update, blockIdx.x, BqD);
}

int bupdate_blocks(const Shape& s) { return (int)((s.M + kBupRows - 1) / kBupRows); }

template <int KP, int NT>
static void bupdate_launch(const Shape& s, float* B, const double* W, const double* V, _Float16* Bq, float* Bsc,
                           double* Gpart, int update, _Float16* BqD, hipStream_t st) {
  const unsigned g = (unsigned)bupdate_blocks(s);
  if (BqD)
    k_bupdate<KP, NT, true><<<g, 256, bup_dyn_lds(s.K, true), st>>>(B, s.M, s.K, W, s.Mpad, V, Bq, Bsc, Gpart, update,
                                                                     BqD);
  else
    k_bupdate<KP, NT, false><<<g, 256, bup_dyn_lds(s.K, false), st>>>(B, s.M, s.K, W, s.Mpad, V, Bq, Bsc, Gpart,
                                                                      update, nullptr);
}

hipError_t bupdate(const Shape& s, float* B, const double* W, const double* V, _Float16* Bq, float* Bsc,
                   double* Gpart, int update, hipStream_t st, _Float16* BqD) {
  if (s.thin) {
    Bq = nullptr;
    Bsc = nullptr;
    BqD = nullptr;
  } else if (!update) {  // an iteration's column pass clears the maxima of its B update
    k_zero_f32<<<1, 64, 0, st>>>(Bsc, s.KP);
  }
  if (s.K <= 16)
    bupdate_launch<32, 1>(s, B, W, V, Bq, Bsc, Gpart, update, BqD, st);
  else if (s.K <= 32)
    bupdate_launch<32, 2>(s, B, W, V, Bq, Bsc, Gpart, update, BqD, st);
  else if (s.K <= 48)
    bupdate_launch<64, 3>(s, B, W, V, Bq, Bsc, Gpart, update, BqD, st);
  else
    bupdate_launch<64, 4>(s, B, W, V, Bq, Bsc, Gpart, update, BqD, st);
  return hipGetLastError();
}

// E order of C, 32 kPackTiles columns a block.
template <int KP>
__global__ __launch_bounds__(256) void k_packc(const float* __restrict__ C, f32x4* __restrict__ Cq, int64_t N, int K) {
  constexpr int J = 32 * kPackTiles;
  extern __shared__ float Ct[];  // J * K floats
  __shared__ int cs[256];
  const int64_t j0 = (int64_t)blockIdx.x * J;
  const int nv = (int)((N - j0) < J ? (N - j0) : J);
  block_copy(Ct, C + j0 * K, nv * K);
  __syncthreads();
  pack_block<KP>(Cq, j0, nv, Ct, K, (N + 31) / 32, cs);
}

template <int KP, int NT, int U>
static void sweep_launch_u(const Shape& s, const float* Hin, float* C, f32x4* q, float* Csc, const double* G,
                           f32x4* qd, hipStream_t st) {
  const unsigned g = (unsigned)sweep_blocks(s.N);
  if (qd)
    k_sweep<KP, NT, U, true><<<g, 256, sweep_dyn_lds(s.K, U, true), st>>>(Hin, s.csplit, C, q, Csc, s.N, s.K, G, qd);
  else
    k_sweep<KP, NT, U, false><<<g, 256, sweep_dyn_lds(s.K, U, false), st>>>(Hin, s.csplit, C, q, Csc, s.N, s.K, G, nullptr);
}

template <int KP, int NT>
static void sweep_launch(const Shape& s, const float* Hin, float* C, f32x4* q, float* Csc, const double* G, f32x4* qd,
                         hipStream_t st) {
  if (sweep_u(s.N) == 1)
    sweep_launch_u<KP, NT, 1>(s, Hin, C, q, Csc, G, qd, st);
  else
    sweep_launch_u<KP, NT, 4>(s, Hin, C, q, Csc, G, qd, st);
}

hipError_t sweep(const Shape& s, const float* Hin, float* C, void* Cq, float* Csc, const double* G,
                 hipStream_t st, void* CqD) {
  f32x4* q = static_cast<f32x4*>(Cq);
  f32x4* qd = static_cast<f32x4*>(CqD);
  if (s.K <= 16)
    sweep_launch<32, 1>(s, Hin, C, q, Csc, G, qd, st);
  else if (s.K <= 32)
    sweep_launch<32, 2>(s, Hin, C, q, Csc, G, qd, st);
  else if (s.K <= 48)
    sweep_launch<64, 3>(s, Hin, C, q, Csc, G, qd, st);
  else
    sweep_launch<64, 4>(s, Hin, C, q, Csc, G, qd, st);
  return hipGetLastError();
}

hipError_t packc(const Shape& s, const float* C, void* Cq, hipStream_t st) {
  constexpr int J = 32 * kPackTiles;
  const unsigned g = (unsigned)((s.N + J - 1) / J);
  f32x4* q = static_cast<f32x4*>(Cq);
  if (s.KP == 32)
    k_packc<32><<<g, 256, J * s.K * sizeof(float), st>>>(C, q, s.N, s.K);
  else
    k_packc<64><<<g, 256, J * s.K * sizeof(float), st>>>(C, q, s.N, s.K);
  return hipGetLastError();
}

// ------------------------------------------------------------------ W order of C and V = tril(C C^T)
// Each block takes a contiguous run of 32-column tiles, wave w every eighth of them.  A wave
// reads a tile of C (each load coalesced across the lanes, which take consecutive
// coordinates; the next tile's loads are in flight while one is worked on), scales each row
// by the power of two from its maximum in Csc[0, KP), splits it and stores the W-order units;
// block 0 stores the inverse scales into Csc[KP, 2 KP).  The units in its registers are also
// the MFMA operands of the tile's contribution to V: for one coordinate kk, eight columns,
// which is both the A fragment (rows kk, reduction over columns) and the B fragment
// (reduction over columns, columns kk').  The lower 32 x 32 blocks (b1 >= b2) are formed in
// float32 within the tile, in units of 2^(w_a + w_b), and added to float64 accumulators; the
// waves' sums are unscaled (exactly), added in a fixed order and written as tril pairs.
// (As two kernels, the second reading the units back: 89 and 81 us at N = 10^6, K = 50; one:
// 89 us, and one launch less.)
constexpr int kVBlocks = 256;
constexpr int kVWaves = 8;

template <int KP>
struct PackvLds {
  double v[kVWaves / 2][KP * (KP + 1) / 2];
  float inv[KP];  // 2^-w_kk
};

// AHEAD: the next tile's loads are issued before a tile is worked on (not in the grouped
// kernel, where the registers would spill).
template <int KP, bool AHEAD>
__device__ __forceinline__ void packv_body(PackvLds<KP>& S, const float* __restrict__ C, f32x4* __restrict__ Cq,
                                           float* __restrict__ Csc, int64_t N, int K, double* __restrict__ Vpart,
                                           int64_t bid, int64_t nblk) {
  constexpr int NB = KP / 32;
  constexpr int UE = CqL<KP>::E;  // E-order units and scales of a packed C tile
  constexpr int UT = CqL<KP>::T;
  constexpr int NBL = NB * (NB + 1) / 2;  // lower blocks (b1 >= b2)
  // the wave index is uniform: from a scalar register, so that wave-based addresses stay scalar
  const int tid = item_tid(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, half = l >> 5,
            lc = l & 31;
  const int NP = g_pairs(K);
  const int64_t ntiles = (N + 31) / 32, per = (ntiles + nblk - 1) / nblk;
  const int64_t t0 = bid * per;
  const int64_t t1 = (t0 + per < ntiles) ? t0 + per : ntiles;
  float ws[NB];  // 2^w_kk of this lane's coordinates
#pragma unroll
  for (int b = 0; b < NB; ++b) ws[b] = pow2f(32 * b + lc < K ? scale_exp(Csc[32 * b + lc]) : 0);
  if (bid == 0 && tid < KP) Csc[KP + tid] = pow2f(-(tid < K ? scale_exp(Csc[tid]) : 0));
  float x[2][NB][8];  // [q][b][t]: C[32 b + lc][column row32(8 q + t, half) of the tile]
  auto load = [&](int64_t T) {
    const float* const ct = C + T * 32 * K;
    const int nv = N - T * 32 < 32 ? (int)(N - T * 32) : 32;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int t = 0; t < 8; ++t)
          x[q][b][t] = ct[(uint32_t)(min(row32(8 * q + t, half), nv - 1) * K + min(32 * b + lc, K - 1))];
  };
  double acc[NBL][16];
#pragma unroll
  for (int k = 0; k < NBL; ++k)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[k][i] = 0.0;
  if (AHEAD && t0 + wave < t1) load(t0 + wave);
#pragma clang loop unroll(disable)
  for (int64_t T = t0 + wave; T < t1; T += kVWaves) {
    if (!AHEAD) load(T);
    const int nv = N - T * 32 < 32 ? (int)(N - T * 32) : 32;
    f32x4* const wu = Cq + T * UT + UE + l;
    f16x8 w[2][NB][2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        float v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t)
          v[t] = (32 * b + lc < K && row32(8 * q + t, half) < nv) ? x[q][b][t] * ws[b] : 0.0f;
        const Split2 sp = split2(v);
#pragma unroll
        for (int p = 0; p < 2; ++p) w[q][b][p] = sp.p[p];
      }
    if (AHEAD && T + kVWaves < t1) load(T + kVWaves);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int p = 0; p < 2; ++p) wu[((b * 2 + q) * 2 + p) * 64] = f16_as_f32x4(w[q][b][p]);
    int k = 0;
#pragma unroll
    for (int b1 = 0; b1 < NB; ++b1)
#pragma unroll
      for (int b2 = 0; b2 <= b1; ++b2, ++k) {
        f32x16 v;
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = 0.0f;
#pragma unroll
        for (int q = 0; q < 2; ++q) v = mfma_x3(w[q][b1], w[q][b2], v);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[k][i] += (double)v[i];
      }
  }
  // unscaled sums: waves 4..7 through LDS, then waves 0..3 add theirs, then the four in order
  if (tid < KP) S.inv[tid] = pow2f(-(tid < K ? scale_exp(Csc[tid]) : 0));
  __syncthreads();
#pragma clang loop unroll(disable)
  for (int turn = 0; turn < 2; ++turn) {
    if ((wave >= kVWaves / 2) == (turn == 0)) {
      double* const vs = S.v[wave & (kVWaves / 2 - 1)];
      int k = 0;
#pragma unroll
      for (int b1 = 0; b1 < NB; ++b1)
#pragma unroll
        for (int b2 = 0; b2 <= b1; ++b2, ++k)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int a = 32 * b1 + row32(i, half), b = 32 * b2 + lc;
            const double v = acc[k][i] * (double)S.inv[a] * (double)S.inv[b];
            if (a >= b) vs[a * (a + 1) / 2 + b] = turn ? v + vs[a * (a + 1) / 2 + b] : v;
          }
    }
    __syncthreads();
  }
  for (int q = tid; q < NP; q += 64 * kVWaves) {
    double v = S.v[0][q];
#pragma unroll
    for (int w = 1; w < kVWaves / 2; ++w) v += S.v[w][q];
    Vpart[bid * NP + q] = v;
  }
}

// A tile per wave at least (blocks of one tile each, as for N <= 8192 before, spent most of a
// batch's launch on their sums: 127 us for 9 jobs at K > 32, 61 us as whole blocks).
int64_t vgram_blocks(const Shape& s) {
  const int64_t t = (n_tiles32(s) + kVWaves - 1) / kVWaves;
  return t < kVBlocks ? t : kVBlocks;
}

// ------------------------------------------------------------------ row pass
// Block = 4 waves; wave w owns the 32-row chunk c = 4*sg + w of slab group sg and column
// range r.  Per 32-column tile T of the range (transposed tiles, rows = columns of X):
//   P    = (C[:, tile] 2^t)^T (-B[chunk, :] 2^s)^T  (scaled fp16 steps, as in the column pass)
//   acc  = X[chunk, tile]^T + P 2^-(t_j + s_m)       -> E'^T with E' = X - B C'
//   WT  += (C[:, tile] 2^w) (acc 2^v)                -> (E' C'^T)^T for this chunk, scaled
// where w is the packed per-row scale of C' and v, per row of E' (per lane), the running
// scale of the column pass's H: chosen per tile from the tile's largest |E'| in the row and
// never raised, the running WT being rescaled exactly when it drops.  The packed C' tile
// (both operand orders, already split and scaled) is copied into LDS for the next tile
// (double buffer shared by the four waves; straight from global memory into LDS, with no
// staging registers) and X of the next tile is prefetched into registers.
// Blocks are dealt to the eight XCDs round-robin; each XCD takes an equal run of the (range,
// slab group) pairs, ranges first, so that the slab groups of a range share its C' tiles in
// one L2 (whole ranges per XCD left XCDs idle at few ranges: 10304 x 575, K = 25, measured at 4
// ranges, 34.6 us, as runs 22.0; the bound on its scratch leaves that shape one range).
//
// RW (the carried-residual form): X is the column-major float32 residual R = X - B C of
// the column pass, the E-order operand of each tile comes from CqE (delta C, stride
// CqL<KP>::E units per tile) while the W-order operand comes from Cq, so that
// E' = R - B delta C, and E' is stored back into R in place.
template <int KP, typename XT, bool RW = false>
__device__ __forceinline__ void rowpass_body(const XT* X, int64_t M, int64_t N, int K,
                                             const f32x4* __restrict__ Cq, const float* __restrict__ Csc,
                                             const _Float16* __restrict__ Bq,
                                             float* __restrict__ Wpart, int64_t Mpad, int64_t nchunks,
                                             const int64_t* __restrict__ tb, int R, int nsg, int64_t bid,
                                             const f32x4* __restrict__ CqE = nullptr, float* Rout = nullptr) {
  constexpr int NB = KP / 32;
  constexpr int KS = KP / 16;
  constexpr int UE0 = CqL<KP>::E0;     // 16-byte units of the E'^T A operand per tile
  constexpr int UE = CqL<KP>::E;       // ... followed by the tile's inverse column scales
  constexpr int UT = CqL<KP>::T;       // then the W A operand
  constexpr int64_t UC = BqL<KP>::C;   // units per packed B chunk
  constexpr int UBS = BqL<KP>::S;      // the chunk's 32 row scales
  __shared__ f32x4 sc[2][UT];
  const int64_t total = (int64_t)R * nsg, lin = (bid & 7) * ((total + 7) / 8) + (bid >> 3);
  if (lin >= total) return;  // whole block
  const int r = (int)(lin / nsg), sg = (int)(lin - (int64_t)r * nsg);
  // the wave index is uniform: from a scalar register, so that wave-based addresses stay scalar
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, half = l >> 5,
            lc = l & 31;
  const int64_t c = (int64_t)sg * 4 + wave;
  const bool active = c < nchunks;  // inactive waves still take part in staging and barriers
  const int64_t tlo = tb[r], thi = tb[r + 1];
  const int64_t hi = (thi * 32 < N) ? thi * 32 : N;  // column end of the range
  const int64_t m0 = (active ? c : 0) * 32, mrow = m0 + lc;
  const bool rowok = active && mrow < M;

  f16x8 bP[KS][2];  // pieces of -B[m0 + l%32][16s + 8*half + t] 2^s_m
  float bs;         // 2^-s_m of this lane's row
  {
    const f32x4* pe = reinterpret_cast<const f32x4*>(Bq) + (active ? c : 0) * UC;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int p = 0; p < 2; ++p) bP[s][p] = as_f16x8(pe[(s * 2 + p) * 64 + l]);
    bs = fabsf(reinterpret_cast<const float*>(pe + UBS)[lc]);  // row 0's may carry the uniform flag
  }
  f32x16 WT[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) WT[b][i] = 0.0f;
  int vcur = 126;  // current scale exponent of this row's E' operand (never raised)

  // tile T's packed C units straight into LDS buffer buf, as the column pass stages B
  constexpr int NX = RW ? 0 : x_loads<XT>::value;
  auto cdma = [&](int64_t T, int buf) {
    stage_units<UT, 4, !RW>(&sc[buf][0], wave, l, [&](int u) {
      const f32x4* src = Cq + T * UT + u;
      if constexpr (RW)
        if (u < UE) src = CqE + T * UE + u;
      return src;
    });
    load_order();
  };
  const uint32_t loff = (uint32_t)(4 * half * M + mrow);  // lane offset within a tile
  const bool rowsfull = active && m0 + 32 <= M;            // wave-uniform
  auto xload = [&](int64_t T) {
    f32x16 v;
    if constexpr (x_is_tiled<XT>::value) {  // tiled copy XR
      return ld_tile(X + ((active ? c : 0) * ((N + 31) / 32) + T) * 1024, l);
    } else {  // column-major float32 X
      const int64_t j0 = T * 32;
      const float* xt = X + j0 * M;  // wave-uniform
      if (rowsfull && j0 + 32 <= hi) {  // wave-uniform
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = xt[(int64_t)(8 * (i >> 2) + (i & 3)) * M + loff];
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int64_t j = j0 + row32(i, half);
          v[i] = (rowok && j < hi) ? X[j * M + mrow] : 0.0f;
        }
      }
      return v;
    }
  };

  // One tile: compute tile T from the X tile in xc (loaded one tile earlier) and the
  // staged C' operands in LDS buffer buf; meanwhile stage tile T+1 and load its X tile
  // into xn.
  auto step = [&](int64_t T, int buf, const f32x16& xc, f32x16& xn) {
    const int64_t Tn = T + 1 < thi ? T + 1 : T;
    cdma(Tn, buf ^ 1);
    xn = xload(Tn);
    load_order();
    if (active) {
      f32x16 acc;  // E' of the tile (the X tile in xc stays as loaded)
      {
        const f32x4* ue = &sc[buf][0] + l;
        f16x8 a[2], an[2];
        f32x16 P;
#pragma unroll
        for (int i = 0; i < 16; ++i) P[i] = 0.0f;
#pragma unroll
        for (int p = 0; p < 2; ++p) a[p] = as_f16x8(ue[p * 64]);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          if (s + 1 < KS) {
#pragma unroll
            for (int p = 0; p < 2; ++p) an[p] = as_f16x8(ue[((s + 1) * 2 + p) * 64]);
          }
          P = mfma_x3(a, bP[s], P);
          if (s + 1 < KS) {
#pragma unroll
            for (int p = 0; p < 2; ++p) a[p] = an[p];
          }
        }
        // rows row32(4q + e, half) = 8q + 4 half + e of the tile: inverse scales in unit 2q + half.
        // A negative first scale flags a tile whose columns share one scale (the C packing):
        // one multiplier for the whole tile.
        const f32x4* ts = &sc[buf][UE0];
        const float t0 =
            __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, ts[0][0])));
        if (t0 < 0.0f) {
          const float mu = -t0 * bs;
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[i] = fmaf(P[i], mu, xc[i]);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 t4 = ts[2 * q + half];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * q + e] = fmaf(P[4 * q + e], t4[e] * bs, xc[4 * q + e]);
          }
        }
      }
      if constexpr (RW) {  // E' back into the residual, where it was read
        const int64_t j0 = T * 32;
        float* rt = Rout + j0 * M;
        if (rowsfull && j0 + 32 <= hi) {
#pragma unroll
          for (int i = 0; i < 16; ++i) rt[(int64_t)(8 * (i >> 2) + (i & 3)) * M + loff] = acc[i];
        } else {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int64_t j = j0 + row32(i, half);
            if (rowok && j < hi) Rout[j * M + mrow] = acc[i];
          }
        }
      }
      // scale of this tile's E' operand: the largest |E'| of the row over the tile (the
      // lane and its partner l ^ 32 hold the row's 32 columns)
      float em = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) em = fmaxf(em, fabsf(acc[i]));
      em = fmaxf(em, __shfl_xor(em, 32, 64));
      int v = scale_exp(em);
      v = (em > 0.0f && v < vcur) ? v : vcur;
      if (__ballot(v != vcur)) {  // wave-uniform: rescale only when some row's scale drops
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i) WT[b][i] = ldexpf(WT[b][i], v - vcur);
        vcur = v;
      }
      const f32x4* uw = &sc[buf][UE] + l;
      f16x8 w[2], wn[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) w[p] = as_f16x8(uw[p * 64]);
      f16x8 eP[2][2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float y[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) y[t] = ldexpf(acc[8 * q + t], v);
        const Split2 sp = split2(y);
#pragma unroll
        for (int p = 0; p < 2; ++p) eP[q][p] = sp.p[p];
      }
#pragma unroll
      for (int gg = 0; gg < NB * 2; ++gg) {  // accumulators alternate, as in the column pass
        if (gg + 1 < NB * 2) {
          const int un = (((gg + 1) % NB) * 2 + (gg + 1) / NB) * 2;
#pragma unroll
          for (int p = 0; p < 2; ++p) wn[p] = as_f16x8(uw[(un + p) * 64]);
        }
        WT[gg % NB] = mfma_x3(w, eP[gg / NB], WT[gg % NB]);
        if (gg + 1 < NB * 2) {
#pragma unroll
          for (int p = 0; p < 2; ++p) w[p] = wn[p];
        }
      }
    }
    stage_barrier<NX>();
  };

  if (tlo < thi) {
    f32x16 x0 = xload(tlo);
    cdma(tlo, 0);
    stage_barrier<0>();
    f32x16 x1;
    for (int64_t T = tlo; T < thi; T += 2) {
      step(T, 0, x0, x1);
      if (T + 1 < thi) step(T + 1, 1, x1, x0);
    }
  }
  if (active) {
    float* wp = Wpart + (int64_t)r * K * Mpad;
    const float* inv = Csc + KP;  // 2^-w_kk, loaded together as the column pass's scales
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float kv[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) kv[i] = inv[32 * b + row32(i, half)];
      load_order();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int kk = 32 * b + row32(i, half);
        if (kk < K) wp[(int64_t)kk * Mpad + m0 + lc] = ldexpf(WT[b][i], -vcur) * kv[i];
      }
    }
  }
}

template <int KP, typename XT>
__global__ __launch_bounds__(256, 2) void k_rowpass(const XT* X, int64_t M, int64_t N, int K,
                                                    const f32x4* __restrict__ Cq, const float* __restrict__ Csc,
                                                    const _Float16* __restrict__ Bq, float* __restrict__ Wpart,
                                                    int64_t Mpad, int64_t nchunks, const int64_t* __restrict__ tb,
                                                    int R, int nsg) {
  rowpass_body<KP, XT>(X, M, N, K, Cq, Csc, Bq, Wpart, Mpad, nchunks, tb, R, nsg, blockIdx.x);
}

template <int KP>
__global__ __launch_bounds__(256, 2) void k_rowpass_rw(float* Rr, int64_t M, int64_t N, int K,
                                                       const f32x4* __restrict__ Cq, const f32x4* __restrict__ CqD,
                                                       const float* __restrict__ Csc,
                                                       const _Float16* __restrict__ Bq, float* __restrict__ Wpart,
                                                       int64_t Mpad, int64_t nchunks, const int64_t* __restrict__ tb,
                                                       int R, int nsg) {
  rowpass_body<KP, float, true>(Rr, M, N, K, Cq, Csc, Bq, Wpart, Mpad, nchunks, tb, R, nsg, blockIdx.x, CqD, Rr);
}

hipError_t rowpass_carry(const Shape& s, float* Rr, const void* Cqv, const void* CqDv, const float* Csc,
                         const _Float16* Bq, float* Wpart, const int64_t* tb, int R, hipStream_t st) {
  const f32x4* Cq = static_cast<const f32x4*>(Cqv);
  const f32x4* CqD = static_cast<const f32x4*>(CqDv);
  const int nsg = (int)((s.nchunks + 3) / 4);
  const unsigned g = (unsigned)(((int64_t)nsg * R + 7) / 8 * 8);
  if (s.KP == 32)
    k_rowpass_rw<32><<<g, 256, 0, st>>>(Rr, s.M, s.N, s.K, Cq, CqD, Csc, Bq, Wpart, s.Mpad, s.nchunks, tb, R, nsg);
  else
    k_rowpass_rw<64><<<g, 256, 0, st>>>(Rr, s.M, s.N, s.K, Cq, CqD, Csc, Bq, Wpart, s.Mpad, s.nchunks, tb, R, nsg);
  return hipGetLastError();
}

template <typename XT>
static void rowpass_launch(const Shape& s, const XT* X, const f32x4* Cq, const float* Csc, const _Float16* Bq,
                           float* Wpart, const int64_t* tb, int R, hipStream_t st) {
  const int nsg = (int)((s.nchunks + 3) / 4);
  const unsigned g = (unsigned)(((int64_t)nsg * R + 7) / 8 * 8);
  if (s.KP == 32)
    k_rowpass<32, XT><<<g, 256, 0, st>>>(X, s.M, s.N, s.K, Cq, Csc, Bq, Wpart, s.Mpad, s.nchunks, tb, R, nsg);
  else
    k_rowpass<64, XT><<<g, 256, 0, st>>>(X, s.M, s.N, s.K, Cq, Csc, Bq, Wpart, s.Mpad, s.nchunks, tb, R, nsg);
}

hipError_t rowpass(const Shape& s, const void* X, const void* Cqv, const float* Csc, const _Float16* Bq,
                   float* Wpart, const int64_t* tb, int R, hipStream_t st) {
  const f32x4* Cq = static_cast<const f32x4*>(Cqv);
  if (s.xbf16)
    rowpass_launch(s, static_cast<const __bf16*>(X), Cq, Csc, Bq, Wpart, tb, R, st);
  else if (s.xtiled)
    rowpass_launch(s, static_cast<const xtf32*>(X), Cq, Csc, Bq, Wpart, tb, R, st);
  else
    rowpass_launch(s, static_cast<const float*>(X), Cq, Csc, Bq, Wpart, tb, R, st);
  return hipGetLastError();
}

// ------------------------------------------------------------------ reductions
// The fixed-order sums below issue the loads of their terms in groups ahead of the
// additions, which still take the terms one at a time in order: a thread then waits for one
// memory round trip per group instead of one per term (a plain loop over a run-time count
// is compiled as load, wait, add).

// W[kk][m] = sum_r Wpart[r][kk][m], r ascending, float64 (blocks of 256 entries).
__device__ __forceinline__ void reduce_w_body(const float* __restrict__ Wpart, int R, int64_t n,
                                              double* __restrict__ W, int64_t bid) {
  const int64_t i = bid * 256 + threadIdx.x;
  if (i >= n) return;
  constexpr int G = 16;
  const float* wp = Wpart + i;
  double s = 0.0;
  int r = 0;
  for (; r + G <= R; r += G) {
    float v[G];
#pragma unroll
    for (int u = 0; u < G; ++u) v[u] = wp[(int64_t)(r + u) * n];
#pragma unroll
    for (int u = 0; u < G; ++u) s += (double)v[u];
  }
  for (; r < R; ++r) s += (double)wp[(int64_t)r * n];
  W[i] = s;
}

// full[a][b] = full[b][a] = sum_p part[p][pair(a,b)] over the NP pairs of the partials (a < KP;
// entries of full past them keep their value), in a fixed order.  A block of 256
// threads takes kSymPairs consecutive pairs with 32 threads each: thread (t, qi) =
// (tid / 8, tid % 8) adds the partials p = t, t + 32, t + 64, ... in turn, then the 32
// sums of a pair are combined by a fixed tree (xor shuffles within each wave, then the
// four waves in order).  Every thread reaches the barrier.
constexpr int kSymPairs = 8;
__device__ __forceinline__ void reduce_sym_body(const double* __restrict__ part, int64_t P, int NP, int KP,
                                                double* __restrict__ full, int64_t bid) {
  __shared__ double ws[4][kSymPairs];
  const int tid = threadIdx.x, qi = tid & (kSymPairs - 1), t = tid / kSymPairs, wave = tid >> 6;
  const int q = (int)bid * kSymPairs + qi;
  double s = 0.0;
  if (q < NP) {
    constexpr int64_t D = 256 / kSymPairs;  // stride between a thread's partials
    constexpr int G = 8;
    int64_t p = t;
    for (; p + (G - 1) * D < P; p += G * D) {
      double v[G];
#pragma unroll
      for (int u = 0; u < G; ++u) v[u] = part[(p + u * D) * NP + q];
#pragma unroll
      for (int u = 0; u < G; ++u) s += v[u];
    }
    for (; p < P; p += D) s += part[p * NP + q];
  }
  // lanes qi + 8 t' of a wave (t' = t % 8) hold the same pair
  s += __shfl_xor(s, 8, 64);
  s += __shfl_xor(s, 16, 64);
  s += __shfl_xor(s, 32, 64);
  if ((tid & 63) < kSymPairs) ws[wave][qi] = s;
  __syncthreads();
  if (tid < kSymPairs && q < NP) {
    const double v = (ws[0][qi] + ws[1][qi]) + (ws[2][qi] + ws[3][qi]);
    int a, b;
    pair_of(q, a, b);
    full[a * KP + b] = v;
    full[b * KP + a] = v;
  }
}

// scale * sum_p part[p] by a block of TB threads: each thread sums a strided subset in order,
// then a fixed tree over the block; the result is returned to every thread.
template <int TB>
__device__ __forceinline__ double reduce_f_body(const double* __restrict__ part, int64_t P, double scale) {
  __shared__ double s[TB];
  constexpr int G = 8;
  double a = 0.0;
  int64_t p = threadIdx.x;
  for (; p + (G - 1) * TB < P; p += G * TB) {
    double v[G];
#pragma unroll
    for (int u = 0; u < G; ++u) v[u] = part[p + u * TB];
#pragma unroll
    for (int u = 0; u < G; ++u) a += v[u];
  }
  for (; p < P; p += TB) a += part[p];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int w = TB / 2; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  const double r = scale * s[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(256) void k_reduce_f(const double* __restrict__ part, int64_t P, double* out,
                                                  double scale) {
  const double r = reduce_f_body<256>(part, P, scale);
  if (threadIdx.x == 0) *out = r;
}

hipError_t reduce_f(const double* part, int64_t P, double* out, double scale, hipStream_t st) {
  k_reduce_f<<<1, 256, 0, st>>>(part, P, out, scale);
  return hipGetLastError();
}

// The objective of an iteration into the history ring at the device iteration counter,
// which then advances: no host value is baked into the launch, so a captured iteration
// can be replayed.  fcur (may be null) receives the objective too.
template <int TB>
__device__ __forceinline__ void f_hist_body(const double* __restrict__ part, int64_t P, double* __restrict__ fhist,
                                            int64_t cap, int64_t* __restrict__ tdev, double* __restrict__ fcur) {
  const double r = reduce_f_body<TB>(part, P, 0.5);
  if (threadIdx.x == 0) {
    const int64_t t = *tdev;
    fhist[t % cap] = r;
    *tdev = t + 1;
    if (fcur) *fcur = r;
  }
}

// Launches of several small stages that wait for the same one: the W order of C with V's
// partials and the objective (last block); the sums of the W and V partials; the sum of G's
// partials with the H order of B.  (As kernels of their own these and two clears of the maxima
// made thirteen launches per iteration, 2 to 4.6 us each beside the work; now seven.)
template <int KP>
__global__ __launch_bounds__(64 * kVWaves, 2) void k_packv(const float* __restrict__ C, f32x4* __restrict__ Cq,
                                                           float* __restrict__ Csc, int64_t N, int K,
                                                           double* __restrict__ Vpart, int nblk,
                                                           const double* __restrict__ fpart, int64_t P,
                                                           double* __restrict__ fhist, int64_t cap,
                                                           int64_t* __restrict__ tdev) {
  __shared__ PackvLds<KP> S;
  if ((int)blockIdx.x < nblk)
    packv_body<KP, true>(S, C, Cq, Csc, N, K, Vpart, blockIdx.x, nblk);
  else
    f_hist_body<64 * kVWaves>(fpart, P, fhist, cap, tdev, nullptr);
}

hipError_t packv(const Shape& s, const float* C, void* Cq, float* Csc, double* Vpart, const double* fpart,
                 double* fhist, int64_t cap, int64_t* tdev, hipStream_t st) {
  const int g = (int)vgram_blocks(s);
  f32x4* q = static_cast<f32x4*>(Cq);
  if (s.KP == 32)
    k_packv<32><<<g + 1, 64 * kVWaves, 0, st>>>(C, q, Csc, s.N, s.K, Vpart, g, fpart, colpass_blocks(s), fhist, cap, tdev);
  else
    k_packv<64><<<g + 1, 64 * kVWaves, 0, st>>>(C, q, Csc, s.N, s.K, Vpart, g, fpart, colpass_blocks(s), fhist, cap, tdev);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_reduce_wv(const float* __restrict__ Wpart, int R, int64_t n,
                                                   double* __restrict__ W, const double* __restrict__ Vpart,
                                                   int64_t P, int NP, int KP, double* __restrict__ V) {
  const int64_t nw = (n + 255) / 256;
  if (blockIdx.x < nw)
    reduce_w_body(Wpart, R, n, W, blockIdx.x);
  else
    reduce_sym_body(Vpart, P, NP, KP, V, blockIdx.x - nw);
}

hipError_t reduce_wv(const Shape& s, const float* Wpart, int R, double* W, const double* Vpart, double* V,
                     hipStream_t st) {
  const int64_t n = (int64_t)s.K * s.Mpad;
  const int NP = g_pairs(s.K);
  const int64_t g = (n + 255) / 256 + (NP + kSymPairs - 1) / kSymPairs;
  k_reduce_wv<<<(unsigned)g, 256, 0, st>>>(Wpart, R, n, W, Vpart, vgram_blocks(s), NP, s.KP, V);
  return hipGetLastError();
}

template <int KP>
__device__ __forceinline__ void finish_b_body(const double* __restrict__ Gpart, int64_t P, double* __restrict__ G,
                                              const float* __restrict__ B, int64_t M, int K, int64_t nchunks,
                                              _Float16* __restrict__ Bq, float* __restrict__ Bsc, int64_t bid) {
  const int np = g_pairs(K);
  const int64_t ng = (np + kSymPairs - 1) / kSymPairs;
  if (bid < ng)
    reduce_sym_body(Gpart, P, np, KP, G, bid);
  else
    packh_body<KP>(B, M, K, nchunks, Bq, Bsc, bid - ng);
}

template <int KP>
__global__ __launch_bounds__(256) void k_finish_b(const double* __restrict__ Gpart, int64_t P, double* __restrict__ G,
                                                  const float* __restrict__ B, int64_t M, int K, int64_t nchunks,
                                                  _Float16* __restrict__ Bq, float* __restrict__ Bsc) {
  finish_b_body<KP>(Gpart, P, G, B, M, K, nchunks, Bq, Bsc, blockIdx.x);
}

hipError_t finish_b(const Shape& s, const double* Gpart, double* G, const float* B, _Float16* Bq, float* Bsc,
                    hipStream_t st) {
  const int64_t ng = (g_pairs(s.K) + kSymPairs - 1) / kSymPairs;
  const int64_t P = bupdate_blocks(s);
  const unsigned g = (unsigned)(ng + (s.thin ? 0 : P));  // the thin path packs nothing
  if (s.KP == 32)
    k_finish_b<32><<<g, 256, 0, st>>>(Gpart, P, G, B, s.M, s.K, s.nchunks, Bq, Bsc);
  else
    k_finish_b<64><<<g, 256, 0, st>>>(Gpart, P, G, B, s.M, s.K, s.nchunks, Bq, Bsc);
  return hipGetLastError();
}

// ------------------------------------------------------------------ batched form
// Grouped persistent kernels: block b takes items b, b + grid, b + 2 grid, ... of the
// stage's concatenated item list, finds the owning instance by binary search over the
// item prefix, and runs the stage's device code for that instance and local block index.
// The row pass's items of each instance start at a multiple of 8 and every grid is a
// multiple of 8, so an item's XCD (block index mod 8) is the same as in the instance's
// own launch.
__device__ __forceinline__ int ginst_find(const GTable* __restrict__ g, int st, int64_t w) {
  int lo = 0, hi = g->n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (g->begin[st][mid] <= w)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// A pointer of the table (generic, wave-uniform) as one into global memory; through an integer
// that the compiler cannot see through, or it folds the casts away and emits flat accesses.
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
  uint64_t u = (uint64_t)(uintptr_t)p;
  asm("" : "+s"(u));
  return (T*)(__attribute__((address_space(1))) T*)u;
}

#define DID_GROUP_LOOP(ST)                                                     \
  const int64_t total_ = g->total[ST];                                        \
  for (int64_t w_ = blockIdx.x; w_ < total_; w_ += gridDim.x) {               \
    const int i_ = ginst_find(g, ST, w_);                                      \
    const GInst& d = g->inst[i_];                                              \
    const int64_t bid = w_ - g->begin[ST][i_];

#define DID_GROUP_END \
  __syncthreads();    \
  }

template <int KP, typename XT, int WPB>
__global__ __launch_bounds__(64 * WPB, 8 / WPB) void kg_colpass(const GTable* __restrict__ g) {
  DID_GROUP_LOOP(GS_COL)
  // global pointers (the table's are generic): after a flat load every wait would be for all
  // loads, and the passes count theirs
  colpass_body<KP, true, XT, false, WPB>(as_global(static_cast<const XT*>(d.X)), d.M, d.N, d.K,
                                         as_global(static_cast<const f32x4*>(d.Cq)), as_global(d.Bq), as_global(d.Bsc),
                                         as_global(d.Csc), as_global(d.H), as_global(d.fpart), d.nchunks, d.csplit, bid);
  DID_GROUP_END
}

template <int KP>
__global__ __launch_bounds__(256, 2) void kg_sweep(const GTable* __restrict__ g) {
  constexpr int NL = KP / 16 - 1;  // 16-coordinate blocks of the class's smaller half
  __shared__ union {
    SweepLds<NL> lo;
    SweepLds<NL + 1> hi;
  } S;
  extern __shared__ __align__(16) float lines[];
  DID_GROUP_LOOP(GS_SWEEP)
  // the table's pointers are generic: as global ones the many loads take scalar bases
  const float* H = as_global(d.H);
  float* C = as_global(d.C);
  f32x4* Cq = as_global(static_cast<f32x4*>(d.Cq));
  const double* G = as_global(d.G);
  if (d.K <= 16 * NL) {
    if (sweep_u(d.N) == 1)
      sweep_body<KP, NL, 1, false>(S.lo, lines, H, d.csplit, C, Cq, d.Csc, d.N, d.K, G, bid, nullptr);
    else
      sweep_body<KP, NL, 4, false>(S.lo, lines, H, d.csplit, C, Cq, d.Csc, d.N, d.K, G, bid, nullptr);
  } else {
    if (sweep_u(d.N) == 1)
      sweep_body<KP, NL + 1, 1, false>(S.hi, lines, H, d.csplit, C, Cq, d.Csc, d.N, d.K, G, bid, nullptr);
    else
      sweep_body<KP, NL + 1, 4, false>(S.hi, lines, H, d.csplit, C, Cq, d.Csc, d.N, d.K, G, bid, nullptr);
  }
  DID_GROUP_END
}

template <int KP>
__global__ __launch_bounds__(64 * kVWaves, 2) void kg_packv(const GTable* __restrict__ g) {
  __shared__ PackvLds<KP> S;
  DID_GROUP_LOOP(GS_PACKV)
  if (bid < d.vblocks)
    packv_body<KP, false>(S, as_global(d.C), as_global(static_cast<f32x4*>(d.Cq)), as_global(d.Csc), d.N, d.K,
                          d.Vpart, bid, d.vblocks);
  else
    f_hist_body<64 * kVWaves>(d.fpart, d.colblocks, d.fhist, d.hist_cap, d.tdev, d.fcur);
  DID_GROUP_END
}

template <int KP, typename XT>
__global__ __launch_bounds__(256, 2) void kg_rowpass(const GTable* __restrict__ g) {
  DID_GROUP_LOOP(GS_ROW)
  rowpass_body<KP, XT>(as_global(static_cast<const XT*>(d.XR)), d.M, d.N, d.K,
                       as_global(static_cast<const f32x4*>(d.Cq)), as_global(d.Csc), as_global(d.Bq),
                       as_global(d.Wpart), d.Mpad, d.nchunks, as_global(d.tb), d.R, d.nsg, bid);
  DID_GROUP_END
}

template <int KP>
__global__ __launch_bounds__(256) void kg_reduce_wv(const GTable* __restrict__ g) {
  DID_GROUP_LOOP(GS_REDWV)
  const int64_t n = (int64_t)d.K * d.Mpad, nw = (n + 255) / 256;
  if (bid < nw)
    reduce_w_body(d.Wpart, d.R, n, d.W, bid);
  else
    reduce_sym_body(d.Vpart, d.vblocks, g_pairs(d.K), KP, d.V, bid - nw);
  DID_GROUP_END
}

template <int KP>
__global__ __launch_bounds__(256, 2) void kg_bupdate(const GTable* __restrict__ g) {
  constexpr int NL = KP / 16 - 1;
  __shared__ union {
    BupLds<NL> lo;
    BupLds<NL + 1> hi;
  } S;
  extern __shared__ __align__(16) float lines[];
  DID_GROUP_LOOP(GS_BUP)
  float* B = as_global(d.B);
  const double* W = as_global(d.W);
  const double* V = as_global(d.V);
  if (d.K <= 16 * NL)
    bupdate_body<KP, NL, false>(S.lo, lines, B, d.M, d.K, W, d.Mpad, V, d.Bq, d.Bsc, d.Gpart, 1, bid, nullptr);
  else
    bupdate_body<KP, NL + 1, false>(S.hi, lines, B, d.M, d.K, W, d.Mpad, V, d.Bq, d.Bsc, d.Gpart, 1, bid, nullptr);
  DID_GROUP_END
}

template <int KP>
__global__ __launch_bounds__(256) void kg_finish_b(const GTable* __restrict__ g) {
  DID_GROUP_LOOP(GS_FIN)
  finish_b_body<KP>(d.Gpart, d.bupblocks, d.G, d.B, d.M, d.K, d.nchunks, d.Bq, d.Bsc, bid);
  DID_GROUP_END
}

#undef DID_GROUP_LOOP
#undef DID_GROUP_END

void ginst_items(const Shape& s, int R, int64_t items[GS_N]) {
  const int64_t ng = (g_pairs(s.K) + kSymPairs - 1) / kSymPairs;
  const int64_t nsg = (s.nchunks + 3) / 4;
  items[GS_COL] = colpass_blocks(s);
  items[GS_SWEEP] = sweep_blocks(s.N);
  items[GS_PACKV] = vgram_blocks(s) + 1;
  items[GS_ROW] = (nsg * R + 7) / 8 * 8;
  items[GS_REDWV] = ((int64_t)s.K * s.Mpad + 255) / 256 + ng;
  items[GS_BUP] = bupdate_blocks(s);
  items[GS_FIN] = ng + bupdate_blocks(s);
}

template <int KP, typename XT, int WPB>
static hipError_t group_grids_t(int64_t grids[GS_N]) {
  int dev = 0, cus = 0;
  hipError_t e;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  auto occ = [&](const void* fn, int threads, size_t lds, int64_t* out) {
    int per = 0;
    hipError_t r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, threads, lds);
    // multiple of 8 (one block per XCD round), at least one round
    *out = ((int64_t)std::max(per, 1) * cus + 7) / 8 * 8;
    return r;
  };
  if ((e = occ((const void*)kg_colpass<KP, XT, WPB>, 64 * WPB, 0, &grids[GS_COL])) != hipSuccess) return e;
  if ((e = occ((const void*)kg_sweep<KP>, 256, sweep_dyn_lds(KP, 4, false), &grids[GS_SWEEP])) != hipSuccess) return e;
  if ((e = occ((const void*)kg_packv<KP>, 64 * kVWaves, 0, &grids[GS_PACKV])) != hipSuccess) return e;
  if ((e = occ((const void*)kg_rowpass<KP, XT>, 256, 0, &grids[GS_ROW])) != hipSuccess) return e;
  if ((e = occ((const void*)kg_reduce_wv<KP>, 256, 0, &grids[GS_REDWV])) != hipSuccess) return e;
  if ((e = occ((const void*)kg_bupdate<KP>, 256, bup_dyn_lds(KP, false), &grids[GS_BUP])) != hipSuccess) return e;
  if ((e = occ((const void*)kg_finish_b<KP>, 256, 0, &grids[GS_FIN])) != hipSuccess) return e;
  return hipSuccess;
}

template <int KP, typename XT>
static hipError_t group_grids_k(int cwpb, int64_t grids[GS_N]) {
  return cwpb == 8 ? group_grids_t<KP, XT, 8>(grids) : group_grids_t<KP, XT, 4>(grids);
}

hipError_t group_grids(int KP, int xkind, int cwpb, int64_t grids[GS_N]) {
  if (KP == 32) {
    if (xkind == XK_BF16) return group_grids_k<32, __bf16>(cwpb, grids);
    if (xkind == XK_F32_TILED) return group_grids_k<32, xtf32>(cwpb, grids);
    return group_grids_k<32, float>(cwpb, grids);
  }
  if (xkind == XK_BF16) return group_grids_k<64, __bf16>(cwpb, grids);
  if (xkind == XK_F32_TILED) return group_grids_k<64, xtf32>(cwpb, grids);
  return group_grids_k<64, float>(cwpb, grids);
}

template <int KP, typename XT, int WPB>
static void group_iteration_t(const GTable* t, const int64_t* gr, hipStream_t st) {
  kg_colpass<KP, XT, WPB><<<(unsigned)gr[GS_COL], 64 * WPB, 0, st>>>(t);
  kg_sweep<KP><<<(unsigned)gr[GS_SWEEP], 256, sweep_dyn_lds(KP, 4, false), st>>>(t);
  kg_packv<KP><<<(unsigned)gr[GS_PACKV], 64 * kVWaves, 0, st>>>(t);
  kg_rowpass<KP, XT><<<(unsigned)gr[GS_ROW], 256, 0, st>>>(t);
  kg_reduce_wv<KP><<<(unsigned)gr[GS_REDWV], 256, 0, st>>>(t);
  kg_bupdate<KP><<<(unsigned)gr[GS_BUP], 256, bup_dyn_lds(KP, false), st>>>(t);
  kg_finish_b<KP><<<(unsigned)gr[GS_FIN], 256, 0, st>>>(t);
}

template <int KP, typename XT>
static void group_iteration_k(int cwpb, const GTable* t, const int64_t* gr, hipStream_t st) {
  if (cwpb == 8)
    group_iteration_t<KP, XT, 8>(t, gr, st);
  else
    group_iteration_t<KP, XT, 4>(t, gr, st);
}

hipError_t group_iteration(int KP, int xkind, int cwpb, const GTable* dtab, const int64_t grids[GS_N],
                           hipStream_t st) {
  if (KP == 32) {
    if (xkind == XK_BF16)
      group_iteration_k<32, __bf16>(cwpb, dtab, grids, st);
    else if (xkind == XK_F32_TILED)
      group_iteration_k<32, xtf32>(cwpb, dtab, grids, st);
    else
      group_iteration_k<32, float>(cwpb, dtab, grids, st);
  } else {
    if (xkind == XK_BF16)
      group_iteration_k<64, __bf16>(cwpb, dtab, grids, st);
    else if (xkind == XK_F32_TILED)
      group_iteration_k<64, xtf32>(cwpb, dtab, grids, st);
    else
      group_iteration_k<64, float>(cwpb, dtab, grids, st);
  }
  return hipGetLastError();
}

}  // namespace didk
