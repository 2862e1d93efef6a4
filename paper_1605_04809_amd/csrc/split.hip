// split.hip -- fp32 products on the fp16 matrix cores (gfx950).
//
// The fp32 matrix pipe does 1/16 of the fp16 one's flops per cycle.  Here an
// fp32 value x, scaled by a power of two, is held as two fp16 halves
// hi = fp16(x) and lo = fp16(x - hi), 22 significant bits and a sign, and a
// product is three fp16 MFMAs into one fp32 accumulator:
//     x y = x_lo y_hi + x_hi y_lo + x_hi y_hi
// (x_lo y_lo, 2^-22 of the product, is dropped).  The dropped bits err by
// about 2^-23.7 rms per term, independently from term to term, and the
// accumulator is rounded once per 16 terms and product instead of once per
// two terms, so the sum errs less than the fp32 MFMA's own: against 64-bit
// sums of N(0,1/K) weights and tanh(N(0,1)) activations 2.6e-7 against
// 4.1e-7 relative at K = 504, 3.5e-7 against 5.7e-7 at K = 1,024 and 5.0e-7
// against 8.1e-7 at K = 2,048.
//
// Range.  fp16 holds 2^-24 .. 65504, so both sides are scaled: a weight
// matrix by the power of two that puts its largest magnitude in [2^14, 2^15),
// activations by a fixed one (their magnitudes are at most 1: GRU states,
// annotations and tanh readouts).  An element's absolute error then is at
// most 2^-39 of its matrix's largest element, below fp32's own rounding of
// any column whose largest element is within 2^-14 of the matrix's; models
// with other weights (and non-finite ones) keep the fp32 MFMA kernels
// (split_scale, checked when the model is made).  A row of activations the
// halves would hold less precisely than fp32 (a caller's states or
// annotations can hold any fp32 value) is found while it is staged, and
// computed again with the fp32 MFMA (k_gemm_sp's rows outside the range).
// Readouts and the encoder's states need no such check: they come out of
// tanhf_ or a cell with an absolute error of a few 2^-24, next to which the
// halves' 2^-39 and 2^-37 do not count.  The splitting of an operand into
// the parts a narrower format holds is Dekker's (1971); on matrix units see
// Markidis et al. (2018) and Ootomo and Yokota (2022).
//
// Weights are packed by the wave: [32-column block][16-k step][hi, lo]
// [k half][column][8 halves], so a wave's fragment is one contiguous 1 KB
// load and its whole column block one contiguous stream.
#include <algorithm>
#include <cmath>

#include "internal.hpp"

namespace nmt {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma16(const f32x4& a, const f32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Eight fp32 values times `scale` as fp16 halves (16 raw bytes each).  The
// scaled value is kept in a register (the empty asm), or the compiler rounds
// it to fp16 a second time for the remainder: two conversions per pair and
// one mixed-precision subtraction per value.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split8(const f32x4& x0, const f32x4& x1, float scale, f32x4& hi, f32x4& lo) {
  f16x8 h, l;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    f32x2 x;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      x[u] = (e + u < 4 ? x0[e + u] : x1[e + u - 4]) * scale;
      asm("" : "+v"(x[u]));
    }
    const f16x2 y = __builtin_convertvector(x, f16x2);
    h[e] = y[0];
    h[e + 1] = y[1];
    l[e] = (_Float16)(x[0] - (float)y[0]);
    l[e + 1] = (_Float16)(x[1] - (float)y[1]);
  }
  hi = __builtin_bit_cast(f32x4, h);
  lo = __builtin_bit_cast(f32x4, l);
}

// --------------------------------------------------------- packing

// A wave's share of a matrix's range: the largest of its lanes' magnitudes
// (bits of |x|, so inf and NaN sort above every finite value) and the
// smallest that is not zero.
__device__ __forceinline__ void add_range(uint32_t m, MagRange* __restrict__ r) {
  uint32_t most = m, least = m ? m : ~0u;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    most = max(most, (uint32_t)__shfl_xor(most, o, 64));
    least = min(least, (uint32_t)__shfl_xor(least, o, 64));
  }
  if ((threadIdx.x & 63) == 0 && most) {
    atomicMax(&r->most, most);
    atomicMin(&r->least, least);
  }
}

// The largest magnitude of a vector's first n elements.  (Each element goes
// through a float of its own: __builtin_bit_cast of a vector's element takes
// the vector's first element whatever the index.)
__device__ __forceinline__ uint32_t vec_magnitude(const f32x4& x, int n) {
  uint32_t m = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float f = x[e];
    const uint32_t b = __builtin_bit_cast(uint32_t, f) & 0x7fffffffu;
    m = e < n ? max(m, b) : m;
  }
  return m;
}

// Range of the packed columns' largest magnitudes over W's first K rows, W
// [Kpad/4][Npad][4].  16 waves share the rows of 64 columns: one thread per
// column, its loads one after another, took 190 us a matrix on average over a
// model's matrices at the paper's sizes.
__global__ __launch_bounds__(1024) void k_column_range(const f32x4* __restrict__ W, int64_t Npad, int K,
                                                       MagRange* __restrict__ out) {
  __shared__ uint32_t part[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n = (int64_t)blockIdx.x * 64 + lane;
  uint32_t m = 0;
  if (n < Npad)
    for (int v = wave; 4 * v < K; v += 16) m = max(m, vec_magnitude(W[(int64_t)v * Npad + n], K - 4 * v));
  part[wave][lane] = m;
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int w = 1; w < 16; ++w) m = max(m, part[w][lane]);
  add_range(m, out);
}

// The same of the rows of a row-major [rows x E] table, E a multiple of 4: a
// wave takes every (16 gridDim.x)-th row and keeps its lanes' largest, then
// smallest, row.
__global__ __launch_bounds__(1024) void k_row_range(const float* __restrict__ x, int64_t rows, int E,
                                                    MagRange* __restrict__ out) {
  __shared__ uint32_t most_s[16], least_s[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t most = 0, least = ~0u;
  for (int64_t r = (int64_t)blockIdx.x * 16 + wave; r < rows; r += (int64_t)gridDim.x * 16) {
    uint32_t m = 0;
    for (int k = 4 * lane; k < E; k += 256) m = max(m, vec_magnitude(*(const f32x4*)(x + r * E + k), 4));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = max(m, (uint32_t)__shfl_xor(m, o, 64));
    most = max(most, m);
    if (m) least = min(least, m);
  }
  if (lane == 0) {
    most_s[wave] = most;
    least_s[wave] = least;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < 16; ++w) {
    most = max(most, most_s[w]);
    least = min(least, least_s[w]);
  }
  if (most) {
    atomicMax(&out->most, most);
    atomicMin(&out->least, least);
  }
}

// Range of the finite magnitudes of packed row krow (the output bias).
__global__ __launch_bounds__(256) void k_bias_range(const float* __restrict__ W, int64_t Npad, int krow,
                                                    MagRange* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const float f = i < Npad ? W[((int64_t)(krow / 4) * Npad + i) * 4 + krow % 4] : 0.f;
  const uint32_t b = __builtin_bit_cast(uint32_t, f) & 0x7fffffffu;
  add_range(b < 0x7f800000u ? b : 0, out);
}

__global__ void k_no_range(MagRange* __restrict__ r, int n) {
  if ((int)threadIdx.x < n) r[threadIdx.x] = MagRange{0, ~0u};
}

hipError_t launch_no_range(MagRange* r, int n, hipStream_t st) {
  if (n > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_no_range, dim3(1), dim3(64), 0, st, r, n);
  return hipGetLastError();
}
hipError_t launch_column_range(const Packed& W, int K, MagRange* out, hipStream_t st) {
  hipLaunchKernelGGL(k_column_range, dim3(ceil_div(W.Npad, 64)), dim3(1024), 0, st, (const f32x4*)W.d, W.Npad, K, out);
  return hipGetLastError();
}
hipError_t launch_row_range(const float* x, int64_t rows, int E, MagRange* out, hipStream_t st) {
  const int blocks = (int)std::min<int64_t>((rows + 15) / 16, 2048);
  hipLaunchKernelGGL(k_row_range, dim3(blocks), dim3(1024), 0, st, x, rows, E, out);
  return hipGetLastError();
}
hipError_t launch_bias_range(const Packed& W, MagRange* out, hipStream_t st) {
  hipLaunchKernelGGL(k_bias_range, dim3(ceil_div(W.Npad, 256)), dim3(256), 0, st, (const float*)W.d, W.Npad, W.Krows, out);
  return hipGetLastError();
}

int split_scale(MagRange r) {
  if (r.most >= 0x7f800000u) return kNoSplit;  // inf or NaN
  if (r.most == 0) return 0;
  const float most = __builtin_bit_cast(float, r.most), least = __builtin_bit_cast(float, r.least);
  if (least < std::ldexp(most, -14)) return kNoSplit;
  int e = 0;
  (void)std::frexp(most, &e);  // most = f 2^e, f in [1/2, 1)
  const int s = 15 - e;
  return (s < -60 || s > 60) ? kNoSplit : s;
}

int split_steps(int K, bool vocab) {
  const int n = ceil_div(K, 16);
  // the tile GEMMs walk K in whole chunks (one or two to a long K's 16
  // steps); the vocabulary kernel in blocks of four steps, or of two for a
  // short K, at least two blocks
  if (!vocab) return (int)round_up(n, K < kSpLongK ? kSpShortChunk : kSpLongChunk);
  return n >= 8 ? (int)round_up(n, 4) : std::max(4, (int)round_up(n, 2));
}
int64_t split_bytes(int64_t blocks, int steps) { return blocks * steps * 2048; }

// Block b, step s of the split copy.  gru_hb > 0: the source's packed column
// tiles hold [r | z | n] of gru_hb units, the copy's blocks r, z, n of 32.
__global__ __launch_bounds__(256) void k_split_pack(const float* __restrict__ W, int64_t Npad, int K, int steps,
                                                    int gru_hb, float scale, char* __restrict__ out, int64_t n_all) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (block, step, half, column)
  if (i >= n_all) return;  // (six steps of an odd number of blocks: half a thread block too many)
  const int col = (int)(i & 31), h = (int)(i >> 5) & 1;
  const int64_t bs = i >> 6;
  const int s = (int)(bs % steps);
  const int64_t b = bs / steps;
  int64_t n = b * 32 + col;
  if (gru_hb > 0) {
    const int64_t u = b / 3 * 32;  // first unit
    n = u / gru_hb * 3 * gru_hb + (b % 3) * gru_hb + u % gru_hb + col;
  }
  f32x4 x[2];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = s * 16 + h * 8 + e;
    x[e / 4][e % 4] = (n < Npad && k < K) ? W[((int64_t)(k / 4) * Npad + n) * 4 + k % 4] : 0.f;
  }
  f32x4 hi, lo;
  split8(x[0], x[1], scale, hi, lo);
  char* o = out + bs * 2048 + h * 512 + col * 16;
  *(f32x4*)o = hi;
  *(f32x4*)(o + 1024) = lo;
}

hipError_t launch_split_pack(const Packed& W, int K, int steps, int64_t blocks, int gru_hb, int scale, void* out,
                             hipStream_t st) {
  const int64_t n = blocks * steps * 64;
  hipLaunchKernelGGL(k_split_pack, dim3((unsigned)(n / 256 + (n % 256 != 0))), dim3(256), 0, st, (const float*)W.d,
                     W.Npad, K, steps, gru_hb, std::ldexp(1.f, scale), (char*)out, n);
  return hipGetLastError();
}

// The output bias in the accumulators' units: row Krows of the packed fp32 matrix times 2^scale.
__global__ void k_scaled_bias(const float* __restrict__ W, int64_t Npad, int krow, float scale, int64_t n,
                              float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = i < Npad ? W[((int64_t)(krow / 4) * Npad + i) * 4 + krow % 4] * scale : 0.f;
}
hipError_t launch_scaled_bias(const Packed& W, int scale, int64_t n, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_scaled_bias, dim3(ceil_div(n, 256)), dim3(256), 0, st, (const float*)W.d, W.Npad, W.Krows,
                     std::ldexp(1.f, scale), n, out);
  return hipGetLastError();
}

// ------------------------------------------------------- tile GEMM
//
// The other products of fp32 models (both decoder GRUs with the cell fused,
// the query, the readout, the source's keys and projections, the encoder and
// the per-word tables): out = epilogue(A W), A fp32 rows (gathered by an
// index or not), W packed in halves.  A block of 8 waves covers 32 RF WM
// rows and 32 CF WN columns (GRU: CF = 3, the r, z and candidate columns of
// 32 units), with each chunk's k steps shared between KS groups of waves
// whose sums meet in LDS at the end, in a fixed order.  The activations are
// split into halves as they go through registers into one of two LDS stages
// (rows XOR-swizzled by vector), a chunk of CH steps at a time; the weights
// stream from L2 straight into registers, each fragment feeding RF row
// fragments and three products.  The MFMA takes the weights as its row
// operand, so a lane's accumulator registers are runs of four consecutive
// columns (units) of one batch row and the epilogues load and store 16 bytes.
//
// What bounds it: the operands' way from L2 (544 MB a launch for a GRU of
// 2,000 rows) and the fixed ends of a block (first chunk, sums of the k
// groups, the cell's operands).  A GRU of 2,000 rows, 1,024 units: 104.2 us
// with fp32 MFMAs, 57 us here.
//
// Which tile: a larger one reads its operands from L2 less often, smaller
// ones trade that for more blocks; the k groups keep 8 waves on a CU whatever
// the tile.  The GRU takes the tile whose launch is shortest by rounds of
// blocks times their measured length (launch_gru_sp), the plain products the
// largest tile that gives every CU a block (launch_plain_sp).  K below
// kSpLongK takes one k group and short chunks, whose sums do not depend on
// the tile.
//
// Rows outside the range.  A row with an element at or beyond the halves'
// range (or an infinity), and one whose largest element is below the least
// that they hold to 2^-25 of it, is computed again by the fp32 MFMA from the
// fp32 row and the fp32 weights, and only that row's values are replaced, so
// a row's results never depend on its neighbours.  NaN needs no such path: it
// fills its row's products either way.
struct SpProblem {
  SpA A;
  const char* W;
  int64_t wbytes;
  int32_t steps, blocks;
  const f32x4* w32;
  int64_t n32;
  int32_t hb;
  float ascale, inv;
  GruEpi g;
  PlainEpi p;
};
struct SpBatch {
  SpProblem p[2];
};

__device__ __forceinline__ int table_row_sp(const int32_t* idx, int nrows, int row) {
  if (!idx) return row;
  const int r = idx[row];
  return r >= 0 && r < nrows ? r : -1;
}

// What the epilogues read besides the sums, for four consecutive columns of
// one row: loaded for several rows before any is used, so that an epilogue
// waits for memory once or twice and not once per row.
struct CellOps {
  f32x4 hp, xr, xz, xn;
};
struct PlainOps {
  f32x4 add, add2;
};
__device__ __forceinline__ f32x4 load4_or0(const float* base, int64_t off, bool ok) {
  const f32x4 v = *(const f32x4*)(base + (ok ? off : 0));
  return f32x4{ok ? v[0] : 0.f, ok ? v[1] : 0.f, ok ? v[2] : 0.f, ok ? v[3] : 0.f};
}

// The largest of N consecutive lanes' values, in all of them.
template <int N>
__device__ __forceinline__ float lanes_max(float v) {
  static_assert(N == 8 || N == 16 || N == 32, "lanes of a row");
  auto with = [&](auto ctrl) {
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf,
                                                                    0xf, true)));
  };
  with(std::integral_constant<int, 0xB1>{});              // lane ^ 1
  with(std::integral_constant<int, 0x4E>{});              // lane ^ 2
  with(std::integral_constant<int, 0x141>{});             // 7 - lane of 8
  if constexpr (N >= 16) with(std::integral_constant<int, 0x140>{});  // 15 - lane of 16
  if constexpr (N >= 32) v = fmaxf(v, __shfl_xor(v, 16, 64));
  return v;
}

template <int RF, int CF, int WM, int WN, int KS, int CH>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_sp(SpBatch batch, int nrow,
                                                                                        int ntile) {
  static_assert(WM * WN * KS == 8 && CH % KS == 0, "eight waves");
  constexpr int TM = 32 * RF * WM, NT = 512, VPC = 2 * CH;   // rows, threads, vectors per row per chunk
  constexpr int NA = TM * VPC / NT, RP = NT / VPC;            // vectors per thread per chunk, rows per pass
  constexpr int NKL = CH / KS;                                // steps per wave and chunk
  constexpr int VPF = CF == 3 ? 2 : (NKL < 4 ? NKL : 4);      // weight steps in flight
  constexpr bool GRU = CF == 3;
  static_assert(NA >= 1 && TM * VPC % NT == 0 && NKL % VPF == 0, "whole vectors, ring slots fixed within a chunk");
  __shared__ f32x4 As[2 * 2 * VPC * TM];  // [stage][vector][hi, lo][row ^ vector]
  __shared__ float row_max[TM];
  constexpr int STG = 2 * VPC * TM;
  const SpProblem& Pb = batch.p[blockIdx.y];
  const SpA A = Pb.A;
  // Blocks with ids congruent mod 8 share an XCD: each XCD takes a run of
  // tiles, rows fastest, so its L2 holds few columns' weights.
  int tile = blockIdx.x;
  if (ntile % 8 == 0) tile = (tile & 7) * (ntile / 8) + (tile >> 3);
  const int m0 = tile % nrow * TM;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int h = lane >> 5, l32 = lane & 31;
  const int wr = wave % WM, wn = wave / WM % WN, kg = wave / (WM * WN);
  const int cb0 = (tile / nrow * WN + wn) * CF;  // the wave's first 32-column block
  // the biases of the block's columns, and the rows that this lane's epilogue reads
  constexpr int BC = 32 * WN * (GRU ? 4 : CF);
  __shared__ float bias_s[BC];
  if constexpr (GRU) {
    for (int i = threadIdx.x; i < BC; i += NT) {
      const int g = i / (32 * WN), j = tile / nrow * WN * 32 + i % (32 * WN), H = Pb.g.H;
      const float* b = g < 2 ? Pb.g.brz + g * H : (g == 2 ? Pb.g.bni : Pb.g.bns);
      bias_s[i] = j < H ? b[j] : 0.f;
    }
  } else {
    for (int i = threadIdx.x; i < BC; i += NT) {
      const int n = tile / nrow * WN * CF * 32 + i;
      bias_s[i] = Pb.p.bias && n < Pb.p.N ? Pb.p.bias[n] : 0.f;
    }
  }
  int row_i[RF], ext0[RF], ext1[RF];  // GRU: rows of h and xin; plain: row of add
#pragma unroll
  for (int i = 0; i < RF; ++i) {
    const int row = m0 + 32 * (RF * wr + i) + l32;
    row_i[i] = row;
    const int rc = row < A.M ? row : 0;
    if constexpr (GRU) {
      ext0[i] = Pb.g.h && row < A.M ? table_row_sp(Pb.g.hrow, Pb.g.hrows, rc) : -1;
      ext1[i] = Pb.g.xin && row < A.M ? table_row_sp(Pb.g.xrow, Pb.g.xrows, rc) : -1;
    } else {
      ext0[i] = Pb.p.add && row < A.M ? table_row_sp(Pb.p.add_row, Pb.p.add_rows, rc) : -1;
      ext1[i] = 0;
    }
  }
  const int steps = Pb.steps, nch = (A.K > 0 && A.M > 0) ? steps / CH : 0, last = steps - 1;
  const int M = A.M, r0 = 32 * RF * wr;

  const __amdgpu_buffer_rsrc_t wres = buffer_rsrc(Pb.W, Pb.wbytes);
  int wo[CF];
#pragma unroll
  for (int f = 0; f < CF; ++f) wo[f] = cb0 + f < Pb.blocks ? lane * 16 + f * steps * 2048 : kNoLoad;
  const int wbase = cb0 < Pb.blocks ? cb0 * steps * 2048 : 0;
  auto wload = [&](f32x4 (&d)[CF][2], int c, int j) {
    const int gs = c * CH + kg * NKL + j;
    const int so = wbase + (gs < last ? gs : last) * 2048;  // past the end: re-read the last step (unused)
#pragma unroll
    for (int f = 0; f < CF; ++f) {
      d[f][0] = buf_load(wres, wo[f], so);
      d[f][1] = buf_load(wres, wo[f] + 1024, so);
    }
  };

  // staging: this thread's vectors are rows tid / VPC + RP i, vector tid % VPC of each chunk
  const __amdgpu_buffer_rsrc_t ares = buffer_rsrc(A.p, (int64_t)(A.gather ? A.gmax : M) * A.ld * 4);
  const int kin = 8 * ((int)threadIdx.x % VPC), arow = (int)threadIdx.x / VPC;
  auto row_off = [&](int row) {
    if (row >= M) return kNoLoad;
    const int r = table_row_sp(A.gather, A.gmax, row);
    return r < 0 ? kNoLoad : (int)((int64_t)r * A.ld * 4);
  };
  int aoff[NA];
  float amax[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    aoff[i] = nch > 0 ? row_off(m0 + arow + RP * i) : kNoLoad;
    amax[i] = 0.f;
  }
  f32x4 ra[NA], rb[NA];
  auto aload = [&](int c) {
    const int k = c * CH * 16 + kin;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int o = aoff[i] + kin * 4;
      ra[i] = buf_load(ares, k < A.K ? o : kNoLoad, c * CH * 64);
      rb[i] = buf_load(ares, k + 4 < A.K ? o + 16 : kNoLoad, c * CH * 64);
    }
  };
  const int sv = (int)threadIdx.x % VPC, st_base = sv * 2 * TM;
  auto astore = [&](int stage) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      f32x4 hi, lo;
      split8(ra[i], rb[i], Pb.ascale, hi, lo);
#pragma unroll
      for (int e = 0; e < 4; ++e) amax[i] = fmaxf(amax[i], fmaxf(fabsf(ra[i][e]), fabsf(rb[i][e])));
      const int r = (arow + RP * i) ^ (sv & 31);
      As[stage * STG + st_base + r] = hi;
      As[stage * STG + st_base + TM + r] = lo;
    }
  };
  auto afrag = [&](f32x4 (&d)[RF][2], int stage, int j) {
    const int v = 2 * (kg * NKL + j) + h;
    const f32x4* s = As + stage * STG + v * 2 * TM + r0 + (l32 ^ (v & 31));
#pragma unroll
    for (int i = 0; i < RF; ++i) {
      d[i][0] = s[32 * i];
      d[i][1] = s[TM + 32 * i];
    }
  };

  f32x16 acc[RF][CF];
#pragma unroll
  for (int i = 0; i < RF; ++i)
#pragma unroll
    for (int f = 0; f < CF; ++f) acc[i][f] = f32x16{};

  if (nch > 0) {  // (without a product every row's largest is 0: in range)
    f32x4 ring[VPF][CF][2];
#pragma unroll
    for (int p = 0; p < VPF; ++p) wload(ring[p], p / NKL, p % NKL);
    aload(0);
    astore(0);
    aload(nch > 1 ? 1 : 0);
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
      const int st = c & 1;
      f32x4 a[RF][2];
      afrag(a, st, 0);
      static_for<NKL>([&](auto jc) {
        constexpr int j = decltype(jc)::value, slot = j % VPF;
        f32x4 an[RF][2];
        if constexpr (j + 1 < NKL) {
          afrag(an, st, j + 1);
        }
#pragma unroll
        for (int f = 0; f < CF; ++f)
#pragma unroll
          for (int i = 0; i < RF; ++i) acc[i][f] = mfma16(ring[slot][f][1], a[i][0], acc[i][f]);
#pragma unroll
        for (int f = 0; f < CF; ++f)
#pragma unroll
          for (int i = 0; i < RF; ++i) acc[i][f] = mfma16(ring[slot][f][0], a[i][1], acc[i][f]);
#pragma unroll
        for (int f = 0; f < CF; ++f)
#pragma unroll
          for (int i = 0; i < RF; ++i) acc[i][f] = mfma16(ring[slot][f][0], a[i][0], acc[i][f]);
        wload(ring[slot], c + (j + VPF) / NKL, (j + VPF) % NKL);  // refill the slot, VPF steps ahead
        // one MFMA, the next step's fragment reads, the other MFMAs, the refill
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (j + 1 < NKL) __builtin_amdgcn_sched_group_barrier(0x100, 2 * RF, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 3 * RF * CF - 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 2 * CF, 0);
        if constexpr (j + 1 < NKL) {
#pragma unroll
          for (int i = 0; i < RF; ++i) {
            a[i][0] = an[i][0];
            a[i][1] = an[i][1];
          }
        }
      });
      if (c + 1 < nch) astore(st ^ 1);
      aload(c + 2 < nch ? c + 2 : nch - 1);
      __syncthreads();
    }
  }

  // Rows outside the halves' range: each wave computes its share of K for
  // them from fp32, 32 k of loads in flight.  (After the sums, the whole of K
  // to a wave and a load at a time, one such row took a step of 1,000 rows
  // from 136 to 520 us; 205 now, 278 where every row is one, 231 with every
  // product on the fp32 MFMA.)
  bool own[RF];  // this lane's rows: the sums are in their own units
#pragma unroll
  for (int i = 0; i < RF; ++i) own[i] = false;
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const float mx = lanes_max<VPC>(amax[i]);
    if (sv == 0) row_max[arow + RP * i] = mx;
  }
  __syncthreads();  // (the biases are there too)
  if (nch > 0) {
#pragma unroll
    for (int i = 0; i < RF; ++i) {
      const float mx = row_max[r0 + 32 * i + l32];
      own[i] = mx >= A.most || (mx > 0.f && mx < A.least);
      if (__builtin_amdgcn_ballot_w64(own[i]) == 0) continue;
      constexpr int U = 4;
      const int ro = row_off(m0 + r0 + 32 * i + l32);
      const int kw = ((A.K + KS - 1) / KS + 8 * U - 1) / (8 * U) * (8 * U), k_end = min(A.K, (kg + 1) * kw);
      int64_t n[CF];
      f32x16 s[CF];
#pragma unroll
      for (int f = 0; f < CF; ++f) {
        const int b = cb0 + f < Pb.blocks ? cb0 + f : 0;
        n[f] = (int64_t)b * 32 + l32;
        if constexpr (GRU) {
          const int u = b / 3 * 32;
          n[f] = (int64_t)(u / Pb.hb) * 3 * Pb.hb + (b % 3) * Pb.hb + u % Pb.hb + l32;
        }
        s[f] = f32x16{};
      }
      // (the packed fp32 rows go on to a multiple of 32, so every k0 has 32)
      for (int k0 = kg * kw; k0 < k_end; k0 += 8 * U) {  // lane half h holds k 4 h .. 4 h + 3 of eight
        f32x4 x[U], w[U][CF];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = k0 + 8 * u + 4 * h;
          x[u] = buf_load(ares, k < A.K ? ro + k * 4 : kNoLoad, 0);
#pragma unroll
          for (int f = 0; f < CF; ++f) w[u][f] = Pb.w32[(int64_t)(k0 / 4 + 2 * u + h) * Pb.n32 + n[f]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int f = 0; f < CF; ++f) s[f] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[u][f][e], x[u][e], s[f], 0, 0, 0);
      }
#pragma unroll
      for (int f = 0; f < CF; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][f][r] = own[i] ? s[f][r] : acc[i][f][r];
    }
  }

  // Epilogue.  A wave's sums are NP pieces (row fragment i, columns 8 q + 4 h
  // .. + 3 of each block); each of the KS waves that share them finishes NPK
  // pieces, adding the k groups' sums from LDS in order, one column block at
  // a time over two LDS regions.
  constexpr int NP = RF * 4, NPK = NP >= KS ? NP / KS : 1, WB = WM * WN;
  constexpr int NB = KS == 1 && GRU ? 2 : (NPK < 4 ? NPK : 4);  // pieces whose operands are in flight together
  const bool busy = KS == 1 || kg * NPK < NP;
  auto piece_i = [&](int t) { return KS == 1 ? t / 4 : (kg * NPK + t) / 4 % RF; };
  auto piece_q = [&](int t) { return KS == 1 ? t % 4 : (kg * NPK + t) % 4; };
  // (by value: an array picked from at run time becomes LDS storage, addressed
  // through the dispatch packet in host memory)
  const int row_0 = row_i[0], row_1 = row_i[RF - 1], e0_0 = ext0[0], e0_1 = ext0[RF - 1], e1_0 = ext1[0],
            e1_1 = ext1[RF - 1];
  const bool own_0 = own[0], own_1 = own[RF - 1];
  auto pick = [](auto x0, auto x1, int i) { return RF == 1 || i == 0 ? x0 : x1; };
  CellOps cop[GRU ? NB : 1];
  PlainOps pop[GRU ? 1 : NB][GRU ? 1 : CF];
  auto load_ops = [&](int t0) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int i = piece_i(t0 + b), q = piece_q(t0 + b);
      if constexpr (GRU) {
        const int H = Pb.g.H, j = cb0 / 3 * 32 + 8 * q + 4 * h;
        const int hr = pick(e0_0, e0_1, i), xq = pick(e1_0, e1_1, i);
        CellOps& o = cop[b];
        o.hp = o.xr = o.xz = o.xn = zero4();
        if (Pb.g.h) o.hp = load4_or0(Pb.g.h, (int64_t)hr * Pb.g.ldh + j, hr >= 0 && j < H);
        if (Pb.g.xin) {
          const bool ok = xq >= 0 && j < H;
          const int64_t x = (int64_t)xq * Pb.g.ldx + j;
          o.xr = load4_or0(Pb.g.xin, x, ok);
          o.xz = load4_or0(Pb.g.xin, x + H, ok);
          o.xn = load4_or0(Pb.g.xin, x + 2 * H, ok);
        }
      } else {
        const int ar = pick(e0_0, e0_1, i), row = pick(row_0, row_1, i);
#pragma unroll
        for (int f = 0; f < CF; ++f) {
          const int n = (cb0 + f) * 32 + 8 * q + 4 * h;
          PlainOps& o = pop[b][f];
          o.add = o.add2 = zero4();
          if (Pb.p.add) o.add = load4_or0(Pb.p.add, (int64_t)ar * Pb.p.ld_add + n, ar >= 0 && n < Pb.p.N);
          if (Pb.p.add2) o.add2 = load4_or0(Pb.p.add2, (int64_t)row * Pb.p.ld_add2 + n, row < M && n < Pb.p.N);
        }
      }
    }
  };
  if constexpr (KS > 1) load_ops(0);

  f32x4 sum[NPK][CF];
  if constexpr (KS > 1) {
    static_assert(2 * 8 * NP * 64 <= 2 * STG, "two regions of every wave's pieces fit the stages");
    f32x4* red = As;
#pragma unroll
    for (int f = 0; f < CF; ++f) {
      f32x4* reg = red + (f & 1) * 8 * NP * 64;
#pragma unroll
      for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          reg[(wave * NP + i * 4 + q) * 64 + lane] =
              f32x4{acc[i][f][4 * q], acc[i][f][4 * q + 1], acc[i][f][4 * q + 2], acc[i][f][4 * q + 3]};
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NPK; ++t) {
        f32x4 v = zero4();
        if (busy)
#pragma unroll
          for (int g = 0; g < KS; ++g) v += reg[((g * WB + wave % WB) * NP + kg * NPK + t) * 64 + lane];
        sum[t][f] = v;
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < NPK; ++t)
#pragma unroll
      for (int f = 0; f < CF; ++f) {
        const int i = t / 4, q = t % 4;
        sum[t][f] = f32x4{acc[i][f][4 * q], acc[i][f][4 * q + 1], acc[i][f][4 * q + 2], acc[i][f][4 * q + 3]};
      }
  }
  if (!busy) return;
#pragma unroll
  for (int t = 0; t < NPK; ++t) {
    const float inv = pick(own_0, own_1, piece_i(t)) ? 1.f : Pb.inv;
#pragma unroll
    for (int f = 0; f < CF; ++f) sum[t][f] *= inv;
  }

#pragma unroll
  for (int t0 = 0; t0 < NPK; t0 += NB) {
    if constexpr (KS == 1) load_ops(t0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int t = t0 + b, i = piece_i(t), q = piece_q(t), row = pick(row_0, row_1, i);
      if constexpr (GRU) {
        const GruEpi& ep = Pb.g;
        const int jl = 32 * wn + 8 * q + 4 * h, j = cb0 / 3 * 32 + 8 * q + 4 * h;
        const f32x4 br = *(const f32x4*)(bias_s + jl), bz = *(const f32x4*)(bias_s + 32 * WN + jl);
        const f32x4 bni = *(const f32x4*)(bias_s + 64 * WN + jl), bns = *(const f32x4*)(bias_s + 96 * WN + jl);
        const CellOps& o = cop[b];
        if (row >= M || j >= ep.H) continue;
        const bool keep = !ep.mask_len || ep.mask_pos < ep.mask_len[row];
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float rg = sigmoidf_(sum[t][0][e] + br[e] + o.xr[e]);
          const float zg = sigmoidf_(sum[t][1][e] + bz[e] + o.xz[e]);
          const float ng = tanhf_(bni[e] + o.xn[e] + rg * (sum[t][CF - 1][e] + bns[e]));
          const float hn = zg * o.hp[e] + (1.f - zg) * ng;
          v[e] = keep ? hn : 0.f;
        }
        *(f32x4*)(ep.out + (int64_t)row * ep.ldo + j) = v;
      } else {
        const PlainEpi& ep = Pb.p;
        const bool masked = ep.mask_len && row < M && (row % ep.mask_T) >= ep.mask_len[row / ep.mask_T];
#pragma unroll
        for (int f = 0; f < CF; ++f) {
          const int n = (cb0 + f) * 32 + 8 * q + 4 * h;
          const f32x4 bn = *(const f32x4*)(bias_s + (wn * CF + f) * 32 + 8 * q + 4 * h);
          f32x4 v = sum[t][f] + (pop[b][f].add + pop[b][f].add2);
          v += bn;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (ep.act == 1) v[e] = tanhf_(v[e]);
            if (masked) v[e] = 0.f;
          }
          if (row < M && n < ep.N) *(f32x4*)(ep.out + (int64_t)row * ep.ldo + n) = v;
        }
      }
    }
  }
}

template <int RF, int CF, int WM, int WN, int KS, int CH>
static void run_gemm_sp(const SpBatch& b, int nprob, int M, int blocks, hipStream_t st) {
  const int nrow = ceil_div(M, 32 * RF * WM), ncol = ceil_div(blocks, CF * WN);
  hipLaunchKernelGGL((k_gemm_sp<RF, CF, WM, WN, KS, CH>), dim3((unsigned)(nrow * ncol), nprob), dim3(512), 0, st, b,
                     nrow, nrow * ncol);
  g_gemm_streamed.fetch_add(1, std::memory_order_relaxed);
}

static bool sp_problem(SpProblem& P, const SpA& A, const SplitW& W) {
  P.A = A;
  P.W = (const char*)W.d;
  P.wbytes = split_bytes(W.blocks, W.steps);
  P.steps = W.steps;
  P.blocks = (int)W.blocks;
  P.A.most = std::ldexp(65504.f, -A.scale);
  P.A.least = std::ldexp(1.f, -A.scale);
  P.w32 = (const f32x4*)W.w32;
  P.n32 = W.n32;
  P.hb = W.gru_hb;
  P.ascale = std::ldexp(1.f, A.scale);
  P.inv = std::ldexp(1.f, -(A.scale + W.scale));
  if (!W.d || !W.w32 || P.wbytes >= ((int64_t)1 << 31) || A.K % 4 || A.ld % 4) return false;
  if (A.K <= 0) return true;  // no product: the epilogue alone
  return A.p && (!A.gather || A.gmax >= 1) && W.steps * 16 >= A.K && W.steps == split_steps(W.K, false) &&
         (int64_t)(A.gather ? A.gmax : A.M) * A.ld * 4 < ((int64_t)1 << 31);
}

// Blocks of a launch with 32 RF WM rows and CF WN column blocks to the tile.
static int64_t sp_blocks(int M, int blocks, int tm, int cw) { return (int64_t)ceil_div(M, tm) * ceil_div(blocks, cw); }

hipError_t launch_gru_sp(const SpA* A, const SplitW* const* W, const GruEpi* ep, int nprob, int cus, hipStream_t st) {
  if (nprob < 1 || nprob > 2) return hipErrorInvalidValue;
  SpBatch b{};
  int M = 0;
  for (int i = 0; i < nprob; ++i) {
    if (!sp_problem(b.p[i], A[i], *W[i]) || W[i]->blocks % 3 || W[i]->K != W[0]->K || W[i]->blocks != W[0]->blocks)
      return hipErrorInvalidValue;
    b.p[i].g = ep[i];
    M = std::max(M, A[i].M);
  }
  if (M <= 0) return hipSuccess;
  const int blocks = (int)W[0]->blocks;
  if (W[0]->K < kSpLongK) return hipErrorInvalidValue;  // models of fewer units keep the fp32 MFMA (kSplitMinH)
  // The tile whose launch is shortest: rounds of one block per CU, each as
  // long as one block (measured at K = 1,024, in units of the smallest
  // tile's 14.5 us: 64 x 32 21 us, 128 x 32 33 us, 128 x 64 57 us; two
  // rounds of the smallest tile, 257 to 512 rows, 26 us against 21).
  const struct {
    int tm, wn;
    double cost;
  } tiles[] = {{128, 4, 7.4}, {128, 2, 3.9}, {128, 1, 2.3}, {64, 1, 1.45}, {32, 1, 1.0}};
  int best = 0;
  double best_cost = 0;
  for (int i = 0; i < 5; ++i) {
    const double c = ceil_div(nprob * sp_blocks(M, blocks, tiles[i].tm, 3 * tiles[i].wn), cus) * tiles[i].cost;
    if (i == 0 || c < best_cost) {
      best = i;
      best_cost = c;
    }
  }
  if (best == 0)
    run_gemm_sp<2, 3, 2, 4, 1, 8>(b, nprob, M, blocks, st);
  else if (best == 1)
    run_gemm_sp<2, 3, 2, 2, 2, 8>(b, nprob, M, blocks, st);
  else if (best == 2)
    run_gemm_sp<2, 3, 2, 1, 4, 8>(b, nprob, M, blocks, st);
  else if (best == 3)
    run_gemm_sp<2, 3, 1, 1, 8, 16>(b, nprob, M, blocks, st);
  else
    run_gemm_sp<1, 3, 1, 1, 8, 16>(b, nprob, M, blocks, st);
  return hipGetLastError();
}

hipError_t launch_plain_sp(const SpA& A, const SplitW& W, const PlainEpi& ep, int cus, hipStream_t st) {
  if (A.M <= 0 || ep.N <= 0) return hipSuccess;
  SpBatch b{};
  const int blocks = ceil_div(ep.N, 32);
  if (!sp_problem(b.p[0], A, W) || blocks > W.blocks || ep.N % 4 || ep.ldo % 4 || ep.out16 || ep.ksplit > 1)
    return hipErrorInvalidValue;
  b.p[0].p = ep;
  const int M = A.M;
  auto fills = [&](int tm, int cw) { return sp_blocks(M, blocks, tm, cw) >= cus; };
  if (W.K < kSpLongK) {
    if (M > 64)
      run_gemm_sp<2, 1, 2, 4, 1, kSpShortChunk>(b, 1, M, blocks, st);
    else
      run_gemm_sp<1, 1, 2, 4, 1, kSpShortChunk>(b, 1, M, blocks, st);
  } else if (fills(128, 8)) {
    run_gemm_sp<2, 2, 2, 4, 1, 8>(b, 1, M, blocks, st);
  } else if (fills(128, 4)) {
    run_gemm_sp<2, 2, 2, 2, 2, 8>(b, 1, M, blocks, st);
  } else if (fills(128, 2)) {
    run_gemm_sp<2, 2, 2, 1, 4, 8>(b, 1, M, blocks, st);
  } else if (fills(128, 1)) {
    run_gemm_sp<2, 1, 2, 1, 4, 8>(b, 1, M, blocks, st);
  } else if (fills(64, 1)) {
    run_gemm_sp<2, 1, 1, 1, 8, 16>(b, 1, M, blocks, st);
  } else {
    run_gemm_sp<1, 1, 1, 1, 8, 16>(b, 1, M, blocks, st);
  }
  return hipGetLastError();
}

// ------------------------------------------------ vocabulary projection
//
// The vocabulary kernel of fp32 models, in the form of k_vocab_lse: a block
// of 8 waves owns VTM rows of t, kept in LDS for the whole kernel, and one
// slice of the vocabulary; each wave streams the packed halves of its 32
// column blocks, two at a time, from L2 into a register ring VPF steps deep,
// with no barrier in the main loop, and folds each group's logits into a
// running (max, sum) per row.  One step is 12 MFMAs (two column blocks, two
// row fragments, three products) for four 16-byte weight loads and four LDS
// fragment reads, 64 rows deep because a row's halves take 2 KB of LDS.  The
// bias enters as the accumulators' first term, one fp32 MFMA per
// accumulator (exact, any magnitude; 2 % of the group's MFMA cycles).
//
// What bounds it: power.  By counters at 2,000 rows, E = 500, V = 100,000 the
// matrix cores are busy 80 % of the launch, 88 % of the cycles in which a CU
// holds its block, at a core clock of about 1.55 GHz, where the chip held 2.39
// under the fp32 MFMA's form (profiles/step_counters_enru_b2000.md).  1,393 us
// with fp32 MFMAs; here 461 us with weights of sigma 0.01 and 522 us with
// unit-gain ones (383 TFLOP/s of fp32 products); 1,000 rows and V = 50,000:
// 136 us.
constexpr int kSvWaves = 8, kSvFN = 2;
constexpr int kSvVectors = 9216;  // LDS vectors of the activation tile (144 KB)

template <int VPF, int VTM>
__global__ __launch_bounds__(kSvWaves * 64) void k_vocab_sp(const float* __restrict__ t, int M, int E, int NK,
                                                            const char* __restrict__ Wp, int64_t wbytes,
                                                            const float* __restrict__ bias, int V, int nM, int nS,
                                                            float ascale, float inv, float2* __restrict__ part,
                                                            const int32_t* __restrict__ req1,
                                                            const int32_t* __restrict__ req_off, int nreq,
                                                            float* __restrict__ zreq) {
  constexpr int VNW = kSvWaves, VFN = kSvFN, FM = VTM / 32;
  __shared__ f32x4 As[kSvVectors * VTM / 64];  // [step][half][hi, lo][row]
  __shared__ float2 red[VNW][VTM];
  const int id = blockIdx.x, xcd = id & 7, slot = id >> 3;
  const int slice = (slot / nM) * 8 + xcd, mt = slot % nM;
  if (slice >= nS) return;
  const int m0 = mt * VTM;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, h = lane >> 5, l32 = lane & 31;
  const int NB = (V + 31) / 32;
  const int cb_begin = (int)((int64_t)NB * slice / nS), cb_end = (int)((int64_t)NB * (slice + 1) / nS);
  const int ngrp = (cb_end - cb_begin + VFN - 1) / VFN;
  const float kz = kLog2e * inv;  // the fold's exponents in the accumulators' units

  float run_m[FM], run_s[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    run_m[i] = -INFINITY;
    run_s[i] = 0.f;
  }
  // the requested word of each row slot with exactly one, and its group if
  // this lane will hold its logit (see k_vocab_lse)
  int rq[FM], rq_g[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = m0 + 32 * i + l32;
    rq[i] = -1;
    if (req1 && row < M) {
      if (!req_off) {
        rq[i] = req1[row];
      } else {
        const int j0 = req_off[row], j1 = req_off[row + 1];
        if (0 <= j0 && j1 == j0 + 1 && j1 <= nreq) rq[i] = req1[j0];
      }
    }
    const int cb = rq[i] >> 5;
    rq_g[i] = (rq[i] >= 0 && cb >= cb_begin && cb < cb_end && ((rq[i] >> 2) & 1) == h) ? (cb - cb_begin) / VFN : -1;
  }

  // Fragment (block, step, half-plane): one contiguous KB at a scalar offset.
  // The packed matrix has one spare zero block, so a group's missing second
  // block reads inside it.
  const __amdgpu_buffer_rsrc_t wres = buffer_rsrc(Wp, wbytes);
  const __amdgpu_buffer_rsrc_t bres = buffer_rsrc(bias, (int64_t)(NB + 1) * 128);
  const int cbytes = NK * 2048;
  const int lo0 = lane * 16, lo1 = lane * 16 + cbytes;
  const int blo = h == 0 ? l32 * 4 : kNoLoad;  // the bias rides on k = 0 of its MFMA
  auto gbase = [&](int g) { return g < ngrp ? cb_begin + g * VFN : cb_begin; };
  auto load = [&](f32x4 (&d)[VFN][2], int soff) {
    d[0][0] = buf_load(wres, lo0, soff);
    d[0][1] = buf_load(wres, lo0 + 1024, soff);
    d[1][0] = buf_load(wres, lo1, soff);
    d[1][1] = buf_load(wres, lo1 + 1024, soff);
  };
  auto load_bias = [&](float (&b)[VFN], int cb) {
#pragma unroll
    for (int f = 0; f < VFN; ++f)
      b[f] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(bres, blo, (cb + f) * 128, 0));
  };
  int sbase = gbase(wave) * cbytes;
  f32x4 ring[VPF][VFN][2];
  float bnext[VFN];
  load_bias(bnext, gbase(wave));
#pragma unroll
  for (int p = 0; p < VPF; ++p) load(ring[p], sbase + p * 2048);

  for (int idx = threadIdx.x; idx < 2 * NK * VTM; idx += VNW * 64) {
    const int m = idx % VTM, v = idx / VTM, row = m0 + m, k = 8 * v;
    f32x4 x0 = zero4(), x1 = zero4();
    if (row < M) {
      const float* r = t + (int64_t)row * E;
      if (k < E) x0 = *(const f32x4*)(r + k);
      if (k + 4 < E) x1 = *(const f32x4*)(r + k + 4);
    }
    f32x4 hi, lo;
    split8(x0, x1, ascale, hi, lo);
    As[(2 * v) * VTM + m] = hi;
    As[(2 * v + 1) * VTM + m] = lo;
  }
  __syncthreads();
  const f32x4* arow = As + h * 2 * VTM + l32;  // + 4 VTM per step, + VTM for lo
  f32x4 ae[FM][2], ao[FM][2];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    ae[i][0] = arow[32 * i];
    ae[i][1] = arow[VTM + 32 * i];
  }
  static_assert(VPF % 2 == 0, "even/odd fragment sets");

  for (int gcur = wave; gcur < ngrp; gcur += VNW) {
    f32x16 acc[FM][VFN];
    const int nbase = gbase(gcur + VNW) * cbytes;
    // accumulators start from the bias
#pragma unroll
    for (int f = 0; f < VFN; ++f)
#pragma unroll
      for (int i = 0; i < FM; ++i) acc[i][f] = __builtin_amdgcn_mfma_f32_32x32x2f32(bnext[f], 1.f, f32x16{}, 0, 0, 0);
    load_bias(bnext, gbase(gcur + VNW));
    auto kstep = [&](const f32x4* ablk, auto pc, auto last_blk, int soff) {
      constexpr int p = decltype(pc)::value;
      const f32x4* an = (decltype(last_blk)::value && p == VPF - 1) ? arow : ablk + p * 4 * VTM;
      f32x4 a[FM][2];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          if constexpr (p % 2 == 0) {
            ao[i][z] = an[z * VTM + 32 * i];
            a[i][z] = ae[i][z];
          } else {
            ae[i][z] = an[z * VTM + 32 * i];
            a[i][z] = ao[i][z];
          }
        }
#pragma unroll
      for (int f = 0; f < VFN; ++f)
#pragma unroll
        for (int i = 0; i < FM; ++i) acc[i][f] = mfma16(ring[p][f][1], a[i][0], acc[i][f]);
#pragma unroll
      for (int f = 0; f < VFN; ++f)
#pragma unroll
        for (int i = 0; i < FM; ++i) acc[i][f] = mfma16(ring[p][f][0], a[i][1], acc[i][f]);
#pragma unroll
      for (int f = 0; f < VFN; ++f)
#pragma unroll
        for (int i = 0; i < FM; ++i) acc[i][f] = mfma16(ring[p][f][0], a[i][0], acc[i][f]);
      load(ring[p], soff);
      constexpr int NMF = 3 * FM * VFN;
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2 * FM, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, NMF - 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 2 * VFN, 0);
    };
    __builtin_amdgcn_s_setprio(1);
    for (int ks0 = 0; ks0 < NK - VPF; ks0 += VPF) {
      const int s0 = sbase + (ks0 + VPF) * 2048;
      const f32x4* ablk = arow + (ks0 + 1) * 4 * VTM;
      static_for<VPF>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        kstep(ablk, pc, std::false_type{}, s0 + p * 2048);
      });
    }
    {
      const f32x4* ablk = arow + (NK - VPF + 1) * 4 * VTM;
      static_for<VPF>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        kstep(ablk, pc, std::true_type{}, nbase + p * 2048);
      });
    }
    __builtin_amdgcn_s_setprio(0);
    sbase = nbase;

    const int cb0 = cb_begin + gcur * VFN;
    if ((cb0 + VFN) * 32 > V || cb0 + VFN > cb_end) {
#pragma unroll
      for (int f = 0; f < VFN; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool ok = cb0 + f < cb_end && (cb0 + f) * 32 + acc_row(r, h) < V;
#pragma unroll
          for (int i = 0; i < FM; ++i) acc[i][f][r] = ok ? acc[i][f][r] : -INFINITY;
        }
    }
    bool hit = false;
#pragma unroll
    for (int i = 0; i < FM; ++i) hit |= rq_g[i] == gcur;
    if (__builtin_amdgcn_ballot_w64(hit)) {
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if (rq_g[i] == gcur) {
          const int d = rq[i] - 32 * cb0;
          const int idx = (d >> 5) * 16 + ((d & 31) >> 3) * 4 + (d & 3);
          float z = 0.f;
#pragma unroll
          for (int f = 0; f < VFN; ++f)
#pragma unroll
            for (int r = 0; r < 16; ++r) z = idx == 16 * f + r ? acc[i][f][r] : z;
          zreq[m0 + 32 * i + l32] = z * inv;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      float bm = acc[i][0][0];
#pragma unroll
      for (int f = 0; f < VFN; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) bm = fmaxf(bm, acc[i][f][r]);
      const float mn = fmaxf(run_m[i], bm);
      const bool none = mn == -INFINITY;
      const float sc = none ? 1.f : __builtin_amdgcn_exp2f((run_m[i] - mn) * kz);
      const float nm = none ? 0.f : -mn * kz;
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int f = 0; f < VFN; ++f)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          s0 += __builtin_amdgcn_exp2f(fmaf(acc[i][f][r], kz, nm));
          s1 += __builtin_amdgcn_exp2f(fmaf(acc[i][f][r + 1], kz, nm));
        }
      run_s[i] = fmaf(run_s[i], sc, s0 + s1);
      run_m[i] = mn;
    }
  }

#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const float om = __shfl_xor(run_m[i], 32, 64), os = __shfl_xor(run_s[i], 32, 64);
    const float mx = fmaxf(run_m[i], om);
    float s = 0.f;
    if (mx != -INFINITY)
      s = run_s[i] * __builtin_amdgcn_exp2f((run_m[i] - mx) * kz) + os * __builtin_amdgcn_exp2f((om - mx) * kz);
    if (h == 0) red[wave][32 * i + l32] = float2{mx, s};
  }
  __syncthreads();
  for (int rl = threadIdx.x; rl < VTM; rl += VNW * 64) {
    const int row = m0 + rl;
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < VNW; ++w) mx = fmaxf(mx, red[w][rl].x);
    float s = 0.f;
    if (mx != -INFINITY) {
#pragma unroll
      for (int w = 0; w < VNW; ++w) {
        const float mw = red[w][rl].x;
        if (mw != -INFINITY) s += red[w][rl].y * __builtin_amdgcn_exp2f((mw - mx) * kz);
      }
    }
    if (row < M) part[(int64_t)slice * M + row] = float2{mx * inv, s};
  }
}

// Launch time of nM row tiles in nS slices, in column blocks of a 64-row
// tile: rounds of one block per CU, each as long as its busiest SIMD's whole
// groups (two column blocks; four SIMDs share a block's groups) plus a fixed
// cost.  A 32-row tile does half the MFMAs per weight load and takes 0.6 of
// a 64-row tile's time per column block.
static double sv_cost(int nM, int nS, int NB, int cus, int tm) {
  const double rounds = (double)ceil_div((int64_t)nM * nS, cus);
  const double groups = 4.0 * ceil_div(ceil_div(ceil_div(NB, nS), kSvFN), 4);
  return rounds * (kSvFN * groups * (tm < 64 ? 0.6 : 1.0) + 8.0);
}

void split_vocab_shape(int M, int V, int cus, int* tm, int* nS) {
  const int NB = (V + 31) / 32;
  double best = 0;
  *nS = 0;
  for (int m : {64, 32}) {
    if (m < 64 && M > 1024) break;
    const int nM = ceil_div(M, m);
    for (int s = 8; s <= 256 && (s == 8 || s <= NB); s += 8) {
      const double c = sv_cost(nM, s, NB, cus, m);
      // equal times: the larger tile, and more slices (shorter blocks on average)
      if (*nS == 0 || c < best || (c == best && *tm == m)) {
        best = c;
        *nS = s;
        *tm = m;
      }
    }
  }
}

bool split_vocab_fits(int E, int64_t blocks) {
  const int nk = split_steps(E, true);
  return 4 * nk * 64 <= kSvVectors && split_bytes(blocks, nk) < ((int64_t)1 << 31);
}

hipError_t launch_vocab_sp(const float* t, int M, int E, const SplitW& W, int V, float2* part, int nS, int tm,
                           const int32_t* req1, const int32_t* req_off, int nreq, float* zreq, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!W.d || !W.bias || W.steps != split_steps(E, true) || 4 * W.steps * 64 > kSvVectors || E % 4 ||
      W.blocks < (V + 31) / 32 + 1 || (req1 && !zreq) || nS % 8 || nS < 8)
    return hipErrorInvalidValue;
  const float ascale = std::ldexp(1.f, kSplitReadout), inv = std::ldexp(1.f, -(kSplitReadout + W.scale));
  const int nM = ceil_div(M, tm);
  const dim3 grid((unsigned)(nS * nM)), block(kSvWaves * 64);
  const int64_t bytes = split_bytes(W.blocks, W.steps);
  auto run = [&](auto vpf, auto vtm) {
    hipLaunchKernelGGL((k_vocab_sp<decltype(vpf)::value, decltype(vtm)::value>), grid, block, 0, st, t, M, E, W.steps,
                       (const char*)W.d, bytes, W.bias, V, nM, nS, ascale, inv, part, req1, req_off, nreq, zreq);
  };
  constexpr std::integral_constant<int, 2> I2{};
  constexpr std::integral_constant<int, 4> I4{};
  constexpr std::integral_constant<int, 8> I8{};
  constexpr std::integral_constant<int, 32> T32{};
  constexpr std::integral_constant<int, 64> T64{};
  const int nk = W.steps;
  if (tm == 64) {
    if (nk % 4 == 0 && nk >= 8)
      run(I4, T64);
    else
      run(I2, T64);
  } else if (tm == 32) {
    if (nk % 8 == 0 && nk >= 16)
      run(I8, T32);
    else if (nk % 4 == 0 && nk >= 8)
      run(I4, T32);
    else
      run(I2, T32);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace nmt
