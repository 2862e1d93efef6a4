// encode.hip -- the encoder's recurrence as one launch (gfx950).
//
// A position of the recurrence is a [S x H] x [H x 3H] product and the GRU
// cell, per direction.  As a chain of launches it cost about 13 us a
// position (fp32 halves) to 27 us (bf16: a split product and a cell kernel)
// whatever S: launching, reading 25 MB of weights again, and the round trips
// of a kernel's first and last accesses.  Here the weights stay in registers
// for all positions: a block of 8 waves holds 16 hidden units of one
// direction (48 gate columns, 196 KB as halves at H = 1,024; each wave an
// eighth of K), computes them for up to 32 sentences per position, and hands
// the new states to the other blocks through memory.
//
// Which wave sums which steps.  fp32: eight runs of equal length.  bf16: the
// chain of launches' K splits, one to a wave, so that every sum has the
// chain's terms in the chain's order and the states are the chain's bit for
// bit (a 16x16x32 MFMA adds like two 32x32x16 ones): a state that rounds to
// bf16 the other way would travel through the rest of the sentence.
//
// Handing over.  The states of a position travel as 8-byte words (two units'
// halves, or four bf16 units) in the MFMA's operand order, written and read
// by relaxed device-scope atomics.  Every word starts as all ones, a NaN
// pattern that no state is ever stored as (NaN states are made canonical
// first), so a word says itself whether it has arrived: a reader repeats its
// loads until none is all ones.  No flag, barrier or fence orders one
// location after another, and every position has words of its own, so none
// is overwritten while it may be read.
//
// The blocks wait for one another, so all of them must be resident: the
// kernel is launched cooperatively, which the runtime refuses where they do
// not fit.  A wait is bounded all the same (kScanPolls, about a quarter of a
// second, where another process's kernels hold the CUs); a block that gives
// up sets a flag and runs on without waiting, and the kernel after it, which
// needs no other block (k_enc_alone), computes the recurrence again.
#include <algorithm>
#include <cmath>

#include "internal.hpp"

namespace nmt {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kScanMaxH = 1024;
constexpr int kScanUnits = 16;   // hidden units per block
constexpr int kScanRows = 32;    // sentences per block
constexpr int kScanPolls = 1 << 18;
constexpr uint64_t kNotYet = ~0ull;

// Weights [direction][block of 16 units][gate][32-k step][hi, lo (fp32 models)][lane][8 halves]: lane l holds
// unit l % 16, k = 8 (l / 16) + 0 .. 7 of the step.  src: the GRU packing [Kpad/KV][Npad][KV], units in tiles of hb.
__global__ __launch_bounds__(256) void k_scan_pack(const void* __restrict__ W, int bf16, int64_t Npad, int H, int hb,
                                                   int nks, float scale, f32x4* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (block, gate, step, lane)
  if (i >= n) return;
  const int lane = (int)(i & 63), s = (int)((i >> 6) % nks), g = (int)((i >> 6) / nks % 3);
  const int u = (int)((i >> 6) / nks / 3) * kScanUnits + lane % 16;
  const int64_t col = (int64_t)(u / hb) * 3 * hb + (int64_t)g * hb + u % hb;
  const int64_t vec = i >> 6;  // this lane's fragment
  if (bf16) {
    typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
    u16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = s * 32 + 8 * (lane / 16) + e;
      v[e] = u < H && k < H ? ((const unsigned short*)W)[((int64_t)(k / 8) * Npad + col) * 8 + k % 8] : (unsigned short)0;
    }
    out[vec * 64 + lane] = __builtin_bit_cast(f32x4, v);
  } else {
    f16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = s * 32 + 8 * (lane / 16) + e;
      const float x = (u < H && k < H ? ((const float*)W)[((int64_t)(k / 4) * Npad + col) * 4 + k % 4] : 0.f) * scale;
      hi[e] = (_Float16)x;
      lo[e] = (_Float16)(x - (float)hi[e]);
    }
    out[(2 * vec) * 64 + lane] = __builtin_bit_cast(f32x4, hi);
    out[(2 * vec + 1) * 64 + lane] = __builtin_bit_cast(f32x4, lo);
  }
}

__global__ void k_fill_words(uint64_t* __restrict__ p, int64_t n2, int* __restrict__ gave_up) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n2) ((ulong2*)p)[i] = make_ulong2(kNotYet, kNotYet);
  if (i == 0) *gave_up = 0;
}

struct ScanArgs {
  const f32x4* W;
  const float* xp;   // [S * Tpad x 6H] input-side pre-activations, forward then backward
  float* ctx;        // [S x Tpad x 2H]
  const int32_t* len;
  uint64_t* words;   // [Tpad][direction][group][row tile][step][word][lane]
  int* gave_up;      // set by a block whose wait ran out
  const float *brz, *bni, *bns;
  int32_t S, Tpad, H, nks;
  int32_t splits;    // waves that share the steps
  int32_t polls;     // bound of a wait
  float hscale, inv;
};

// The first step of wave w's run: fp32 an equal share; bf16 that of K split w
// of the chain, which splits chunks of two steps.
__host__ __device__ inline int scan_first(bool bf16, int nks, int splits, int w) {
  return bf16 ? min(2 * ((nks + 1) / 2 * w / splits), nks) : min((nks + splits - 1) / splits * w, nks);
}

template <bool BF16>
struct Scan {
  static constexpr int NPL = BF16 ? 1 : 2;  // planes of a weight fragment
  static constexpr int NA = BF16 ? 2 : 4;   // words per lane and step
  static constexpr int UPT = BF16 ? 4 : 2;  // units per word
  typedef float fu __attribute__((ext_vector_type(UPT)));

  // Fragment of gate g, step s, plane p of unit block ub.
  static __device__ __forceinline__ f32x4 weight(const ScanArgs& a, int dir, int nub, int ub, int g, int s, int p,
                                                 int lane) {
    return a.W[(((((int64_t)dir * nub + ub) * 3 + g) * a.nks + s) * NPL + p) * 64 + lane];
  }
  // One step's products of the three gates.
  static __device__ __forceinline__ void step(const f32x4 (&w)[3][NPL], const uint64_t (&x)[NA], f32x4 (&acc)[3]) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    if constexpr (BF16) {
      const u32x4 v = {(uint32_t)x[0], (uint32_t)(x[0] >> 32), (uint32_t)x[1], (uint32_t)(x[1] >> 32)};
#pragma unroll
      for (int g = 0; g < 3; ++g)
        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[g][0]),
                                                         __builtin_bit_cast(bf16x8, v), acc[g], 0, 0, 0);
    } else {
      const u32x4 vh = {(uint32_t)x[0], (uint32_t)x[1], (uint32_t)x[2], (uint32_t)x[3]};
      const u32x4 vl = {(uint32_t)(x[0] >> 32), (uint32_t)(x[1] >> 32), (uint32_t)(x[2] >> 32), (uint32_t)(x[3] >> 32)};
      const f16x8 hh = __builtin_bit_cast(f16x8, vh), hl = __builtin_bit_cast(f16x8, vl);
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        f32x4& d = acc[g];
        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w[g][NPL - 1]), hh, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w[g][0]), hl, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w[g][0]), hh, d, 0, 0, 0);
      }
    }
  }
  // The states of UPT units from their gates' sums.
  static __device__ __forceinline__ fu cell(const ScanArgs& a, const fu& sr, const fu& sz, const fu& sn, const fu& br,
                                            const fu& bz, const fu& bni, const fu& bns, const fu& xr, const fu& xz,
                                            const fu& xn, const fu& hp, bool keep) {
    fu o;
#pragma unroll
    for (int e = 0; e < UPT; ++e) {
      const float inv = BF16 ? 1.f : a.inv;
      const float hn = gru_cell(sr[e] * inv, sz[e] * inv, 0.f, sn[e] * inv, br[e], bz[e], bni[e], bns[e], xr[e], xz[e],
                                xn[e], hp[e]);
      o[e] = keep ? hn : 0.f;
    }
    return o;
  }
  // Their word as an operand, never all ones.
  static __device__ __forceinline__ uint64_t word(const ScanArgs& a, const fu& o) {
    auto canon = [](float v) { return v == v ? v : __builtin_nanf(""); };
    uint32_t lo32, hi32;
    if constexpr (BF16) {
      const f32x2 c0 = f32x2{canon(o[0]), canon(o[1])}, c1 = f32x2{canon(o[UPT - 2]), canon(o[UPT - 1])};
      lo32 = __builtin_bit_cast(uint32_t, __builtin_convertvector(c0, bf16x2));
      hi32 = __builtin_bit_cast(uint32_t, __builtin_convertvector(c1, bf16x2));
    } else {
      const f32x2 c0 = f32x2{canon(o[0]) * a.hscale, canon(o[1]) * a.hscale};
      const f16x2 hi = __builtin_convertvector(c0, f16x2);
      const f32x2 c1 = f32x2{c0[0] - (float)hi[0], c0[1] - (float)hi[1]};
      lo32 = __builtin_bit_cast(uint32_t, hi);
      hi32 = __builtin_bit_cast(uint32_t, __builtin_convertvector(c1, f16x2));
    }
    return (uint64_t)hi32 << 32 | lo32;
  }
  // The place of the word of units j .. j+UPT-1, row r of a tile: step j / 32, lane group (j % 32) / 8.
  static __device__ __forceinline__ int place(int j, int r) {
    return (j / 32 * NA + j % 8 / UPT) * 64 + j % 32 / 8 * 16 + r;
  }
};

template <bool BF16, int WK>  // WK: 32-k steps per wave, at most
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_enc_scan(ScanArgs a) {
  using K = Scan<BF16>;
  using fu = typename K::fu;
  constexpr int NPL = K::NPL, NA = K::NA, UPT = K::UPT;
  __shared__ f32x4 red[2][8][3][2][64];     // [position parity][wave][gate][row tile][lane]
  const int ub = blockIdx.x, dir = blockIdx.y, grp = blockIdx.z;
  const int nub = gridDim.x, ngrp = gridDim.z;
  const int H = a.H, nks = a.nks, Tpad = a.Tpad;
  const int row0 = grp * kScanRows, rows = min(kScanRows, a.S - row0);
  const int nrt = rows > 16 ? 2 : 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

  // this wave's weights: steps s0 .. s1 - 1
  const int s0 = wave < a.splits ? scan_first(BF16, nks, a.splits, wave) : nks;
  const int s1 = wave < a.splits ? scan_first(BF16, nks, a.splits, wave + 1) : nks;
  f32x4 w[WK][3][NPL];
#pragma unroll
  for (int i = 0; i < WK; ++i)
#pragma unroll
    for (int g = 0; g < 3; ++g)
#pragma unroll
      for (int p = 0; p < NPL; ++p) w[i][g][p] = s0 + i < s1 ? K::weight(a, dir, nub, ub, g, s0 + i, p, lane) : zero4();

  // the cell: thread tid owns UPT units of one sentence
  const int tid = threadIdx.x, cl = tid & 63;
  const int crt = BF16 ? tid >> 6 : tid >> 7, part = BF16 ? 0 : (tid >> 6) & 1;  // row tile, pair of the lane's quad
  const int crow = row0 + crt * 16 + (cl & 15), ju = 4 * (cl >> 4) + UPT * part, j = ub * kScanUnits + ju;
  const bool cell = crt < nrt && crow < a.S && j < H;
  const int L = cell ? a.len[crow] : 0;
  fu br{}, bz{}, bni{}, bns{}, hp{};
  if (cell) {
    br = *(const fu*)(a.brz + j);
    bz = *(const fu*)(a.brz + H + j);
    bni = *(const fu*)(a.bni + j);
    bns = *(const fu*)(a.bns + j);
  }
  const int64_t tile_words = (int64_t)nks * NA * 64;           // words of one row tile of a position
  const int64_t pos_words = 2 * (int64_t)ngrp * 2 * tile_words;  // words of a position
  uint64_t* const base = a.words + (dir * ngrp + grp) * 2 * tile_words;
  const int64_t my_word = crt * tile_words + K::place(j, cl & 15);
  bool waiting = true;  // false once a wait has run out

  for (int t = 0; t < Tpad; ++t) {
    const int pos = dir == 0 ? t : Tpad - 1 - t;
    fu xr{}, xz{}, xn{};
    if (cell) {
      const float* x = a.xp + ((int64_t)crow * Tpad + pos) * 6 * H + dir * 3 * H + j;
      xr = *(const fu*)x;
      xz = *(const fu*)(x + H);
      xn = *(const fu*)(x + 2 * H);
    }
    fu sr{}, sz{}, sn{};
    if (t > 0) {
      const uint64_t* src = base + (t - 1) * pos_words;
      static_for<2>([&](auto rtc) {
        constexpr int rt = decltype(rtc)::value;
        if (rt >= nrt) return;
        const bool live = rt * 16 + (lane & 15) < rows;
        // words of rows and units that do not exist are never written: they
        // read another word of the tile and count as zeros (units past H
        // meet zero weights)
        const uint64_t* tsrc = src + rt * tile_words;
        int off[WK][NA];
        uint64_t x[WK][NA];
#pragma unroll
        for (int i = 0; i < WK; ++i)
#pragma unroll
          for (int q = 0; q < NA; ++q) {
            const int s = s0 + i;
            off[i][q] = live && s < s1 && s * 32 + 8 * (lane >> 4) + q * UPT < H ? (s * NA + q) * 64 + lane : -1;
          }
        for (int polls = 0;; ++polls) {
          bool ok = true;
#pragma unroll
          for (int i = 0; i < WK; ++i)
#pragma unroll
            for (int q = 0; q < NA; ++q)
              x[i][q] = __hip_atomic_load(
                  (const uint64_t*)((const char*)tsrc + (uint32_t)(off[i][q] >= 0 ? off[i][q] * 8 : 0)), __ATOMIC_RELAXED,
                  __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int i = 0; i < WK; ++i)
#pragma unroll
            for (int q = 0; q < NA; ++q) ok = ok && (off[i][q] < 0 || x[i][q] != kNotYet);
          if (__builtin_amdgcn_ballot_w64(!ok) == 0 || !waiting) break;
          if (polls >= a.polls) {
            waiting = false;
            if (lane == 0) atomicOr(a.gave_up, 1);
          }
          // Half a microsecond between polls: the polls of 1,024 waves share
          // the path of the stores they wait for (sleeps of 64, 512, 1,024 and
          // 1,536 cycles: 30 positions of one sentence 244, 233, 228 and 221 us
          // a source, 80 of 32 bf16 ones 513, 504, 496 and 504 us).
          __builtin_amdgcn_s_sleep(16);
        }
        f32x4 acc[3] = {zero4(), zero4(), zero4()};
#pragma unroll
        for (int i = 0; i < WK; ++i) {
#pragma unroll
          for (int q = 0; q < NA; ++q) x[i][q] = off[i][q] < 0 ? 0 : x[i][q];
          K::step(w[i], x[i], acc);
        }
#pragma unroll
        for (int g = 0; g < 3; ++g) red[t & 1][wave][g][rt][lane] = acc[g];
      });
      __syncthreads();
      if (cell) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          sr += *(const fu*)((const float*)&red[t & 1][v][0][crt][cl] + UPT * part);
          sz += *(const fu*)((const float*)&red[t & 1][v][1][crt][cl] + UPT * part);
          sn += *(const fu*)((const float*)&red[t & 1][v][2][crt][cl] + UPT * part);
        }
      }
    }
    if (cell) {
      hp = K::cell(a, sr, sz, sn, br, bz, bni, bns, xr, xz, xn, hp, pos < L);
      *(fu*)(a.ctx + ((int64_t)crow * Tpad + pos) * 2 * H + dir * H + j) = hp;
      if (t + 1 < Tpad)
        __hip_atomic_store(base + t * pos_words + my_word, K::word(a, hp), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The same recurrence with no block waiting for another, after a launch of
// k_enc_scan in which a wait ran out (else it ends at once): a block computes
// every unit of 16 sentences of one direction, position after position, its
// states in LDS in k_enc_scan's words and the weights read again from L2 for
// every position (0.2 to 0.3 ms a position at H = 1,024), with the same sums in the same
// order.
template <bool BF16>
__global__ __launch_bounds__(512) void k_enc_alone(ScanArgs a) {
  using K = Scan<BF16>;
  using fu = typename K::fu;
  constexpr int NPL = K::NPL, NA = K::NA, UPT = K::UPT;
  __shared__ uint64_t state[2][kScanMaxH / 32 * NA * 64];  // [position parity]
  __shared__ f32x4 red[8][3][64];
  if (*a.gave_up == 0) return;
  const int row0 = blockIdx.x * 16, dir = blockIdx.y;
  const int H = a.H, nks = a.nks, Tpad = a.Tpad, nub = (H + kScanUnits - 1) / kScanUnits;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int s0 = wave < a.splits ? scan_first(BF16, nks, a.splits, wave) : nks;
  const int s1 = wave < a.splits ? scan_first(BF16, nks, a.splits, wave + 1) : nks;
  const int tid = threadIdx.x, cl = tid & 63, part = BF16 ? 0 : (tid >> 6) & 1;
  const int crow = row0 + (cl & 15), ju = 4 * (cl >> 4) + UPT * part;
  const bool crow_ok = tid < 64 * (4 / UPT) && crow < a.S;
  const int L = crow_ok ? a.len[crow] : 0;
  for (int i = tid; i < nks * NA * 64; i += 512) state[0][i] = state[1][i] = 0;  // rows and units that do not exist
  for (int t = 0; t < Tpad; ++t) {
    const int pos = dir == 0 ? t : Tpad - 1 - t;
    const uint64_t* prev = state[(t + 1) & 1];
    for (int ub = 0; ub < nub; ++ub) {
      __syncthreads();  // the last sums are read, the last position's states are there
      if (t > 0) {
        f32x4 acc[3] = {zero4(), zero4(), zero4()};
        for (int s = s0; s < s1; ++s) {
          f32x4 w[3][NPL];
          uint64_t x[NA];
#pragma unroll
          for (int g = 0; g < 3; ++g)
#pragma unroll
            for (int p = 0; p < NPL; ++p) w[g][p] = K::weight(a, dir, nub, ub, g, s, p, lane);
#pragma unroll
          for (int q = 0; q < NA; ++q) x[q] = prev[(s * NA + q) * 64 + lane];
          K::step(w, x, acc);
        }
#pragma unroll
        for (int g = 0; g < 3; ++g) red[wave][g][lane] = acc[g];
        __syncthreads();
      }
      const int j = ub * kScanUnits + ju;
      if (!crow_ok || j >= H) continue;
      fu sr{}, sz{}, sn{}, hp{};
      float* out = a.ctx + ((int64_t)crow * Tpad + pos) * 2 * H + dir * H + j;
      if (t > 0) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          sr += *(const fu*)((const float*)&red[v][0][cl] + UPT * part);
          sz += *(const fu*)((const float*)&red[v][1][cl] + UPT * part);
          sn += *(const fu*)((const float*)&red[v][2][cl] + UPT * part);
        }
        hp = *(const fu*)(out + (dir == 0 ? -2 * H : 2 * H));  // this thread's own store of the last position
      }
      const float* x = a.xp + ((int64_t)crow * Tpad + pos) * 6 * H + dir * 3 * H + j;
      const fu o = K::cell(a, sr, sz, sn, *(const fu*)(a.brz + j), *(const fu*)(a.brz + H + j), *(const fu*)(a.bni + j),
                           *(const fu*)(a.bns + j), *(const fu*)x, *(const fu*)(x + H), *(const fu*)(x + 2 * H), hp,
                           pos < L);
      *(fu*)out = o;
      state[t & 1][K::place(j, cl & 15)] = K::word(a, o);
    }
  }
}

static int scan_steps(int H) { return ceil_div(H, 32); }
static int scan_blocks(int H) { return ceil_div(H, kScanUnits); }

size_t scan_weight_bytes(int H, bool bf16) {
  return (size_t)2 * scan_blocks(H) * 3 * scan_steps(H) * (bf16 ? 1 : 2) * 1024;
}

hipError_t launch_scan_pack(const Packed (&U)[2], int H, bool bf16, int hb, int scale, void* out, hipStream_t st) {
  const int nks = scan_steps(H);
  const int64_t n = (int64_t)scan_blocks(H) * 3 * nks * 64;
  for (int d = 0; d < 2; ++d) {
    hipLaunchKernelGGL(k_scan_pack, dim3(ceil_div(n, 256)), dim3(256), 0, st, U[d].d, bf16 ? 1 : 0, U[d].Npad, H, hb,
                       nks, bf16 ? 1.f : std::ldexp(1.f, scale),
                       (f32x4*)((char*)out + d * (scan_weight_bytes(H, bf16) / 2)), n);
  }
  return hipGetLastError();
}

// Sentences per launch: as many groups of 32 as are resident at once, at most two.
static int scan_groups(int H, int cus) { return std::min(2, cus / (2 * scan_blocks(H))); }

// Waves that share K, and the steps that the longest run of one has.  fp32 weights take twice the registers, so four
// steps a wave (H of at most 1,024) against eight.
constexpr int kScanLongF32 = 4, kScanLongBF16 = 8;
static_assert(kScanMaxH == 32 * 8 * kScanLongF32, "eight waves' runs hold K");
static int scan_splits(bool bf16, int chain_ks) { return bf16 ? chain_ks : 8; }
static int scan_longest(int H, bool bf16, int splits) {
  int n = 0;
  for (int w = 0; w < splits; ++w)
    n = std::max(n, scan_first(bf16, scan_steps(H), splits, w + 1) - scan_first(bf16, scan_steps(H), splits, w));
  return n;
}

size_t scan_words_bytes(int S, int Tpad, int H, bool bf16, int chain_ks, int cus) {
  const int splits = scan_splits(bf16, chain_ks);
  if (H > kScanMaxH || splits > 8 || scan_longest(H, bf16, splits) > (bf16 ? kScanLongBF16 : kScanLongF32)) return 0;
  const int g = scan_groups(H, cus);
  if (g < 1 || S > 4 * kScanRows) return 0;  // more sentences fill the chip as a chain of launches
  const size_t n = (size_t)Tpad * 2 * std::min(g, ceil_div(S, kScanRows)) * 2 * scan_steps(H) * (bf16 ? 2 : 4) * 512;
  return n > ((size_t)128 << 20) ? 0 : n;
}

hipError_t launch_enc_scan(const void* W, const float* xp, float* ctx, const int32_t* len, void* words, int* gave_up,
                           int form, const GruEpi& bias, int S, int Tpad, int H, bool bf16, int chain_ks, int scale, int cus,
                           hipStream_t st) {
  const int g = scan_groups(H, cus), per = std::min(g, ceil_div(S, kScanRows)) * kScanRows;
  const int64_t bytes = (int64_t)scan_words_bytes(S, Tpad, H, bf16, chain_ks, cus);
  if (bytes <= 0) return hipErrorInvalidValue;
  const int splits = scan_splits(bf16, chain_ks);
  const void* kernel = !bf16 ? (const void*)k_enc_scan<false, kScanLongF32>
                             : (scan_longest(H, bf16, splits) <= 4 ? (const void*)k_enc_scan<true, 4>
                                                                   : (const void*)k_enc_scan<true, kScanLongBF16>);
  for (int s0 = 0; s0 < S; s0 += per) {
    hipLaunchKernelGGL(k_fill_words, dim3(ceil_div(bytes / 16, 256)), dim3(256), 0, st, (uint64_t*)words, bytes / 16,
                       gave_up);
    ScanArgs a{};
    a.W = (const f32x4*)W;
    a.xp = xp + (int64_t)s0 * Tpad * 6 * H;
    a.ctx = ctx + (int64_t)s0 * Tpad * 2 * H;
    a.len = len + s0;
    a.words = (uint64_t*)words;
    a.gave_up = gave_up;
    a.polls = form == 2 ? 0 : kScanPolls;
    a.brz = bias.brz;
    a.bni = bias.bni;
    a.bns = bias.bns;
    a.S = std::min(per, S - s0);
    a.Tpad = Tpad;
    a.H = H;
    a.nks = scan_steps(H);
    a.splits = splits;
    a.hscale = std::ldexp(1.f, kSplitState);
    a.inv = bf16 ? 1.f : std::ldexp(1.f, -(kSplitState + scale));
    void* args[] = {&a};
    const dim3 grid(scan_blocks(H), 2, ceil_div(a.S, kScanRows));
    const hipError_t e = hipLaunchCooperativeKernel(kernel, grid, dim3(512), args, 0, st);
    if (e != hipSuccess) return e;
    const dim3 rest(ceil_div(a.S, 16), 2);
    if (bf16)
      hipLaunchKernelGGL(k_enc_alone<true>, rest, dim3(512), 0, st, a);
    else
      hipLaunchKernelGGL(k_enc_alone<false>, rest, dim3(512), 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace nmt
