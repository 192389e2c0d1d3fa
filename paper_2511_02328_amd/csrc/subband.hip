// subband.hip -- the paper's own dedispersion path on gfx950: stage 2 of the
// two-stage subband method, the zero-DM filter and square-law downsampling.
//
// Stage 1 (Eq. stage1: per coarse DM, shift and sum the channels of each
// subband) is brute-force dedispersion restricted to a subband's channels
// over the coarse DM grid, so it runs on the dedispersion kernel of
// dedisperse.hip, once per subband.  Stage 2 (Eq. stage2) sums the subband
// series of the coarse group j(m) = floor(m / n0) with the residual shifts
// R[m][s] of Eq. (residual).
#include "sps_internal.h"

namespace sps {
namespace {

constexpr int kS2Threads = 256;
constexpr int kS2Out = 4;  // outputs per thread

// Stage 2, Y[m][t] = sum_s I[s][j(m)][t + R[m][s]], one workgroup per coarse
// group j and 1024 output samples.  The subband loop is outside and up to
// GM fine DMs of the group are accumulated together, so the GM overlapping
// windows of one subband row (a few KB) are read back to back and served
// from L1, and each word of I leaves L2 about once per tile.  Rt: the
// residual table transposed, [nsub][ndm], so the GM shifts of one subband
// are one scalar load.
//
// Whole groups of GM trials on whole tiles take a branch-free path: thread i
// owns outputs t0 + 4 i .. t0 + 4 i + 3 and reads each trial's window with
// one 16-byte load at its (dword-aligned) offset; all GM loads of a subband
// are issued before the first add, and two subbands are in flight.  Group
// and tile edges take the guarded loop, in which thread i owns outputs
// t0 + i + 256 b (b < 4).
template <int GM>
__global__ __launch_bounds__(kS2Threads) void subband_stage2_blocked_kernel(
    const uint32_t *__restrict__ I, int64_t len1, int ncoarse, int nsub,
    const int32_t *__restrict__ Rt, int ndm, int n0, uint32_t *__restrict__ Y, int64_t nout,
    int64_t nchunks) {
  const int64_t blk = blockIdx.x;
  const int j = (int)(blk / nchunks);
  const int64_t t0 = (blk - (int64_t)j * nchunks) * kS2Threads * kS2Out;
  const int64_t t = t0 + threadIdx.x;
  const bool full_tile = t0 + kS2Threads * kS2Out <= nout;
  const int mend = min((j + 1) * n0, ndm);
  const int64_t plane = (int64_t)ncoarse * len1;
  const uint32_t *base = I + (int64_t)j * len1 + t;
  for (int m0 = j * n0; m0 < mend; m0 += GM) {
    const int gm = min(GM, mend - m0);
    uint32_t acc[GM][kS2Out];
#pragma unroll
    for (int a = 0; a < GM; ++a)
#pragma unroll
      for (int b = 0; b < kS2Out; ++b) acc[a][b] = 0u;
    if (gm == GM && full_tile) {
      // Lane-consecutive outputs here: the thread owns t0 + 4 tid .. + 3 and
      // reads each trial's window with one 16-byte load at its dword offset
      // (four times fewer load instructions than one dword per output).
      static_assert(kS2Out == 4, "one 16-byte load per trial");
      const uint32_t *base4 = I + (int64_t)j * len1 + t0 + 4 * (int64_t)threadIdx.x;
#pragma unroll 2
      for (int sb = 0; sb < nsub; ++sb) {
        const uint32_t *row = base4 + (int64_t)sb * plane;
        const int32_t *Rs = Rt + (int64_t)sb * ndm + m0;
        u32x4_a4 v[GM];
#pragma unroll
        for (int a = 0; a < GM; ++a) v[a] = *(const SPS_GLOBAL u32x4_a4 *)gmem(row + Rs[a]);
#pragma unroll
        for (int a = 0; a < GM; ++a) {
          acc[a][0] += v[a].x;
          acc[a][1] += v[a].y;
          acc[a][2] += v[a].z;
          acc[a][3] += v[a].w;
        }
      }
      const bool vec = ((reinterpret_cast<uintptr_t>(Y) & 15) == 0) && (nout & 3) == 0;
#pragma unroll
      for (int a = 0; a < GM; ++a) {
        SPS_GLOBAL uint32_t *Ym = gmem(Y + (int64_t)(m0 + a) * nout + t0 + 4 * (int64_t)threadIdx.x);
        if (vec) {
          *(SPS_GLOBAL u32x4 *)Ym = u32x4{acc[a][0], acc[a][1], acc[a][2], acc[a][3]};
        } else {
#pragma unroll
          for (int b = 0; b < 4; ++b) Ym[b] = acc[a][b];
        }
      }
      continue;
    } else if (t < nout) {
      for (int sb = 0; sb < nsub; ++sb) {
        const uint32_t *row = base + (int64_t)sb * plane;
        for (int a = 0; a < gm; ++a) {
          const uint32_t *w = row + Rt[(int64_t)sb * ndm + m0 + a];
#pragma unroll
          for (int b = 0; b < kS2Out; ++b)
            if (t + b * kS2Threads < nout) acc[a][b] += w[b * kS2Threads];
        }
      }
    }
    if (t < nout) {
#pragma unroll
      for (int a = 0; a < GM; ++a) {
        if (a < gm) {
          uint32_t *Ym = Y + (int64_t)(m0 + a) * nout + t;
#pragma unroll
          for (int b = 0; b < kS2Out; ++b)
            if (t + b * kS2Threads < nout) Ym[b * kS2Threads] = acc[a][b];
        }
      }
    }
  }
}

// The same with each subband row staged in LDS, so that its words cross L1
// once per GM trials: a tile's window from the smallest to the largest of the
// group's shifts.  Thread i owns outputs t0 + i + 256 b (b < 4); the next
// subband's row is in registers while the current one is summed.  Bound by
// reading I and writing Y once (20.6 GB, 4.1 ms at the rate of a large copy, on
// 32 subbands x 257 coarse and 2048 fine trials x 500,000 outputs): 4.05 ms,
// where the form above, bound by L1, takes 5.95 ms.
constexpr int kS2Span = 1024;  // largest difference of two shifts
constexpr int kS2Row = kS2Threads * kS2Out + kS2Span;

template <int GM>
__global__ __launch_bounds__(kS2Threads) void subband_stage2_lds_kernel(
    const uint32_t *__restrict__ I, int64_t len1, int ncoarse, int nsub,
    const int32_t *__restrict__ Rt, int ndm, int n0, uint32_t *__restrict__ Y, int64_t nout,
    int64_t nchunks) {
  static_assert(kS2Out == 4 && kS2Row <= 8 * kS2Threads, "two vectors per thread and row");
  __shared__ __attribute__((aligned(16))) uint32_t rowbuf[2][kS2Row];
  const int64_t blk = blockIdx.x;
  const int j = (int)(blk / nchunks);
  const int64_t t0 = (blk - (int64_t)j * nchunks) * kS2Threads * kS2Out;
  const int i = threadIdx.x;
  const int mend = min((j + 1) * n0, ndm);
  const int64_t plane = (int64_t)ncoarse * len1;
  const SPS_GLOBAL uint32_t *base = gmem(I + (int64_t)j * len1);
  for (int m0 = j * n0; m0 < mend; m0 += GM) {
    uint32_t acc[GM][kS2Out];
#pragma unroll
    for (int a = 0; a < GM; ++a)
#pragma unroll
      for (int b = 0; b < kS2Out; ++b) acc[a][b] = 0u;
    // trials past the group repeat its last
    auto shift = [&](int sb, int a) { return Rt[(int64_t)sb * ndm + min(m0 + a, mend - 1)]; };
    auto low = [&](int sb) {
      int lo = shift(sb, 0);
#pragma unroll
      for (int a = 1; a < GM; ++a) lo = min(lo, shift(sb, a));
      return lo;
    };
    auto high = [&](int sb) {
      int hi = shift(sb, 0);
#pragma unroll
      for (int a = 1; a < GM; ++a) hi = max(hi, shift(sb, a));
      return hi;
    };
    u32x4 v[2];
    auto load = [&](int sb) {
      const int lo = low(sb);
      const int64_t first = t0 + lo;
      const int words = kS2Threads * kS2Out + high(sb) - lo;
      const SPS_GLOBAL uint32_t *src = base + (int64_t)sb * plane + first;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int w = 4 * (i + u * kS2Threads);
        if (w < words) {
          if (first + w + 4 <= len1) {
            v[u] = *(const SPS_GLOBAL u32x4_a4 *)(src + w);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[u][q] = first + w + q < len1 ? src[w + q] : 0u;
          }
        }
      }
    };
    __syncthreads();  // the rows of the trials before are read
    load(0);
    for (int sb = 0; sb < nsub; ++sb) {
      uint32_t *row = rowbuf[sb & 1];
      const int lo = low(sb), words = kS2Threads * kS2Out + high(sb) - lo;
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (4 * (i + u * kS2Threads) < words)
          *reinterpret_cast<u32x4 *>(row + 4 * (i + u * kS2Threads)) = v[u];
      __syncthreads();
      if (sb + 1 < nsub) load(sb + 1);
#pragma unroll
      for (int a = 0; a < GM; ++a) {
        const uint32_t *r = row + (shift(sb, a) - lo) + i;
#pragma unroll
        for (int b = 0; b < kS2Out; ++b) acc[a][b] += r[b * kS2Threads];
      }
    }
#pragma unroll
    for (int a = 0; a < GM; ++a) {
      if (m0 + a >= mend) break;
      SPS_GLOBAL uint32_t *Ym = gmem(Y + (int64_t)(m0 + a) * nout);
#pragma unroll
      for (int b = 0; b < kS2Out; ++b)
        if (t0 + i + b * kS2Threads < nout) Ym[t0 + i + b * kS2Threads] = acc[a][b];
    }
  }
}

// Zero-DM filter: X'[c][t] = clip(X[c][t] - m(t) + 128, 0, 255) with m(t) the
// channel mean rounded half up.
//
// HBM bound: 1 B read and 1 B written per sample.  A workgroup owns 16 COLS
// consecutive samples of every channel: COLS lanes cover a row with 16-byte
// accesses, so THREADS take THREADS / COLS rows at a time.  Byte sums run in
// packed 16-bit halves, are reduced across the workgroup (unless a thread has
// whole columns) and the samples are corrected in packed 16-bit arithmetic.
// Up to STEPS THREADS / COLS rows the samples stay in registers between the two
// passes; with STEPS = 0 (more rows than the registers hold) they are read
// again, while the tile is still in the Infinity Cache.
// One thread per 4 samples, reading both passes with 4-byte loads, took 2.22
// ms for 2048 channels x 573,440 samples (1.6 TB/s of 3.5 GB); this form takes
// 0.53 ms (4.4 TB/s of 2.35 GB).
typedef short i16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t zero_dm_apply(uint32_t w, uint32_t ce, uint32_t co) {
  const i16x2 lo = {0, 0}, hi = {255, 255};
  const uint32_t e = w & 0x00FF00FFu, o = (w >> 8) & 0x00FF00FFu;
  const i16x2 a = __builtin_elementwise_min(
      __builtin_elementwise_max(__builtin_bit_cast(i16x2, e) + __builtin_bit_cast(i16x2, ce), lo), hi);
  const i16x2 b = __builtin_elementwise_min(
      __builtin_elementwise_max(__builtin_bit_cast(i16x2, o) + __builtin_bit_cast(i16x2, co), lo), hi);
  return __builtin_bit_cast(uint32_t, a) | __builtin_bit_cast(uint32_t, b) << 8;
}

template <int COLS, int THREADS, int STEPS>
__global__ __launch_bounds__(THREADS) void zero_dm_kernel(const uint8_t *X, int64_t pitch,
                                                          int64_t nsamp, int nchan, uint8_t *Xo,
                                                          int64_t pitch_out) {
  constexpr int kTile = 16 * COLS, kRows = THREADS / COLS;
  static_assert(THREADS % COLS == 0 && 64 % COLS == 0, "a wave holds whole rows");
  __shared__ uint32_t total[kRows > 1 ? kTile : 1];
  const int tid = threadIdx.x, col = tid % COLS, r0 = tid / COLS;
  const int64_t t = (int64_t)blockIdx.x * kTile + 16 * col;
  const bool live = t < nsamp;  // rows are 16-byte multiples, so a whole vector lies in the row
  if constexpr (kRows > 1)
    for (int i = tid; i < kTile; i += THREADS) total[i] = 0u;
  u32x4 keep[STEPS > 0 ? STEPS : 1];
  uint32_t even[4] = {0u, 0u, 0u, 0u}, odd[4] = {0u, 0u, 0u, 0u};  // bytes 0, 2 / 1, 3 of each dword
  auto add = [&](u32x4 v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      even[q] += v[q] & 0x00FF00FFu;
      odd[q] += (v[q] >> 8) & 0x00FF00FFu;
    }
  };
  // the rows of a wave, still packed (at most 8 x 16 of them: 8 x 16 x 255 <
  // 2^16), then the waves
  static_assert(COLS >= 8 && STEPS <= 16, "packed sums");
  auto reduce = [&]() {
    if constexpr (kRows == 1) return;  // a thread holds whole columns
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t e = even[q], o = odd[q];
#pragma unroll
      for (int m = COLS; m < 64; m <<= 1) {
        e += __shfl_xor(e, m, 64);
        o += __shfl_xor(o, m, 64);
      }
      if ((tid & 63) < COLS) {
        uint32_t *c = total + 16 * col + 4 * q;
        atomicAdd(c, e & 0xFFFFu);
        atomicAdd(c + 1, o & 0xFFFFu);
        atomicAdd(c + 2, e >> 16);
        atomicAdd(c + 3, o >> 16);
      }
      even[q] = odd[q] = 0u;
    }
  };
  __syncthreads();
  if constexpr (STEPS > 0) {
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      const int r = r0 + kRows * i;
      keep[i] = u32x4{0u, 0u, 0u, 0u};
      if (live && r < nchan) keep[i] = *(const SPS_GLOBAL u32x4 *)gmem(X + (int64_t)r * pitch + t);
    }
#pragma unroll
    for (int i = 0; i < STEPS; ++i) add(keep[i]);
    reduce();
  } else {
    for (int64_t base = 0; base < nchan; base += 16 * kRows) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int64_t r = base + r0 + kRows * i;
        if (live && r < nchan) add(*(const SPS_GLOBAL u32x4 *)gmem(X + r * pitch + t));
      }
      reduce();
    }
  }
  const auto shift = [&](uint32_t sum) {  // 128 - m
    return 128u - (sum + (uint32_t)(nchan / 2)) / (uint32_t)nchan;
  };
  if constexpr (kRows > 1) {
    __syncthreads();
    for (int i = tid; i < kTile; i += THREADS) total[i] = shift(total[i]);
    __syncthreads();
  }
  if (!live) return;
  uint32_t ce[4], co[4];  // 128 - m as 16-bit halves of bytes 0, 2 / 1, 3
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if constexpr (kRows > 1) {
      const uint32_t *c = total + 16 * col + 4 * q;
      ce[q] = (c[0] & 0xFFFFu) | c[2] << 16;
      co[q] = (c[1] & 0xFFFFu) | c[3] << 16;
    } else {
      ce[q] = (shift(even[q] & 0xFFFFu) & 0xFFFFu) | shift(even[q] >> 16) << 16;
      co[q] = (shift(odd[q] & 0xFFFFu) & 0xFFFFu) | shift(odd[q] >> 16) << 16;
    }
  }
  const bool whole = t + 16 <= nsamp;
  auto put = [&](int r, u32x4 v) {
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = zero_dm_apply(v[q], ce[q], co[q]);
    uint8_t *out = Xo + (int64_t)r * pitch_out + t;
    if (whole) {
      *(SPS_GLOBAL u32x4 *)gmem(out) = o;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t left = nsamp - t - 4 * q;
        if (left >= 4) {
          *(SPS_GLOBAL uint32_t *)gmem(out + 4 * q) = o[q];
        } else {
#pragma unroll
          for (int b = 0; b < 3; ++b)
            if (b < left) out[4 * q + b] = (uint8_t)(o[q] >> (8 * b));
        }
      }
    }
  };
  if constexpr (STEPS > 0) {
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      // opaque: otherwise the widened bytes of the first pass stay live
      asm volatile("" : "+v"(keep[i]));
      if (r0 + kRows * i < nchan) put(r0 + kRows * i, keep[i]);
    }
  } else {
#pragma unroll 8
    for (int r = r0; r < nchan; r += kRows)
      put(r, *(const SPS_GLOBAL u32x4 *)gmem(X + (int64_t)r * pitch + t));
  }
}

// Square-law downsampling (Sec. 2.2): out = min(sqrt(255 S / N), 255), S the
// sum of a bin of N samples, rounded half up.  A float square root gives a
// first guess, at most 1 off; the rounding is then settled exactly:
// (2r - 1)^2 N <= 4 * 255 S < (2r + 1)^2 N.
//
// N <= 16: every term is an integer below 2^24, so binary32 arithmetic is
// exact ((2r + 1)^2 N <= 511^2 16).
__device__ __forceinline__ uint32_t sqrt_bin_small(uint32_t S, float N, float inv_n) {
  const float s = (float)S, v = 1020.0f * s;
  float r = __builtin_floorf(__builtin_amdgcn_sqrtf(255.0f * s * inv_n) + 0.5f);
  const float a = 2.0f * r + 1.0f, b = 2.0f * r - 1.0f;
  r += a * a * N <= v ? 1.0f : 0.0f;
  r -= b > 0.0f && b * b * N > v ? 1.0f : 0.0f;
  return (uint32_t)fminf(r, 255.0f);
}

// U: 32 bits hold every term up to N = 2^12 (4 * 255 * 255 N < 2^31), 64 bits
// above.
template <typename U>
__device__ __forceinline__ uint32_t sqrt_bin(U S, U N, float inv_n) {
  const U V = 255;
  U r = (U)(__builtin_amdgcn_sqrtf((float)(V * S) * inv_n) + 0.5f);
  while ((2 * r + 1) * (2 * r + 1) * N <= 4 * V * S) ++r;
  while (r > 0 && (2 * r - 1) * (2 * r - 1) * N > 4 * V * S) --r;
  return (uint32_t)(r > V ? V : r);
}

// dwords and 16-byte vectors at any byte address (rows need no alignment)
typedef unsigned int u32_a1 __attribute__((aligned(1)));
typedef unsigned int u32x4_a1 __attribute__((ext_vector_type(4), aligned(1)));

// Factors up to 16: a thread makes Q outputs (a multiple of 4, stored as
// dwords) from their Q N consecutive bytes, read as whole dwords; which bytes
// make up a bin is known at compile time.  HBM bound: N B read and 1 B
// written per output.  One thread per output with byte loads and 64-bit
// rounding took 1.82 ms for 2048 channels x 573,440 samples at N = 4 (0.8
// TB/s); this form takes 0.27 ms (5.4 TB/s).
template <int N, int Q>
__global__ __launch_bounds__(256) void downsample_sqrt_kernel(const uint8_t *X, int64_t pitch,
                                                              int64_t nout, uint8_t *Xo,
                                                              int64_t pitch_out) {
  static_assert(Q % 4 == 0, "whole dwords in and out");
  constexpr int ND = Q * N / 4;  // dwords read
  const int64_t t = Q * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  if (t >= nout) return;
  const uint8_t *row = X + (int64_t)blockIdx.y * pitch + t * N;
  uint8_t *out = Xo + (int64_t)blockIdx.y * pitch_out + t;
  if (t + Q <= nout) {
    uint32_t w[ND];
#pragma unroll
    for (int k = 0; k < ND / 4; ++k) {
      const u32x4_a1 v = ((const SPS_GLOBAL u32x4_a1 *)gmem(row))[k];
      w[4 * k] = v.x;
      w[4 * k + 1] = v.y;
      w[4 * k + 2] = v.z;
      w[4 * k + 3] = v.w;
    }
#pragma unroll
    for (int k = ND / 4 * 4; k < ND; ++k) w[k] = ((const SPS_GLOBAL u32_a1 *)gmem(row))[k];
#pragma unroll
    for (int q = 0; q < Q / 4; ++q) {
      uint32_t o = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int first = (4 * q + b) * N;
        uint32_t S = 0;
#pragma unroll
        for (int k = first / 4; 4 * k < first + N; ++k) {
          // the bytes of dword k that belong to the bin
          const int lo = first > 4 * k ? first - 4 * k : 0;
          const int hi = first + N < 4 * k + 4 ? first + N - 4 * k : 4;
          const uint32_t mask = (hi == 4 ? 0xFFFFFFFFu : (1u << (8 * hi)) - 1u) & ~((1u << (8 * lo)) - 1u);
          S = __builtin_amdgcn_sad_u8(w[k] & mask, 0u, S);
        }
        o |= sqrt_bin_small(S, (float)N, 1.0f / N) << (8 * b);
      }
      ((SPS_GLOBAL u32_a1 *)gmem(out))[q] = o;
    }
    return;
  }
  for (int64_t i = 0; t + i < nout; ++i) {
    uint32_t S = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) S += row[i * N + k];
    out[i] = (uint8_t)sqrt_bin_small(S, (float)N, 1.0f / N);
  }
}

// Any factor: one thread per output.
template <typename U>
__global__ __launch_bounds__(256) void downsample_sqrt_any_kernel(const uint8_t *X, int64_t pitch,
                                                                  int factor, int64_t nout,
                                                                  uint8_t *Xo, int64_t pitch_out) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= nout) return;
  const uint8_t *row = X + (int64_t)blockIdx.y * pitch + t * factor;
  uint32_t S = 0;  // at most 255 x 2^20
  int k = 0;
  for (; k + 16 <= factor; k += 16) {
    const u32x4_a1 v = *(const SPS_GLOBAL u32x4_a1 *)gmem(row + k);
    S = __builtin_amdgcn_sad_u8(v.x, 0u, S);
    S = __builtin_amdgcn_sad_u8(v.y, 0u, S);
    S = __builtin_amdgcn_sad_u8(v.z, 0u, S);
    S = __builtin_amdgcn_sad_u8(v.w, 0u, S);
  }
  for (; k + 4 <= factor; k += 4)
    S = __builtin_amdgcn_sad_u8(*(const SPS_GLOBAL u32_a1 *)gmem(row + k), 0u, S);
  for (; k < factor; ++k) S += row[k];
  Xo[(int64_t)blockIdx.y * pitch_out + t] =
      (uint8_t)sqrt_bin<U>((U)S, (U)factor, 1.0f / (float)factor);
}

}  // namespace

hipError_t launch_subband_stage2(const uint32_t *I, int64_t len1, int ncoarse, int nsub,
                                 const int32_t *Rt, int rmax, int ndm, int n0, uint32_t *Y,
                                 int64_t nout, hipStream_t stream) {
  const int64_t per_block = (int64_t)kS2Threads * kS2Out;
  const int64_t nchunks = (nout + per_block - 1) / per_block;
  const int64_t grid = nchunks * ncoarse;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  // shifts are 0 .. rmax; past kS2Span a staged window is more than twice its
  // tile (and the two vectors per thread)
  if (rmax <= kS2Span) {
    hipLaunchKernelGGL(subband_stage2_lds_kernel<8>, dim3((unsigned)grid), dim3(kS2Threads), 0,
                       stream, I, len1, ncoarse, nsub, Rt, ndm, n0, Y, nout, nchunks);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(subband_stage2_blocked_kernel<8>, dim3((unsigned)grid), dim3(kS2Threads), 0,
                     stream, I, len1, ncoarse, nsub, Rt, ndm, n0, Y, nout, nchunks);
  return hipGetLastError();
}

hipError_t launch_zero_dm(const uint8_t *X, int64_t pitch, int64_t nsamp, int nchan, uint8_t *Xo,
                          int64_t pitch_out, hipStream_t stream) {
  if (nsamp == 0) return hipSuccess;
  // The widest tile whose rows fill the workgroup and its registers: with tiles
  // of 128 samples (8 columns of 1024 threads) for any number of channels, most
  // of a workgroup had no row.  2^20 samples of 4, 16, 64 and 128 channels: 58,
  // 58, 63 and 69 us so, 7.4, 7.6, 22 and 44 us now (one thread per 4 samples:
  // 7.5, 9.2, 49 and 96 us).
  auto go = [&](auto kern, int cols, int threads) {
    const int64_t grid = (nsamp + 16 * cols - 1) / (16 * cols);
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3((unsigned)threads), 0, stream, X, pitch,
                       nsamp, nchan, Xo, pitch_out);
    return hipGetLastError();
  };
  if (nchan <= 8) return go(zero_dm_kernel<64, 64, 8>, 64, 64);
  if (nchan <= 16) return go(zero_dm_kernel<64, 64, 16>, 64, 64);
  if (nchan <= 64) return go(zero_dm_kernel<32, 128, 16>, 32, 128);
  if (nchan <= 128) return go(zero_dm_kernel<32, 256, 16>, 32, 256);
  if (nchan <= 256) return go(zero_dm_kernel<8, 1024, 2>, 8, 1024);
  if (nchan <= 512) return go(zero_dm_kernel<8, 1024, 4>, 8, 1024);
  if (nchan <= 2048) return go(zero_dm_kernel<8, 1024, 16>, 8, 1024);
  return go(zero_dm_kernel<8, 1024, 0>, 8, 1024);
}

hipError_t launch_downsample_sqrt(const uint8_t *X, int64_t pitch, int64_t nsamp, int nchan,
                                  int factor, uint8_t *Xo, int64_t pitch_out,
                                  hipStream_t stream) {
  const int64_t nout = nsamp / factor;
  if (nchan > 65535) return hipErrorInvalidValue;
  auto grid = [&](int64_t per_block) { return (nout + per_block - 1) / per_block; };
  if (grid(256) > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (nout == 0) return hipSuccess;
  auto go = [&](auto kern, int q) {
    hipLaunchKernelGGL(kern, dim3((unsigned)grid(256 * q), (unsigned)nchan), dim3(256), 0, stream, X,
                       pitch, nout, Xo, pitch_out);
    return hipGetLastError();
  };
  switch (factor) {  // at least 16 bytes read per thread
    case 1: return go(downsample_sqrt_kernel<1, 16>, 16);
    case 2: return go(downsample_sqrt_kernel<2, 8>, 8);
    case 3: return go(downsample_sqrt_kernel<3, 8>, 8);
    case 4: return go(downsample_sqrt_kernel<4, 4>, 4);
    case 5: return go(downsample_sqrt_kernel<5, 4>, 4);
    case 6: return go(downsample_sqrt_kernel<6, 4>, 4);
    case 7: return go(downsample_sqrt_kernel<7, 4>, 4);
    case 8: return go(downsample_sqrt_kernel<8, 4>, 4);
    case 9: return go(downsample_sqrt_kernel<9, 4>, 4);
    case 10: return go(downsample_sqrt_kernel<10, 4>, 4);
    case 11: return go(downsample_sqrt_kernel<11, 4>, 4);
    case 12: return go(downsample_sqrt_kernel<12, 4>, 4);
    case 13: return go(downsample_sqrt_kernel<13, 4>, 4);
    case 14: return go(downsample_sqrt_kernel<14, 4>, 4);
    case 15: return go(downsample_sqrt_kernel<15, 4>, 4);
    case 16: return go(downsample_sqrt_kernel<16, 4>, 4);
    default: break;
  }
  auto any = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)grid(256), (unsigned)nchan), dim3(256), 0, stream, X,
                       pitch, factor, nout, Xo, pitch_out);
    return hipGetLastError();
  };
  return factor <= 4096 ? any(downsample_sqrt_any_kernel<uint32_t>)
                        : any(downsample_sqrt_any_kernel<int64_t>);
}

}  // namespace sps
