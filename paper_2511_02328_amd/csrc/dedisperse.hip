// dedisperse.hip -- brute-force incoherent dedispersion on gfx950.
//
// Computes Y[d][t] = sum_c X[c][t + D[d][c]] (ASTROFLOW Sec. 2.3, the direct
// method of cost N_DM N_t N_f; samples at or past nsamp_in count as zero as in
// Eq. stage1) exactly in integers, as products of the data with 0/1 matrices
// on the matrix cores.
//
// Design (CDNA4, wave64):
//  * A workgroup owns a block of nd = nw * dpw consecutive trials and a time
//    tile of nt = 512 m - 16 outputs.  Channels are processed in slabs of cs
//    rows; for each channel the slab row holds the input window that the
//    block's trials need, from t0 + D[d_lo][c] rounded down to 16, loaded with
//    coalesced 16-byte reads (one wave per row), zero-filled past nsamp_in and
//    stored with the top bit of every byte inverted: as a signed byte it is
//    the sample minus 128, and 128 per summed row is added back once.
//  * A wave's trial reads aligned 16-byte chunks of a row: chunk q covers the
//    samples that fall, after a delay v = 16 a + r (r < 16), on outputs
//    16 (q - a) - r .. 16 (q - a) - r + 15, i.e. on two output chunks.  One
//    sparse product v_smfmac_i32_32x32x64_i8 takes 32 chunks (columns) of
//    each of 4 channels and adds every byte once: row i of the 0/1 operand
//    selects byte i - 16 + r of a channel's chunk, so rows 0..15 are the sums
//    for the output chunk before and rows 16..31 for the one the chunk
//    starts.  The operand has at most one 1 per row and channel, so it fits
//    the 4:2 structured form and costs half the dense product.  The two
//    halves meet in the epilogue; the last chunk of a tile lacks its
//    successor, hence the 16 outputs less.
//  * No byte is shifted or widened on the vector units, and a wave reads each
//    16-byte chunk from LDS with one aligned read: 1 B of LDS reads per
//    sample-add, lanes on consecutive chunks (no bank conflicts).  Per group
//    of 4 channels a wave spends about 14 vector instructions on addresses
//    and the 0/1 operand, for 2 m LDS reads and m products.
//  * The delay table is read in a staged form built once per tiling
//    (stage_delays): per (trial, 4 channels, half wave) the LDS offsets of
//    the two chunk rows the half reads and the remainders r its operand rows
//    need.  A lane holds the entries of one group; the row broadcast of the
//    consuming instruction (DPP row_newbcast) picks the current one.
//  * Workgroups are dealt to the 8 XCDs round-robin by the hardware; the
//    logical index is remapped so that each XCD walks a contiguous range in
//    panels of a few DM blocks (DM block fastest inside a panel, then time),
//    so the workgroups resident on one XCD share their staged delay rows and
//    most of their input windows in that XCD's L2.
//
// What bounds it: the matrix cores and LDS at the part's power limit.  On
// 4096 channels x 2048 trials x 2^18 outputs the products alone (operands in
// registers) would take 21 ms at noise-like data, products with their LDS
// reads 29 ms (0.6 of the matrix cores' cycles at a clock that falls to
// 1.9 GHz), the whole kernel takes 36 ms; the form it replaces (byte permutes
// and packed 16-bit adds on the vector units) took 55 ms.
#include <math.h>

#include "sps_internal.h"

namespace sps {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
// four dwords stored at any dword-aligned address (one 16-byte store)
typedef unsigned int u32x4_s4 __attribute__((ext_vector_type(4), aligned(4)));

// v of lane Q of the lane's row of 16; folded into the instruction that uses
// it as its first operand.
template <int Q>
__device__ __forceinline__ uint32_t row_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + Q, 0xF, 0xF, true);
}

// Adds one group of 4 channels.  a0, b0: LDS byte addresses of this lane's
// first chunk of its half's first and second channel; u: 4 (i + r) of row
// i = lane & 31 for the two channels whose operand rows this lane holds (low
// and high 16 bits); sel: (i & 3) + (r & 3) of the same, each twice.
//
// Row i of a channel selects byte k = i - 16 + r if 0 <= k < 16, i.e. if bit
// 6 of u is set.  In the 4:2 form byte k is value slot 2 (k / 4) with index
// k mod 4: a 64-bit value with the byte at bit 16 (k / 4), and a 2-bit index
// repeated over the slots (the other slots hold zeros).
template <int J>
__device__ __forceinline__ void add_group(i32x16 (&acc)[J], const char *lds, uint32_t a0,
                                          uint32_t b0, uint32_t u, uint32_t sel) {
  const int idx = (int)__builtin_amdgcn_perm(0xFFAA5500u, 0xFFAA5500u, sel);
  const uint64_t a = (uint64_t)__builtin_amdgcn_ubfe(u, 6, 1) << (u & 0x30u);
  const uint64_t b = (uint64_t)__builtin_amdgcn_ubfe(u, 22, 1) << ((u >> 16) & 0x30u);
  const i32x4 A = {(int)a, (int)(a >> 32), (int)b, (int)(b >> 32)};
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const i32x4 x = *(const i32x4 *)(lds + a0 + 512 * j);
    const i32x4 y = *(const i32x4 *)(lds + b0 + 512 * j);
    const i32x8 B = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    acc[j] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(A, B, acc[j], idx, 0, 0);
  }
}

// Accumulators to start from: 128 per row to be summed, in the half (rows
// 16..31) that is added once per output.
template <int J>
__device__ __forceinline__ void reset_acc(i32x16 (&acc)[J], int rows) {
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = i < 8 ? 0 : 128 * rows;
}

// Writes trial d's outputs of a tile.  Lane (n = lane & 31, h = lane >> 5)
// holds rows 8 (i / 4) + 4 h + i % 4 of chunk 32 j + n's column; rows 0..15
// of the next chunk (lane n + 1, or lane 0 of step j + 1) complete it.
template <int J>
__device__ __forceinline__ void store_acc(const i32x16 (&acc)[J], uint32_t *__restrict__ Y,
                                          int64_t nout, int ndm, int d, int lane, int64_t t0) {
  const int n = lane & 31, h = lane >> 5;
  SPS_GLOBAL uint32_t *Yd = gmem(Y + (int64_t)d * nout);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    uint32_t nx[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int own = n == 0 && j + 1 < J ? acc[j + 1 < J ? j + 1 : 0][i] : acc[j][i];
      nx[i] = (uint32_t)__shfl(own, (lane & 32) | ((n + 1) & 31));
    }
    if (d >= ndm || (j == J - 1 && n == 31)) continue;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t t = t0 + 16 * (32 * j + n) + 8 * q + 4 * h;
      uint32_t o[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) o[b] = (uint32_t)acc[j][8 + 4 * q + b] + nx[4 * q + b];
      if (t + 4 <= nout) {
        *(SPS_GLOBAL u32x4_s4 *)(Yd + t) = u32x4_s4{o[0], o[1], o[2], o[3]};
      } else {
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (t + b < nout) Yd[t + b] = o[b];
      }
    }
  }
}

// One workgroup's share: trials [d_lo, d_lo + nw dpw) of DM block dblk x
// outputs [t0, t0 + 512 m - 16) of one filterbank.  P, B: the staged delay
// table of this tiling (StagedDelays).  With seg > 0 (a multiple of CS) the
// channels form consecutive groups of seg and group g's partial sums go to
// plane Y + g seg_stride instead of one total (the first stage of subband
// dedispersion in one pass over all channels).
//
// Rows are double-buffered: the next slab's loads are issued before the
// current slab is summed and stored to the other buffer after it.  INTERIOR:
// every staged window lies below nsamp_in and every slab is whole, so loads
// need no guard.
template <int J, int DPW, int NW, int CS, int KMAX, bool SEG = false, bool INTERIOR = false>
__device__ __forceinline__ void dedisperse_block(
    const uint8_t *__restrict__ X, int64_t pitch, int64_t nsamp_in, const uint4 *__restrict__ P,
    int pcols, const int2 *__restrict__ B, int nchan, int ndm, uint32_t *__restrict__ Y,
    int64_t nout, int lds_pitch, int64_t t0, int dblk, u32x4 *smem, int seg = 0,
    int64_t seg_stride = 0) {
  static_assert(CS == NW, "each wave stages one row of a slab");
  constexpr int GPS = CS / 4;  // groups of a slab
  static_assert(CS % 4 == 0 && GPS <= 4, "a lane row of 16 holds a slab's groups");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int n = lane & 31, h = lane >> 5;
  const int dw0 = dblk * (NW * DPW) + wave * DPW;
  const int buf_bytes = CS * lds_pitch;
  const int nslab = pcols / CS;
  const uint32_t row4 = (uint32_t)n * 0x00040004u, row_sel = (uint32_t)(n & 3) * 0x01010101u;
  char *lds = reinterpret_cast<char *>(smem);

  i32x16 acc[DPW][J];
#pragma unroll
  for (int k = 0; k < DPW; ++k) reset_acc<J>(acc[k], SEG ? seg : pcols);

  // Trials past the last one (a partial DM block) repeat the last trial's
  // entries, so the channel loop has no per-trial branch; store_acc drops
  // them.
  const SPS_GLOBAL u32x4 *Pl[DPW];
#pragma unroll
  for (int k = 0; k < DPW; ++k)
    Pl[k] = (const SPS_GLOBAL u32x4 *)gmem(P) + (int64_t)min(dw0 + k, ndm - 1) * (pcols / 2) +
            2 * (lane & (GPS - 1)) + h;
  // this wave's row of 64 slabs at a time: lane l holds slab 64 i + l's
  const SPS_GLOBAL u32x2 *Bw = (const SPS_GLOBAL u32x2 *)gmem(B) + (int64_t)dblk * pcols + wave;
  auto rows_of = [&](int i) { return Bw[(int64_t)min(64 * i + lane, nslab - 1) * CS]; };
  u32x2 rows = rows_of(0);

  u32x4 st[KMAX];
  auto stage_load = [&](int s) {
    const int c = s * CS + wave;
    const int first = __builtin_amdgcn_readlane((int)rows[0], s & 63);
    const int nv = __builtin_amdgcn_readlane((int)rows[1], s & 63) + 32 * J;
    if constexpr (INTERIOR) {
      const SPS_GLOBAL u32x4 *src =
          (const SPS_GLOBAL u32x4 *)(gmem(X) + (int64_t)c * pitch + t0 + first);
      // every lane loads; lanes past the row repeat its last vector, which
      // stage_store skips
#pragma unroll
      for (int u = 0; u < KMAX; ++u)
        st[u] = src[64 * u + 63 < 32 * J ? lane + 64 * u : min(lane + 64 * u, nv - 1)];
    } else {
#pragma unroll
      for (int u = 0; u < KMAX; ++u) {
        st[u] = u32x4{0u, 0u, 0u, 0u};
        const int k = lane + 64 * u;
        const int64_t s0 = t0 + first + 16 * (int64_t)k;
        if (c < nchan && k < nv && s0 < nsamp_in) {
          u32x4 v = *(const SPS_GLOBAL u32x4 *)(gmem(X) + (int64_t)c * pitch + s0);
          const int64_t left = nsamp_in - s0;
          if (left < 16) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int64_t keep = left - 4 * q;
              v[q] = keep >= 4 ? v[q] : (keep <= 0 ? 0u : (v[q] & ((1u << (8 * keep)) - 1u)));
            }
          }
          st[u] = v;
        }
      }
    }
  };
  auto stage_store = [&](int s, int buf) {
    const int nv = __builtin_amdgcn_readlane((int)rows[1], s & 63) + 32 * J;
    u32x4 *dst = reinterpret_cast<u32x4 *>(lds + buf * buf_bytes + wave * lds_pitch);
#pragma unroll
    for (int u = 0; u < KMAX; ++u)
      if (64 * u + 63 < 32 * J || lane + 64 * u < nv) dst[lane + 64 * u] = st[u] ^ 0x80808080u;
  };

  u32x4 ent[DPW];
#pragma unroll
  for (int k = 0; k < DPW; ++k) ent[k] = Pl[k][0];
  stage_load(0);
  stage_store(0, 0);
  __syncthreads();

  int buf = 0;
#pragma unroll 1
  for (int s = 0; s < nslab;) {
    const int s1 = SEG ? s + seg / CS : nslab;
#pragma unroll 1
    for (; s < s1; ++s) {
      const bool more = s + 1 < nslab;
      if (more) {
        if (((s + 1) & 63) == 0) rows = rows_of((s + 1) >> 6);
        stage_load(s + 1);
      }
      u32x4 next[DPW];
#pragma unroll
      for (int k = 0; k < DPW; ++k) next[k] = Pl[k][2 * GPS * (int64_t)min(s + 1, nslab - 1)];
      const uint32_t base = (uint32_t)(16 * n + buf * buf_bytes);
#pragma unroll
      for (int k = 0; k < DPW; ++k) {
        const u32x4 e = ent[k];
#define SPS_ADD_GROUP(q)                                                                \
  if constexpr (q < GPS)                                                                \
    add_group<J>(acc[k], lds, row_lane<q>(e[0]) + base, row_lane<q>(e[1]) + base,       \
                 row_lane<q>(e[2]) + row4, row_lane<q>(e[3]) + row_sel);
        SPS_ADD_GROUP(0)
        SPS_ADD_GROUP(1)
        SPS_ADD_GROUP(2)
        SPS_ADD_GROUP(3)
#undef SPS_ADD_GROUP
      }
      if (more) stage_store(s + 1, buf ^ 1);
      __syncthreads();
      buf ^= 1;
#pragma unroll
      for (int k = 0; k < DPW; ++k) ent[k] = next[k];
    }
#pragma unroll
    for (int k = 0; k < DPW; ++k) {
      store_acc<J>(acc[k], SEG ? Y + (int64_t)(s * CS / seg - 1) * seg_stride : Y, nout, ndm,
                   dw0 + k, lane, t0);
      if constexpr (SEG) reset_acc<J>(acc[k], seg);
    }
  }
}

// DM blocks per panel of the workgroup order.  The workgroups resident on an
// XCD then cover a few DM blocks x time tiles: their staged delay rows stay
// in the XCD's L2 and the input windows of neighbouring blocks and tiles
// overlap.  Measured on the full-scale channels and trials at 2^18 outputs:
// panels of 4, 8, 16 and 32 blocks 37.4, 36.5, 36.7 and 37.8 ms.
constexpr int kPanel = 8;

template <int J, int DPW, int NW, int CS, int KMAX, int WPE, bool SEG>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(WPE))) void
dedisperse_kernel(const uint8_t *__restrict__ X, int64_t pitch, int64_t nsamp_in,
                  const uint4 *__restrict__ P, int pcols, const int2 *__restrict__ B, int nchan,
                  int ndm, uint32_t *__restrict__ Y, int64_t nout, int lds_pitch, int ntiles,
                  int ndmb, int per_xcd, int seg, int64_t seg_stride, int dmax) {
  extern __shared__ u32x4 smem[];  // two slab buffers of CS rows x lds_pitch bytes
  const int blk = blockIdx.x;
  const int logical = (blk & 7) * per_xcd + (blk >> 3);
  if (logical >= ntiles * ndmb) return;
  // panels of kPanel DM blocks: DM block fastest inside a panel, then the
  // time tile, then the next panel
  const int panel = logical / (ntiles * kPanel);
  const int pd = min(kPanel, ndmb - panel * kPanel);
  const int rem = logical - panel * (ntiles * kPanel);
  const int tile = rem / pd;
  const int dblk = panel * kPanel + rem % pd;
  const int64_t t0 = (int64_t)tile * (512 * J - 16);
  // every staged row starts at or below t0 + dmax and spans lds_pitch bytes
  if (nchan % CS == 0 && t0 + dmax + lds_pitch <= nsamp_in)
    dedisperse_block<J, DPW, NW, CS, KMAX, SEG, true>(X, pitch, nsamp_in, P, pcols, B, nchan, ndm,
                                                      Y, nout, lds_pitch, t0, dblk, smem, seg,
                                                      seg_stride);
  else
    dedisperse_block<J, DPW, NW, CS, KMAX, SEG, false>(X, pitch, nsamp_in, P, pcols, B, nchan,
                                                       ndm, Y, nout, lds_pitch, t0, dblk, smem,
                                                       seg, seg_stride);
}

// Many filterbanks that share a plan (beams of one receiver, chunks of
// different lengths): the work items (beam, time tile, DM block) form one
// flat range, DM block fastest, and each workgroup takes one item.  The item
// numbering gives each XCD a contiguous share, so the workgroups resident on
// an XCD cover neighbouring time tiles of all DM blocks of a beam.
template <int J, int DPW, int NW, int CS, int KMAX, int WPE>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(WPE))) void
dedisperse_batch_kernel(const BeamWork *__restrict__ beams, int nbeams, int64_t total_items,
                        int64_t per_xcd, const uint4 *__restrict__ P, int pcols,
                        const int2 *__restrict__ B, int nchan, int ndm, int lds_pitch,
                        int ndmb, int dmax) {
  extern __shared__ u32x4 smem[];
  const int64_t item = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (item >= total_items) return;
  const BeamWork &bw = beams[find_beam<&BeamWork::dd_begin>(beams, nbeams, item)];
  const int64_t local = item - bw.dd_begin;
  const int dblk = (int)(local % ndmb);
  const int64_t tile = local / ndmb;
  const int64_t t0 = tile * (512 * J - 16);
  if (nchan % CS == 0 && t0 + dmax + lds_pitch <= bw.nsamp_in)
    dedisperse_block<J, DPW, NW, CS, KMAX, false, true>(bw.X, bw.pitch, bw.nsamp_in, P, pcols, B,
                                                        nchan, ndm, bw.Y, bw.nout, lds_pitch, t0,
                                                        dblk, smem);
  else
    dedisperse_block<J, DPW, NW, CS, KMAX, false, false>(bw.X, bw.pitch, bw.nsamp_in, P, pcols,
                                                         B, nchan, ndm, bw.Y, bw.nout, lds_pitch,
                                                         t0, dblk, smem);
}

// Staged form of the delay table for blocks of nd trials and slabs of cs rows
// of row_bytes bytes (see StagedDelays).  One thread per (trial, group of 4 columns); columns past
// the last channel (up to pcols, a multiple of cs) read the start of their
// zeroed slab row.  Delays are non-decreasing in the trial, so a trial's
// offset from its block's first staged sample is >= 0.
__global__ __launch_bounds__(256) void stage_delays_kernel(const int32_t *__restrict__ D,
                                                           int nchan, int ndm, int pcols, int nd,
                                                           int cs, int row_bytes,
                                                           uint4 *__restrict__ P,
                                                           int2 *__restrict__ B) {
  const int groups = pcols / 4;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)ndm * groups) return;
  const int d = (int)(i / groups);
  const int c0 = 4 * (int)(i - (int64_t)d * groups);
  const int dlo = d - d % nd;
  uint32_t off[4], r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = c0 + k;
    int32_t first = 0, v = 0, last = 0;
    if (c < nchan) {
      first = D[(int64_t)dlo * nchan + c] & ~15;
      v = D[(int64_t)d * nchan + c] - first;
      last = D[(int64_t)min(dlo + nd - 1, ndm - 1) * nchan + c] - first;
    }
    off[k] = (uint32_t)((c % cs) * row_bytes + (v & ~15));
    r[k] = (uint32_t)(v & 15);
    if (d == dlo) B[(int64_t)(d / nd) * pcols + c] = make_int2(first, last >> 4);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
    P[2 * i + h] = make_uint4(off[h], off[2 + h], 4 * r[2 * h] | (4 * r[2 * h + 1]) << 16,
                              (r[2 * h] & 3) * 0x00000101u | (r[2 * h + 1] & 3) * 0x01010000u);
}

// Plain fallback for delay spreads too wide to stage in LDS: one thread sums
// four consecutive outputs of one trial straight from global memory.
__global__ __launch_bounds__(256) void dedisperse_direct_kernel(
    const uint8_t *__restrict__ X, int64_t pitch, int64_t nsamp_in,
    const int32_t *__restrict__ D, int nchan, int ndm, uint32_t *__restrict__ Y, int64_t nout) {
  const int64_t t = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  if (t >= nout) return;
  for (int d = blockIdx.y; d < ndm; d += gridDim.y) {
    const int32_t *Dd = D + (int64_t)d * nchan;
    uint32_t acc[4] = {0u, 0u, 0u, 0u};
    for (int c = 0; c < nchan; ++c) {
      const uint8_t *row = X + (int64_t)c * pitch;
      const int64_t s = t + Dd[c];
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (s + b < nsamp_in) acc[b] += row[s + b];
    }
    uint32_t *Yd = Y + (int64_t)d * nout;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if (t + b < nout) Yd[t + b] = acc[b];
  }
}

// Bytes of LDS of a launch; above 64 KiB the kernel has to ask for them.
template <typename K>
hipError_t allow_lds(K kern, size_t lds) {
  if (lds <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

template <int J, int DPW, int NW, int CS, int KMAX, int WPE, bool SEG>
hipError_t launch_cfg(int lds_pitch, const uint8_t *X, int64_t pitch, int64_t nsamp_in,
                      const StagedDelays &sd, int nchan, int ndm, uint32_t *Y, int64_t nout,
                      hipStream_t stream, int seg, int64_t seg_stride) {
  constexpr int NT = 512 * J - 16;
  constexpr int ND = NW * DPW;
  if (lds_pitch > 16 * 64 * KMAX || lds_pitch % 16 != 0) return hipErrorInvalidValue;
  if (SEG != (seg > 0) || (SEG && (seg % CS != 0 || nchan % seg != 0)))
    return hipErrorInvalidValue;
  const int64_t ntiles64 = (nout + NT - 1) / NT;
  const int ndmb = (ndm + ND - 1) / ND;
  const int64_t total = ntiles64 * ndmb;
  if (total > (int64_t)0x7FFFFFFF - 8) return hipErrorInvalidValue;
  const int per_xcd = (int)((total + 7) / 8);
  const int grid = per_xcd * 8;
  const size_t lds = 2 * (size_t)CS * (size_t)lds_pitch;
  auto kern = dedisperse_kernel<J, DPW, NW, CS, KMAX, WPE, SEG>;
  const hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), lds, stream, X, pitch, nsamp_in, sd.P,
                     sd.pcols, sd.B, nchan, ndm, Y, nout, lds_pitch, (int)ntiles64, ndmb, per_xcd,
                     seg, seg_stride, sd.dmax);
  return hipGetLastError();
}

template <int J, int DPW, int NW, int CS, int KMAX, int WPE>
hipError_t launch_batch_cfg(int lds_pitch, const BeamWork *beams, int nbeams, int64_t total,
                            const StagedDelays &sd, int nchan, int ndm, int grid,
                            hipStream_t stream) {
  constexpr int ND = NW * DPW;
  // one workgroup per item: grid = 8 ceil(total / 8)
  if (lds_pitch > 16 * 64 * KMAX || lds_pitch % 16 != 0 || grid % 8 != 0 ||
      (int64_t)grid < total)
    return hipErrorInvalidValue;
  const int ndmb = (ndm + ND - 1) / ND;
  const size_t lds = 2 * (size_t)CS * (size_t)lds_pitch;
  auto kern = dedisperse_batch_kernel<J, DPW, NW, CS, KMAX, WPE>;
  const hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), lds, stream, beams, nbeams, total,
                     (int64_t)(grid / 8), sd.P, sd.pcols, sd.B, nchan, ndm, lds_pitch, ndmb,
                     sd.dmax);
  return hipGetLastError();
}

}  // namespace

int64_t dedisp_lds_pitch(const DedispConfig &cfg, int spread) {
  // A row starts up to 15 samples before its block's first window; a window
  // is read as 32 m whole 16-byte chunks.
  return (((int64_t)spread + 15) & ~(int64_t)15) + 512 * cfg.m;
}

int dedisp_block_spread(const int32_t *Dh, int nchan, int ndm, int nd) {
  int spread = 0;
  for (int d0 = 0; d0 < ndm; d0 += nd) {
    const int d1 = (d0 + nd < ndm ? d0 + nd : ndm) - 1;
    const int32_t *lo = Dh + (int64_t)d0 * nchan;
    const int32_t *hi = Dh + (int64_t)d1 * nchan;
    for (int c = 0; c < nchan; ++c) {
      const int s = hi[c] - lo[c];
      if (s > spread) spread = s;
    }
  }
  return spread;
}

// Compiled tilings: (m, dpw, nw, cs, kmax, waves per EU).  kmax bounds the
// staged row length (lds_pitch <= 1024 kmax bytes).
#define SPS_DEDISP_CONFIGS(X) \
  X(4, 1, 16, 16, 3, 4)       \
  X(3, 1, 16, 16, 3, 4)       \
  X(4, 1, 8, 8, 4, 4)         \
  X(2, 1, 16, 16, 3, 4)       \
  X(4, 1, 8, 8, 6, 2)         \
  X(4, 1, 8, 8, 9, 2)         \
  X(1, 1, 16, 16, 3, 4)

bool dedisp_config_supported(const DedispConfig &c) {
#define SPS_MATCH(m_, dpw_, nw_, cs_, kmax_, wpe_)                                      \
  if (c.m == m_ && c.dpw == dpw_ && c.nw == nw_ && c.cs == cs_ && c.kmax == kmax_ && \
      c.wpe == wpe_)                                                                  \
    return true;
  SPS_DEDISP_CONFIGS(SPS_MATCH)
#undef SPS_MATCH
  return false;
}

// The time tile for spans of nouts[0 .. n) outputs: any m up to c.m reads the
// table and rows staged for c.  A workgroup of m steps costs WG[m] (relative;
// measured on 4096 channels x 2048 trials x 2^18 outputs: 57, 53, 45 and 32 T
// sample-adds/s at m = 4, 3, 2 and 1), and one workgroup runs on each of 256
// CUs at a time: long spans take c.m, a span of few workgroups smaller tiles
// that fill the chip, and one that ends early in its last tile the tiles that
// waste least.
// RULE_FIGURES
DedispConfig dedisp_for_span(const DedispConfig &c, int ndm, const int64_t *nouts, int n) {
  static const double WG[5] = {0.0, 1.7, 2.47, 3.18, 4.0};
  DedispConfig best = c;
  if (c.m < 2 || c.m > 4) return best;
  double best_cost = -1.0;
  for (int m = c.m; m >= 1; --m) {
    DedispConfig q = c;
    q.m = m;
    if (!dedisp_config_supported(q)) continue;
    double items = 0.0;
    for (int i = 0; i < n; ++i) items += (double)dedisp_batch_items(q, ndm, nouts[i]);
    const double rounds = items / 256.0;
    const double cost = (rounds < 16.0 ? ceil(rounds) : rounds) * WG[m];
    if (best_cost < 0.0 || cost < best_cost) {
      best = q;
      best_cost = cost;
    }
  }
  return best;
}

int64_t dedisp_batch_items(const DedispConfig &c, int ndm, int64_t nout) {
  const int64_t nt = c.nt(), nd = c.nd();
  return ((nout + nt - 1) / nt) * ((ndm + nd - 1) / nd);
}

hipError_t launch_dedisperse_batch(const DedispConfig &c, int lds_pitch, const BeamWork *beams,
                                   int nbeams, int64_t total_items, const StagedDelays &sd,
                                   int nchan, int ndm, int grid, hipStream_t stream) {
  if (!sd.matches(c, lds_pitch, nchan, ndm)) return hipErrorInvalidValue;
#define SPS_BLAUNCH(m_, dpw_, nw_, cs_, kmax_, wpe_)                                          \
  if (c.m == m_ && c.dpw == dpw_ && c.nw == nw_ && c.cs == cs_ && c.kmax == kmax_ &&         \
      c.wpe == wpe_)                                                                          \
    return launch_batch_cfg<m_, dpw_, nw_, cs_, kmax_, wpe_>(lds_pitch, beams, nbeams,        \
                                                             total_items, sd, nchan, ndm, grid, \
                                                             stream);
  SPS_DEDISP_CONFIGS(SPS_BLAUNCH)
#undef SPS_BLAUNCH
  return hipErrorInvalidValue;
}

hipError_t launch_dedisperse(const DedispConfig &c, int lds_pitch, const uint8_t *X,
                             int64_t pitch, int64_t nsamp_in, const int32_t *D,
                             const StagedDelays *sd, int nchan, int ndm, uint32_t *Y,
                             int64_t nout, hipStream_t stream, int seg, int64_t seg_stride) {
  if (c.m == 0) {
    if (seg != 0) return hipErrorInvalidValue;
    const int64_t nthreads = (nout + 3) / 4;
    const int64_t gx = (nthreads + 255) / 256;
    if (gx > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int gy = ndm < 65535 ? ndm : 65535;
    hipLaunchKernelGGL(dedisperse_direct_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0,
                       stream, X, pitch, nsamp_in, D, nchan, ndm, Y, nout);
    return hipGetLastError();
  }
  if (!sd || !sd->matches(c, lds_pitch, nchan, ndm)) return hipErrorInvalidValue;
#define SPS_LAUNCH(m_, dpw_, nw_, cs_, kmax_, wpe_)                                      \
  if (c.m == m_ && c.dpw == dpw_ && c.nw == nw_ && c.cs == cs_ && c.kmax == kmax_ &&     \
      c.wpe == wpe_)                                                                      \
    return seg > 0 ? launch_cfg<m_, dpw_, nw_, cs_, kmax_, wpe_, true>(                  \
                         lds_pitch, X, pitch, nsamp_in, *sd, nchan, ndm, Y, nout, stream, seg, \
                         seg_stride)                                                         \
                   : launch_cfg<m_, dpw_, nw_, cs_, kmax_, wpe_, false>(                     \
                         lds_pitch, X, pitch, nsamp_in, *sd, nchan, ndm, Y, nout, stream, 0, 0);
  SPS_DEDISP_CONFIGS(SPS_LAUNCH)
#undef SPS_LAUNCH
  return hipErrorInvalidValue;
}

void free_staged(StagedDelays &sd) {
  if (sd.P) (void)hipFree(sd.P);
  if (sd.B) (void)hipFree(sd.B);
  sd = StagedDelays{};
}

hipError_t stage_delays(StagedDelays &sd, const DedispConfig &c, int lds_pitch, const int32_t *D,
                        int nchan, int ndm, int32_t dmax) {
  if (c.m == 0) {
    free_staged(sd);
    return hipSuccess;
  }
  if (sd.matches(c, lds_pitch, nchan, ndm) && sd.dmax == dmax) return hipSuccess;
  if (nchan < 1 || ndm < 1 || lds_pitch % 16 != 0 || c.nd() < 1 || c.cs < 4 || c.cs % 4 != 0)
    return hipErrorInvalidValue;
  const int pcols = (nchan + c.cs - 1) / c.cs * c.cs;
  const int64_t n = (int64_t)ndm * (pcols / 4);
  const int64_t nb = (int64_t)((ndm + c.nd() - 1) / c.nd()) * pcols;
  if ((n + 255) / 256 > 0x7FFFFFFF) return hipErrorInvalidValue;
  free_staged(sd);
  hipError_t e = hipMalloc(&sd.P, 2 * sizeof(uint4) * (size_t)n);
  if (e == hipSuccess) e = hipMalloc(&sd.B, sizeof(int2) * (size_t)nb);
  if (e != hipSuccess) {
    free_staged(sd);
    return e;
  }
  // null stream, waited for: callers may launch on any stream afterwards
  hipLaunchKernelGGL(stage_delays_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, nullptr,
                     D, nchan, ndm, pcols, c.nd(), c.cs, lds_pitch, sd.P, sd.B);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  if (e != hipSuccess) {
    free_staged(sd);
    return e;
  }
  sd.nchan = nchan;
  sd.dmax = dmax;
  sd.pcols = pcols;
  sd.ndm = ndm;
  sd.nd = c.nd();
  sd.cs = c.cs;
  sd.pitch = lds_pitch;
  return hipSuccess;
}

}  // namespace sps
