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
// 1.9 GHz), the whole kernel takes 37 ms channel by channel; the form it
// replaces (byte permutes and packed 16-bit adds on the vector units) took 55
// ms.
#include <math.h>

#include <type_traits>

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

// The 16 samples from s0 (a multiple of 16) of a row, those at or past
// nsamp_in zero.
__device__ __forceinline__ u32x4 load_below(const uint8_t *row, int64_t s0, int64_t nsamp_in) {
  const int64_t left = nsamp_in - s0;
  if (left <= 0) return u32x4{0u, 0u, 0u, 0u};
  u32x4 v = *(const SPS_GLOBAL u32x4 *)(gmem(row) + s0);
  if (left < 16) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t keep = left - 4 * q;
      v[q] = keep >= 4 ? v[q] : (keep <= 0 ? 0u : (v[q] & ((1u << (8 * keep)) - 1u)));
    }
  }
  return v;
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
        if (c < nchan && k < nv) {
          st[u] = load_below(X + (int64_t)c * pitch, s0, nsamp_in);
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

// ---- channels in pairs ----
//
// The delays of neighbouring channels differ by nearly the same amount over a
// block of 16 trials: by r or r + 1.  So a workgroup forms the sums of a
// channel pair (c, c + 1) at both distances once and every trial reads one of
// them in place of two rows: half the products and half the LDS reads.  A
// slab of 16 channels then stages 8 pairs x 2 distances = 16 rows, one pair
// by each of 8 waves of two trials.
//
// A sum is held as a signed byte, (x - 128) + (y - 128).  Where a row's sums
// leave that range, a pair has more than two distances in the block, or its
// window reaches past nsamp_in, the rows hold channel c alone and a bit in LDS
// says so; when all slabs are done the second channels of those pairs are
// summed one by one over the trials that read such a row (their other trials
// read zeros).  The same pass takes the channels past the last whole slab and,
// when most rows so far did not hold sums, all channels from there on.
//
// What bounds it: about as much time goes into the rows (two loads, ~200 vector
// instructions and 6 LDS stores per wave and slab) as into the products, and
// the two overlap by half; either alone would take 21 to 24 ms where both take
// 30 (4096 channels x 2048 trials x 2^18 outputs, 37 ms channel by channel).
// Loads run two slabs ahead (one ahead: 46 ms), their table entries come from
// LDS so that no wait drains them (31.4 against 39.4 ms).
//
// The byte holds sums of 128 to 383, so the gain depends on the data's level.
// Gaussian noise, the same case, in pairs and channel by channel: sigma 16 at
// levels 128 and 140 30.5 and 37 ms, at 150 39 and 36 ms, at 80 to 100 41 and
// 37 ms; sigma 11 at 181 (noise after square-law downsampling) 41 and 36 ms;
// sigma 24 at 128 44 and 38 ms; uniform random bytes 43 and 39 ms.  256 channels
// x 1024 trials: 1.25 and 1.42 ms at 128, 1.75 and 1.4 ms at 80 to 100 and 181.
// The form before the matrix cores took 55 and 1.88 ms on all of them.
constexpr int kPairWaves = 8;  // of two trials each
constexpr int kPairKmax = 3;   // staged rows of at most 1024 kPairKmax bytes
constexpr int kZeroRow = 2048; // bytes of zeros a trial reads for nothing

// LDS of the paired kernel: two slab buffers, zeros, the block's pairs (B2), a
// word of row bits per slab, the list of single channels and its length.
constexpr size_t pair_lds_bytes(int lds_pitch, int nchan) {
  return 32 * (size_t)lds_pitch + kZeroRow + 8 * 8 * (size_t)(nchan / 16) +
         4 * (size_t)(nchan / 16) + 4 * (size_t)(nchan / 2) + 16;
}

typedef unsigned int u32x4_a1 __attribute__((ext_vector_type(4), aligned(1)));

template <int J>
__device__ __forceinline__ void pair_block(const uint8_t *__restrict__ X, int64_t pitch,
                                           int64_t nsamp_in, const uint4 *__restrict__ P,
                                           const int2 *__restrict__ B,
                                           const int32_t *__restrict__ D, int nchan, int ndm,
                                           uint32_t *__restrict__ Y, int64_t nout, int lds_pitch,
                                           int64_t t0, int dblk, u32x4 *smem) {
  constexpr int NW = kPairWaves, DPW = 16 / NW, CS = 16, KMAX = kPairKmax;
  static_assert(NW == 8, "a wave stages one pair of a slab");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int n = lane & 31, h = lane >> 5;
  const int dlo = dblk * 16, dw0 = dlo + wave * DPW;
  const int buf_bytes = CS * lds_pitch;
  const int nslab = nchan / CS;  // whole slabs, summed in pairs
  const uint32_t row4 = (uint32_t)n * 0x00040004u, row_sel = (uint32_t)(n & 3) * 0x01010101u;
  char *lds = reinterpret_cast<char *>(smem);
  char *zeros = lds + 2 * buf_bytes;
  u32x2 *info = reinterpret_cast<u32x2 *>(zeros + kZeroRow);
  uint32_t *bits = reinterpret_cast<uint32_t *>(info + 8 * nslab);
  uint32_t *list = bits + nslab;
  uint32_t *count = list + nchan / 2;

  i32x16 acc[DPW][J];
#pragma unroll
  for (int k = 0; k < DPW; ++k) reset_acc<J>(acc[k], nchan);
  for (int i = threadIdx.x; i < kZeroRow / 4; i += NW * 64)
    reinterpret_cast<uint32_t *>(zeros)[i] = 0u;
  for (int i = threadIdx.x; i < nslab; i += NW * 64) bits[i] = 0u;
  if (threadIdx.x == 0) *count = 0u;

  int s = 0;
  // an input of less than one vector, which a row may not even hold: channel by
  // channel, where nothing past nsamp_in is read
  if (nslab > 0 && nsamp_in >= 16) {
    // entries of 8 slabs at a time: lane i of a row of 16 holds group i & 1 of
    // slab 8 i' + i / 2; the row is turned by a slab after each
    const int ngroup = 2 * nslab;
    auto entries_of = [&](int k, int i) {
      const SPS_GLOBAL u32x4 *Pl =
          (const SPS_GLOBAL u32x4 *)gmem(P) + (int64_t)min(dw0 + k, ndm - 1) * (2 * ngroup) + h;
      return Pl[2 * min(16 * i + (lane & 15), ngroup - 1)];
    };
    // the block's pairs; read from LDS, so that no wait for them is a wait for
    // the rows in flight
    for (int i = threadIdx.x; i < 8 * nslab; i += NW * 64)
      info[i] = ((const SPS_GLOBAL u32x2 *)gmem(B))[(int64_t)dblk * nslab * 8 + i];
    __syncthreads();
    u32x4 sa[2][KMAX], sb[2][KMAX];
    // An entry of the pairs' table, wave-uniform, for this tile.
    struct Row {
      int first, dist, nv;
      bool edge, single;  // not wholly below nsamp_in; not to hold sums
    };
    auto row_of = [&](u32x2 o) {
      Row r;
      const int w = __builtin_amdgcn_readfirstlane((int)o[1]);
      r.first = __builtin_amdgcn_readfirstlane((int)o[0]);
      r.dist = w >> 9;
      r.nv = (w & 255) + 32 * J;
      r.edge = t0 + r.first + max(r.dist, 0) + 1 + 16 * r.nv > nsamp_in;
      r.single = r.edge || (w & 256) != 0;
      return r;
    };
    // both rows of the wave's pair of slab s1; at an edge any vectors of the
    // same rows (check_rows loads such a row itself)
    auto stage_load = [&](int s1, u32x2 o, auto set) {
      constexpr int Q = decltype(set)::value;
      const Row r = row_of(o);
      const int last = r.edge ? max((int)min(nsamp_in >> 4, (int64_t)r.nv) - 1, 0) : r.nv - 1;
      const SPS_GLOBAL uint8_t *row =
          gmem(X) + (int64_t)(s1 * CS + 2 * wave) * pitch + (r.edge ? (int64_t)0 : t0 + r.first);
      const SPS_GLOBAL u32x4 *x = (const SPS_GLOBAL u32x4 *)row;
      const SPS_GLOBAL u32x4_a1 *y =
          (const SPS_GLOBAL u32x4_a1 *)(row + pitch + (r.edge ? 0 : r.dist));
#pragma unroll
      for (int u = 0; u < KMAX; ++u) {
        const int k = min(lane + 64 * u, last);
        sa[Q][u] = x[k];
        sb[Q][u] = y[k];
      }
    };
    // Vectors U0 .. U1 - 1 of each lane of the next slab's row sums: bytewise
    // sums with y, and with y one sample on (the byte after a lane's 16 is the
    // next lane's first; after the row's last it is never used).  lerp gives (x
    // + y) >> 1, in 64 .. 191 where the sum is in the range of a signed byte
    // plus 256; the low byte of the sum is twice that plus the low bit of x ^ y.
    // in: the AND of what has each byte's top bit set where it is in range.
    uint32_t in0, in1;
    auto sum_rows = [&](int nv, int buf, auto set, auto from, auto to) {
      constexpr int Q = decltype(set)::value, U0 = decltype(from)::value, U1 = decltype(to)::value;
      u32x4 *dst = reinterpret_cast<u32x4 *>(lds + buf * buf_bytes + 2 * wave * lds_pitch);
      u32x4 *dst1 = reinterpret_cast<u32x4 *>(lds + buf * buf_bytes + (2 * wave + 1) * lds_pitch);
      const auto add = [](uint32_t x, uint32_t y, uint32_t &in) {
        const uint32_t half = __builtin_amdgcn_lerp(x, y, 0u);
        in &= half + 0x40404040u;
        return ((half << 1) & 0xFEFEFEFEu) | ((x ^ y) & 0x01010101u);
      };
#pragma unroll
      for (int u = U0; u < U1; ++u) {
        const uint32_t over = __builtin_amdgcn_readlane((int)sb[Q][u + 1 < KMAX ? u + 1 : u][0], 0);
        const uint32_t nx = (uint32_t)__builtin_amdgcn_update_dpp(
            (int)over, (int)sb[Q][u][0], 0x130, 0xF, 0xF, false);
        u32x4 v0, v1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t x = sa[Q][u][q], y = sb[Q][u][q];
          v0[q] = add(x, y, in0);
          v1[q] = add(x, __builtin_amdgcn_alignbyte(q < 3 ? sb[Q][u][q < 3 ? q + 1 : q] : nx, y, 1),
                      in1);
        }
        // lanes past the row store its last vector once more
        const int k = 64 * u + 63 < 32 * J ? lane + 64 * u : min(lane + 64 * u, nv - 1);
        dst[k] = v0;
        dst1[k] = v1;
      }
    };
    // Marks and replaces the rows that do not hold sums.
    auto check_rows = [&](int s1, const Row &r, int buf, auto set) {
      constexpr int Q = decltype(set)::value;
      const bool out0 = r.single || __any((in0 & 0x80808080u) != 0x80808080u);
      const bool out1 = r.single || __any((in1 & 0x80808080u) != 0x80808080u);
      if (out0 || out1) {
        if (lane == 0) atomicOr(&bits[s1], ((out0 ? 1u : 0u) | (out1 ? 2u : 0u)) << (2 * wave));
        u32x4 *dst = reinterpret_cast<u32x4 *>(lds + buf * buf_bytes + 2 * wave * lds_pitch);
        u32x4 *dst1 = reinterpret_cast<u32x4 *>(lds + buf * buf_bytes + (2 * wave + 1) * lds_pitch);
        const uint8_t *row = X + (int64_t)(s1 * CS + 2 * wave) * pitch;
#pragma unroll
        for (int u = 0; u < KMAX; ++u)
          if (lane + 64 * u < r.nv) {
            u32x4 x = sa[Q][u];
            if (r.edge) x = load_below(row, t0 + r.first + 16 * (int64_t)(lane + 64 * u), nsamp_in);
            if (out0) dst[lane + 64 * u] = x ^ 0x80808080u;
            if (out1) dst1[lane + 64 * u] = x ^ 0x80808080u;
          }
      }
    };
    auto pair_of = [&](int s1) { return info[8 * min(s1, nslab - 1) + wave]; };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, KMAX> c3{};

    u32x4 ent[DPW], next[DPW];
#pragma unroll
    for (int k = 0; k < DPW; ++k) next[k] = ent[k] = entries_of(k, 0);
    // loads of slabs past the last repeat it, so that every slab has the same
    // count of them in flight
    stage_load(0, pair_of(0), c0);
    stage_load(min(1, nslab - 1), pair_of(1), c1);
    {
      const Row r = row_of(pair_of(0));
      in0 = in1 = ~0u;
      sum_rows(r.nv, 0, c0, c0, c3);
      check_rows(0, r, 0, c0);
      stage_load(min(2, nslab - 1), pair_of(2), c0);
    }
    __syncthreads();

    int single = 0, end = nslab;
    // Slab s in buffer buf, and the sums of the next one's rows (the last slab
    // again past the end: stored, never read) among the products: the vector
    // units work on the rows while the matrix cores are busy.
    auto products = [&](int buf) {
      const uint32_t base = (uint32_t)(16 * n + buf * buf_bytes);
#pragma unroll
      for (int k = 0; k < DPW; ++k) {
        const u32x4 e = ent[k];
        add_group<J>(acc[k], lds, row_lane<0>(e[0]) + base, row_lane<0>(e[1]) + base,
                     row_lane<0>(e[2]) + row4, row_lane<0>(e[3]) + row_sel);
        add_group<J>(acc[k], lds, row_lane<1>(e[0]) + base, row_lane<1>(e[1]) + base,
                     row_lane<1>(e[2]) + row4, row_lane<1>(e[3]) + row_sel);
      }
    };
    // set: the registers of the next slab's loads
    auto step = [&](int buf, auto set) {
      const uint32_t held = bits[s];
      const u32x2 o1 = pair_of(s + 1), o3 = pair_of(s + 3);
      const Row r = row_of(o1);
      in0 = in1 = ~0u;
      products(buf);
      sum_rows(r.nv, buf ^ 1, set, c0, c2);
      if (r.nv > 128) sum_rows(r.nv, buf ^ 1, set, c2, c3);
      if (s + 1 < nslab) check_rows(s + 1, r, buf ^ 1, set);
      // the entries to come are loaded here, ahead of the rows, and taken over
      // below: a wait for them then leaves the rows in flight
      if ((s & 7) == 4) {
#pragma unroll
        for (int k = 0; k < DPW; ++k) next[k] = entries_of(k, (s >> 3) + 1);
      }
      stage_load(min(s + 3, nslab - 1), o3, set);
      single += __popc(__builtin_amdgcn_readfirstlane(held));
      __syncthreads();
      ++s;
      if ((s & 7) == 0) {
#pragma unroll
        for (int k = 0; k < DPW; ++k) ent[k] = next[k];
        // same in every wave: the bits of the slabs summed are complete
        if (single > 8 * s) end = s;
      } else {
#pragma unroll
        for (int k = 0; k < DPW; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            ent[k][i] = (uint32_t)__builtin_amdgcn_mov_dpp((int)ent[k][i], 0x12E, 0xF, 0xF, true);
      }
    };
#pragma unroll 1
    while (s < end) {
      step(0, c1);
      if (s < end) step(1, c0);
    }
    // the second channels of the rows that held their first alone; which of
    // the two distances: the low bit of the distance tells them apart
    for (int p = threadIdx.x; p < 8 * s; p += NW * 64) {
      const uint32_t m = (bits[p >> 3] >> (2 * (p & 7))) & 3u;
      if (m != 0u) {
        const uint32_t odd = (info[p][1] >> 9) & 1u;  // of the first row's distance
        const uint32_t need = odd ? (m >> 1) | ((m & 1u) << 1) : m;
        list[atomicAdd(count, 1u)] = (uint32_t)(2 * p + 1) | need << 30;
      }
    }
  }
  __syncthreads();

  // Channels one by one: the list, then all from the first slab not summed.
  const int nlist = __builtin_amdgcn_readfirstlane((int)*count);
  const int rest = CS * s, nsingle = nlist + nchan - rest;
  if (nsingle > 0) {
    const int ns = (nsingle + CS - 1) / CS;
    const SPS_GLOBAL int32_t *Dlo = gmem(D + (int64_t)dlo * nchan);
    const SPS_GLOBAL int32_t *Dhi = gmem(D + (int64_t)min(dlo + 15, ndm - 1) * nchan);
    // channel and, in the top bits, the distances (even, odd) that need it;
    // 0 past the last
    auto channel = [&](int k) {
      if (k >= nsingle) return 0u;
      return k < nlist ? list[k] : (uint32_t)(rest + k - nlist) | 3u << 30;
    };
    // this wave's two rows, 32 slabs at a time: lane l holds row l & 1 of slab
    // 32 i + l / 2
    u32x2 rows;
    uint32_t row_ch;
    auto rows_of = [&](int i) {
      row_ch = channel((32 * i + (lane >> 1)) * CS + 2 * wave + (lane & 1));
      const int c = (int)(row_ch & 0x3FFFFFFFu);
      const int first = Dlo[c] & ~15;
      rows = u32x2{(uint32_t)first, (uint32_t)((Dhi[c] - first) >> 4)};
    };
    u32x4 st[2][KMAX];
    auto stage_load = [&](int s1) {
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const int i = 2 * (s1 & 31) + w;
        const int c = __builtin_amdgcn_readlane((int)row_ch, i) & 0x3FFFFFFF;
        const int first = __builtin_amdgcn_readlane((int)rows[0], i);
        const int nv = __builtin_amdgcn_readlane((int)rows[1], i) + 32 * J;
        const uint8_t *row = X + (int64_t)c * pitch;
        if (t0 + first + 16 * nv <= nsamp_in) {
          // every lane loads; lanes past the row repeat its last vector
          const SPS_GLOBAL u32x4 *src = (const SPS_GLOBAL u32x4 *)(gmem(row) + t0 + first);
#pragma unroll
          for (int u = 0; u < KMAX; ++u) st[w][u] = src[min(lane + 64 * u, nv - 1)];
        } else {
#pragma unroll
          for (int u = 0; u < KMAX; ++u) {
            st[w][u] = u32x4{0u, 0u, 0u, 0u};
            const int k = lane + 64 * u;
            if (k < nv) st[w][u] = load_below(row, t0 + first + 16 * (int64_t)k, nsamp_in);
          }
        }
      }
    };
    auto stage_store = [&](int s1, int buf) {
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const int nv = __builtin_amdgcn_readlane((int)rows[1], 2 * (s1 & 31) + w) + 32 * J;
        u32x4 *dst = reinterpret_cast<u32x4 *>(lds + buf * buf_bytes + (2 * wave + w) * lds_pitch);
#pragma unroll
        for (int u = 0; u < KMAX; ++u)
          if (64 * u + 63 < 32 * J || lane + 64 * u < nv)
            dst[lane + 64 * u] = st[w][u] ^ 0x80808080u;
      }
    };
    // Entries: lane i of a row of 16 loads for slab row i; off is then moved
    // to where add_group's halves expect it (group g's rows 4 g + h and 4 g + 2
    // + h at lanes 4 g and 4 g + 2), r likewise (rows 4 g + 2 h and the next
    // at lanes 4 g and 4 g + 1, in the forms of the low and the high 16 bits).
    const int i16 = lane & 15;
    uint32_t er = 0, elo = 0, evd[DPW], eprev[DPW], off[DPW], rem[DPW], rsel[DPW];
    auto entry_load = [&](int s1) {
      er = channel(s1 * CS + i16);
      const int c = (int)(er & 0x3FFFFFFFu);
      elo = (uint32_t)Dlo[c];
#pragma unroll
      for (int k = 0; k < DPW; ++k) {
        const SPS_GLOBAL int32_t *Dd = gmem(D + (int64_t)min(dw0 + k, ndm - 1) * nchan);
        evd[k] = (uint32_t)Dd[c];
        eprev[k] = (uint32_t)Dd[max(c - 1, 0)];
      }
    };
    auto entry_make = [&](int buf) {
#pragma unroll
      for (int k = 0; k < DPW; ++k) {
        const uint32_t v = evd[k] - (elo & ~15u);
        const bool use = ((er >> 30) >> ((evd[k] - eprev[k]) & 1u)) & 1u;
        const uint32_t o = use ? (uint32_t)(i16 * lds_pitch) + (v & ~15u)
                               : (uint32_t)((2 - buf) * buf_bytes);  // zeros
        const uint32_t o1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)o, 0xB1, 0xF, 0xF, true);
        const uint32_t r1 =
            (uint32_t)__builtin_amdgcn_mov_dpp((int)(v & 15u), 0x4E, 0xF, 0xF, true);
        const uint32_t r = h ? r1 : v & 15u;
        off[k] = h ? o1 : o;
        rem[k] = 4 * r << ((lane & 1) * 16);
        rsel[k] = (r & 3u) * 0x0101u << ((lane & 1) * 16);
      }
    };
    rows_of(0);
    entry_load(0);
    stage_load(0);
    entry_make(0);
    stage_store(0, 0);
    __syncthreads();
    int buf = 0;
#pragma unroll 1
    for (int q = 0; q < ns; ++q) {
      const bool more = q + 1 < ns;
      if (more) {
        if (((q + 1) & 31) == 0) rows_of((q + 1) >> 5);
        stage_load(q + 1);
        entry_load(q + 1);
      }
      const uint32_t base = (uint32_t)(16 * n + buf * buf_bytes);
#pragma unroll
      for (int k = 0; k < DPW; ++k) {
        const uint32_t o = off[k], r = rem[k], rs = rsel[k];
#define SPS_ADD_GROUP(g)                                                                  \
  add_group<J>(acc[k], lds, row_lane<4 * g>(o) + base, row_lane<4 * g + 2>(o) + base,     \
               row_lane<4 * g>(r) + (row_lane<4 * g + 1>(r) + row4),                      \
               row_lane<4 * g>(rs) + (row_lane<4 * g + 1>(rs) + row_sel));
        SPS_ADD_GROUP(0)
        SPS_ADD_GROUP(1)
        SPS_ADD_GROUP(2)
        SPS_ADD_GROUP(3)
#undef SPS_ADD_GROUP
      }
      if (more) {
        stage_store(q + 1, buf ^ 1);
        entry_make(buf ^ 1);
      }
      __syncthreads();
      buf ^= 1;
    }
  }
#pragma unroll
  for (int k = 0; k < DPW; ++k) store_acc<J>(acc[k], Y, nout, ndm, dw0 + k, lane, t0);
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

template <int J>
__global__ __launch_bounds__(64 * kPairWaves) __attribute__((amdgpu_waves_per_eu(2))) void
dedisperse_pairs_kernel(const uint8_t *__restrict__ X, int64_t pitch, int64_t nsamp_in,
                        const uint4 *__restrict__ P, const int2 *__restrict__ B,
                        const int32_t *__restrict__ D, int nchan, int ndm,
                        uint32_t *__restrict__ Y, int64_t nout, int lds_pitch, int ntiles,
                        int ndmb, int per_xcd) {
  extern __shared__ u32x4 smem[];  // pair_lds_bytes
  const int blk = blockIdx.x;
  const int logical = (blk & 7) * per_xcd + (blk >> 3);
  if (logical >= ntiles * ndmb) return;
  const int panel = logical / (ntiles * kPanel);
  const int pd = min(kPanel, ndmb - panel * kPanel);
  const int rem = logical - panel * (ntiles * kPanel);
  const int tile = rem / pd;
  const int dblk = panel * kPanel + rem % pd;
  const int64_t t0 = (int64_t)tile * (512 * J - 16);
  pair_block<J>(X, pitch, nsamp_in, P, B, D, nchan, ndm, Y, nout, lds_pitch, t0, dblk, smem);
}

template <int J>
__global__ __launch_bounds__(64 * kPairWaves) __attribute__((amdgpu_waves_per_eu(2))) void
dedisperse_pairs_batch_kernel(const BeamWork *__restrict__ beams, int nbeams, int64_t total_items,
                              int64_t per_xcd, const uint4 *__restrict__ P,
                              const int2 *__restrict__ B, const int32_t *__restrict__ D, int nchan,
                              int ndm, int lds_pitch, int ndmb) {
  extern __shared__ u32x4 smem[];
  const int64_t item = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (item >= total_items) return;
  const BeamWork &bw = beams[find_beam<&BeamWork::dd_begin>(beams, nbeams, item)];
  const int64_t local = item - bw.dd_begin;
  const int dblk = (int)(local % ndmb);
  const int64_t t0 = (local / ndmb) * (512 * J - 16);
  pair_block<J>(bw.X, bw.pitch, bw.nsamp_in, P, B, D, nchan, ndm, bw.Y, bw.nout, lds_pitch, t0,
                dblk, smem);
}

// The pairs' table for blocks of 16 trials (see StagedDelays): one thread per
// (DM block, pair) of the whole slabs.  over: counts the pairs with more than
// two distances, or whose second row would start before its channel's.
__global__ __launch_bounds__(256) void stage_pairs_kernel(const int32_t *__restrict__ D, int nchan,
                                                          int ndm, int row_bytes,
                                                          uint4 *__restrict__ P,
                                                          int2 *__restrict__ B,
                                                          unsigned long long *over) {
  const int nslab = nchan / 16, groups = 2 * nslab;  // groups of 4 pairs
  const int nblk = (ndm + 15) / 16;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)nblk * groups) return;
  const int blk = (int)(i / groups), g = (int)(i - (int64_t)blk * groups);
  const int dlo = 16 * blk, dn = min(16, ndm - dlo);
  int first[4], rmin[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int p = 4 * g + k;
    const int32_t *col = D + (int64_t)dlo * nchan + 2 * p;
    int lo = col[1] - col[0], hi = lo;
    for (int d = 1; d < dn; ++d) {
      const int r = col[(int64_t)d * nchan + 1] - col[(int64_t)d * nchan];
      lo = min(lo, r);
      hi = max(hi, r);
    }
    first[k] = col[0] & ~15;
    rmin[k] = lo;
    const int last = (col[(int64_t)(dn - 1) * nchan] - first[k]) >> 4;
    const bool bad = hi - lo > 1 || first[k] + lo < 0 || lo < -(1 << 22) || lo >= 1 << 22;
    if (bad) atomicAdd(over, 1ull);
    B[(int64_t)blk * nslab * 8 + p] = make_int2(first[k], last | (bad ? 256 : lo * 512));
  }
  for (int d = 0; d < dn; ++d) {
    uint32_t off[4], r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int p = 4 * g + k;
      const int32_t *row = D + (int64_t)(dlo + d) * nchan + 2 * p;
      const int v = row[0] - first[k];
      off[k] = (uint32_t)((2 * (p % 8) + ((row[1] - row[0] - rmin[k]) & 1)) * row_bytes +
                          (v & ~15));
      r[k] = (uint32_t)(v & 15);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      P[2 * ((int64_t)(dlo + d) * groups + g) + h] =
          make_uint4(off[h], off[2 + h], 4 * r[2 * h] | (4 * r[2 * h + 1]) << 16,
                     (r[2 * h] & 3) * 0x00000101u | (r[2 * h + 1] & 3) * 0x01010000u);
  }
}

// Staged form of the delay table for blocks of nd trials and slabs of cs rows
// of row_bytes bytes (see StagedDelays).  One thread per (trial, group of 4
// columns); columns past the last channel (up to pcols, a multiple of cs) read
// the start of their zeroed slab row.  Delays are non-decreasing in the trial, so a trial's
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

template <int J>
hipError_t launch_pairs(int lds_pitch, const uint8_t *X, int64_t pitch, int64_t nsamp_in,
                        const StagedDelays &sd, int nchan, int ndm, uint32_t *Y, int64_t nout,
                        hipStream_t stream) {
  constexpr int NT = 512 * J - 16;
  if (lds_pitch > 1024 * kPairKmax || lds_pitch % 16 != 0) return hipErrorInvalidValue;
  const int64_t ntiles = (nout + NT - 1) / NT;
  const int ndmb = (ndm + 15) / 16;
  const int64_t total = ntiles * ndmb;
  if (total > (int64_t)0x7FFFFFFF - 8) return hipErrorInvalidValue;
  const int per_xcd = (int)((total + 7) / 8);
  const size_t lds = pair_lds_bytes(lds_pitch, nchan);
  auto kern = dedisperse_pairs_kernel<J>;
  const hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(64 * kPairWaves), lds, stream, X, pitch,
                     nsamp_in, sd.P2, sd.B2, sd.D, nchan, ndm, Y, nout, lds_pitch, (int)ntiles, ndmb, per_xcd);
  return hipGetLastError();
}

template <int J>
hipError_t launch_pairs_batch(int lds_pitch, const BeamWork *beams, int nbeams, int64_t total,
                              const StagedDelays &sd, int nchan, int ndm, int grid,
                              hipStream_t stream) {
  if (lds_pitch > 1024 * kPairKmax || lds_pitch % 16 != 0 || grid % 8 != 0 ||
      (int64_t)grid < total)
    return hipErrorInvalidValue;
  const size_t lds = pair_lds_bytes(lds_pitch, nchan);
  auto kern = dedisperse_pairs_batch_kernel<J>;
  const hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kPairWaves), lds, stream, beams, nbeams, total,
                     (int64_t)(grid / 8), sd.P2, sd.B2, sd.D, nchan, ndm, lds_pitch,
                     (ndm + 15) / 16);
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
  X(4, 1, 8, 8, 5, 4)         \
  X(3, 1, 8, 8, 5, 4)         \
  X(2, 1, 8, 8, 5, 4)         \
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
// table and rows staged for c.  A workgroup of m steps costs WG (relative;
// measured on 4096 channels x 2048 trials x 2^18 outputs: 57, 53, 45 and 32 T
// sample-adds/s at m = 4, 3, 2 and 1; with channels in pairs 73, 64, 47 and
// 25, hence pairs from m = 3), and one workgroup runs on each of 256 CUs at a
// time: long spans take c.m, a span of few workgroups smaller tiles that fill
// the chip, and one that ends early in its last tile the tiles that waste least.
// The costs are used for every channel count, and with 8 waves where a smaller
// m is compiled.
DedispConfig dedisp_for_span(const DedispConfig &c, int ndm, const int64_t *nouts, int n,
                             const StagedDelays &sd) {
  static const double kWG[5] = {0.0, 1.7, 2.47, 3.18, 4.0};
  static const double kPaired[5] = {0.0, 0.0, 0.0, 2.65, 3.11};
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
    const double cost =
        (rounds < 16.0 ? ceil(rounds) : rounds) * (sd.paired(m) ? kPaired[m] : kWG[m]);
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
  if (sd.paired(c.m)) {
#define SPS_PLAUNCH(m_)                                                                     \
  if (c.m == m_)                                                                            \
    return launch_pairs_batch<m_>(lds_pitch, beams, nbeams, total_items, sd, nchan, ndm, grid, \
                                  stream);
    SPS_PLAUNCH(4) SPS_PLAUNCH(3)
#undef SPS_PLAUNCH
    return hipErrorInvalidValue;
  }
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
  if (seg == 0 && sd->paired(c.m)) {
#define SPS_PLAUNCH(m_)                                                                       \
  if (c.m == m_)                                                                              \
    return launch_pairs<m_>(lds_pitch, X, pitch, nsamp_in, *sd, nchan, ndm, Y, nout, stream);
    SPS_PLAUNCH(4) SPS_PLAUNCH(3)
#undef SPS_PLAUNCH
    return hipErrorInvalidValue;
  }
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

void free_pairs(StagedDelays &sd) {
  if (sd.P2) (void)hipFree(sd.P2);
  if (sd.B2) (void)hipFree(sd.B2);
  sd.P2 = nullptr;
  sd.B2 = nullptr;
}

void free_staged(StagedDelays &sd) {
  if (sd.P) (void)hipFree(sd.P);
  if (sd.B) (void)hipFree(sd.B);
  free_pairs(sd);
  sd = StagedDelays{};
}

// Channels from which pairs pay: with fewer slabs the longer prologue is not
// made up (1024 trials x 500,000 outputs: 64 channels 1.16 ms without and 1.26
// with, 128 channels 1.68 and 1.70, 256 channels 2.72 and 2.55).
constexpr int kPairChannels = 256;

// Builds the pairs' table into sd where it pays: blocks of 16 trials of 16
// waves, enough channels, room in LDS, and at most an eighth of the pairs with
// more than two distances in their block, since their second channels are
// summed one by one.  2^18 outputs of level 128: 4096 channels x 2048 trials (1%
// such pairs) 37.5 ms without, 30.5 ms with; 1024 channels x 1024 trials (15%)
// 5.0 and 4.7 ms, but no gain once a twentieth of the channels is disturbed.
// The delays alone decide, not the data (see pair_block for other levels).
static hipError_t stage_pairs(StagedDelays &sd, const DedispConfig &c, int lds_pitch,
                              const int32_t *D, int nchan, int ndm) {
  if (c.nw != 16 || c.dpw != 1 || c.cs != 16 || nchan < kPairChannels || nchan >= 1 << 30 ||
      lds_pitch > 1024 * kPairKmax || pair_lds_bytes(lds_pitch, nchan) > 160 * 1024)
    return hipSuccess;
  const int nslab = nchan / 16, nblk = (ndm + 15) / 16;
  const int64_t threads = (int64_t)nblk * 2 * nslab;
  if ((threads + 255) / 256 > 0x7FFFFFFF) return hipSuccess;
  unsigned long long *over = nullptr, n = 0;
  hipError_t e = hipMalloc(&sd.P2, 4 * sizeof(uint4) * (size_t)ndm * (size_t)nslab);
  if (e == hipSuccess) e = hipMalloc(&sd.B2, 8 * sizeof(int2) * (size_t)nblk * (size_t)nslab);
  if (e == hipSuccess) e = hipMalloc(&over, sizeof(*over));
  const bool room = e == hipSuccess;
  if (room) e = hipMemset(over, 0, sizeof(*over));
  if (e == hipSuccess) {
    hipLaunchKernelGGL(stage_pairs_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0,
                       nullptr, D, nchan, ndm, lds_pitch, sd.P2, sd.B2, over);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpy(&n, over, sizeof(n), hipMemcpyDeviceToHost);
  if (over) (void)hipFree(over);
  if (e != hipSuccess || n > (unsigned long long)nblk * (unsigned long long)nslab) free_pairs(sd);
  if (!room) {  // no memory to spare: channel by channel
    (void)hipGetLastError();
    return hipSuccess;
  }
  return e;
}

hipError_t stage_delays(StagedDelays &sd, const DedispConfig &c, int lds_pitch, const int32_t *D,
                        int nchan, int ndm, int32_t dmax, bool segments) {
  if (c.m == 0) {
    free_staged(sd);
    return hipSuccess;
  }
  const bool pairs = !segments && c.m >= kPairSteps;  // smaller tiles read no P2, B2
  if (sd.matches(c, lds_pitch, nchan, ndm) && sd.dmax == dmax && (sd.pairs_seen || !pairs))
    return hipSuccess;
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
  if (e == hipSuccess && pairs) e = stage_pairs(sd, c, lds_pitch, D, nchan, ndm);
  if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  if (e != hipSuccess) {
    free_staged(sd);
    return e;
  }
  sd.D = D;
  sd.nchan = nchan;
  sd.dmax = dmax;
  sd.pcols = pcols;
  sd.ndm = ndm;
  sd.nd = c.nd();
  sd.cs = c.cs;
  sd.pitch = lds_pitch;
  sd.pairs_seen = pairs;
  return hipSuccess;
}

}  // namespace sps
