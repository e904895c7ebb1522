// Block encoders from 8-bit texel values, for the paper's export path (Sec. 3.4, last
// paragraph of Feature Map Compression): after training, F_uv and F_uvt are reconstructed
// from their parameters, quantised to 8 bits and block-compressed; the supplementary
// ablation's "w/o BC simulation" arm compresses a directly optimised map the same way.  The
// paper names no encoder.  Two are built, both integer-only and deterministic:
//
// * BC4 (one channel of 16 texels): the optimum in summed squared error over all 65536
//   endpoint pairs (both palette modes), each texel at its nearest palette entry; ties go to
//   the lowest pair e0 * 256 + e1, and per texel to the lowest selector.  One wave per block:
//   the pairs are walked by their difference, whose palette offsets fix a table of errors, and
//   pairs whose interval alone leaves texels too far out are skipped.
//
// * BC7 mode 6 (4 channels of 16 texels): its 2^58 endpoint settings are too many to try, so
//   the encoder is a fixed search.  (1) Endpoints at the corners of the texels' bounding box
//   along its principal diagonal: the channel of largest spread is the reference, and a
//   channel runs from its minimum to its maximum when its covariance with the reference is
//   >= 0, else from maximum to minimum.  (2) Both target endpoints quantised for each of the
//   four p-bit pairs, v = clamp(floor((x - p + 1) / 2), 0, 127); a candidate replaces the
//   current block only when strictly better.  (3) Twice: the least-squares endpoints of the
//   current indices (per channel the 2 x 2 normal equations of
//   sum ((64 - w) E0 + w E1 - 64 x)^2, solved exactly in integers, rounded half up, clamped to
//   0..255), quantised as in (2).  (4) Best-improvement local search at steps 8, 4, 2, 1, at
//   most 64 rounds per step, over 22 moves in a fixed order (each 7-bit value of endpoint 0,
//   then of endpoint 1, by -s and +s; all four values of endpoint 0, then of endpoint 1, by
//   -s and +s; the p-bit of endpoint 0, then of endpoint 1, flipped; a move leaving 0..127 is
//   not taken); the first strictly best move is taken while it improves.  (5) When texel 0's
//   index has its top bit set (the anchor index has 3 bits) the endpoints swap and every
//   index J becomes 15 - J, which decodes identically.  Every candidate's indices are
//   refitted: each texel takes its least-error index, the lowest on ties.
//
// * BC7 with several modes (Sec. 3.4: the BC7 compression may pick among the format's modes): after the
//   mode-6 search, every block tries mode 5 under each of its 4 rotations and mode 4 under
//   each rotation and both index selections, and keeps the candidate of least summed squared
//   error (ties: mode 6, then mode 5 by rotation, then mode 4 by rotation then selection).  A
//   rotation r > 0 encodes the texels with channel r - 1 and channel 3 exchanged.  Modes 5
//   and 4 fit their colour (3 channels) and alpha (1 channel) endpoints apart, each by the
//   same fixed search at its endpoint precision n and index width b: (1) the bounding-box
//   diagonal (one channel: its minimum and maximum), each 8-bit target quantised to the
//   n-bit value whose expansion is nearest (ties to the lower; the candidates are
//   round(x (2^n - 1) / 255) and its neighbours); (2) twice, the least-squares endpoints of
//   the current indices, quantised as in (1); (3) best-improvement local search at steps
//   2^(n - 4) .. 1 over each value of each endpoint -s and +s, then (several channels) all
//   values of one endpoint -s and +s, at most 64 rounds per step; (4) the anchor swap of
//   endpoints and indices J -> 2^b - 1 - J when texel 0's index has its top bit set.
#include <climits>

#include "bcsim.hpp"
#include "internal.hpp"

namespace ndgi {

// The 4 channels (0..255) of texel s of footprint f.
__device__ __forceinline__ void src_texel4(const TexSrc& S, int64_t f, int s, int q[4]) {
  if (S.u8) {
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = c < S.C ? (int)S.u8[(f * 16 + s) * S.C + c] : 0;
    return;
  }
  const int wb = S.W >> 2;
  const int64_t per = (int64_t)(S.H >> 2) * wb;
  const int64_t sl = f / per, rem = f - sl * per;
  const int x = 4 * (int)(rem % wb) + (s & 3), y = 4 * (int)(rem / wb) + (s >> 2);
  const int cw = S.codec ? 1 : 4;
  map_texel_u8(S.ep + f * 8, S.w + ((sl * S.H + y) * S.W + x) * cw, S.kind, S.codec, q);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kRor = 0x120;                       // row_ror:n = kRor + n (rows of 16 lanes)
constexpr int kQuadX1 = 0xB1, kQuadX2 = 0x4E;     // quad_perm [1,0,3,2] and [2,3,0,1]
constexpr int kHalfMirror = 0x141;                // lanes 0..7 of a half row reversed
// Sum, or, minimum and maximum over each row of 16 lanes, returned in all of them.
__device__ __forceinline__ int row_sum(int v) {
  v += (int)dpp_mov<kRor + 8>((uint32_t)v);
  v += (int)dpp_mov<kRor + 4>((uint32_t)v);
  v += (int)dpp_mov<kRor + 2>((uint32_t)v);
  return v + (int)dpp_mov<kRor + 1>((uint32_t)v);
}
__device__ __forceinline__ uint32_t row_or(uint32_t v) {
  v |= dpp_mov<kRor + 8>(v);
  v |= dpp_mov<kRor + 4>(v);
  v |= dpp_mov<kRor + 2>(v);
  return v | dpp_mov<kRor + 1>(v);
}
__device__ __forceinline__ uint32_t row_min(uint32_t v) {
  v = min(v, dpp_mov<kRor + 8>(v));
  v = min(v, dpp_mov<kRor + 4>(v));
  v = min(v, dpp_mov<kRor + 2>(v));
  return min(v, dpp_mov<kRor + 1>(v));
}
__device__ __forceinline__ uint32_t row_max(uint32_t v) { return ~row_min(~v); }
// The same over each half row (8 lanes).
template <typename Op>
__device__ __forceinline__ uint32_t half_reduce(uint32_t v, Op op) {
  v = op(v, dpp_mov<kQuadX1>(v));
  v = op(v, dpp_mov<kQuadX2>(v));
  return op(v, dpp_mov<kHalfMirror>(v));   // the quads are uniform by now
}
__device__ __forceinline__ int half_sum(int v) {
  return (int)half_reduce((uint32_t)v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t half_min(uint32_t v) {
  return half_reduce(v, [](uint32_t a, uint32_t b) { return min(a, b); });
}
__device__ __forceinline__ uint32_t half_or(uint32_t v) {
  return half_reduce(v, [](uint32_t a, uint32_t b) { return a | b; });
}
__device__ __forceinline__ int lane_of(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

// --------------------------------------------------------------------------------- BC4
__device__ __forceinline__ void bc4_palette8(int e0, int e1, int p[8]) {
  p[0] = e0;
  p[1] = e1;
  if (e0 > e1) {
#pragma unroll
    for (int j = 1; j <= 6; ++j) p[j + 1] = ((7 - j) * e0 + j * e1 + 3) / 7;
  } else {
#pragma unroll
    for (int j = 1; j <= 4; ++j) p[j + 1] = ((5 - j) * e0 + j * e1 + 2) / 5;
    p[6] = 0;
    p[7] = 255;
  }
}

// The palette of a pair depends on its lower endpoint only through an offset: with D the
// endpoints' difference, the 8-value palette (e0 > e1) is e1 + floor((k D + 3) / 7), k = 0..7,
// and the 6-value one (e0 <= e1) e0 + floor((k D + 2) / 5), k = 0..5, with 0 and 255.  So a
// texel's squared error is a table of its distance t from the lower endpoint, one table a
// difference: bc4_table(D, t) for t = -255..255 (without 0 and 255).
template <bool SIX>
__device__ __forceinline__ uint32_t bc4_table(int D, int t) {
  uint32_t best = 0xffffffffu;
#pragma unroll
  for (int k = 0; k <= (SIX ? 5 : 7); ++k) {
    const int d = t - (SIX ? (k * D + 2) / 5 : (k * D + 3) / 7);
    best = min(best, (uint32_t)(d * d));
  }
  return best;
}

// Bounds of a block.
struct Bc4Bounds {
  uint32_t below[256], above[256];   // error of the texels below / above an interval that starts / ends at i
};
// Texels X (uniform) and, for the 6-value mode, their least squared distance Z to 0 and 255.
template <bool SIX>
__device__ __forceinline__ void bc4_bound(const uint32_t X[16], const uint32_t Z[16], int v, Bc4Bounds& B) {
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    const int d = v - (int)X[s];
    uint32_t d2 = (uint32_t)(d * d);
    if (SIX) d2 = min(d2, Z[s]);
    lo += d > 0 ? d2 : 0u;
    hi += d < 0 ? d2 : 0u;
  }
  B.below[v] = lo;
  B.above[v] = hi;
}

__device__ __forceinline__ uint32_t wave_umin(uint32_t v) {
  const int r = (int)row_min(v);
  return min(min((uint32_t)lane_of(r, 0), (uint32_t)lane_of(r, 16)), min((uint32_t)lane_of(r, 32), (uint32_t)lane_of(r, 48)));
}

// A wave's part of difference D of one mode: lane takes lower endpoint 64 c + lane of chunk c;
// tab: the 511 errors of D.  The texels outside the pair's interval bound its error from below
// (texel by texel an entry outside the interval is 0 or 255 at best), and a chunk whose bounds
// all exceed the least error so far (lim) is skipped.
template <bool SIX>
__device__ __forceinline__ void bc4_pairs(const uint32_t X[16], const uint32_t Z[16], const Bc4Bounds& B,
                                          const uint16_t* tab, int D, int lane, uint32_t& best, uint32_t& pair,
                                          uint32_t& lim) {
#pragma unroll 1
  for (int c = 0; 64 * c < 256 - D; ++c) {
    const int e = 64 * c + lane;
    const bool in = e + D < 256;
    const uint32_t bound = B.below[in ? e : 255] + B.above[in ? e + D : 0];
    if (!__any(in && bound <= lim)) continue;
    const uint16_t* const at = tab + 255 - (in ? e : 0);
    uint32_t sse = 0;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const uint32_t d = at[X[s]];
      sse += SIX ? min(d, Z[s]) : d;
    }
    const uint32_t p = SIX ? (uint32_t)(e * 257 + D) : (uint32_t)(e * 257 + 256 * D);   // e0 * 256 + e1
    if (in && (sse < best || (sse == best && p < pair))) {
      best = sse;
      pair = p;
    }
    if (__any(best < lim)) lim = wave_umin(best);
  }
}

// Every pair of one mode, by difference.  A wave to a block (PRIV false): f holds two tables,
// filled by the workgroup one difference ahead of their use.  A workgroup to a block (PRIV): wave
// w of nw takes every nw-th difference with a table of its own, f[w].
template <bool SIX, bool PRIV>
__device__ __forceinline__ void bc4_mode(const uint32_t X[16], const uint32_t Z[16], const Bc4Bounds& B,
                                         uint16_t (*f)[512], int tid, bool live, int nw, uint32_t& best,
                                         uint32_t& pair, uint32_t& lim) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (PRIV) {
#pragma unroll 1
    for (int D = (SIX ? 0 : 1) + wave; D < 256; D += nw) {
      uint16_t* const tab = f[wave];
      wave_sync();   // the previous difference is read
      for (int i = lane; i < 511; i += 64) tab[i] = (uint16_t)bc4_table<SIX>(D, i - 255);
      wave_sync();
      bc4_pairs<SIX>(X, Z, B, tab, D, lane, best, pair, lim);
    }
  } else {
#pragma unroll 1
    for (int D = SIX ? 0 : 1; D < 256; ++D) {
      uint16_t* const tab = f[D & 1];
      for (int i = tid; i < 511; i += 256) tab[i] = (uint16_t)bc4_table<SIX>(D, i - 255);
      __syncthreads();   // filled; and the other table's readers are done
      if (live) bc4_pairs<SIX>(X, Z, B, tab, D, lane, best, pair, lim);
    }
  }
}

// Texel (lane & 15) of block i of the two jobs.
__device__ __forceinline__ uint32_t bc4_source(const EncodeJob& job, int64_t b, int lane) {
  if (job.src.u8) return job.src.u8[b * 16 + (lane & 15)];
  int q[4];
  src_texel4(job.src, b >> 2, lane & 15, q);
  const int c = (int)(b & 3);
  return (uint32_t)(c == 0 ? q[0] : (c == 1 ? q[1] : (c == 2 ? q[2] : q[3])));
}
// X and Z, and the least error so far from the texels' own range.
__device__ __forceinline__ uint32_t bc4_setup(uint32_t x, uint32_t X[16], uint32_t Z[16]) {
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    X[s] = (uint32_t)lane_of((int)x, s);
    Z[s] = min(X[s] * X[s], (255u - X[s]) * (255u - X[s]));
  }
  const uint32_t hi = (uint32_t)lane_of((int)row_max(x), 0), lo = (uint32_t)lane_of((int)row_min(x), 0);
  const uint32_t e = hi > lo ? bc4_table<false>((int)(hi - lo), (int)x - (int)lo) : 0u;
  return (uint32_t)lane_of(row_sum((int)e), 0);
}
// The wave's least error, then its lowest pair, as one key.
__device__ __forceinline__ uint64_t bc4_key(uint32_t best, uint32_t pair) {
  uint64_t key = ((uint64_t)best << 32) | pair;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t o = __shfl_xor(key, off, 64);
    key = o < key ? o : key;
  }
  return key;
}
// The block of a key's pair; x as above, all lanes of the wave take part.
__device__ __forceinline__ void bc4_write(uint64_t key, uint32_t x, int lane, uint8_t* out) {
  const int E0 = (int)((key >> 8) & 255u), E1 = (int)(key & 255u);
  int p[8];
  bc4_palette8(E0, E1, p);
  int code = 0, m = INT_MAX;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int d = p[c] - (int)x;
    if (d * d < m) {
      m = d * d;
      code = c;
    }
  }
  // gather the 16 selectors and pack
  uint64_t field = (uint64_t)code << (3 * (lane & 15));
  field = (uint64_t)row_or((uint32_t)field) | ((uint64_t)row_or((uint32_t)(field >> 32)) << 32);
  if (lane == 0) {
    const uint32_t lo = (uint32_t)E0 | ((uint32_t)E1 << 8) | ((uint32_t)(field & 0xffffu) << 16);
    *(uint2*)out = make_uint2(lo, (uint32_t)(field >> 16));
  }
}

// Block b: channel b % 4 of footprint b / 4 of a map source, or 16 texels at u8 + 16 b; the
// blocks of two maps in one launch.  A wave takes one block, four waves share the tables.
// Bound by VALU and LDS issue: 16 table reads a pair (consecutive lanes, consecutive entries)
// instead of 16 x 8 palette distances with a thread to an e0; 40,000 blocks took 22-24 ms that
// way and take 3.9-5.4 ms.
__global__ __launch_bounds__(256) void k_encode_bc4(EncodeJob ja, EncodeJob jb) {
  __shared__ uint16_t f[2][512];
  __shared__ Bc4Bounds bounds[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t n = ja.n + jb.n;
  for (int64_t i0 = 4 * (int64_t)blockIdx.x; i0 < n; i0 += 4 * (int64_t)gridDim.x) {
    const bool live = i0 + wave < n;
    const int64_t i = live ? i0 + wave : n - 1;
    const EncodeJob& job = i < ja.n ? ja : jb;
    const int64_t b = i < ja.n ? i : i - ja.n;
    const uint32_t x = bc4_source(job, b, lane);
    uint32_t X[16], Z[16], best = 0xffffffffu, pair = 0xffffffffu, lim = bc4_setup(x, X, Z);
    Bc4Bounds& B = bounds[wave];   // private to the wave
    __syncthreads();               // the previous block's readers of f are done
#pragma unroll 1
    for (int k = 0; k < 4; ++k) bc4_bound<false>(X, Z, 64 * k + lane, B);
    wave_sync();
    bc4_mode<false, false>(X, Z, B, f, tid, live, 4, best, pair, lim);
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < 4; ++k) bc4_bound<true>(X, Z, 64 * k + lane, B);
    wave_sync();
    bc4_mode<true, false>(X, Z, B, f, tid, live, 4, best, pair, lim);
    const uint64_t key = bc4_key(best, pair);
    if (live) bc4_write(key, x, lane, job.out + b * 8);
  }
}

// The same with a workgroup of 16 waves to a block, for launches that would leave most of the chip
// idle: the differences are dealt out over the waves, which then wait for each other once a block
// instead of 511 times.  Each wave fills tables that four blocks share above, so many blocks are
// better off there.  Constant to random texels, above and here: 256 blocks 360-517 and 50-64 us, 2048
// blocks 430-600 and 375-470, 3000 blocks 500-680 and 555-690.
constexpr int kBc4OneWaves = 16;
constexpr int64_t kBc4OnePerCu = 8;   // blocks a CU up to which a workgroup takes one
__global__ __launch_bounds__(64 * kBc4OneWaves) void k_encode_bc4_one(EncodeJob ja, EncodeJob jb) {
  __shared__ uint16_t f[kBc4OneWaves][512];
  __shared__ Bc4Bounds bounds[2];   // of each mode
  __shared__ uint64_t keys[kBc4OneWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int64_t i = blockIdx.x; i < ja.n + jb.n; i += gridDim.x) {
    const EncodeJob& job = i < ja.n ? ja : jb;
    const int64_t b = i < ja.n ? i : i - ja.n;
    const uint32_t x = bc4_source(job, b, lane);
    uint32_t X[16], Z[16], best = 0xffffffffu, pair = 0xffffffffu, lim = bc4_setup(x, X, Z);
    if (wave < 4) bc4_bound<false>(X, Z, tid, bounds[0]);
    else if (wave < 8) bc4_bound<true>(X, Z, tid - 256, bounds[1]);
    __syncthreads();
    bc4_mode<false, true>(X, Z, bounds[0], f, tid, true, kBc4OneWaves, best, pair, lim);
    bc4_mode<true, true>(X, Z, bounds[1], f, tid, true, kBc4OneWaves, best, pair, lim);
    const uint64_t key = bc4_key(best, pair);
    if (lane == 0) keys[wave] = key;
    __syncthreads();   // and the readers of the bounds are done
    if (wave == 0) {
      uint64_t k = keys[0];
#pragma unroll
      for (int w = 1; w < kBc4OneWaves; ++w) k = keys[w] < k ? keys[w] : k;
      bc4_write(k, x, lane, job.out + b * 8);
    }
    __syncthreads();   // the keys may be written again
  }
}

// ------------------------------------------------------------------------------- BC7
// One workgroup of six waves per block, one wave per family of searches, so that the 25
// searches of a block (one of mode 6; colour and alpha of mode 5 under 4 rotations, of mode 4
// under 4 rotations and 2 selections) run side by side:
//   wave 0  mode 6            lane = (half of the texels, move): 22 moves x 2
//   wave 1  mode 5 colour     16-lane row = rotation, lane = move (16 of them)
//   wave 2  mode 4 colour, 2-bit indices     as wave 1
//   wave 3  mode 4 colour, 3-bit indices     as wave 1
//   wave 4  the 8 alpha searches of 2-bit indices: 8 lanes each (4 moves x 2 parts)
//   wave 5  the 4 alpha searches of 3-bit indices: 16 lanes each (4 moves x 4 parts)
// A round of the local search costs one evaluation: each lane prices its own move over the
// block's texels and the best (error, move) is a minimum over the row (DPP, no LDS).  The
// steps outside the local search put one texel on each lane of a row instead.  A candidate is
// priced from its palette, packed as 4 bytes an entry p: a texel x is |x|^2 - max over entries
// of (2 p.x - |p|^2) away, one v_dot4 and one shift-add an entry, with the 16 packed texels
// uniform over the wave.  Bound by VALU issue (integer; 62% of the issue rate on a 128^2
// tile's 1792 blocks, whose last workgroups run alone).  An earlier kernel, a wave to a block
// that walked its 25 searches with 64 lanes to a candidate and shuffle sums, took 3.1 ms for
// those blocks in two launches, a chain of LDS-routed shuffles at one wave a SIMD; this one
// takes 0.086 ms in one launch, and 1.4-4.0 ms against 12-32 ms for 40,000 blocks (constant
// to random texels).
typedef uint16_t us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t us2_bits(us2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ us2 us2_of(int a, int b) { return (us2){(uint16_t)a, (uint16_t)b}; }

// The format's weight of a b-bit index.
template <int IB>
__host__ __device__ constexpr int bc7_weight(int j) {
  return (64 * j + ((1 << IB) - 1) / 2) / ((1 << IB) - 1);
}

// Palette of 8-bit endpoints (channel slots 0, 1 in E?a and 2, 3 in E?b): entry j's bytes
// p[j], placed by the byte selector sel, and n[j] = -|p[j]|^2.  ((64 - w) E0 + w E1 + 32) >> 6
// is the high byte of 256 E0 + 128 + 4 w (E1 - E0), which fits 16 bits.
template <int IB>
__device__ __forceinline__ void bc7_palette(us2 E0a, us2 E0b, us2 E1a, us2 E1b, uint32_t sel, uint32_t p[1 << IB],
                                            int n[1 << IB]) {
  const us2 ba = E0a * (us2)((uint16_t)256) + (us2)((uint16_t)128), da = E1a - E0a;
  const us2 bb = E0b * (us2)((uint16_t)256) + (us2)((uint16_t)128), db = E1b - E0b;
#pragma unroll
  for (int j = 0; j < (1 << IB); ++j) {
    const us2 w = (us2)((uint16_t)(4 * bc7_weight<IB>(j)));
    p[j] = __builtin_amdgcn_perm(us2_bits(bb + db * w), us2_bits(ba + da * w), sel);
    n[j] = -(int)__builtin_amdgcn_udot4(p[j], p[j], 0u, false);
  }
}

// max over entries of 2 p.x - |p|^2: |x|^2 minus it is the texel's least squared error.
template <int IB>
__device__ __forceinline__ int bc7_nearest(const uint32_t p[1 << IB], const int n[1 << IB], uint32_t x) {
  int best = INT_MIN;
#pragma unroll
  for (int j = 0; j < (1 << IB); ++j)
    best = max(best, (int)(__builtin_amdgcn_udot4(p[j], x, 0u, false) << 1) + n[j]);
  return best;
}
// The same with the entry that reaches it (the lowest on ties).
template <int IB>
__device__ __forceinline__ int bc7_nearest_index(const uint32_t p[1 << IB], const int n[1 << IB], uint32_t x, int& J) {
  int best = INT_MIN;
  J = 0;
#pragma unroll
  for (int j = 0; j < (1 << IB); ++j) {
    const int v = (int)(__builtin_amdgcn_udot4(p[j], x, 0u, false) << 1) + n[j];
    J = v > best ? j : J;
    best = max(best, v);
  }
  return best;
}

// Rounded least-squares endpoint floor((2 num + det) / (2 det)) clamped to 0..255: the exact
// integers (below 2^42) divided in FP64, whose quotient never rounds up to an integer (it would
// have to be within 2^-53 of one relative, and is at least 1 / (2 det) > 2^-34 away).
__device__ __forceinline__ int bc7_ls_endpoint(double num, double det) {
  return (int)fmin(fmax(floor((2.0 * num + det) / (2.0 * det)), 0.0), 255.0);
}

__device__ __forceinline__ int bc7_xpand(int v, int n) { return (v << (8 - n)) | (v >> (2 * n - 8)); }

// The n-bit value whose expansion is nearest to the 8-bit target x (ties to the lower).
__device__ __forceinline__ int bc7_quant(int x, int n) {
  const int top = (1 << n) - 1;
  const int g = min(max((x * top + 127) / 255, 0), top);
  int best = 0, bd = INT_MAX;
#pragma unroll
  for (int dv = -1; dv <= 1; ++dv) {
    const int v = min(max(g + dv, 0), top);
    const int d = abs(bc7_xpand(v, n) - x);
    if (d < bd || (d == bd && v < best)) {
      best = v;
      bd = d;
    }
  }
  return best;
}

// OR value v (< 256) into the 128-bit block (lo, hi) at bit pos.
__device__ __forceinline__ void bc7_put(uint64_t& lo, uint64_t& hi, uint32_t v, int pos) {
  if (pos >= 64) {
    hi |= (uint64_t)v << (pos - 64);
  } else {
    lo |= (uint64_t)v << pos;
    if (pos > 56) hi |= (uint64_t)v >> (64 - pos);
  }
}
// Index J of texel s into an index set of b-bit indices starting at bit pos (texel 0 has b - 1
// bits).
__device__ __forceinline__ void bc7_put_index(uint64_t& lo, uint64_t& hi, int J, int s, int pos, int b) {
  bc7_put(lo, hi, (uint32_t)J, s ? pos + b - 1 + b * (s - 1) : pos);
}

// What the searches of a block leave for its last step: each one's error and its share of the
// block's bits.  Search 0 is mode 6; 1 + 4 f + r is family f under rotation r, the families
// being mode 5 colour, mode 4 colour (2-bit, 3-bit indices), mode 5 alpha, mode 4 alpha
// (3-bit, 2-bit indices).
struct Bc7Found {
  int sse[25];
  uint32_t w[25][4];
};
__device__ __forceinline__ void bc7_found(Bc7Found& F, int k, int sse, uint64_t lo, uint64_t hi) {
  F.sse[k] = sse;
  F.w[k][0] = (uint32_t)lo;
  F.w[k][1] = (uint32_t)(lo >> 32);
  F.w[k][2] = (uint32_t)hi;
  F.w[k][3] = (uint32_t)(hi >> 32);
}

// ---- mode 6.  x = texel (lane & 15) packed, X[s] = texel s (uniform).
__device__ __forceinline__ void m6_search(uint32_t x, const uint32_t X[16], int lane, Bc7Found& F) {
  constexpr uint32_t kSel = 0x07050301u;
  const int row = lane >> 4;
  const int x2 = (int)__builtin_amdgcn_udot4(x, x, 0u, false);
  const int sum_x2 = lane_of(row_sum(x2), 0);
  // the current block: packed 7-bit values (slots 0, 1 | 2, 3), p-bits, error (uniform)
  us2 v0a = us2_of(0, 0), v0b = v0a, v1a = v0a, v1b = v0a;
  int p0 = 0, p1 = 0, sse = INT_MAX;
  auto expand = [](us2 v, int p) { return (v << (us2)((uint16_t)1)) | (us2)((uint16_t)p); };
  // this lane's texel index under the current block
  auto index = [&]() {
    uint32_t p[16];
    int n[16], J;
    bc7_palette<4>(expand(v0a, p0), expand(v0b, p0), expand(v1a, p1), expand(v1b, p1), kSel, p, n);
    bc7_nearest_index<4>(p, n, x, J);
    return J;
  };
  // targets A, B (8-bit, per channel, uniform) quantised for the four p-bit pairs: row q
  // prices pair q, and the least error in pair order is taken when strictly better
  auto quantised = [&](const int A[4], const int B[4]) {
    auto q7 = [](int t, int p) { return min(max((t - p + 1) >> 1, 0), 127); };
    const int q0 = row >> 1, q1 = row & 1;
    const us2 a0 = us2_of(q7(A[0], q0), q7(A[1], q0)), b0 = us2_of(q7(A[2], q0), q7(A[3], q0));
    const us2 a1 = us2_of(q7(B[0], q1), q7(B[1], q1)), b1 = us2_of(q7(B[2], q1), q7(B[3], q1));
    uint32_t p[16];
    int n[16];
    bc7_palette<4>(expand(a0, q0), expand(b0, q0), expand(a1, q1), expand(b1, q1), kSel, p, n);
    const int key = (row_sum(x2 - bc7_nearest<4>(p, n, x)) << 2) | row;
    const int best = min(min(lane_of(key, 0), lane_of(key, 16)), min(lane_of(key, 32), lane_of(key, 48)));
    if ((best >> 2) < sse) {
      sse = best >> 2;
      p0 = (best >> 1) & 1;
      p1 = best & 1;
      v0a = us2_of(q7(A[0], p0), q7(A[1], p0));
      v0b = us2_of(q7(A[2], p0), q7(A[3], p0));
      v1a = us2_of(q7(B[0], p1), q7(B[1], p1));
      v1b = us2_of(q7(B[2], p1), q7(B[3], p1));
    }
  };
  // (1)-(2): the bounding box's principal diagonal
  {
    int A[4], B[4], D[4], var[4], lo[4], hi[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int v = (int)((x >> (8 * c)) & 0xffu);
      lo[c] = lane_of((int)row_min((uint32_t)v), 0);
      hi[c] = lane_of((int)row_max((uint32_t)v), 0);
      D[c] = 16 * v - row_sum(v);
      var[c] = lane_of(row_sum(D[c] * D[c]), 0);
    }
    int vr = var[0], Dr = D[0];
#pragma unroll
    for (int c = 1; c < 4; ++c)
      if (var[c] > vr) {
        vr = var[c];
        Dr = D[c];
      }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int cov = lane_of(row_sum(D[c] * Dr), 0);
      A[c] = cov >= 0 ? lo[c] : hi[c];
      B[c] = cov >= 0 ? hi[c] : lo[c];
    }
    quantised(A, B);
  }
  // (3): least-squares endpoints of the current indices, twice; row c solves channel c
#pragma unroll 1
  for (int it = 0; it < 2; ++it) {
    const int w = (64 * index() + 7) / 15, a = 64 - w;
    const int v = (int)((x >> (8 * row)) & 0xffu);
    const double Aa = row_sum(a * a), Bab = row_sum(a * w), Cb = row_sum(w * w);
    const double r0 = 64.0 * row_sum(a * v), r1 = 64.0 * row_sum(w * v);
    const double det = Aa * Cb - Bab * Bab;
    int E0 = 0, E1 = 0;
    const bool solve = det > 0.0;   // uniform: every row holds the same indices
    if (solve) {
      E0 = bc7_ls_endpoint(Cb * r0 - Bab * r1, det);
      E1 = bc7_ls_endpoint(Aa * r1 - Bab * r0, det);
    }
    int A[4], B[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const us2 v0 = c < 2 ? v0a : v0b, v1 = c < 2 ? v1a : v1b;
      A[c] = solve ? lane_of(E0, 16 * c) : 2 * (int)v0[c & 1] + p0;
      B[c] = solve ? lane_of(E1, 16 * c) : 2 * (int)v1[c & 1] + p1;
    }
    quantised(A, B);
  }
  // (4): local search, coarse to fine.  Lane (half, mv): move mv over texels 8 half .. + 7.
  {
    const int mv = lane & 31, half = lane >> 5;
    const uint32_t sgn = (mv & 1) ? 1u : 0xffffu;      // +1, -1
    const bool all = mv >= 16;
    const int k = all ? (mv - 16) >> 1 : mv >> 3, c = (mv >> 1) & 3;
    const bool val = mv < 20;
    auto unit = [&](int e, int ch) { return (uint16_t)(val && k == e && (all || c == ch) ? sgn : 0u); };
    const us2 u0a = {unit(0, 0), unit(0, 1)}, u0b = {unit(0, 2), unit(0, 3)};
    const us2 u1a = {unit(1, 0), unit(1, 1)}, u1b = {unit(1, 2), unit(1, 3)};
    const int f0 = mv == 20 ? 1 : 0, f1 = mv == 21 ? 1 : 0;
    uint32_t Y[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const uint32_t lo8 = X[s], hi8 = X[8 + s];   // values first: a choice of addresses would keep X in memory
      Y[s] = half ? hi8 : lo8;
    }
#pragma unroll 1
    for (int st = 8; st >= 1; st >>= 1) {
      const us2 sv = (us2)((uint16_t)st);
#pragma unroll 1
      for (int round = 0; round < 64; ++round) {
        const us2 t0a = v0a + u0a * sv, t0b = v0b + u0b * sv, t1a = v1a + u1a * sv, t1b = v1b + u1b * sv;
        const uint32_t over = (us2_bits(t0a) | us2_bits(t0b) | us2_bits(t1a) | us2_bits(t1b)) & 0xff80ff80u;
        const int q0 = p0 ^ f0, q1 = p1 ^ f1;
        uint32_t p[16];
        int n[16];
        bc7_palette<4>(expand(t0a, q0), expand(t0b, q0), expand(t1a, q1), expand(t1b, q1), kSel, p, n);
        int near = 0;
#pragma unroll
        for (int s = 0; s < 8; ++s) near += bc7_nearest<4>(p, n, Y[s]);
        const auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)near, (uint32_t)near, false, false);
        near = (int)sw[0] + (int)sw[1];   // both halves of the move
        uint32_t key = ((uint32_t)(sum_x2 - near) << 5) | (uint32_t)mv;
        key = row_min(over != 0u || mv >= 22 ? 0xffffffffu : key);
        const uint32_t best = min((uint32_t)lane_of((int)key, 0), (uint32_t)lane_of((int)key, 16));
        if (best == 0xffffffffu || (int)(best >> 5) >= sse) break;
        sse = (int)(best >> 5);
        const int b = (int)(best & 31u);
        v0a = __builtin_bit_cast(us2, (uint32_t)lane_of((int)us2_bits(t0a), b));
        v0b = __builtin_bit_cast(us2, (uint32_t)lane_of((int)us2_bits(t0b), b));
        v1a = __builtin_bit_cast(us2, (uint32_t)lane_of((int)us2_bits(t1a), b));
        v1b = __builtin_bit_cast(us2, (uint32_t)lane_of((int)us2_bits(t1b), b));
        p0 ^= b == 20 ? 1 : 0;
        p1 ^= b == 21 ? 1 : 0;
      }
    }
  }
  // (5): anchor and bits
  const int J0 = index();
  const bool swap = lane_of(J0, 0) >= 8;
  const int J = swap ? 15 - J0 : J0;
  const int s = lane & 15;
  uint64_t hi = s ? (uint64_t)J << (4 * s) : (uint64_t)J << 1;
  hi = (uint64_t)row_or((uint32_t)hi) | ((uint64_t)row_or((uint32_t)(hi >> 32)) << 32);
  if (lane == 0) {
    const us2 aa = swap ? v1a : v0a, ab = swap ? v1b : v0b, za = swap ? v0a : v1a, zb = swap ? v0b : v1b;
    uint64_t lo = 0x40;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lo |= (uint64_t)(c < 2 ? aa[c & 1] : ab[c & 1]) << (7 + 14 * c);
      lo |= (uint64_t)(c < 2 ? za[c & 1] : zb[c & 1]) << (14 + 14 * c);
    }
    lo |= (uint64_t)(swap ? p1 : p0) << 63;
    hi |= (uint64_t)(swap ? p0 : p1);
    bc7_found(F, 0, sse, lo, hi);
  }
}

// ---- colour of mode 5 (N = 7) or 4 (N = 5) under the four rotations: row r is rotation r.
// Colour slot c is the texel's byte c, or byte 3 when c == r - 1; the byte left over (alpha's)
// is zero in the palette.  E0POS, STEP: bit positions of the endpoint values; IPOS: indices.
template <int N, int IB, int STEP, int IPOS>
__device__ __forceinline__ void col_search(uint32_t x, const uint32_t X[16], int lane, Bc7Found& F, int first) {
  constexpr int top = (1 << N) - 1;
  const int rot = lane >> 4, lead = lane & 48;
  // bytes taken from the palette's 16-bit slots (high bytes 1, 3, 5), 0x0c = zero
  const uint32_t sel = rot == 0 ? 0x0c050301u : (rot == 1 ? 0x0105030cu : (rot == 2 ? 0x03050c01u : 0x050c0301u));
  const uint32_t cmask = rot == 0 ? 0x00ffffffu : ~(0xffu << (8 * (rot - 1)));
  int Y[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) Y[c] = (int)((x >> (c == rot - 1 ? 24 : 8 * c)) & 0xffu);
  const int x2 = (int)__builtin_amdgcn_udot4(x & cmask, x & cmask, 0u, false);
  const int sum_x2 = row_sum(x2);
  us2 v0a = us2_of(0, 0), v0b = v0a, v1a = v0a, v1b = v0a;   // the row's current endpoints
  int sse = INT_MAX, J = 0;
  auto expand = [](us2 v) { return (v << (us2)((uint16_t)(8 - N))) | (v >> (us2)((uint16_t)(2 * N - 8))); };
  // candidate (a0, b0 | a1, b1) priced with a texel a lane, taken when strictly better
  auto take = [&](us2 a0, us2 b0, us2 a1, us2 b1) {
    uint32_t p[1 << IB];
    int n[1 << IB], j;
    bc7_palette<IB>(expand(a0), expand(b0), expand(a1), expand(b1), sel, p, n);
    const int e = row_sum(x2 - bc7_nearest_index<IB>(p, n, x, j));
    if (e < sse) {
      sse = e;
      J = j;
      v0a = a0;
      v0b = b0;
      v1a = a1;
      v1b = b1;
    }
  };
  // (1) bounding-box diagonal
  {
    int D[3], q0[3], q1[3], vr = -1, Dr = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      D[c] = 16 * Y[c] - row_sum(Y[c]);
      const int var = row_sum(D[c] * D[c]);
      if (var > vr) {
        vr = var;
        Dr = D[c];
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int lo = (int)row_min((uint32_t)Y[c]), hi = (int)row_max((uint32_t)Y[c]);
      const bool up = row_sum(D[c] * Dr) >= 0;
      q0[c] = bc7_quant(up ? lo : hi, N);
      q1[c] = bc7_quant(up ? hi : lo, N);
    }
    take(us2_of(q0[0], q0[1]), us2_of(q0[2], 0), us2_of(q1[0], q1[1]), us2_of(q1[2], 0));
  }
  // (2) least-squares endpoints of the current indices, twice
#pragma unroll 1
  for (int it = 0; it < 2; ++it) {
    const int w = (64 * J + ((1 << IB) - 1) / 2) / ((1 << IB) - 1), a = 64 - w;
    const double Aa = row_sum(a * a), Bab = row_sum(a * w), Cb = row_sum(w * w);
    const double det = Aa * Cb - Bab * Bab;
    int q0[3], q1[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double r0 = 64.0 * row_sum(a * Y[c]), r1 = 64.0 * row_sum(w * Y[c]);
      const int e0 = bc7_xpand(c < 2 ? v0a[c & 1] : v0b[0], N), e1 = bc7_xpand(c < 2 ? v1a[c & 1] : v1b[0], N);
      const double d = det > 0.0 ? det : 1.0;
      q0[c] = bc7_quant(det > 0.0 ? bc7_ls_endpoint(Cb * r0 - Bab * r1, d) : e0, N);
      q1[c] = bc7_quant(det > 0.0 ? bc7_ls_endpoint(Aa * r1 - Bab * r0, d) : e1, N);
    }
    take(us2_of(q0[0], q0[1]), us2_of(q0[2], 0), us2_of(q1[0], q1[1]), us2_of(q1[2], 0));
  }
  // (3) local search, coarse to fine; each row keeps its own step and round count
  {
    // packed unit steps of move mv: value slots (0, 1 | 2) of endpoint 0, then of endpoint 1
    auto unit = [](int mv, us2& u0a, us2& u0b, us2& u1a, us2& u1b) {
      const bool all = mv >= 12;
      const int k = all ? (mv - 12) >> 1 : (mv >= 6 ? 1 : 0);
      const int c = (mv >> 1) - (mv >= 6 ? 3 : 0);
      const uint16_t s = (mv & 1) ? 1u : 0xffffu;
      const us2 a = {(uint16_t)(all || c == 0 ? s : 0u), (uint16_t)(all || c == 1 ? s : 0u)};
      const us2 b = {(uint16_t)(all || c == 2 ? s : 0u), (uint16_t)0};
      const us2 z = {0, 0};
      u0a = k ? z : a;
      u0b = k ? z : b;
      u1a = k ? a : z;
      u1b = k ? b : z;
    };
    const int mv = lane & 15;
    us2 u0a, u0b, u1a, u1b;
    unit(mv, u0a, u0b, u1a, u1b);
    int st = 1 << (N - 4), round = 0;
    while (__any(st > 0)) {
      const us2 sv = (us2)((uint16_t)st);
      const us2 t0a = v0a + u0a * sv, t0b = v0b + u0b * sv, t1a = v1a + u1a * sv, t1b = v1b + u1b * sv;
      const uint32_t over = (us2_bits(t0a) | us2_bits(t0b) | us2_bits(t1a) | us2_bits(t1b)) & (0x00010001u * (0xffffu ^ top));
      uint32_t p[1 << IB];
      int n[1 << IB];
      bc7_palette<IB>(expand(t0a), expand(t0b), expand(t1a), expand(t1b), sel, p, n);
      int near = 0;
#pragma unroll
      for (int s = 0; s < 16; ++s) near += bc7_nearest<IB>(p, n, X[s]);
      const uint32_t key = row_min(over != 0u ? 0xffffffffu : ((uint32_t)(sum_x2 - near) << 4) | (uint32_t)mv);
      if (key == 0xffffffffu || (int)(key >> 4) >= sse) {   // the same in the whole row
        st >>= 1;
        round = 0;
      } else if (st > 0) {
        sse = (int)(key >> 4);
        us2 b0a, b0b, b1a, b1b;
        unit((int)(key & 15u), b0a, b0b, b1a, b1b);
        v0a += b0a * sv;
        v0b += b0b * sv;
        v1a += b1a * sv;
        v1b += b1b * sv;
        if (++round == 64) {
          st >>= 1;
          round = 0;
        }
      }
    }
  }
  // (4) indices, anchor and bits
  {
    uint32_t p[1 << IB];
    int n[1 << IB];
    bc7_palette<IB>(expand(v0a), expand(v0b), expand(v1a), expand(v1b), sel, p, n);
    bc7_nearest_index<IB>(p, n, x, J);
  }
  const bool swap = __shfl(J, lead, 64) >= (1 << (IB - 1));
  if (swap) J = (1 << IB) - 1 - J;
  uint64_t lo = 0, hi = 0;
  bc7_put_index(lo, hi, J, lane & 15, IPOS, IB);
  lo = (uint64_t)row_or((uint32_t)lo) | ((uint64_t)row_or((uint32_t)(lo >> 32)) << 32);
  hi = (uint64_t)row_or((uint32_t)hi) | ((uint64_t)row_or((uint32_t)(hi >> 32)) << 32);
  if (lane == lead) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint32_t a = c < 2 ? v0a[c & 1] : v0b[0], z = c < 2 ? v1a[c & 1] : v1b[0];
      bc7_put(lo, hi, swap ? z : a, 8 + STEP * 2 * c);
      bc7_put(lo, hi, swap ? a : z, 8 + STEP + STEP * 2 * c);
    }
    bc7_found(F, first + rot, sse, lo, hi);
  }
}

// ---- the alpha searches of one index width: with 3-bit indices the 4 rotations of mode 4
// (6-bit values), a row of 16 lanes each; with 2-bit indices the 4 rotations of mode 5 (8-bit
// values), then of mode 4 (6-bit), 8 lanes each.  Alpha is the texel's byte rot - 1 (rot = 0:
// byte 3).  In the local search lane l of a search prices move l / P over part l % P of the
// texels (P = 2 or 4 parts), so that both widths price 32 (texel, entry) pairs a lane: one wave
// for all 12 searches, a whole block's texels to a lane, took 81 us for a 128^2 tile's maps
// where each of the two takes less than the other roles' 41-58.
template <int IB>
__device__ __forceinline__ void alpha_search(uint32_t x, const uint32_t X[16], int lane, Bc7Found& F) {
  constexpr int NE = 1 << IB, GL = IB == 2 ? 8 : 16, P = GL / 4, T = 16 / P, OWN = 16 / GL;
  const int l = lane & (GL - 1), grp = lane / GL, part = l % P, mv = l / P, rot = grp & 3;
  const int fam = IB == 3 ? 1 : (grp >> 2) * 2;
  const int N = IB == 2 && fam == 0 ? 8 : 6, top = (1 << N) - 1;
  const uint32_t sh = rot == 0 ? 24u : 8u * (uint32_t)(rot - 1);
  auto gsum = [](int v) { return IB == 3 ? row_sum(v) : half_sum(v); };
  auto gmin = [](uint32_t v) { return IB == 3 ? row_min(v) : half_min(v); };
  auto gor = [](uint32_t v) { return IB == 3 ? row_or(v) : half_or(v); };
  // the lane's own texels outside the local search: l (and l + 8)
  int own[OWN];
  {
    const int a = (int)((x >> sh) & 0xffu), b = (int)((dpp_mov<kRor + 8>(x) >> sh) & 0xffu);
    if constexpr (IB == 3) {
      own[0] = a;
    } else {
      own[0] = (lane & 8) ? b : a;
      own[1] = (lane & 8) ? a : b;
    }
  }
  int part_x[T];   // its texels T part .. of the local search
#pragma unroll
  for (int i = 0; i < T; ++i) {
    uint32_t v = X[i];
#pragma unroll
    for (int q = 1; q < P; ++q) {
      const uint32_t o = X[T * q + i];
      v = part == q ? o : v;
    }
    part_x[i] = (int)((v >> sh) & 0xffu);
  }
  int v0 = 0, v1 = 0, sse = INT_MAX;
  auto palette = [&](int a, int z, int p[NE]) {
    const int E0 = bc7_xpand(a, N), d = bc7_xpand(z, N) - E0;
#pragma unroll
    for (int j = 0; j < NE; ++j) p[j] = E0 + ((bc7_weight<IB>(j) * d + 32) >> 6);
  };
  auto nearest = [](const int p[NE], int v) {   // least |p - v|
    int m = INT_MAX;
#pragma unroll
    for (int j = 0; j < NE; ++j) m = min(m, (int)__builtin_amdgcn_sad_u16((uint32_t)p[j], (uint32_t)v, 0u));
    return m;
  };
  auto nearest_index = [](const int p[NE], int v) {
    int m = INT_MAX, J = 0;
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const int e = abs(p[j] - v);
      J = e < m ? j : J;
      m = min(m, e);
    }
    return J;
  };
  auto take = [&](int a, int z) {
    int p[NE], e = 0;
    palette(a, z, p);
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
      const int m = nearest(p, own[i]);
      e += m * m;
    }
    e = gsum(e);
    if (e < sse) {
      sse = e;
      v0 = a;
      v1 = z;
    }
  };
  // (1) minimum and maximum
  {
    const int lo = OWN == 1 ? own[0] : min(own[0], own[OWN - 1]), hi = OWN == 1 ? own[0] : max(own[0], own[OWN - 1]);
    take(bc7_quant((int)gmin((uint32_t)lo), N), bc7_quant((int)~gmin(~(uint32_t)hi), N));
  }
  // (2) least-squares endpoints of the current indices, twice
#pragma unroll 1
  for (int it = 0; it < 2; ++it) {
    int p[NE], aa = 0, ab = 0, cb = 0, ra = 0, rw = 0;
    palette(v0, v1, p);
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
      const int j = nearest_index(p, own[i]);
      const int w = (64 * j + (NE - 1) / 2) / (NE - 1), a = 64 - w;
      aa += a * a;
      ab += a * w;
      cb += w * w;
      ra += a * own[i];
      rw += w * own[i];
    }
    const double Aa = gsum(aa), Bab = gsum(ab), Cb = gsum(cb);
    const double r0 = 64.0 * gsum(ra), r1 = 64.0 * gsum(rw);
    const double det = Aa * Cb - Bab * Bab, d = det > 0.0 ? det : 1.0;
    const int E0 = det > 0.0 ? bc7_ls_endpoint(Cb * r0 - Bab * r1, d) : bc7_xpand(v0, N);
    const int E1 = det > 0.0 ? bc7_ls_endpoint(Aa * r1 - Bab * r0, d) : bc7_xpand(v1, N);
    take(bc7_quant(E0, N), bc7_quant(E1, N));
  }
  // (3) local search: move mv = (endpoint mv >> 1, sign mv & 1)
  {
    int st = 1 << (N - 4), round = 0;
    const int u0 = mv < 2 ? ((mv & 1) ? 1 : -1) : 0, u1 = mv < 2 ? 0 : ((mv & 1) ? 1 : -1);
    while (__any(st > 0)) {
      const int t0 = v0 + u0 * st, t1 = v1 + u1 * st;
      const bool over = t0 < 0 || t0 > top || t1 < 0 || t1 > top;
      int p[NE], e = 0;
      palette(min(max(t0, 0), top), min(max(t1, 0), top), p);
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int m = nearest(p, part_x[i]);
        e += m * m;
      }
      e += (int)dpp_mov<kQuadX1>((uint32_t)e);                        // the move's parts
      if constexpr (P == 4) e += (int)dpp_mov<kQuadX2>((uint32_t)e);
      const uint32_t key = gmin(over ? 0xffffffffu : ((uint32_t)e << 2) | (uint32_t)mv);
      if (key == 0xffffffffu || (int)(key >> 2) >= sse) {
        st >>= 1;
        round = 0;
      } else if (st > 0) {
        sse = (int)(key >> 2);
        const int b = (int)(key & 3u), dv = (b & 1) ? st : -st;
        if (b < 2) v0 += dv;
        else v1 += dv;
        if (++round == 64) {
          st >>= 1;
          round = 0;
        }
      }
    }
  }
  // (4) indices, anchor and bits
  int p[NE], J[OWN];
  palette(v0, v1, p);
#pragma unroll
  for (int i = 0; i < OWN; ++i) J[i] = nearest_index(p, own[i]);
  const bool swap = __shfl(J[0], lane & ~(GL - 1), 64) >= NE / 2;
  const int ipos = fam == 0 ? 97 : (fam == 1 ? 81 : 50);
  uint64_t lo = 0, hi = 0;
#pragma unroll
  for (int i = 0; i < OWN; ++i) bc7_put_index(lo, hi, swap ? NE - 1 - J[i] : J[i], l + 8 * i, ipos, IB);
  lo = (uint64_t)gor((uint32_t)lo) | ((uint64_t)gor((uint32_t)(lo >> 32)) << 32);
  hi = (uint64_t)gor((uint32_t)hi) | ((uint64_t)gor((uint32_t)(hi >> 32)) << 32);
  if (l == 0) {
    bc7_put(lo, hi, (uint32_t)(swap ? v1 : v0), fam == 0 ? 50 : 38);
    bc7_put(lo, hi, (uint32_t)(swap ? v0 : v1), fam == 0 ? 58 : 44);
    bc7_found(F, 13 + 4 * fam + rot, sse, lo, hi);
  }
}

// Blocks of up to two maps (ja, then jb) in one launch.  80 registers: six waves a SIMD hold four
// workgroups a CU (3% faster than 96 registers and three, in spite of four spilled values).
constexpr int kBc7Threads = 384;
__global__ __launch_bounds__(kBc7Threads, 6) void k_encode_bc7(EncodeJob ja, EncodeJob jb) {
  __shared__ Bc7Found F;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  for (int64_t i = blockIdx.x; i < ja.n + jb.n; i += gridDim.x) {
    const EncodeJob& job = i < ja.n ? ja : jb;
    const int64_t f = i < ja.n ? i : i - ja.n;
    uint8_t* const out = job.out;
    int q[4];
    src_texel4(job.src, f, lane & 15, q);
    const uint32_t x = (uint32_t)q[0] | (uint32_t)q[1] << 8 | (uint32_t)q[2] << 16 | (uint32_t)q[3] << 24;
    uint32_t X[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) X[s] = (uint32_t)lane_of((int)x, s);
    // an opaque copy of the lane per block: what a role derives from it would otherwise be
    // hoisted out of this loop and held through every role (161 registers against 105 for the
    // largest role alone)
    int ln = lane;
    asm volatile("" : "+v"(ln));
    if (wave == 0) m6_search(x, X, ln, F);
    else if (wave == 1) col_search<7, 2, 7, 66>(x, X, ln, F, 1);
    else if (wave == 2) col_search<5, 2, 5, 50>(x, X, ln, F, 5);
    else if (wave == 3) col_search<5, 3, 5, 81>(x, X, ln, F, 9);
    else if (wave == 4) alpha_search<2>(x, X, ln, F);
    else alpha_search<3>(x, X, ln, F);
    __syncthreads();
    if (wave == 0) {
      // candidates in order: mode 6, mode 5 by rotation, mode 4 by rotation then selection; a
      // later one replaces an earlier one only when strictly better
      const int o = min(lane & 15, 12);
      const int rot = o < 5 ? o - 1 : (o - 5) >> 1, sel = (o - 5) & 1;
      const int kc = o == 0 ? 0 : (o < 5 ? 1 + rot : 5 + 4 * sel + rot);
      const int ka = o == 0 ? 0 : (o < 5 ? 13 + rot : 17 + 4 * sel + rot);
      const uint32_t sse = (uint32_t)F.sse[kc] + (o == 0 ? 0u : (uint32_t)F.sse[ka]);
      const int win = (int)(row_min((sse << 4) | (uint32_t)o) & 15u);
      if (lane == win) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = F.w[kc][i] | F.w[ka][i];
        if (o > 0) w[0] |= o < 5 ? (uint32_t)((1 << 5) | (rot << 6)) : (uint32_t)((1 << 4) | (rot << 5) | (sel << 7));
        *(u4v*)(out + f * 16) = (u4v){w[0], w[1], w[2], w[3]};
      }
    }
    __syncthreads();   // F may be written again
  }
}

int launch_encode(const EncodeJob& ja, const EncodeJob& jb, int codec, int n_cu, hipStream_t s) {
  const int64_t n = ja.n + jb.n;
  if (n <= 0) return NDGI_OK;
  if (codec == NDGI_CODEC_BC7) {
    const int64_t cap = (int64_t)n_cu * 64;
    hipLaunchKernelGGL(k_encode_bc7, dim3((unsigned)(n < cap ? n : cap)), dim3(kBc7Threads), 0, s, ja, jb);
  } else if (n <= (int64_t)n_cu * kBc4OnePerCu) {
    hipLaunchKernelGGL(k_encode_bc4_one, dim3((unsigned)n), dim3(64 * kBc4OneWaves), 0, s, ja, jb);
  } else {
    const int64_t wgs = (n + 3) / 4, cap = (int64_t)n_cu * 64;
    hipLaunchKernelGGL(k_encode_bc4, dim3((unsigned)(wgs < cap ? wgs : cap)), dim3(256), 0, s, ja, jb);
  }
  NDGI_HIP(hipGetLastError());
  return NDGI_OK;
}

}  // namespace ndgi

using namespace ndgi;

extern "C" {

int ndgi_bc4_encode_blocks(const uint8_t* texels, int64_t n, uint8_t* out, hipStream_t s) {
  clear_error();
  if (n < 0) return fail(NDGI_ERR_INVALID_ARG, "bc4_encode_blocks: n < 0");
  if (n > 0 && (!texels || !out)) return fail(NDGI_ERR_INVALID_ARG, "bc4_encode_blocks: NULL pointer");
  if (((uintptr_t)out & 7u) != 0) return fail(NDGI_ERR_INVALID_ARG, "bc4_encode_blocks: out not 8-byte aligned");
  int dev = 0, n_cu = 0;
  NDGI_HIP(hipGetDevice(&dev));
  NDGI_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  EncodeJob job = {};
  job.src.u8 = texels;
  job.src.C = 1;
  job.n = n;
  job.out = out;
  return launch_encode(job, EncodeJob{}, NDGI_CODEC_BC4, n_cu, s);
}

int ndgi_bc7_encode_blocks(const uint8_t* texels, int64_t n, uint8_t* out, hipStream_t s) {
  clear_error();
  if (n < 0) return fail(NDGI_ERR_INVALID_ARG, "bc7_encode_blocks: n < 0");
  if (n > 0 && (!texels || !out)) return fail(NDGI_ERR_INVALID_ARG, "bc7_encode_blocks: NULL pointer");
  if (((uintptr_t)out & 15u) != 0) return fail(NDGI_ERR_INVALID_ARG, "bc7_encode_blocks: out not 16-byte aligned");
  int dev = 0, n_cu = 0;
  NDGI_HIP(hipGetDevice(&dev));
  NDGI_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  EncodeJob job = {};
  job.src.u8 = texels;
  job.src.C = 4;
  job.n = n;
  job.out = out;
  return launch_encode(job, EncodeJob{}, NDGI_CODEC_BC7, n_cu, s);
}

}  // extern "C"
