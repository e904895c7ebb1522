// Decode kernels: BC4 block decoder, random-access query decode, persistent page decode.
#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

namespace ndgi {

// ------------------------------------------------------------------------ BC4 blocks
// IMPL selects the texel decoder: 0 the integer bc4_texel, 1 the float bc4_texel_f of the query
// kernels (both layouts), 2 the row decode bc4_rows of the binned and hybrid page kernels (the page
// kernel's bc4_rows4 shares its palette and its pick and takes all four rows).
template <int IMPL>
__global__ __launch_bounds__(256) void k_bc4_blocks(const uint8_t* __restrict__ blocks, int64_t n,
                                                     uint8_t* __restrict__ out) {
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n; b += (int64_t)gridDim.x * blockDim.x) {
    const uint2 w = ((const uint2*)blocks)[b];
    uint32_t o[4];
    if constexpr (IMPL == 2) {
      bc4_rows(w.x, w.y, 0, o[0], o[1]);
      bc4_rows(w.x, w.y, 1, o[2], o[3]);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint32_t v = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t t = IMPL == 1 ? (uint32_t)bc4_texel_f(w.x, w.y, 4 * r + c) : bc4_texel(w.x, w.y, 4 * r + c);
          v |= t << (8 * c);
        }
        o[r] = v;
      }
    }
    ((uint4*)out)[b] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

int launch_bc4_blocks(const uint8_t* blocks, int64_t n, uint8_t* out, int impl, hipStream_t s) {
  const int64_t want = (n + 255) / 256;
  const int grid = (int)(want < 65536 ? want : 65536);
  if (impl == 1) hipLaunchKernelGGL(k_bc4_blocks<1>, dim3(grid), dim3(256), 0, s, blocks, n, out);
  else if (impl == 2) hipLaunchKernelGGL(k_bc4_blocks<2>, dim3(grid), dim3(256), 0, s, blocks, n, out);
  else hipLaunchKernelGGL(k_bc4_blocks<0>, dim3(grid), dim3(256), 0, s, blocks, n, out);
  NDGI_HIP(hipGetLastError());
  return NDGI_OK;
}

// ------------------------------------------------------------------- query decode
// Each wave takes passes of 64 consecutive queries (phase A: one query per lane; phase B:
// the decoder after the register handoff); 4 waves per workgroup; grid-stride.
// FP32 on an FP16 grid is held to three waves a SIMD: for a fourth the compiler gave up the registers
// in which the grid's eight loads are in flight together, and small calls took 8.3 us instead of 7.4.
template <int PREC, int GDT>
constexpr int query_waves() { return PREC == NDGI_PREC_F32 && GDT == NDGI_DTYPE_F16 ? 3 : 8; }
template <int PREC, int GDT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, query_waves<PREC, GDT>())))
void k_decode_query(ndgi_model m, const float* __restrict__ uvt, int64_t n, void* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  Dec<PREC> dec;
  dec.load(m.mlp, m.mlp_dtype, lane);
  const int64_t passes = (n + 63) >> 6;
  const int64_t wave0 = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  for (int64_t p = wave0; p < passes; p += nwaves) {
    const int64_t mine = (p << 6) + lane;
    float u = 0.5f, v = 0.5f, t = 0.0f;
    if (mine < n) {
      u = uvt[mine * 3 + 0];
      v = uvt[mine * 3 + 1];
      t = uvt[mine * 3 + 2];
    }
    float sp[8], gr[8];
    spatial8_global(m, coord_axis(u, m.W), coord_axis(v, m.H), sp);
    query_grid8<GDT>(m, u, v, t, gr);
    const f4v acc = decode_regs<PREC>(dec, sp, gr);
    if (mine < n) store_rgb<PREC>(out, (size_t)mine, acc, !(isfinite(u) && isfinite(v) && isfinite(t)));
  }
}

int launch_decode(ndgi_ctx* ctx, const ndgi_model& m, const float* uvt, int64_t n, void* out, int prec,
                  hipStream_t s) {
  if (n == 0) return NDGI_OK;
  const int64_t passes = (n + 63) / 64;
  int64_t wgs = (passes + 3) / 4;
  const bool g16 = m.grid_dtype == NDGI_DTYPE_F16;
  const void* kern = (prec == NDGI_PREC_F16)
                         ? (g16 ? (const void*)k_decode_query<NDGI_PREC_F16, NDGI_DTYPE_F16>
                                : (const void*)k_decode_query<NDGI_PREC_F16, NDGI_DTYPE_F32>)
                         : (g16 ? (const void*)k_decode_query<NDGI_PREC_F32, NDGI_DTYPE_F16>
                                : (const void*)k_decode_query<NDGI_PREC_F32, NDGI_DTYPE_F32>);
  // Waves read from all over the maps, and more of them in flight than hide the latency only evict
  // each other's lines: workgroups a CU where all that is resident would be slower (us, all resident
  // and this):
  //  * FP16, FP16 grid: 2 (1M queries of 256^2 x 24 60.7 and 54.2, of 1024^2 115 and 103, 16M of
  //    4096^2 2250 and 1990); of a model that lies in the CUs' own caches, on either grid and after some
  //    rounds, all (3M of 64^2 x 8: 108, with two 119).
  //  * FP16, FP32 grid: 3 (1M of 512^2 98.5 and 92.5), or 2 where the model exceeds the chip's 32 MB
  //    of L2 and there are rounds to spread over (1M of 1024^2 128 and 111).
  //  * FP32, FP16 grid: 2 (1M of 4096^2 145 and 133), or 3 for a model within an XCD's L2 and many
  //    rounds, which is bound by the decoder (3M of 256^2: 176, with two 182).
  //  * FP32, FP32 grid: 3 (1M of 512^2 102 and 98), or all for such models and counts (3M of 256^2: 193,
  //    with three 200).
  // Three a CU that take as many rounds as two are two (200003 queries of 1024^2, FP32 grid, FP16: 33.6
  // and 29.3).  In FP16 up to a quarter of a workgroup a CU beyond a round goes with it: as a round of its
  // own it would leave the chip idle (131073 queries on an FP32 grid of 512^2: 16.9, cut into two 20.4).
  // Where the last round would put as many workgroups on some CUs as a full one, the rounds are made
  // equal: no CU takes more for it, and fewer waves are in flight (200003 queries of 2048^2 x 24, FP16,
  // 32.1 and 29.5; 1M 117 and 114).  Where it would put fewer, equal rounds cost a pass on every CU
  // (262145 of 512^2 26.0 and 32.6).
  const int64_t cu = ctx->n_cu, bytes = (int64_t)m.W * m.H * 4 + (int64_t)m.T * m.Gh * m.Gw * (g16 ? 16 : 32);
  const auto rounds_of = [&](int64_t c) { return (wgs + c * cu - 1) / (c * cu); };
  int64_t per_cu, slack = 0;
  if (prec == NDGI_PREC_F16) {
    per_cu = g16 || (bytes > (32 << 20) && wgs > 5 * cu) ? 2 : 3;
    if (bytes <= (128 << 10) && wgs > 9 * cu) per_cu = 4;
    slack = cu / 4;
  } else if (g16) {
    per_cu = bytes <= (2 << 20) && wgs > 12 * cu ? 3 : 2;
  } else {
    per_cu = bytes <= (4 << 20) && wgs > 12 * cu ? 4 : 3;
  }
  if (per_cu == 3 && wgs > 3 * cu + cu / 64 && rounds_of(2) == rounds_of(3)) per_cu = 2;
  const int64_t resident = resident_wgs(ctx, kern);
  const int64_t cap = wgs > per_cu * cu + slack ? std::min(resident, per_cu * cu) : resident;
  if (wgs > cap) {
    const int64_t rounds = (wgs + cap - 1) / cap, last = wgs - (rounds - 1) * cap;
    wgs = last > cap - cu + cu / 64 ? (wgs + rounds - 1) / rounds : cap;
  }
  if (prec == NDGI_PREC_F16 && g16)
    hipLaunchKernelGGL((k_decode_query<NDGI_PREC_F16, NDGI_DTYPE_F16>), dim3((unsigned)wgs), dim3(256), 0, s, m, uvt, n, out);
  else if (prec == NDGI_PREC_F16)
    hipLaunchKernelGGL((k_decode_query<NDGI_PREC_F16, NDGI_DTYPE_F32>), dim3((unsigned)wgs), dim3(256), 0, s, m, uvt, n, out);
  else if (g16)
    hipLaunchKernelGGL((k_decode_query<NDGI_PREC_F32, NDGI_DTYPE_F16>), dim3((unsigned)wgs), dim3(256), 0, s, m, uvt, n, out);
  else
    hipLaunchKernelGGL((k_decode_query<NDGI_PREC_F32, NDGI_DTYPE_F32>), dim3((unsigned)wgs), dim3(256), 0, s, m, uvt, n, out);
  NDGI_HIP(hipGetLastError());
  return NDGI_OK;
}

// -------------------------------------------------------------- persistent page decode
// Work item = (request, sub-tile of 16*tw x 4*th texels).  Every wave of the persistent
// grid takes items round-robin (items cost the same, so a static schedule balances
// without a shared counter).  A sub-tile is walked in slabs of 16 columns, top to bottom, in
// passes of 4 rows: group q of a pass is its row q, lane (g, j) holds channels 2g, 2g+1 of
// column j.
//  * Blocks: two passes are eight BC4 footprints; lane (footprint, channel) decodes one whole
//    block into wave-private LDS (the palette is built once for four rows), from which the
//    groups read their bytes.
//  * Grid: a lane needs, of each grid row, the two nodes around its column at both keys.  The
//    four values are loaded into registers and folded by one set of weights (key x column)
//    into a row sample, one row ahead of use; a texel row is then one lerp between the two
//    row samples around it.  No grid value goes through LDS, and a row sample serves every
//    texel row that it bounds.
// The precision's decoder takes it from there.  FP16: 271 vector instructions a pass, 32 of them
// MFMA (294 by a kernel that staged each pass's time-blended grid window in LDS, beside a second
// kernel, launched after it in any case, for maps off its quarter-resolution FP16 grid).  The VALU is
// busy 73% of the time and the matrix cores 27%; a wave waits 42% of its time to issue and 19% for
// memory.  4096^2 FP16 frame 207 -> 190 us, 2000 pages of 32 maps 437 -> 390 us.  FP32 is bound by
// matrix time (busy 62%): 1600 x 1152 with a grid at an eighth of the texels 125 -> 73 us (there each
// texel took its two texel_axis divisions, two integer block decodes and eight node loads alone).
// Measured and not kept: the passes dealt out in equal contiguous runs, or in rounds of equal
// parts of a run, instead of sub-tiles round-robin (197-209 us for the frame: more slab starts,
// and neighbouring columns' lines written by different waves).

struct PageLds {
  uint32_t sp[2][8 * 20];   // decoded bytes of two passes: [channel][row][16 columns]; a channel
                            // stride of 80 B keeps the four lane groups of a read on distinct banks
};

// The model's buffers are device memory: global address-space pointers let each load take a
// uniform 64-bit base and a 32-bit lane offset (no 64-bit address arithmetic per lane).
typedef const __attribute__((address_space(1))) uint8_t* gbyte_ptr;
template <typename T>
__device__ __forceinline__ T gload(gbyte_ptr base, uint32_t byte_off) {
  return *(const __attribute__((address_space(1))) T*)(base + byte_off);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A grid row as a lane needs it: channels 2g, 2g+1 of the nodes left and right of its column,
// at the keys k0 and k1.
template <int GDT> struct GridRaw;
template <> struct GridRaw<NDGI_DTYPE_F16> { uint32_t v[4]; };
template <> struct GridRaw<NDGI_DTYPE_F32> { float2 v[4]; };
template <int GDT> struct GridCols {
  static constexpr uint32_t kNode = GDT == NDGI_DTYPE_F16 ? 16u : 32u;   // bytes of a node
  gbyte_ptr k0, k1;     // the keys' planes
  uint32_t row;         // bytes of a grid row
  uint32_t o0, o1;      // the lane's two nodes within a row
  float w[4];           // (key, column) weights
};

template <int GDT>
__device__ __forceinline__ GridRaw<GDT> grid_row_load(const GridCols<GDT>& c, int r) {
  GridRaw<GDT> o;
  const size_t at = (size_t)(uint32_t)r * c.row;
  o.v[0] = gload<uint32_t>(c.k0 + at, c.o0);
  o.v[1] = gload<uint32_t>(c.k0 + at, c.o1);
  o.v[2] = gload<uint32_t>(c.k1 + at, c.o0);
  o.v[3] = gload<uint32_t>(c.k1 + at, c.o1);
  return o;
}
template <>
__device__ __forceinline__ GridRaw<NDGI_DTYPE_F32> grid_row_load(const GridCols<NDGI_DTYPE_F32>& c, int r) {
  GridRaw<NDGI_DTYPE_F32> o;
  const size_t at = (size_t)(uint32_t)r * c.row;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned long long b = gload<unsigned long long>((i & 2 ? c.k1 : c.k0) + at, i & 1 ? c.o1 : c.o0);
    o.v[i] = make_float2(__uint_as_float((uint32_t)b), __uint_as_float((uint32_t)(b >> 32)));
  }
  return o;
}

__device__ __forceinline__ float2 half2_bits(uint32_t w) {
  return make_float2((float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu)),
                     (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16)));
}
__device__ __forceinline__ float2 half2_bits(float2 v) { return v; }

template <int GDT>
__device__ __forceinline__ float2 grid_row_sample(const GridCols<GDT>& c, const GridRaw<GDT>& r) {
  float2 o = make_float2(0.0f, 0.0f);
#pragma unroll
  for (int i = 0; i < 4; ++i) {   // the first term as an FMA with a zero addend: the same rounded product
    const float2 v = half2_bits(r.v[i]);
    o.x = fmaf(c.w[i], v.x, o.x);
    o.y = fmaf(c.w[i], v.y, o.y);
  }
  return o;
}

// One sub-tile.  R4: the grid is a quarter of the texel resolution, where a pass's rows lie at
// fixed places between three grid rows; otherwise each texel row's grid rows and weight come
// from texel_axis, 64 rows at a time (one a lane), and the two row samples move on as they do.
template <int PREC, int GDT, bool R4>
__device__ __forceinline__ void page_subtile(const Dec<PREC>& dec, const ndgi_model& m, const ndgi_page_req& rq,
                                             const Keys& k, int page, int ox, int oy, int tw, int th, void* dst,
                                             int64_t pitch, int lane, PageLds& L) {
  typedef typename std::conditional<PREC == NDGI_PREC_F16, _Float16, float>::type OutT;
  const int g = lane >> 4, j = lane & 15;
  const uint8_t* const sp8 = (const uint8_t*)L.sp;
  const int by = page * rq.page_y + oy;
  const uint32_t wb = (uint32_t)m.W >> 2;
  const int bf = lane >> 3, bc = lane & 7;   // this lane's footprint (pass bf >> 2, column bf & 3) and channel
  GridCols<GDT> gc;
  gc.row = (uint32_t)m.Gw * GridCols<GDT>::kNode;
  const size_t plane = (size_t)m.Gh * gc.row;
  gc.k0 = (gbyte_ptr)m.grid + (size_t)k.k0 * plane;
  gc.k1 = (gbyte_ptr)m.grid + (size_t)k.k1 * plane;
#pragma unroll 1
  for (int a = 0; a < tw; ++a) {
    const int bx = page * rq.page_x + ox + 16 * a;
    // this lane's column in the grid
    {
      const Axis cx = texel_axis<R4>(bx + j, m.Gw, m.W);
      gc.o0 = (uint32_t)cx.i0 * GridCols<GDT>::kNode + (uint32_t)g * (GridCols<GDT>::kNode / 4);
      gc.o1 = (uint32_t)cx.i1 * GridCols<GDT>::kNode + (uint32_t)g * (GridCols<GDT>::kNode / 4);
      gc.w[0] = k.w0 * cx.w0;
      gc.w[1] = k.w0 * cx.w1;
      gc.w[2] = k.w1 * cx.w0;
      gc.w[3] = k.w1 * cx.w1;
    }
    // blocks of the pass pair at rows 8 pr (the last pass again past an odd end)
    const gbyte_ptr blocks = (gbyte_ptr)m.bc4 + ((size_t)((uint32_t)by >> 2) * wb + ((uint32_t)bx >> 2)) * 64u;
    auto load_blocks = [&](int b) {
      const uint32_t row = (uint32_t)min(b + (bf >> 2), th - 1);
      return gload<unsigned long long>(blocks, (row * wb + (uint32_t)(bf & 3)) * 64u + 8u * (uint32_t)bc);
    };
    unsigned long long blk = load_blocks(0);
    // grid rows: lo and hi bound the current texel rows, nx is the row after, in flight
    int r_lo, r_hi, rows_packed = 0;
    float rows_w1 = 0.0f;
    auto row_axes = [&](int r0) {   // texel rows r0 .. r0 + 63 of the slab, one a lane
      const Axis ry = texel_axis<false>(min(by + r0 + lane, m.H - 1), m.Gh, m.H);
      rows_packed = ry.i0 | (ry.i1 << 16);
      rows_w1 = ry.w1;
    };
    if constexpr (R4) {
      r_lo = max((by >> 2) - 1, 0);
      r_hi = by >> 2;
    } else {
      row_axes(0);
      const int p = __builtin_amdgcn_readlane(rows_packed, 0);
      r_lo = p & 0xffff;
      r_hi = p >> 16;
    }
    float2 lo, hi;
    GridRaw<GDT> nx;
    {
      const GridRaw<GDT> l0 = grid_row_load<GDT>(gc, r_lo), h0 = grid_row_load<GDT>(gc, r_hi);
      nx = grid_row_load<GDT>(gc, min(r_hi + 1, m.Gh - 1));
      lo = grid_row_sample<GDT>(gc, l0);
      hi = grid_row_sample<GDT>(gc, h0);
    }
    OutT* out = (OutT*)dst + (rq.dst_offset + (int64_t)(oy + g) * pitch + (ox + 16 * a + j)) * 3;
#pragma unroll 1
    for (int b = 0; b < th; ++b) {
      if (!(b & 1)) {
        uint32_t r[4];
        bc4_rows4((uint32_t)blk, (uint32_t)(blk >> 32), r);
        uint32_t* const w = &L.sp[bf >> 2][bc * 20 + (bf & 3)];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[4 * i] = r[i];
        if (b + 2 < th) blk = load_blocks(b + 2);
        wave_sync();
      }
      const uint8_t* const at = sp8 + (b & 1) * 640 + (2 * g) * 80 + j;
      typename Dec<PREC>::Acc acc = dec.start();
      if constexpr (R4) {
        const float2 nw = grid_row_sample<GDT>(gc, nx);
        nx = grid_row_load<GDT>(gc, min((by >> 2) + b + 2, m.Gh - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float w1 = (float)((2 * q - 3) & 7) * 0.125f, w0 = 1.0f - w1;   // texel rows 4n + q
          const float2 s = q < 2 ? lo : hi, e = q < 2 ? hi : nw;
          dec.texel_group(at[16 * q], at[80 + 16 * q], fmaf(w1, e.x, w0 * s.x), fmaf(w1, e.y, w0 * s.y), q, acc);
        }
        lo = hi;
        hi = nw;
      } else {
        if (b > 0 && !(b & 15)) row_axes(4 * b);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int rl = (4 * b + q) & 63;
          const int p = __builtin_amdgcn_readlane(rows_packed, rl), i0 = p & 0xffff, i1 = p >> 16;
          const float w1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(rows_w1), rl)), w0 = 1.0f - w1;
          if (i0 != r_lo || i1 != r_hi) {   // uniform
            if (i0 == r_hi && i1 == min(r_hi + 1, m.Gh - 1)) {   // on by one row: the one in flight
              lo = hi;
              hi = grid_row_sample<GDT>(gc, nx);
            } else {
              const GridRaw<GDT> l0 = grid_row_load<GDT>(gc, i0), h0 = grid_row_load<GDT>(gc, i1);
              lo = grid_row_sample<GDT>(gc, l0);
              hi = grid_row_sample<GDT>(gc, h0);
            }
            r_lo = i0;
            r_hi = i1;
            nx = grid_row_load<GDT>(gc, min(r_hi + 1, m.Gh - 1));
          }
          dec.texel_group(at[16 * q], at[80 + 16 * q], fmaf(w1, hi.x, w0 * lo.x), fmaf(w1, hi.y, w0 * lo.y), q, acc);
        }
      }
      if ((b & 1) || b + 1 == th) wave_sync();   // every lane has read the pair's bytes
      store_rgb<PREC>(out, 0, dec.finish(acc), false);
      out += 12 * pitch;
    }
  }
}

// Request of item `it`: its sub-tile s and its model.  Returns false (and flags the request
// once) when the request is invalid.
struct PageItem {
  ndgi_page_req rq;
  int s;
};

__device__ __forceinline__ bool page_item(const ndgi_model* __restrict__ models, int32_t n_models,
                                          const ndgi_page_req* __restrict__ reqs, int64_t it, int64_t per_req,
                                          int page, int lane, int& cur, ndgi_model& m, PageItem& pi,
                                          uint32_t* __restrict__ flags) {
  const int r = (int)(it / per_req);
  pi.s = (int)(it - (int64_t)r * per_req);
  pi.rq = reqs[r];
  const ndgi_page_req& rq = pi.rq;
  bool ok = rq.model >= 0 && rq.model < n_models && rq.page_x >= 0 && rq.page_y >= 0;
  if (ok && rq.model != cur) {
    m = models[rq.model];
    cur = rq.model;
  }
  ok = ok && (int64_t)page * (rq.page_x + 1) <= m.W && (int64_t)page * (rq.page_y + 1) <= m.H;
  if (!ok && lane == 0 && pi.s == 0) atomicOr(flags, NDGI_FLAG_BAD_PAGE_REQUEST);
  return ok;
}

template <int PREC>
__global__ __launch_bounds__(256, 3) void k_decode_pages(const ndgi_model* __restrict__ models, int32_t n_models,
                                                      const ndgi_page_req* __restrict__ reqs,
                                                      const int32_t* __restrict__ n_reqs_dev, int32_t max_reqs,
                                                      int32_t page, void* __restrict__ dst, int64_t pitch, int tw,
                                                      int th, uint32_t* __restrict__ flags) {
  __shared__ PageLds lds[4];
  const int lane = threadIdx.x & 63;
  PageLds& L = lds[threadIdx.x >> 6];
  int n_req = *n_reqs_dev;
  n_req = n_req < 0 ? 0 : (n_req > max_reqs ? max_reqs : n_req);
  const int sub_w = 16 * tw, sub_h = 4 * th;
  const int nsx = page / sub_w, nsy = page / sub_h;
  const int64_t per_req = (int64_t)nsx * nsy;
  const int64_t total = (int64_t)n_req * per_req;
  const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
  const int64_t wave0 = uniform((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
  Dec<PREC> dec;
  int dmodel = -1, cur = -1;
  ndgi_model m = {};
  PageItem pi;
  for (int64_t it = wave0; it < total; it += nwaves) {
    if (!page_item(models, n_models, reqs, it, per_req, page, lane, cur, m, pi, flags)) continue;
    if (dmodel != pi.rq.model) {
      dec.load_texel(m.mlp, m.mlp_dtype, lane);
      dmodel = pi.rq.model;
    }
    const Keys k = make_keys(pi.rq.t, m.T);
    const int ox = (pi.s % nsx) * sub_w, oy = (pi.s / nsx) * sub_h;
    const bool r4 = m.W == 4 * m.Gw && m.H == 4 * m.Gh;
    if (m.grid_dtype == NDGI_DTYPE_F16) {
      if (r4) page_subtile<PREC, NDGI_DTYPE_F16, true>(dec, m, pi.rq, k, page, ox, oy, tw, th, dst, pitch, lane, L);
      else page_subtile<PREC, NDGI_DTYPE_F16, false>(dec, m, pi.rq, k, page, ox, oy, tw, th, dst, pitch, lane, L);
    } else {
      if (r4) page_subtile<PREC, NDGI_DTYPE_F32, true>(dec, m, pi.rq, k, page, ox, oy, tw, th, dst, pitch, lane, L);
      else page_subtile<PREC, NDGI_DTYPE_F32, false>(dec, m, pi.rq, k, page, ox, oy, tw, th, dst, pitch, lane, L);
    }
  }
}

int launch_pages(ndgi_ctx* ctx, const ndgi_model* models, int32_t n_models, const ndgi_page_req* reqs,
                 const int32_t* n_reqs, int32_t max_reqs, int32_t page, void* dst, int64_t pitch, int prec,
                 hipStream_t s) {
#define NDGI_PAGES(P)                                                                                             \
  hipLaunchKernelGGL(k_decode_pages<P>, dim3(resident_wgs(ctx, (const void*)k_decode_pages<P>)), dim3(256), 0, s, \
                     models, n_models, reqs, n_reqs, max_reqs, page, dst, pitch, ctx->tile_w, ctx->tile_h,        \
                     ctx->flags_dev)
  if (prec == NDGI_PREC_F16) NDGI_PAGES(NDGI_PREC_F16);
  else NDGI_PAGES(NDGI_PREC_F32);
#undef NDGI_PAGES
  NDGI_HIP(hipGetLastError());
  return NDGI_OK;
}

}  // namespace ndgi
