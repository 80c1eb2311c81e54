// Integral image (summed-area table) of a uint8 image, mod 2^32: the
// application of the shuffle scans that Table 1 lists (the row pass and the
// vertical pass of the CUDA scan sample).
//
// Instead of a row pass and a column pass over the whole image (13 bytes
// per pixel: 1 + 4 read, 4 + 4 written), the image is cut into tiles of
// TH rows x TW columns (band b, segment s) and reduced, carried, then
// scanned:
//   k_ii_reduce16 (k_ii_reduce below 16 columns) per tile: column sums
//                (colsum[b][x]), row sums (rowsum[s][y]) and the tile total
//                (total[b][s]);
//   k_ii_colscan per column: colsum[b][x] replaced by its exclusive prefix
//                over the bands above, T[b][x], and total[b][s] likewise (8 waves
//                per 64 columns; with few bands k_ii_scan sums them itself
//                instead);
//   k_ii_scan    per tile: sat[y][x] = rowprefix_x(T[b][.] + column sums
//                of rows y0..y)[x] + corner + sum of L over rows y0..y,
//                with L[y] the row sums of the segments to the left and
//                corner the totals of the tiles above and to the left.
// Every row of a tile is an inclusive scan over TW columns: lane-serial
// over a lane's 4 columns, a shuffle scan over the wave (DPP row shifts), and
// the waves' sums through shared memory.  About 6.1 bytes per pixel
// move (the image is read twice), all in uint32 arithmetic, so the result
// is exact (mod 2^32) whatever the order.
#include "cox_internal.hpp"

namespace cox {

constexpr int II_TH = 64;     // rows per tile
constexpr int II_TW = 1024;   // columns per tile
constexpr int II_BT = 256;    // threads per block, 4 columns each
constexpr int II_RB = 8;      // rows per round of the reduce kernel (its butterfly sums 8)
// wave 0 (64 threads) of the reduce kernel handles the tile's rows: one row
// per thread, two logical warps
static_assert(II_TH == 64 && II_BT >= 64 && II_TW == 4 * II_BT, "tile shape the kernels assume");

// inclusive scan over the 32 lanes of a logical warp
__device__ __forceinline__ uint32_t ii_warp_scan(uint32_t v) {
  v += (uint32_t)dpp<DPP_ROW_SHR1>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_SHR2>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_SHR4>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_SHR8>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_BCAST15, 0xa>(0, (int)v);
  return v;
}

__device__ __forceinline__ uint32_t ii_warp_sum(uint32_t v) {
  v += (uint32_t)xor_lane<16>((int)v);
  v += (uint32_t)xor_lane<8>((int)v);
  v += (uint32_t)xor_lane<4>((int)v);
  v += (uint32_t)xor_lane<2>((int)v);
  v += (uint32_t)xor_lane<1>((int)v);
  return v;
}

struct IiArgs {
  const uint8_t *img;
  uint32_t *sat;
  int64_t H, W;
  int64_t nb, ns;     // bands, segments
  uint32_t *colsum;   // [nb][W]: column sums, then their exclusive prefix T
  uint32_t *rowsum;   // [ns][H]
  uint32_t *total;    // [nb][ns]: tile totals, then their exclusive prefix over the bands
  bool whole;         // k_ii_scan: one segment, all rows above are summed from the image
  bool direct;        // k_ii_scan: colsum and total hold the bands' sums, not yet their prefix
};

// Tile number of work item i: the tiles are handed out so that each XCD
// (blocks b mod 8) walks an eighth of the image that is contiguous in memory.
// In plain order an XCD got the same 1024 columns of every band whenever a row
// has 8 segments, so its traffic met one eighth of the memory channels:
// 8192 x 8192 pixels 89.7 us, 76.4 in this order (8192 x 8000: 80.2 and 79.1,
// 6016 x 6016: 49.4 and 48.9).
__device__ __forceinline__ int64_t ii_tile(int64_t i, int64_t tiles) {
  const int64_t per = tiles >> 3;
  return i < 8 * per ? (i & 7) * per + (i >> 3) : i;
}

// How pixels are loaded: VEC (W % 4 == 0, image 4-byte aligned): aligned
// words; ANY: words at any address, the last lane of a row reading the row's
// last four bytes; NARROW (W < 4): bytes
enum { II_VEC = 0, II_ANY = 1, II_NARROW = 2 };
typedef uint32_t ii_u32u __attribute__((aligned(1)));
typedef uint32_t ii_u32x4u __attribute__((ext_vector_type(4), aligned(4)));

// the cols (1 .. 4) pixels of a lane at p, column j in byte j, zero above
template <int MODE>
__device__ __forceinline__ uint32_t ii_word(const uint8_t *p, int cols) {
  if constexpr (MODE == II_VEC) {
    return ld_stream1(p);
  } else if constexpr (MODE == II_ANY) {
    return *(const ii_u32u *)(p - (4 - cols)) >> (8 * (4 - cols));
  } else {
    return (uint32_t)p[0] | (cols > 1 ? (uint32_t)p[1] << 8 : 0u) | (cols > 2 ? (uint32_t)p[2] << 16 : 0u);
  }
}

// After row r of a tile is requested: the bytes of 8 rows are joined to words
// before those of the next are requested (all of 64 rows' bytes in flight spill to
// scratch: 2^20 rows of 1 / 2 / 3 columns 995 / 1213 / 1411 us, 653 / 732 / 832 so)
template <int MODE, int TH>
__device__ __forceinline__ void ii_join(uint32_t (&px)[TH], int r) {
  if constexpr (MODE == II_NARROW)
    if (r % 8 == 7) {
#pragma unroll
      for (int i = 0; i < 8; i++) asm volatile("" : "+v"(px[r - i]));
    }
}

// the lane's columns x .. x + 3 that lie in the image
__device__ __forceinline__ int ii_cols(const IiArgs &a, int64_t x) {
  return x < a.W ? (a.W - x < 4 ? (int)(a.W - x) : 4) : 0;
}

// The 4 pixels of a thread in row y (columns x .. x + 3; zero past W, and
// zero for rows past the tile).
template <int MODE>
__device__ __forceinline__ void ii_pixels(const IiArgs &a, int64_t y, bool row_ok, int64_t x, int cols,
                                          uint32_t (&p)[4]) {
  const uint32_t w = row_ok && cols ? ii_word<MODE>(a.img + y * a.W + x, cols) : 0u;
#pragma unroll
  for (int j = 0; j < 4; j++) p[j] = (w >> (8 * j)) & 0xffu;
}

// Sums of 8 values over a logical warp, one value per row: a butterfly
// that halves the values a lane holds at every step (xor 16, 8, 4), then
// two plain steps (xor 2, 1).  Returns, in every lane, the warp sum of
// value ((lane >> 2) & 7).
__device__ __forceinline__ uint32_t ii_warp_sum8(const uint32_t (&v)[8]) {
  const int l = llane();
  uint32_t a[4], b[2];
  const bool h16 = (l & 16) != 0, h8 = (l & 8) != 0, h4 = (l & 4) != 0;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const uint32_t send = h16 ? v[i] : v[i + 4];
    a[i] = (h16 ? v[i + 4] : v[i]) + (uint32_t)xor_lane<16>((int)send);
  }
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const uint32_t send = h8 ? a[i] : a[i + 2];
    b[i] = (h8 ? a[i + 2] : a[i]) + (uint32_t)xor_lane<8>((int)send);
  }
  uint32_t c = (h4 ? b[1] : b[0]) + (uint32_t)xor_lane<4>((int)(h4 ? b[0] : b[1]));
  c += (uint32_t)xor_lane<2>((int)c);
  c += (uint32_t)xor_lane<1>((int)c);
  return c;
}

template <int MODE>
__global__ __launch_bounds__(II_BT) void k_ii_reduce(IiArgs a) {
  static_assert(II_RB == 8, "row sums are reduced 8 rows at a time");
  __shared__ uint32_t s_rows[II_BT / 32][II_TH];
  __shared__ uint32_t s_tot[2];
  const int t = threadIdx.x, w = t >> 5, l = t & 31;
  for (int64_t i = blockIdx.x; i < a.nb * a.ns; i += gridDim.x) {
    const int64_t tile = ii_tile(i, a.nb * a.ns), b = tile / a.ns, s = tile % a.ns;
    const int64_t y0 = b * II_TH, x = s * II_TW + 4 * t;
    const int rows = (int)(a.H - y0 < II_TH ? a.H - y0 : II_TH), cols = ii_cols(a, x);
    uint32_t cs[4] = {0u, 0u, 0u, 0u};
    for (int r0 = 0; r0 < rows; r0 += II_RB) {
      uint32_t p[II_RB][4];
#pragma unroll
      for (int r = 0; r < II_RB; r++) ii_pixels<MODE>(a, y0 + r0 + r, r0 + r < rows, x, cols, p[r]);
      uint32_t rp[II_RB];
#pragma unroll
      for (int r = 0; r < II_RB; r++) {
        cs[0] += p[r][0];
        cs[1] += p[r][1];
        cs[2] += p[r][2];
        cs[3] += p[r][3];
        rp[r] = p[r][0] + p[r][1] + p[r][2] + p[r][3];
      }
      const uint32_t rs = ii_warp_sum8(rp);
      const int r = (l >> 2) & 7;
      if ((l & 3) == 0 && r0 + r < rows) s_rows[w][r0 + r] = rs;
    }
#pragma unroll
    for (int j = 0; j < 4; j++)
      if (x + j < a.W) a.colsum[b * a.W + x + j] = cs[j];
    __syncthreads();
    if (t < II_TH) {
      uint32_t v = 0u;
#pragma unroll
      for (int k = 0; k < II_BT / 32; k++) v += s_rows[k][t];
      if (t < rows) a.rowsum[s * a.H + y0 + t] = v;
      // tile total: the first two warps (all of wave 0) sum the row sums
      const uint32_t tot = ii_warp_sum(t < rows ? v : 0u);
      if (l == 0) s_tot[w] = tot;
    }
    __syncthreads();
    if (t == 0) a.total[b * a.ns + s] = s_tot[0] + s_tot[1];
    __syncthreads();
  }
}

// value of lane t ^ 32 of the wave: every lane receives the other half's
// value of the same register
__device__ __forceinline__ uint32_t ii_xor32(uint32_t v) {
  const auto pr = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return lhalf() ? (uint32_t)pr[0] : (uint32_t)pr[1];
}

// Sums of 16 values over the 64 lanes of a wave: a butterfly that halves
// the values a lane holds at every step (xor 32, 16, 8, 4), then two plain
// steps (xor 2, 1).  Returns, in every lane, the wave sum of value
// ((lane >> 2) & 15).
__device__ __forceinline__ uint32_t ii_wave_sum16(const uint32_t (&v)[16]) {
  const int L = (int)__lane_id();
  uint32_t a[8], b[4], c[2];
  const bool h32 = (L & 32) != 0, h16 = (L & 16) != 0, h8 = (L & 8) != 0, h4 = (L & 4) != 0;
#pragma unroll
  for (int i = 0; i < 8; i++) a[i] = (h32 ? v[i + 8] : v[i]) + ii_xor32(h32 ? v[i] : v[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; i++) b[i] = (h16 ? a[i + 4] : a[i]) + (uint32_t)xor_lane<16>((int)(h16 ? a[i] : a[i + 4]));
#pragma unroll
  for (int i = 0; i < 2; i++) c[i] = (h8 ? b[i + 2] : b[i]) + (uint32_t)xor_lane<8>((int)(h8 ? b[i] : b[i + 2]));
  uint32_t d = (h4 ? c[1] : c[0]) + (uint32_t)xor_lane<4>((int)(h4 ? c[0] : c[1]));
  d += (uint32_t)xor_lane<2>((int)d);
  d += (uint32_t)xor_lane<1>((int)d);
  return d;
}

// the 128-bit value w shifted down by sh (0 .. 127) bits
__device__ __forceinline__ u32x4 ii_shift_down(u32x4 w, int sh) {
  uint64_t lo = w.x | (uint64_t)w.y << 32, hi = w.z | (uint64_t)w.w << 32;
  if (sh >= 64) {
    lo = hi;
    hi = 0u;
  }
  sh &= 63;
  lo = lo >> sh | (hi << 1) << (63 - sh);
  hi >>= sh;
  return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}
typedef uint32_t ii_u32x4b __attribute__((ext_vector_type(4), aligned(1)));

// Tile sums with 16-pixel loads (width at least 16).  Lane c of wave g covers
// columns 16c .. 16c + 15 of the tile and rows g, g + 4, .., g + 60, so a
// row's sum is a wave sum; the four waves' column sums meet in shared memory.
// VEC: width a multiple of 16, image 16-byte aligned.  ANY: vectors at any
// address, a row's last, partial lane reading its last 16 bytes (1999 x 3001
// pixels: 21.5 us with 4-pixel loads, 6.6).  Same outputs as k_ii_reduce.
template <int MODE>
__global__ __launch_bounds__(II_BT, 4) void k_ii_reduce16(IiArgs a) {
  static_assert(II_BT == 256 && II_TW == 1024 && II_TH == 64, "4 waves x 64 lanes x 16 columns, 16 rows a wave");
  __shared__ __align__(16) uint32_t s_col[4][II_TW];
  __shared__ uint32_t s_tot[4];
  const int t = threadIdx.x, g = t >> 6, L = t & 63;
  for (int64_t i = blockIdx.x; i < a.nb * a.ns; i += gridDim.x) {
    const int64_t tile = ii_tile(i, a.nb * a.ns), b = tile / a.ns, s = tile % a.ns;
    const int64_t y0 = b * II_TH, x = s * II_TW + 16 * L;
    const int rows = (int)(a.H - y0 < II_TH ? a.H - y0 : II_TH);
    const bool okx = x < a.W;
    const int back = MODE == II_ANY && okx && a.W - x < 16 ? 16 - (int)(a.W - x) : 0;  // of a partial lane
    // column sums packed two to a word (even and odd bytes in 16-bit
    // halves; at most 16 * 255 each, no carry between halves), row sums by
    // v_sad_u8 against zero; rows in two batches of 8 loads
    uint32_t ev[4] = {0u, 0u, 0u, 0u}, od[4] = {0u, 0u, 0u, 0u}, rs[16];
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += 8) {
      u32x4 px[8];
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const int r = g + 4 * (i0 + i);
        const uint8_t *p = a.img + (y0 + (r < rows ? r : 0)) * a.W + (okx ? x - back : 0);
        if constexpr (MODE == II_VEC) px[i] = ld_stream4(p);
        else px[i] = __builtin_nontemporal_load((const ii_u32x4b *)p);
      }
      if constexpr (MODE == II_ANY)
        if (s == a.ns - 1) {
#pragma unroll
          for (int i = 0; i < 8; i++) px[i] = ii_shift_down(px[i], 8 * back);
        }
#pragma unroll
      for (int i = 0; i < 8; i++)
        if (!okx || g + 4 * (i0 + i) >= rows) px[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int i = 0; i < 8; i++) {
        uint32_t sum = 0u;
#pragma unroll
        for (int w = 0; w < 4; w++) {
          const uint32_t word = px[i][w];
          ev[w] += word & 0x00ff00ffu;
          od[w] += (word >> 8) & 0x00ff00ffu;
          sum = __builtin_amdgcn_sad_u8(word, 0u, sum);
        }
        rs[i0 + i] = sum;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t cs[16];
#pragma unroll
    for (int w = 0; w < 4; w++) {
      cs[4 * w + 0] = ev[w] & 0xffffu;
      cs[4 * w + 1] = od[w] & 0xffffu;
      cs[4 * w + 2] = ev[w] >> 16;
      cs[4 * w + 3] = od[w] >> 16;
    }
    // row g + 4 * slot of the tile, slot = (lane >> 2) & 15
    const uint32_t row_sum = ii_wave_sum16(rs);
    const int r = g + 4 * ((L >> 2) & 15);
    if ((L & 3) == 0 && r < rows) a.rowsum[s * a.H + y0 + r] = row_sum;
    // tile total: every row sum once (lanes with (L & 3) == 0), per wave
    uint32_t tv = (L & 3) == 0 && r < rows ? row_sum : 0u;
    tv = ii_warp_sum(tv);
    tv += ii_xor32(tv);
    if (L == 0) s_tot[g] = tv;
#pragma unroll
    for (int j = 0; j < 16; j += 4)
      *(u32x4 *)&s_col[g][16 * L + j] = u32x4{cs[j], cs[j + 1], cs[j + 2], cs[j + 3]};
    __syncthreads();
    {
      const int c0 = 4 * t;  // 4 columns a thread
      const int64_t xc = s * II_TW + c0;
      uint32_t out[4];
#pragma unroll
      for (int j = 0; j < 4; j++) out[j] = s_col[0][c0 + j] + s_col[1][c0 + j] + s_col[2][c0 + j] + s_col[3][c0 + j];
      uint32_t *dst = &a.colsum[b * a.W + xc];
      if constexpr (MODE == II_VEC) {
        if (xc < a.W) *(u32x4 *)dst = u32x4{out[0], out[1], out[2], out[3]};
      } else if (xc + 4 <= a.W) {
        *(ii_u32x4u *)dst = ii_u32x4u{out[0], out[1], out[2], out[3]};
      } else {
#pragma unroll
        for (int j = 0; j < 3; j++)
          if (xc + j < a.W) dst[j] = out[j];
      }
    }
    if (t == 0) a.total[b * a.ns + s] = s_tot[0] + s_tot[1] + s_tot[2] + s_tot[3];
    __syncthreads();
  }
}

// exclusive prefix of every column's band sums, and of every segment's tile
// totals (columns from the next multiple of 64 after W on).  A block takes 64
// columns (one per lane) and batches of 8 x 16 bands: wave g loads and
// sums bands g*16 .. g*16 + 15 of the batch, the 8 group sums meet in
// shared memory, and every wave writes its bands' exclusive prefixes
// (carry of the batches above + groups above + its own bands above).
constexpr int II_CS_WAVES = 8, II_CS_PB = 16;
__global__ __launch_bounds__(64 * II_CS_WAVES) void k_ii_colscan(IiArgs a) {
  __shared__ uint32_t s_grp[II_CS_WAVES][64];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int64_t Wp = (a.W + 63) / 64 * 64;
  for (int64_t x0 = (int64_t)blockIdx.x * 64; x0 < Wp + a.ns; x0 += (int64_t)gridDim.x * 64) {
    uint32_t *const m = x0 < Wp ? a.colsum : a.total;
    const int64_t width = x0 < Wp ? a.W : a.ns, x = (x0 < Wp ? x0 : x0 - Wp) + lane;
    const bool okx = x < width;
    uint32_t carry = 0u;
    for (int64_t b0 = 0; b0 < a.nb; b0 += II_CS_WAVES * II_CS_PB) {
      const int64_t bg = b0 + (int64_t)g * II_CS_PB;
      uint32_t v[II_CS_PB], sum = 0u;
#pragma unroll
      for (int k = 0; k < II_CS_PB; k++) v[k] = okx && bg + k < a.nb ? m[(bg + k) * width + x] : 0u;
#pragma unroll
      for (int k = 0; k < II_CS_PB; k++) sum += v[k];
      s_grp[g][lane] = sum;
      __syncthreads();
      uint32_t off = carry, tot = 0u;
#pragma unroll
      for (int h = 0; h < II_CS_WAVES; h++) {
        const uint32_t u = s_grp[h][lane];
        off += h < g ? u : 0u;
        tot += u;
      }
#pragma unroll
      for (int k = 0; k < II_CS_PB; k++) {
        if (okx && bg + k < a.nb) m[(bg + k) * width + x] = off;
        off += v[k];
      }
      carry += tot;
      __syncthreads();  // s_grp is rewritten by the next batch
    }
  }
}

// inclusive scan over the 64 lanes of the wave
__device__ __forceinline__ uint32_t ii_wave_scan(uint32_t v) {
  v = ii_warp_scan(v);
  v += (uint32_t)dpp<0x143, 0xc>(0, (int)v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// One step of the butterfly below: 2H values to H, lanes exchanging with
// lane ^ M (the lane's bit of M says which half it keeps).
template <int M, int H, int N>
__device__ __forceinline__ void ii_halve(uint32_t (&v)[N], int lane) {
  const bool up = (lane & M) != 0;
#pragma unroll
  for (int i = 0; i < H; i++) {
    const uint32_t keep = up ? v[i + H] : v[i], send = up ? v[i] : v[i + H];
    if constexpr (M == 32) v[i] = keep + ii_xor32(send);
    else v[i] = keep + (uint32_t)xor_lane<M>((int)send);
  }
}

// Tile scans.  Wave w of the block holds columns 256w .. 256w + 255 of the
// tile (4 a lane) and all its TH rows: every pixel is requested before
// anything else, a word a row and lane, so no row waits for memory.  Of the
// other waves it needs the sums of their column carries and their row sums,
// which a butterfly leaves one row per lane, so the block meets at one barrier
// per tile; the carry of row y (corner, segments and waves to the left, over
// the rows up to y) is then a scan over the lanes, and row y takes it from
// lane y.  Bound by the table's stores for large images.  Reading four rows at
// a time, with a barrier and shared-memory warp totals for each four, the
// rounds' latency bound it: the same 70 us whatever the order of the tiles; now
// 55 us for 8192 x 8192 pixels (see ii_tile), 4.9 TB/s of image and table.
//
// TH = 64: the bands of the reduce kernel.  TH = 16 and 32: for images whose
// 64-row tiles leave the chip idle, where the 64 rows' scans of one wave (some
// 10 us) bound the call; the tile adds up the rows of its band above it (at
// most 48, read again from the image) to its column carries.
template <int MODE, int TH>
__global__ __launch_bounds__(II_BT, 4) void k_ii_scan(IiArgs a) {
  static_assert(II_TH == 64 && II_TW == 4 * 256 && II_BT == 256, "a wave per 256 columns, a lane per row");
  static_assert(TH == 64 || TH == 32 || TH == 16, "row sums of 64, 32 or 16 rows");
  __shared__ uint32_t s_rt[4][TH], s_above[4];  // the waves' row sums, sums of their column carries
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int64_t tiles = (a.H + TH - 1) / TH * a.ns;
  for (int64_t i = blockIdx.x; i < tiles; i += gridDim.x) {
    const int64_t tile = ii_tile(i, tiles), bt = tile / a.ns, s = tile % a.ns;
    const int64_t b = TH == II_TH ? bt : a.whole ? 0 : bt / (II_TH / TH);  // band
    const int64_t y0 = bt * TH, x = s * II_TW + 4 * t;
    const int rows = (int)(a.H - y0 < TH ? a.H - y0 : TH), cols = ii_cols(a, x);
    const int over = (int)(y0 - b * II_TH);  // rows of the band above the tile, a multiple of TH
    // pixels of row r (column x + j in byte j); rows and lanes past the image
    // read a valid row or the row's start and are cleared below
    uint32_t px[TH] = {};
    const uint8_t *src = a.img + y0 * a.W + (cols ? x : 0);
    const int load_cols = cols ? cols : (a.W < 4 ? (int)a.W : 4);
    if (MODE != II_NARROW || w == 0) {  // the other waves' columns lie past a narrow image
#pragma unroll
      for (int r = 0; r < TH; r++) {
        px[r] = ii_word<MODE>(src + (r < rows ? r : rows - 1) * a.W, load_cols);
        ii_join<MODE>(px, r);
      }
    }
    // column carries: the band sums above
    uint32_t c[4] = {0u, 0u, 0u, 0u};
    if (TH == II_TH || !a.direct) {
#pragma unroll
      for (int j = 0; j < 4; j++) c[j] = j < cols ? a.colsum[b * a.W + x + j] : 0u;
    } else if (cols) {
      // lanes at the edge read, and drop, columns before their own
      const uint32_t *cp = a.colsum + (cols == 4 || a.W < 4 ? x : a.W - 4);
      for (int64_t k0 = 0; k0 < b; k0 += 8) {
        ii_u32x4u v[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
          const uint32_t *q = cp + (k0 + k < b ? k0 + k : 0) * a.W;
          if constexpr (MODE == II_NARROW) v[k] = ii_u32x4u{q[0], cols > 1 ? q[1] : 0u, cols > 2 ? q[2] : 0u, 0u};
          else v[k] = *(const ii_u32x4u *)q;
        }
#pragma unroll
        for (int k = 0; k < 8; k++)
#pragma unroll
          for (int j = 0; j < 4; j++) c[j] += k0 + k < b ? v[k][j] : 0u;
      }
      if constexpr (MODE == II_ANY)
        if (cols < 4) {
          const int sh = 4 - cols;  // column x is element sh of the vector
          c[0] = sh == 1 ? c[1] : sh == 2 ? c[2] : c[3];
          c[1] = sh == 1 ? c[2] : sh == 2 ? c[3] : 0u;
          c[2] = sh == 1 ? c[3] : 0u;
          c[3] = 0u;
        }
    }
    if constexpr (TH < II_TH) {
      // packed two to a word (at most 64 * 255 each)
      const uint8_t *up = src - over * a.W;
      for (int r0 = 0; r0 < over; r0 += 64) {
        uint32_t ev = 0u, od = 0u;
        for (int r1 = r0; r1 < r0 + 64 && r1 < over; r1 += TH) {
          uint32_t q[TH];
#pragma unroll
          for (int r = 0; r < TH; r++) {
            q[r] = ii_word<MODE>(up + (r1 + r) * a.W, load_cols);
            ii_join<MODE>(q, r);
          }
#pragma unroll
          for (int r = 0; r < TH; r++) {
            ev += q[r] & 0x00ff00ffu;
            od += (q[r] >> 8) & 0x00ff00ffu;
          }
        }
        if (cols) {
          c[0] += ev & 0xffffu;
          c[1] += od & 0xffffu;
          c[2] += ev >> 16;
          c[3] += od >> 16;
        }
      }
    }
    // lane r: row y0 + r's sums of the segments to the left; and the totals of
    // the tiles above and to the left, lane k's those of segment k (added up
    // tile by tile, b s of them, 32768 x 32768 pixels took 2480 us, 1305 so)
    uint32_t left = 0u, cv = 0u;
    for (int64_t k = 0; k < s; k++) {
      if (lane < rows) left += a.rowsum[k * a.H + y0 + lane];
      if (TH < II_TH && lane < over) cv += a.rowsum[k * a.H + b * II_TH + lane];
      if (TH < II_TH && a.direct && lane < b) cv += a.total[lane * a.ns + k];  // at most 40 bands
    }
    if (TH == II_TH || !a.direct)
      for (int64_t k = lane; k < s; k += 64) cv += a.total[b * a.ns + k];
    uint32_t corner = (uint32_t)__builtin_amdgcn_readlane((int)ii_wave_scan(cv), 63);
    const uint32_t above = ii_wave_scan(c[0] + c[1] + c[2] + c[3]);
    if (lane == 63) s_above[w] = above;
#pragma unroll
    for (int r = 0; r < TH; r++)
      if (r >= rows || cols == 0) px[r] = 0u;
    uint32_t v[TH];
#pragma unroll
    for (int r = 0; r < TH; r++) v[r] = __builtin_amdgcn_sad_u8(px[r], 0u, 0u);
    if constexpr (TH == 64) {
      // lane r ends with row r's sum: the halves kept at each step are chosen
      // by the row's bits from the highest down
      ii_halve<32, 32>(v, lane);
      ii_halve<16, 16>(v, lane);
      ii_halve<8, 8>(v, lane);
      ii_halve<4, 4>(v, lane);
      ii_halve<2, 2>(v, lane);
      ii_halve<1, 1>(v, lane);
      s_rt[w][lane] = v[0];
    } else if constexpr (TH == 32) {
      ii_halve<32, 16>(v, lane);
      ii_halve<16, 8>(v, lane);
      ii_halve<8, 4>(v, lane);
      ii_halve<4, 2>(v, lane);
      ii_halve<2, 1>(v, lane);
      v[0] += (uint32_t)xor_lane<1>((int)v[0]);
      if ((lane & 1) == 0) s_rt[w][lane >> 1] = v[0];
    } else {
      const uint32_t rs = ii_wave_sum16(v);
      if ((lane & 3) == 0) s_rt[w][lane >> 2] = rs;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; k++) {
      left += k < w && lane < TH ? s_rt[k][lane & (TH - 1)] : 0u;
      corner += k < w ? s_above[k] : 0u;
    }
    left = corner + ii_wave_scan(left);
    uint32_t *dst = a.sat + y0 * a.W + x;
#pragma unroll
    for (int r = 0; r < TH; r++) {
#pragma unroll
      for (int j = 0; j < 4; j++) c[j] += (px[r] >> (8 * j)) & 0xffu;
      uint32_t q[4];
      q[0] = c[0];
#pragma unroll
      for (int j = 1; j < 4; j++) q[j] = q[j - 1] + c[j];
      const uint32_t off = ii_wave_scan(q[3]) - q[3] + (uint32_t)__builtin_amdgcn_readlane((int)left, r);
      // plain (cached) stores: the table is four times the image, and for
      // write-dominated traffic they beat non-temporal stores
      if constexpr (MODE == II_VEC) {
        if (r < rows && cols) *(u32x4 *)dst = u32x4{q[0] + off, q[1] + off, q[2] + off, q[3] + off};
      } else if (r < rows && cols == 4) {
        *(ii_u32x4u *)dst = ii_u32x4u{q[0] + off, q[1] + off, q[2] + off, q[3] + off};
      } else if (r < rows) {
#pragma unroll
        for (int j = 0; j < 3; j++)
          if (j < cols) dst[j] = q[j] + off;
      }
      dst += a.W;
    }
    __syncthreads();  // s_rt is written again for the next tile
  }
}

}  // namespace cox

namespace cox {

struct IiLayout {
  size_t colsum, rowsum, total, bytes;
};

static IiLayout ii_layout(int64_t H, int64_t W) {
  auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
  const int64_t nb = (H + II_TH - 1) / II_TH, ns = (W + II_TW - 1) / II_TW;
  IiLayout L;
  L.colsum = WS_HEADER;
  L.rowsum = L.colsum + up((size_t)nb * W * 4);
  L.total = L.rowsum + up((size_t)ns * H * 4);
  L.bytes = L.total + up((size_t)nb * ns * 4);
  return L;
}

size_t ii_workspace_bytes(int64_t H, int64_t W) { return ii_layout(H, W).bytes; }

}  // namespace cox

using namespace cox;

extern "C" cox_status cox_integral_image(const uint8_t *img, int64_t height, int64_t width, uint32_t *sat, void *ws,
                                         size_t ws_bytes, void *stream) {
  if (height < 0 || width < 0) return COX_ERR_INVALID;
  if (height == 0 || width == 0) return COX_OK;
  if (!img || !sat) return COX_ERR_INVALID;
  const IiLayout L = ii_layout(height, width);
  if (!ws || ws_bytes < L.bytes) return COX_ERR_WORKSPACE;
  char *w = (char *)ws;
  IiArgs a;
  a.img = img;
  a.sat = sat;
  a.H = height;
  a.W = width;
  a.nb = (height + II_TH - 1) / II_TH;
  a.ns = (width + II_TW - 1) / II_TW;
  a.colsum = (uint32_t *)(w + L.colsum);
  a.rowsum = (uint32_t *)(w + L.rowsum);
  a.total = (uint32_t *)(w + L.total);
  const bool vec = width % 4 == 0 && ((uintptr_t)img & 3u) == 0 && aligned16(sat);
  const bool vec16 = width % 16 == 0 && ((uintptr_t)img & 15u) == 0;
  auto reduce = vec16 ? k_ii_reduce16<II_VEC> : width >= 16 ? k_ii_reduce16<II_ANY>
                : width >= 4 ? k_ii_reduce<II_ANY> : k_ii_reduce<II_NARROW>;
  const int64_t tiles = a.nb * a.ns;
  // Rows per tile of the scan kernel, by the number of 64-row tiles: 64-row
  // tiles leave the chip idle up to about 250 of them, 16-row tiles read the
  // rows above them once too often from 64 on (us per call with 16 / 32 / 64:
  // 1000 x 1000 pixels, 16 tiles, 14.2 / 15.7 / 19.0; 2048 x 2048, 64, 15.0 /
  // 16.5 / 20.8; 2500 x 2500, 120, 22.7 / 20.9 / 23.8; 4000 x 4000, 252, 31.8 /
  // 27.1 / 27.3; 6000 x 6000, 564, 67 / 58 / 52).
  const int th = tiles <= 64 ? 16 : tiles <= 192 ? 32 : 64;
  auto scan = th == 16 ? (vec ? k_ii_scan<II_VEC, 16> : width >= 4 ? k_ii_scan<II_ANY, 16> : k_ii_scan<II_NARROW, 16>)
              : th == 32
                  ? (vec ? k_ii_scan<II_VEC, 32> : width >= 4 ? k_ii_scan<II_ANY, 32> : k_ii_scan<II_NARROW, 32>)
                  : (vec ? k_ii_scan<II_VEC, 64> : width >= 4 ? k_ii_scan<II_ANY, 64> : k_ii_scan<II_NARROW, 64>);
  // One segment and up to 256 rows: the scan kernel alone, adding up the rows
  // above a tile from the image (64 / 256 / 512 rows: 6.1 / 9.5 / 13.9 us, with
  // the reduce kernel 9.6 / 10.5 / 10.8).
  a.whole = th == 16 && a.ns == 1 && height <= 256;
  // Up to 40 bands the scan kernel adds up the bands' column sums itself, and
  // the column kernel's launch is saved (1000 x 1000: 14.2 and 12.0 us; 2048 x
  // 2048 16.1 and 14.9; 47 bands 16.2 and 16.0, 94 bands 14.4 and 16.8).
  a.direct = th < 64 && a.nb <= 40;
  hipStream_t hs = (hipStream_t)stream;
  if (!a.whole) {
    const int g1 = persistent_grid((const void *)reduce, II_BT, tiles, 0, 0, 8);
    hipLaunchKernelGGL(reduce, dim3(g1), dim3(II_BT), 0, hs, a);
    const int64_t gc = (width + 63) / 64 + (a.ns + 63) / 64;
    if (!a.direct)
      hipLaunchKernelGGL(k_ii_colscan, dim3((unsigned)(gc < 65536 ? gc : 65536)), dim3(64 * II_CS_WAVES), 0, hs, a);
  }
  const int g3 = persistent_grid((const void *)scan, II_BT, (height + th - 1) / th * a.ns, 0, 0, 8);
  hipLaunchKernelGGL(scan, dim3(g3), dim3(II_BT), 0, hs, a);
  return launch_status();
}
