// Warp-shuffle reductions.
//
// k_reduce_blocks_i32: sums of 256 elements and positive counts of 32, what the
// SDK reduction pattern that COX's Code 1 simplifies (Sec. 2.3) gives with
// 256-thread blocks of 8 logical warps: shfl_down tree and ballot(x > 0) per
// warp, shared-memory combine of the 8 warp values by warp 0.
//
// k_reduce: chunked sum / dot under the fixed schedule sigma = (k, W)
// (documented in cox.h); persistent blocks walk chunks c = b, b + G, ...;
// every chunk partial is published as a 64-bit word [tag | value bits]
// with a device-scope atomic store (tag = this call's epoch), and the grid's
// last block, once it has published its own, collects the words, waiting for
// each one's tag, and runs the FP64 (or int64) final combine.  A single
// chunk's value is the total at once.  No memory fences are needed: a word
// with the current tag can only hold this call's partial, and the epoch
// advances only after every block's words were seen, whose tags every block
// derived from its own read of the epoch.  A wait that takes too long ends
// with the combine handed over to the block that publishes last (HDR_HAND), so
// the total does not depend on when blocks start.  (With a counter
// of finished blocks, the last of which combines, one or two more round trips
// lay between: sums of 2^20 / 2^24 / 2^28 float32 8.4 / 17.6 / 162.7 us, 6.4 /
// 16.0 / 161 now; dot of 2^28 330.6 and 320.  Looking at HDR_HAND at a block's
// end costs short int32 sums 0.4 us, 65,613 elements 4.8 and 5.3, others nothing;
// partials published by exchanges that would find a request in their place
// arrive 0.4 us later, for every type.)
//
// The shfl_down tree is evaluated at lane 0, which only ever reads
// in-range sources (offset o reads lanes below 2o); the exchanges use the
// xor partner l ^ o, which for every lane l < o is exactly l + o, so lane
// 0's value is the one CUDA's __shfl_down_sync tree produces, bit for bit.
#include <type_traits>

#include "cox_internal.hpp"

namespace cox {

// ---------------------------------------------------------------- K-R0
// A wave takes R = 2 consecutive groups of 256 elements (a reduction block
// each), a 16-byte load per group and lane, requested together: no shared
// memory, no barrier.  Positive counts of the 8 lanes of a logical warp's 32
// elements are bytes of one word; a group's sum is a DPP scan's last lane.  The
// sums are mod 2^32, so any order gives the same.  Bound by the reads: us per
// call at 2^20 / 2^22 / 2^24 / 2^26 elements 3.3 / 5.3 / 13.0 / 44.4 (6.1 TB/s
// at 2^26); with an element per thread, trees through ds_swizzle and a barrier
// 4.3 / 9.9 / 30.1 / 152.  R = 1 / 4 / 8: 53.8 / 45.8 / 45.7 at 2^26.
constexpr int RB_R = 2;
template <bool STREAM>
__global__ __launch_bounds__(256) void k_reduce_blocks_i32(const int32_t *__restrict__ x, int64_t n,
                                                           int32_t *__restrict__ bsum,
                                                           int32_t *__restrict__ wpos) {
  constexpr int R = RB_R;
  static_assert(R <= 4, "an octet's lanes each store one group's count, a byte of one word");
  typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));  // x of any alignment
  const int lane = threadIdx.x & 63;
  const int64_t g0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
  if (256 * g0 >= n) return;
  const int64_t e = 256 * g0 + 4 * lane;
  u32x4a4 q[R];
  if (256 * (g0 + R) <= n) {
#pragma unroll
    for (int r = 0; r < R; r++) {
      const u32x4a4 *p = (const u32x4a4 *)(x + e + 256 * r);
      if constexpr (STREAM) q[r] = __builtin_nontemporal_load(p);
      else q[r] = *p;
    }
  } else {
#pragma unroll
    for (int r = 0; r < R; r++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int64_t i = e + 256 * r + j;
        const uint32_t v = (uint32_t)x[i < n ? i : n - 1];
        q[r][j] = i < n ? v : 0u;
      }
  }
  uint32_t cnt = 0u, out = 0u;
#pragma unroll
  for (int r = 0; r < R; r++) {
    uint32_t c = 0u;
#pragma unroll
    for (int j = 0; j < 4; j++) c += (int32_t)q[r][j] > 0 ? 1u : 0u;
    cnt += c << (8 * r);
    uint32_t v = (q[r][0] + q[r][1]) + (q[r][2] + q[r][3]);
    v += (uint32_t)dpp<DPP_ROW_SHR1>(0, (int)v);
    v += (uint32_t)dpp<DPP_ROW_SHR2>(0, (int)v);
    v += (uint32_t)dpp<DPP_ROW_SHR4>(0, (int)v);
    v += (uint32_t)dpp<DPP_ROW_SHR8>(0, (int)v);
    v += (uint32_t)dpp<DPP_ROW_BCAST15, 0xa>(0, (int)v);
    v += (uint32_t)dpp<0x143, 0xc>(0, (int)v);  // row_bcast:31
    const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    out = lane == r ? sum : out;
  }
  cnt += (uint32_t)xor_lane<1>((int)cnt);
  cnt += (uint32_t)xor_lane<2>((int)cnt);
  cnt += (uint32_t)xor_lane<7>((int)cnt);  // the other quad of the octet
  const int r = lane & 7;                  // lane r of an octet stores group r's count
  const int64_t g = 8 * (g0 + r) + (lane >> 3);
  if (r < R && 32 * g < n) wpos[g] = (int32_t)((cnt >> (8 * (r & 3))) & 0xffu);
  if (lane < R && 256 * (g0 + lane) < n) bsum[g0 + lane] = (int32_t)out;
}

// ---------------------------------------------------------------- chunked reduce
enum { DT_I32 = COX_I32, DT_F32 = COX_F32, DT_BF16 = COX_BF16 };
enum { OP_SUM = 0, OP_DOT = 1 };

template <int DT> struct ElemT;
template <> struct ElemT<DT_I32> { static constexpr int size = 4; };
template <> struct ElemT<DT_F32> { static constexpr int size = 4; };
template <> struct ElemT<DT_BF16> { static constexpr int size = 2; };

// a vector of V elements as it lies in memory: NW words (a 2-byte vector in
// the low half of its word)
template <int BYTES>
__device__ __forceinline__ void load_raw(const char *p, uint32_t (&w)[(BYTES + 3) / 4]) {
  if constexpr (BYTES == 16) {
    const u32x4 q = ld_stream4(p);
    w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
  } else if constexpr (BYTES == 8) {
    const u32x2 q = ld_stream2(p);
    w[0] = q.x; w[1] = q.y;
  } else if constexpr (BYTES == 4) {
    w[0] = ld_stream1(p);
  } else {
    w[0] = ld_stream_h(p);
  }
}

// raw 32-bit value of element v of such a vector (bfloat16 widened)
template <int ESZ, int NW>
__device__ __forceinline__ uint32_t element(const uint32_t (&w)[NW], int v) {
  if constexpr (ESZ == 4) return w[v];
  else return (v & 1) ? (w[v >> 1] & 0xffff0000u) : (w[v >> 1] << 16);
}

// per-lane accumulator
struct Acc {
  float s, c;
  uint32_t i;
};

template <int DT, int ACC>
__device__ __forceinline__ Acc acc_identity() {
  Acc a;
  a.s = -0.0f;
  a.c = -0.0f;
  a.i = 0u;
  return a;
}

__device__ __forceinline__ void two_sum(float a, float b, float &s, float &e) {
  float ss = a + b;
  float bb = ss - a;
  e = (a - (ss - bb)) + (b - bb);
  s = ss;
}

template <int DT, int OP, int ACC>
__device__ __forceinline__ void acc_step(Acc &a, uint32_t xr, uint32_t yr) {
  if constexpr (DT == DT_I32) {
    a.i += xr;
  } else {
    const float xv = i2f((int)xr);
    if constexpr (OP == OP_SUM) {
      if constexpr (ACC == COX_ACC_PLAIN) {
        a.s = a.s + xv;
      } else {
        float s, e;
        two_sum(a.s, xv, s, e);
        a.s = s;
        a.c = a.c + e;
      }
    } else {
      const float yv = i2f((int)yr);
      if constexpr (ACC == COX_ACC_PLAIN) {
        a.s = __builtin_fmaf(xv, yv, a.s);
      } else {
        const float p = xv * yv;
        const float pe = __builtin_fmaf(xv, yv, -p);
        float s, q;
        two_sum(a.s, p, s, q);
        a.s = s;
        a.c = a.c + (pe + q);
      }
    }
  }
}

// combine own value with the partner's (own operand first)
template <int DT, int ACC>
__device__ __forceinline__ Acc acc_combine(Acc a, Acc b) {
  if constexpr (DT == DT_I32) {
    a.i += b.i;
  } else if constexpr (ACC == COX_ACC_PLAIN) {
    a.s = a.s + b.s;
  } else {
    float s, e;
    two_sum(a.s, b.s, s, e);
    a.c = (a.c + b.c) + e;
    a.s = s;
  }
  return a;
}

// a with every 32-bit value in use replaced by f of it
template <int DT, int ACC, class F>
__device__ __forceinline__ Acc acc_map(Acc a, F f) {
  if constexpr (DT == DT_I32) {
    a.i = (uint32_t)f((int)a.i);
  } else {
    a.s = i2f(f(f2i(a.s)));
    if constexpr (ACC == COX_ACC_TWOSUM) a.c = i2f(f(f2i(a.c)));
  }
  return a;
}

// shfl_down tree, offsets 16, 8, 4, 2, 1 (value valid at lane 0)
template <int DT, int ACC>
__device__ __forceinline__ Acc warp_tree(Acc a) {
  const Acc b = acc_map<DT, ACC>(a, [](int v) {
    uint32_t own, partner;
    tree16((uint32_t)v, own, partner);
    return (int)partner;
  });
  a = acc_map<DT, ACC>(a, [](int v) {
    uint32_t own, partner;
    tree16((uint32_t)v, own, partner);
    return (int)own;
  });
  a = acc_combine<DT, ACC>(a, b);
  a = acc_combine<DT, ACC>(a, acc_map<DT, ACC>(a, [](int v) { return xor_lane<8>(v); }));
  a = acc_combine<DT, ACC>(a, acc_map<DT, ACC>(a, [](int v) { return tree4(v); }));
  a = acc_combine<DT, ACC>(a, acc_map<DT, ACC>(a, [](int v) { return xor_lane<2>(v); }));
  a = acc_combine<DT, ACC>(a, acc_map<DT, ACC>(a, [](int v) { return xor_lane<1>(v); }));
  return a;
}

// int64 sum over a logical warp, in every lane
__device__ __forceinline__ long long tree_i64(long long v) {
  auto moved = [&](auto f) {
    uint2 p = __builtin_bit_cast(uint2, v);
    p.x = (uint32_t)f((int)p.x);
    p.y = (uint32_t)f((int)p.y);
    return __builtin_bit_cast(long long, p);
  };
  const uint2 p = __builtin_bit_cast(uint2, v);
  uint2 a, b;
  tree16(p.x, a.x, b.x);
  tree16(p.y, a.y, b.y);
  v = __builtin_bit_cast(long long, a) + __builtin_bit_cast(long long, b);
  v += moved([](int u) { return xor_lane<8>(u); });
  v += moved([](int u) { return tree4(u); });
  v += moved([](int u) { return xor_lane<2>(u); });
  v += moved([](int u) { return xor_lane<1>(u); });
  return v;
}

// chunk partial: optional plain copy for the caller, tagged word(s) for the
// final combine (two words per chunk for TWOSUM: s then c)
template <int DT, int ACC>
__device__ __forceinline__ void store_partial(void *part, uint64_t *pw, uint32_t tag, int64_t c, const Acc &a) {
  const uint64_t hi = (uint64_t)tag << 32;
  if constexpr (DT == DT_I32) {
    if (part) ((int32_t *)part)[c] = (int32_t)a.i;
    st_dev(&pw[c], hi | a.i);
  } else if constexpr (ACC == COX_ACC_PLAIN) {
    if (part) ((float *)part)[c] = a.s;
    st_dev(&pw[c], hi | (uint32_t)f2i(a.s));
  } else {
    if (part) ((float2 *)part)[c] = make_float2(a.s, a.c);
    st_dev(&pw[2 * c], hi | (uint32_t)f2i(a.s));
    st_dev(&pw[2 * c + 1], hi | (uint32_t)f2i(a.c));
  }
}

// a tagged word that did not yet carry `tag` when first read: at most `polls`
// more readings; the caller looks at the tag of what comes back
__device__ __noinline__ uint64_t wait_word(const uint64_t *p, uint32_t tag, uint32_t polls) {
  uint64_t s = 0;
  for (uint32_t spins = 0; spins < polls; spins++) {
    s = ld_dev(p);
    if ((uint32_t)(s >> 32) == tag) break;
    if (spins < 256) __builtin_amdgcn_s_sleep(1);
    else __builtin_amdgcn_s_sleep(32);
  }
  return s;
}

// value bits of FB tagged words p[i0 + b*stride] (b < FB, index < lim):
// all loads are issued first, then any word not yet carrying the tag is
// waited for (late: one did not come; the rest is not waited for);
// out-of-range entries get `pad`
template <int FB>
__device__ __forceinline__ void take_words(const uint64_t *p, int64_t i0, int64_t stride, int64_t lim,
                                           uint32_t tag, uint32_t polls, bool &late, uint32_t pad,
                                           uint32_t (&out)[FB]) {
  uint64_t w[FB];
#pragma unroll
  for (int b = 0; b < FB; b++) {
    const int64_t i = i0 + (int64_t)b * stride;
    w[b] = i < lim ? ld_dev(&p[i]) : (((uint64_t)tag << 32) | pad);
  }
#pragma unroll
  for (int b = 0; b < FB; b++) {
    const int64_t i = i0 + (int64_t)b * stride;
    if ((uint32_t)(w[b] >> 32) != tag) {
      w[b] = wait_word(&p[i], tag, late ? 0u : polls);
      late = late || (uint32_t)(w[b] >> 32) != tag;
    }
    out[b] = (uint32_t)w[b];
  }
}

// whether words [0, nw) all carry the tag (every thread of the block)
__device__ __forceinline__ bool words_there(const uint64_t *p, int64_t nw, uint32_t tag) {
  int missing = 0;
  for (int64_t i = threadIdx.x; i < nw; i += blockDim.x) missing |= (uint32_t)(ld_dev(&p[i]) >> 32) != tag;
  return !__syncthreads_or(missing);
}

// Full chunks c = first + i * gridDim.x run double-buffered: the next
// chunk's vectors are requested before the current chunk is reduced, so loads
// stay in flight across the block's barrier.  A buffer holds the vectors as
// they lie in memory and elements are widened where they are used: widened at
// the load, bfloat16 vectors took twice the registers, and the compiler
// waited for one chunk before it requested the next (dot of 2^28 bfloat16,
// TwoSum: 179 -> 165 us; of 2^28 float32: 373 -> 341; sum: 179 -> 162).  Past the
// block's last full chunk the request is kept (loads stay unconditional) but
// every lane reads the array's first vector: one line, not a chunk.  Buffers of
// more than 32 words a lane (32 float32 elements of two arrays) would spill (dot
// of 2^25 in chunks of 32768 elements, plain / TwoSum: 75 / 73 us, 57 / 57 where
// the compiler loads one at a time), so they hold half of a chunk's rows: 43 / 44.
template <int K, int DT, int OP, int ACC>
__global__ __launch_bounds__(1024) void k_reduce(const void *__restrict__ x, const void *__restrict__ y,
                                                 int64_t n, int64_t nch, void *__restrict__ part,
                                                 void *__restrict__ total, uint32_t *__restrict__ hdr,
                                                 uint32_t polls, int away) {
  constexpr int ESZ = ElemT<DT>::size;
  constexpr int V = K < 16 / ESZ ? K : 16 / ESZ;
  constexpr int R = K / V;
  constexpr int VB = V * ESZ, NW = (VB + 3) / 4;
  constexpr int NA = OP == OP_DOT ? 2 : 1;
  // padding of x (-0.0, or 0 for int32) and y (+0.0), as raw words
  constexpr uint32_t XPAD = DT == DT_I32 ? 0u : DT == DT_BF16 ? 0x80008000u : 0x80000000u;
  __shared__ Acc slot[2][32];
  __shared__ double fin[256];
  __shared__ uint32_t s_epoch, s_late, s_go;

  if ((int)blockIdx.x == away) stay_away();
  const int W = blockDim.x >> 5;
  uint64_t *pw = (uint64_t *)(hdr + HDR_WORDS);
  // thread 0 stores the partials, so it alone needs the epoch until the
  // final combine; its load is not waited for before the data's
  uint32_t epoch = 0u;
  if (threadIdx.x == 0) epoch = ld_dev32(&hdr[HDR_EPOCH]);
  const int w = threadIdx.x >> 5, l = threadIdx.x & 31;
  const int64_t S = (int64_t)blockDim.x * K;
  const bool single = nch == 1 && gridDim.x == 1;  // its value is the total
  int par = 0;

  // Block's first chunk.  Blocks b mod 8 share an XCD; here an XCD's blocks take
  // neighbouring chunks of every round (dot of 2^26 / 2^28 bfloat16, TwoSum:
  // 53.7 / 175 us in plain order, 48.3 / 170; the sums 1 % faster).  Which
  // block reduces a chunk does not change its value.
  const int64_t per_xcd = gridDim.x >> 3;
  const int64_t first = blockIdx.x < 8 * per_xcd ? (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3) : blockIdx.x;

  const int64_t nfull = n / S;
  constexpr int PARTS = NA * R * NW > 32 ? 2 : 1, RP = R / PARTS;  // rows of a buffer
  typedef uint32_t Buf[NA][RP][NW];
  auto load_full = [&](int64_t c, int part, Buf &r) {
    const bool dummy = c >= nfull;
    // one base offset and one row stride per lane (not a select per load)
    const int64_t b0 = (dummy ? 0 : c * S + (int64_t)w * 32 * K + (int64_t)(part * RP * 32 + l) * V) * ESZ;
    const int rs = dummy ? 0 : 32 * VB;
#pragma unroll
    for (int i = 0; i < RP; i++) {
      load_raw<VB>((const char *)x + b0 + i * rs, r[0][i]);
      if constexpr (NA == 2) load_raw<VB>((const char *)y + b0 + i * rs, r[NA - 1][i]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto accumulate = [&](Acc &a, const auto &r) {
#pragma unroll
    for (int i = 0; i < (int)(sizeof(r[0]) / sizeof(r[0][0])); i++)
#pragma unroll
      for (int v = 0; v < V; v++)
        acc_step<DT, OP, ACC>(a, element<ESZ>(r[0][i], v), NA == 2 ? element<ESZ>(r[NA - 1][i], v) : 0u);
  };
  auto finish_chunk = [&](int64_t c, Acc a) {
    a = warp_tree<DT, ACC>(a);
    // two sets of slots: warp 0 reads this chunk's before it comes to the
    // next chunk's barrier, past which they are written again
    if (l == 0) slot[par][w] = a;
    __syncthreads();
    if (w == 0) {
      Acc b = l < W ? slot[par][l] : acc_identity<DT, ACC>();
      b = warp_tree<DT, ACC>(b);
      if (l == 0) {
        if (single) {
          // one chunk: the final combine of its value alone
          if constexpr (DT == DT_I32) {
            if (part) ((int32_t *)part)[0] = (int32_t)b.i;
            *(long long *)total = (long long)(int32_t)b.i;
          } else if constexpr (ACC == COX_ACC_PLAIN) {
            if (part) ((float *)part)[0] = b.s;
            *(double *)total = -0.0 + (double)b.s;
          } else {
            if (part) ((float2 *)part)[0] = make_float2(b.s, b.c);
            *(double *)total = -0.0 + ((double)b.s + (double)b.c);
          }
        } else {
          store_partial<DT, ACC>(part, pw, tag_of_epoch(epoch), c, b);
        }
      }
    }
    par ^= 1;
  };
  if (nfull > 0) {
    Buf A, B;
    int64_t c = first;
    load_full(c, 0, A);
    while (c < nfull) {
      int64_t cn = c + gridDim.x;
      Acc a = acc_identity<DT, ACC>();
      if constexpr (PARTS == 2) {
        load_full(c, 1, B);
        accumulate(a, A);
        load_full(cn, 0, A);
        accumulate(a, B);
        finish_chunk(c, a);
        c = cn;
      } else {
        load_full(cn, 0, B);
        accumulate(a, A);
        finish_chunk(c, a);
        c = cn;
        if (c >= nfull) break;
        cn = c + gridDim.x;
        load_full(cn, 0, A);
        a = acc_identity<DT, ACC>();
        accumulate(a, B);
        finish_chunk(c, a);
        c = cn;
      }
    }
  }
  if (nfull * S < n && first == nfull % gridDim.x) {
    // the partial last chunk, every load unconditional so that all are in
    // flight together: vectors past n read vector 0 and become padding, and
    // every lane reads the elements of the vector that n cuts (at edge)
    const int64_t e0 = nfull * S + (int64_t)w * 32 * K + (int64_t)l * V;
    const int64_t edge = n / V * V;
    uint32_t r[NA][R][NW];
    uint32_t cut[NA][NW];
#pragma unroll
    for (int k = 0; k < NW; k++) {
      cut[0][k] = XPAD;
      if constexpr (NA == 2) cut[NA - 1][k] = 0u;
    }
    if (edge < n) {
      uint32_t h[NA][V];
#pragma unroll
      for (int v = 0; v < V; v++) {
        const int64_t e = edge + v < n ? edge + v : n - 1;
        if constexpr (ESZ == 4) h[0][v] = ((const uint32_t *)x)[e];
        else h[0][v] = ((const uint16_t *)x)[e];
        if constexpr (NA == 2) {
          if constexpr (ESZ == 4) h[NA - 1][v] = ((const uint32_t *)y)[e];
          else h[NA - 1][v] = ((const uint16_t *)y)[e];
        }
      }
#pragma unroll
      for (int v = 0; v < V; v++)
#pragma unroll
        for (int k = 0; k < NA; k++) {
          uint32_t &word = cut[k][v * ESZ / 4];
          const int sh = ESZ == 4 ? 0 : 16 * (v & 1);
          const uint32_t m = (ESZ == 4 ? 0xffffffffu : 0xffffu) << sh;
          if (edge + v < n) word = (word & ~m) | (h[k][v] << sh);
        }
    }
    if (edge > 0) {
#pragma unroll
      for (int i = 0; i < R; i++) {
        const int64_t e = e0 + i * 32 * V, b0 = (e < edge ? e : 0) * ESZ;
        load_raw<VB>((const char *)x + b0, r[0][i]);
        if constexpr (NA == 2) load_raw<VB>((const char *)y + b0, r[NA - 1][i]);
      }
    }
#pragma unroll
    for (int i = 0; i < R; i++) {
      const int64_t e = e0 + i * 32 * V;
      if (e >= edge) {
#pragma unroll
        for (int k = 0; k < NW; k++) {
          r[0][i][k] = e == edge ? cut[0][k] : XPAD;
          if constexpr (NA == 2) r[NA - 1][i][k] = e == edge ? cut[NA - 1][k] : 0u;
        }
      }
    }
    Acc a = acc_identity<DT, ACC>();
    accumulate(a, r);
    finish_chunk(nfull, a);
  }
  if (single) return;

  // the grid's last block combines the chunk partials, or the block that it
  // was handed over to
  const bool last = blockIdx.x == gridDim.x - 1;
  if (threadIdx.x == 0) {
    s_epoch = epoch;
    s_late = 0u;
    if (!last) {
      wait_stores();
      s_go = ld_dev32(&hdr[HDR_HAND]) == tag_of_epoch(epoch) ? 1u : 0u;
    }
  }
  __syncthreads();
  if (!last && !s_go) return;
  epoch = s_epoch;
  const uint32_t tag = tag_of_epoch(epoch);

  // Loads of the partials are issued in batches of FB independent loads per
  // thread before they are added, so the fixed serial order costs one
  // memory latency per batch rather than one per chunk.
  constexpr int FB = ACC == COX_ACC_PLAIN ? 32 : 8;  // TwoSum: two words a chunk, and no spills
  for (bool handed = !last;;) {
    if (handed) {
      if (!words_there(pw, ACC == COX_ACC_PLAIN ? nch : 2 * nch, tag)) return;
      if (threadIdx.x == 0) s_go = hand_taken(hdr, tag) ? 1u : 0u;
      __syncthreads();
      if (!s_go) return;
    }
    bool late = false;
    if constexpr (DT == DT_I32) {
      __shared__ long long isum[32];
      long long s = 0;
      auto batch = [&](auto fb, int64_t c0) {
        constexpr int B = decltype(fb)::value;
        uint32_t buf[B];
        take_words<B>(pw, c0, blockDim.x, nch, tag, polls, late, 0u, buf);
#pragma unroll
        for (int b = 0; b < B; b++) s += (long long)(int32_t)buf[b];
      };
      if (nch <= blockDim.x) batch(std::integral_constant<int, 1>{}, threadIdx.x);
      else
        for (int64_t c0 = threadIdx.x; c0 < nch; c0 += (int64_t)FB * blockDim.x)
          batch(std::integral_constant<int, FB>{}, c0);
      // block sum of int64 (order does not matter for integers)
      s = tree_i64(s);
      if (l == 0) isum[w] = s;
      if (late) s_late = 1u;
      __syncthreads();
      if (!s_late) {
        if (threadIdx.x < 32) {
          long long tot = l < W ? isum[l] : 0;
          tot = tree_i64(tot);
          if (l == 0) {
            *(long long *)total = tot;
            st_dev32(&hdr[HDR_EPOCH], epoch + 1u);
          }
        }
        return;
      }
    } else {
      // FP64 final tree shaped like a 256-thread block (see cox.h); a chain
      // padded with -0.0 at its end is unchanged
      for (int j = threadIdx.x; j < 256; j += blockDim.x) {
        double s = -0.0;
        auto batch = [&](auto fb, int64_t c0) {
          constexpr int B = decltype(fb)::value;
          double buf[B];
          if constexpr (ACC == COX_ACC_PLAIN) {
            uint32_t v[B];
            take_words<B>(pw, c0, 256, nch, tag, polls, late, 0x80000000u, v);
#pragma unroll
            for (int b = 0; b < B; b++) buf[b] = (double)i2f((int)v[b]);
          } else {
            // words 2c (s) and 2c + 1 (c); padding (-0.0, -0.0) adds -0.0
            uint32_t vs[B], vc[B];
            take_words<B>(pw, 2 * c0, 512, 2 * nch, tag, polls, late, 0x80000000u, vs);
            take_words<B>(pw, 2 * c0 + 1, 512, 2 * nch, tag, polls, late, 0x80000000u, vc);
#pragma unroll
            for (int b = 0; b < B; b++) buf[b] = (double)i2f((int)vs[b]) + (double)i2f((int)vc[b]);
          }
#pragma unroll
          for (int b = 0; b < B; b++) s = s + buf[b];
        };
        if (nch <= 256) batch(std::integral_constant<int, 1>{}, j);
        else
          for (int64_t c0 = j; c0 < nch; c0 += (int64_t)FB * 256) batch(std::integral_constant<int, FB>{}, c0);
        // the tree of each group of 32, by its own warp where there are eight
        if (blockDim.x >= 256) {
          s = tree_f64(s);
          if (l == 0) fin[j >> 5] = s;
        } else {
          fin[j] = s;
        }
      }
      if (late) s_late = 1u;
      __syncthreads();
      if (!s_late) {
        if (threadIdx.x < 32) {
          double top = -0.0;
          if (blockDim.x >= 256) {
            if (l < 8) top = fin[l];
          } else {
#pragma unroll 1
            for (int vw = 0; vw < 8; vw++) {
              const double r = tree_f64(fin[32 * vw + l]);
              const double r0 = __shfl(r, 0, 32);
              if (l == vw) top = r0;
            }
          }
          top = tree_f64(top);
          if (l == 0) {
            *(double *)total = top;
            st_dev32(&hdr[HDR_EPOCH], epoch + 1u);
          }
        }
        return;
      }
    }
    // a word did not come in time
    __syncthreads();  // s_late and the sums are written again
    if (threadIdx.x == 0) {
      s_late = 0u;
      st_dev32(&hdr[HDR_HAND], tag);
      wait_stores();
    }
    __syncthreads();
    handed = true;
  }
}

// ---------------------------------------------------------------- dispatch
using reduce_fn = void (*)(const void *, const void *, int64_t, int64_t, void *, void *, uint32_t *, uint32_t, int);

template <int DT, int OP, int ACC>
static reduce_fn pick_k(int k) {
  switch (k) {
  case 1: return k_reduce<1, DT, OP, ACC>;
  case 2: return k_reduce<2, DT, OP, ACC>;
  case 4: return k_reduce<4, DT, OP, ACC>;
  case 8: return k_reduce<8, DT, OP, ACC>;
  case 16: return k_reduce<16, DT, OP, ACC>;
  case 32: return k_reduce<32, DT, OP, ACC>;
  }
  return nullptr;
}

static reduce_fn pick(int dt, int op, int acc, int k) {
  if (dt == DT_I32) return op == OP_SUM && acc == COX_ACC_PLAIN ? pick_k<DT_I32, OP_SUM, COX_ACC_PLAIN>(k) : nullptr;
  if (dt == DT_F32) {
    if (op == OP_SUM) return acc == COX_ACC_PLAIN ? pick_k<DT_F32, OP_SUM, COX_ACC_PLAIN>(k) : pick_k<DT_F32, OP_SUM, COX_ACC_TWOSUM>(k);
    return acc == COX_ACC_PLAIN ? pick_k<DT_F32, OP_DOT, COX_ACC_PLAIN>(k) : pick_k<DT_F32, OP_DOT, COX_ACC_TWOSUM>(k);
  }
  if (dt == DT_BF16) {
    if (op == OP_SUM) return acc == COX_ACC_PLAIN ? pick_k<DT_BF16, OP_SUM, COX_ACC_PLAIN>(k) : pick_k<DT_BF16, OP_SUM, COX_ACC_TWOSUM>(k);
    return acc == COX_ACC_PLAIN ? pick_k<DT_BF16, OP_DOT, COX_ACC_PLAIN>(k) : pick_k<DT_BF16, OP_DOT, COX_ACC_TWOSUM>(k);
  }
  return nullptr;
}

// default persistent grid: about 512 threads per compute unit (measured
// best for streaming reads on MI355X: fewer concurrent streams keep DRAM
// pages open)
static int reduce_blocks_per_cu(int block) { return block >= 512 ? 1 : 512 / block; }

static cox_status reduce_any(const void *x, const void *y, cox_dtype dtype, int op, int64_t n, cox_acc acc,
                             const cox_cfg *cfg, void *chunk_partials, void *total, void *ws,
                             size_t ws_bytes, void *stream, uint32_t polls = HAND_POLLS, int away = -1) {
  if (n < 0 || !total) return COX_ERR_INVALID;
  if (acc != COX_ACC_PLAIN && acc != COX_ACC_TWOSUM) return COX_ERR_DTYPE;
  if (dtype != COX_I32 && dtype != COX_F32 && dtype != COX_BF16) return COX_ERR_DTYPE;
  if (dtype == COX_I32 && (acc != COX_ACC_PLAIN || op != OP_SUM)) return COX_ERR_DTYPE;
  Sigma sg;
  cox_status st = resolve_cfg(op == OP_SUM ? COX_OP_REDUCE : COX_OP_DOT, dtype, cfg, &sg);
  if (st != COX_OK) return st;
  if (n > 0 && (!x || (op == OP_DOT && !y))) return COX_ERR_INVALID;
  if (n > 0 && (!aligned16(x) || (op == OP_DOT && !aligned16(y)))) return COX_ERR_ALIGN;
  const size_t need = cox_workspace_bytes(op == OP_SUM ? COX_OP_REDUCE : COX_OP_DOT, dtype, n, 0, cfg);
  if (!ws || ws_bytes < need) return COX_ERR_WORKSPACE;
  reduce_fn fn = pick(dtype, op, acc, sg.k);
  if (!fn) return COX_ERR_UNSUPPORTED;
  const int block = 32 * sg.W;
  const int64_t S = (int64_t)block * sg.k;
  const int64_t nch = (n + S - 1) / S;
  void *part = chunk_partials;  // optional plain copy; tagged words live in the workspace
  const int grid = persistent_grid((const void *)fn, block, nch > 0 ? nch : 1, sg.G, 0, reduce_blocks_per_cu(block));
  hipLaunchKernelGGL(fn, dim3(grid), dim3(block), 0, (hipStream_t)stream, x, y, n, nch, part, total,
                     (uint32_t *)ws, polls, away);
  return launch_status();
}

}  // namespace cox

using namespace cox;

extern "C" {

cox_status cox_warp_reduce_blocks_i32(const int32_t *x, int64_t n, int32_t *block_sums,
                                      int32_t *warp_pos_count, void *stream) {
  if (n < 0) return COX_ERR_INVALID;
  if (n == 0) return COX_OK;
  if (!x || !block_sums || !warp_pos_count) return COX_ERR_INVALID;
  const int64_t nb = (n + 255) / 256;
  if (nb > 0x7fffffff) return COX_ERR_INVALID;
  // Inputs that the L2 caches can hold are read with ordinary loads (2^20: 3.3
  // us, with streaming ones 3.8; 2^21 3.4 and 4.3), larger ones with streaming
  // loads (2^22: 5.6 and 5.3; 2^26 47.6 and 44.4).
  auto fn = n <= 1 << 21 ? k_reduce_blocks_i32<false> : k_reduce_blocks_i32<true>;
  hipLaunchKernelGGL(fn, dim3((unsigned)((nb + 4 * RB_R - 1) / (4 * RB_R))), dim3(256), 0, (hipStream_t)stream, x, n,
                     block_sums, warp_pos_count);
  return launch_status();
}

cox_status cox_warp_reduce(const void *x, cox_dtype dtype, int64_t n, cox_acc acc, const cox_cfg *cfg,
                           void *chunk_partials, void *total, void *ws, size_t ws_bytes, void *stream) {
  return reduce_any(x, nullptr, dtype, OP_SUM, n, acc, cfg, chunk_partials, total, ws, ws_bytes, stream);
}

cox_status cox_warp_dot(const void *a, const void *b, cox_dtype dtype, int64_t n, cox_acc acc,
                        const cox_cfg *cfg, void *chunk_partials, double *total, void *ws, size_t ws_bytes,
                        void *stream) {
  if (dtype != COX_F32 && dtype != COX_BF16) return COX_ERR_DTYPE;
  return reduce_any(a, b, dtype, OP_DOT, n, acc, cfg, chunk_partials, total, ws, ws_bytes, stream);
}

cox_status cox_warp_reduce_away(const void *x, const void *y, cox_dtype dtype, int64_t n, cox_acc acc,
                                const cox_cfg *cfg, void *chunk_partials, void *total, int32_t away_block,
                                uint32_t polls, void *ws, size_t ws_bytes, void *stream) {
  if (away_block < 0 || polls > HAND_POLLS) return COX_ERR_INVALID;
  if (y && dtype != COX_F32 && dtype != COX_BF16) return COX_ERR_DTYPE;
  return reduce_any(x, y, dtype, y ? OP_DOT : OP_SUM, n, acc, cfg, chunk_partials, total, ws, ws_bytes, stream, polls,
                    away_block);
}

}  // extern "C"
