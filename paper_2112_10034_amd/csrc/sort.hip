// Bitonic tile sort of groups of T = 32 .. 1024 keys.
//
// A group of T consecutive keys lives in LG = T/K consecutive lanes, K keys
// per lane (lane g of the group holds keys gK..gK+K-1, loaded as one
// vector), so key index i = g*K + r.  The network is the bitonic sorter in
// its all-ascending form: for each merge size k2 = 2, 4, .., T a first
// layer compares i with i ^ (k2 - 1) (the mirror inside the k2-block), then
// half-cleaner layers compare i with i ^ j for j = k2/4 .. 1; the smaller
// index always keeps the minimum.  A layer whose partner differs only in
// the low log2(K) bits is a compare-exchange between two registers of one
// lane; every other layer exchanges with partner lane g ^ (mask / K),
// register r ^ (mask mod K), then keeps min or max:
//   - partner in the same 32-lane half: a __shfl_xor_sync (DPP or
//     ds_swizzle; with K = 4 and T = 32 all are DPP quad_perm /
//     row_half_mirror exchanges);
//   - partner in the other half of the wave (a group of 64 lanes, the
//     full-wave sort): the in-half exchange, then v_permlane32_swap;
//   - partner in another wave (groups wider than a wave): through shared
//     memory, between two block barriers.
// Longer inputs in groups of 128 .. 1024 keys at the default 4 keys per lane are
// sorted by k_group_sort instead (below): 32 keys per lane, a group inside one
// wave.
// The layers inside one lane's K registers (every merge size up to K) are
// replaced by Batcher's odd-even merge sort of the K registers, which needs
// fewer comparators.  The sorted result is the unique ascending order, so
// any such network gives the same output as a one-key-per-lane network.
#include "cox_internal.hpp"

namespace cox {

// value of lane t ^ LM of the wave (LM < 64)
template <int LM>
__device__ __forceinline__ uint32_t xor_lane_wave(uint32_t v) {
  if constexpr (LM < 32) {
    return (uint32_t)xor_lane<LM>((int)v);
  } else {
    const uint32_t u = LM == 32 ? v : (uint32_t)xor_lane<LM - 32>((int)v);
    // swaps the upper half of the first operand with the lower half of the
    // second: every lane receives the other half's value
    const auto pr = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return lhalf() ? (uint32_t)pr[0] : (uint32_t)pr[1];
  }
}

template <int K, int PM, int LB, int U>
__device__ __forceinline__ void cx_layer(uint32_t (&key)[U][K], int g, uint32_t *lds) {
  constexpr int RM = PM & (K - 1);  // register part of the partner mask
  constexpr int LM = PM / K;        // lane part
  if constexpr (LM == 0) {
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int r = 0; r < K; r++) {
        const int r2 = r ^ RM;
        if (r < r2) {
          const uint32_t a = key[u][r], b = key[u][r2];
          key[u][r] = a < b ? a : b;
          key[u][r2] = a < b ? b : a;
        }
      }
  } else {
    // the lower lane of a pair keeps min = med3(a, b, 0), the upper one
    // max = med3(a, b, ~0): one exchange and one median per key
    const uint32_t sel = (g & (LB / K)) ? 0xffffffffu : 0u;
    uint32_t other[U][K];
    if constexpr (LM < 64) {
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int r = 0; r < K; r++) other[u][r] = xor_lane_wave<LM>(key[u][r ^ RM]);
    } else {
      const int t = threadIdx.x;
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int r = 0; r < K; r++) lds[(u * 256 + t) * K + r] = key[u][r];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int r = 0; r < K; r++) other[u][r] = lds[u * 256 * K + ((t * K + r) ^ PM)];
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int r = 0; r < K; r++) key[u][r] = med3u(key[u][r], other[u][r], sel);
  }
}

template <int K, int J, int U>
__device__ __forceinline__ void half_cleaners(uint32_t (&key)[U][K], int g, uint32_t *lds) {
  if constexpr (J >= 1) {
    cx_layer<K, J, J, U>(key, g, lds);
    half_cleaners<K, J / 2, U>(key, g, lds);
  }
}

template <int K, int K2, int T, int U>
__device__ __forceinline__ void merge_stages(uint32_t (&key)[U][K], int g, uint32_t *lds) {
  if constexpr (K2 <= T) {
    cx_layer<K, K2 - 1, K2 / 2, U>(key, g, lds);  // mirror layer
    half_cleaners<K, K2 / 4, U>(key, g, lds);
    merge_stages<K, K2 * 2, T, U>(key, g, lds);
  }
}

// compare-exchange of registers a < b of every row (a keeps the minimum)
template <int K, int U>
__device__ __forceinline__ void cx_reg(uint32_t (&key)[U][K], int a, int b) {
#pragma unroll
  for (int u = 0; u < U; u++) {
    const uint32_t x = key[u][a], y = key[u][b];
    key[u][a] = x < y ? x : y;
    key[u][b] = x < y ? y : x;
  }
}

// Batcher's odd-even merge sort of the K registers of each row: 1, 5, 19
// and 63 comparators for K = 2, 4, 8, 16, where the bitonic sorter takes
// 1, 6, 24 and 80.  Any sorting network gives the same sorted block, and
// the bitonic merges of the group continue from sorted blocks of K keys.
template <int K, int U, int LO, int N, int R>
__device__ __forceinline__ void oem_merge(uint32_t (&key)[U][K]) {
  constexpr int M = 2 * R;
  if constexpr (M < N) {
    oem_merge<K, U, LO, N, M>(key);
    oem_merge<K, U, LO + R, N, M>(key);
#pragma unroll
    for (int i = LO + R; i < LO + N - R; i += M) cx_reg<K, U>(key, i, i + R);
  } else {
    cx_reg<K, U>(key, LO, LO + R);
  }
}

template <int K, int U, int LO, int N>
__device__ __forceinline__ void oem_sort(uint32_t (&key)[U][K]) {
  if constexpr (N > 1) {
    oem_sort<K, U, LO, N / 2>(key);
    oem_sort<K, U, LO + N / 2, N / 2>(key);
    oem_merge<K, U, LO, N, 1>(key);
  }
}

// the group's network: the keys of each lane sorted in registers, then
// the bitonic merges of blocks of 2K, 4K, .., T keys
template <int K, int T, int U>
__device__ __forceinline__ void sort_group(uint32_t (&key)[U][K], int g, uint32_t *lds) {
  oem_sort<K, U, 0, K>(key);
  merge_stages<K, 2 * K, T, U>(key, g, lds);
}

template <int K>
__device__ __forceinline__ void load_keys(const uint32_t *__restrict__ p, uint32_t (&key)[K]) {
  if constexpr (K % 4 == 0) {
#pragma unroll
    for (int q = 0; q < K / 4; q++) {
      const u32x4 v = ld_stream4(p + 4 * q);
      key[4 * q] = v.x; key[4 * q + 1] = v.y; key[4 * q + 2] = v.z; key[4 * q + 3] = v.w;
    }
  } else if constexpr (K == 2) {
    const u32x2 v = ld_stream2(p);
    key[0] = v.x; key[1] = v.y;
  } else {
    key[0] = ld_stream1(p);
  }
}

template <int K>
__device__ __forceinline__ void store_keys(uint32_t *__restrict__ p, const uint32_t (&key)[K]) {
  if constexpr (K % 4 == 0) {
#pragma unroll
    for (int q = 0; q < K / 4; q++)
      st_stream4(p + 4 * q, key[4 * q], key[4 * q + 1], key[4 * q + 2], key[4 * q + 3]);
  } else if constexpr (K == 2) {
    st_stream2(p, key[0], key[1]);
  } else {
    st_stream1(p, key[0]);
  }
}

// keys of one round: U rows of 256 lane vectors starting at lane vector
// vbase (row u = vectors vbase + 256u).  A round that runs past n reads element
// by element, the last element in place of those past n, so that every load is
// unconditional and all are in flight together (each waited for, such a round
// took 1.5 us of a call on 2^22 + 17 keys); keys past n become the maximum key.
// Full rounds have loads of their own: with the selection of addresses in them
// 2^28 keys, one per lane, took 595 us in 32-key groups and 461 in 64-key
// groups, 556 and 438 without.
template <int K, int U>
__device__ __forceinline__ void load_round(const uint32_t *keys, int64_t vbase, int64_t n, bool full,
                                           uint32_t (&key)[U][K]) {
  if (full) {
#pragma unroll
    for (int u = 0; u < U; u++) load_keys<K>(keys + (vbase + 256 * u) * K, key[u]);
    return;
  }
  const int64_t b0 = (vbase - threadIdx.x) * K;  // the block's first key
  if (b0 < n) {
    const uint32_t *src = keys + b0;
    const uint32_t rem = (uint32_t)(n - b0);  // below 256 U K
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int r = 0; r < K; r++) {
        const uint32_t o = (threadIdx.x + 256 * u) * K + r;
        key[u][r] = src[o < rem ? o : rem - 1];
      }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int r = 0; r < K; r++)
        if ((threadIdx.x + 256 * u) * K + r >= rem) key[u][r] = 0xffffffffu;
  } else {
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int r = 0; r < K; r++) key[u][r] = 0xffffffffu;
  }
}

template <int K, int U>
__device__ __forceinline__ void store_round(uint32_t *out, int64_t vbase, int64_t n, bool full,
                                            const uint32_t (&key)[U][K]) {
  if (full) {
#pragma unroll
    for (int u = 0; u < U; u++) store_keys<K>(out + (vbase + 256 * u) * K, key[u]);
  } else {
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int64_t e0 = (vbase + 256 * u) * K;
#pragma unroll
      for (int r = 0; r < K; r++)
        if (e0 + r < n) out[e0 + r] = key[u][r];
    }
  }
}

// Grid-stride rounds; in a round a block handles U rows of 256 lane
// vectors (row u = vectors [base + 256u, base + 256u + 256)), and each
// thread first requests its U vectors, then sorts and stores them, so U
// independent loads per lane are in flight.  (Requesting the next round's
// keys before sorting the current ones, in a second register set, measured
// slower: 0.37-0.38 against 0.36 ms at 2^28.)  Every group is held by LG
// aligned lanes of one block row (T <= 256 K).  keys and out may be the
// same buffer (each lane writes back only the positions it read, after its
// whole group has been sorted).
template <int K, int T>
__global__ __launch_bounds__(256) void k_tile_sort(const uint32_t *keys, uint32_t *out, int64_t n) {
  constexpr int LG = T / K;
  static_assert(LG >= 1 && LG <= 256, "a group fits in one block row");
  constexpr int U = K >= 16 ? 1 : 16 / K > 4 ? 4 : 16 / K;
  uint32_t *lds = nullptr;
  if constexpr (LG > 64) {
    __shared__ uint32_t s_x[U * 256 * K];  // the exchanges between waves
    lds = s_x;
  }
  const int g = (int)(threadIdx.x % LG);
  const int64_t nvec = (n + K - 1) / K;
  const int64_t per_round = (int64_t)gridDim.x * 256 * U;
  // the whole block iterates together so that partial groups see full warps
  const int64_t rounds = (nvec + per_round - 1) / per_round;
  for (int64_t it = 0; it < rounds; it++) {
    const int64_t vbase = it * per_round + (int64_t)blockIdx.x * 256 * U + threadIdx.x;
    const bool full = (vbase - threadIdx.x + 256 * U) * K <= n;
    uint32_t key[U][K];
    load_round<K, U>(keys, vbase, n, full, key);
    sort_group<K, T, U>(key, g, lds);
    store_round<K, U>(out, vbase, n, full, key);
  }
}

// ---------------------------------------------------------------- wide groups
// Groups of T = 128 .. 1024 keys, 32 keys per lane: LG = T / 32 lanes hold a
// group, a wave 2048 keys, and no block barrier is needed.
//
// What bounds it: VALU issue.  A compare-exchange inside a lane costs one
// operation per key, one across lanes two (the exchange and the median), so
// layers are run inside lanes where possible.  In layout A lane l of a group
// holds the keys 32l .. 32l + 31 (index bits 4 .. 0 in the register number);
// in layout B the register number holds the index bits from 5 up, and lane l
// the low bits.  The merge of 2^m keys runs its layers for bits m - 1 .. 5
// across lanes by DPP (m <= 7) or in layout B (m >= 8), the others in layout
// A; shared memory turns one layout into the other, 8 vector and 32 word
// accesses a lane, on a pipe of its own.  At T = 1024 that is 55 operations
// per key and 7 turns instead of 77 operations, three block barriers and
// exchanges of every key through shared memory (4 keys per lane, 4 waves per
// group).  2^26 keys in groups of 128 / 256 / 512 / 1024: 95.7 / 95.3 / 112 /
// 129 us against 99 / 119 / 152 / 175 us, the first two at the rate of a plain
// copy.
//
// The network is the bitonic sorter with directions: blocks of 2^m keys are
// sorted alternately up and down (bit m of the index), the last merge up.
// med3(a, b, 0) is the minimum and med3(a, b, ~0) the maximum, so a
// direction that differs between lanes is a mask operand.
constexpr int GROW = 36;  // words of a lane's row in shared memory: 16-byte rows, all banks
template <int T>
struct GroupLds {
  static constexpr int LG = T / 32, GPW = 64 / LG;
  // words of a group; the padding spreads the groups of a wave over the
  // banks when each lane reads its words of layout B
  static constexpr int GS = LG * GROW + (LG == 32 ? 32 : LG == 16 ? 16 : LG == 8 ? 8 : 4);
};

__device__ __forceinline__ void cx_dir(uint32_t &a, uint32_t &b, uint32_t sel) {
  const uint32_t x = a, y = b;
  a = med3u(x, y, sel);
  b = med3u(x, y, ~sel);
}
__device__ __forceinline__ void cx_up(uint32_t &a, uint32_t &b) {
  const uint32_t x = a, y = b;
  a = x < y ? x : y;
  b = x < y ? y : x;
}

template <int LO, int N, int R>
__device__ __forceinline__ void oem_merge_dir(uint32_t (&key)[32], uint32_t sel) {
  constexpr int M = 2 * R;
  if constexpr (M < N) {
    oem_merge_dir<LO, N, M>(key, sel);
    oem_merge_dir<LO + R, N, M>(key, sel);
#pragma unroll
    for (int i = LO + R; i < LO + N - R; i += M) cx_dir(key[i], key[i + R], sel);
  } else {
    cx_dir(key[LO], key[LO + R], sel);
  }
}
template <int LO, int N>
__device__ __forceinline__ void oem_sort_dir(uint32_t (&key)[32], uint32_t sel) {
  if constexpr (N > 1) {
    oem_sort_dir<LO, N / 2>(key, sel);
    oem_sort_dir<LO + N / 2, N / 2>(key, sel);
    oem_merge_dir<LO, N, 1>(key, sel);
  }
}

__device__ __forceinline__ void lds_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// exchange with lane l ^ LM; bit: this lane's bit of LM, dir: downwards
template <int LM>
__device__ __forceinline__ void cx_lanes(uint32_t (&key)[32], bool bit, bool dir) {
  const uint32_t sel = bit != dir ? 0xffffffffu : 0u;
#pragma unroll
  for (int r = 0; r < 32; r++) key[r] = med3u(key[r], (uint32_t)xor_lane<LM>((int)key[r]), sel);
}

// the merge of 2^M keys (6 <= M <= log2 T), layout A before and after
template <int T, int M>
__device__ __forceinline__ void merge_wide(uint32_t (&key)[32], int l, uint32_t *buf) {
  constexpr int LG = T / 32;
  constexpr bool LAST = (1 << M) == T;
  const bool dir = !LAST && ((l >> (M - 5)) & 1);
  if constexpr (M == 6) {
    cx_lanes<1>(key, l & 1, dir);
  } else if constexpr (M == 7) {
    cx_lanes<2>(key, l & 2, dir);
    cx_lanes<1>(key, l & 1, dir);
  } else {
    // layout B: register hi * P + p holds index 32 hi + LG p + l
    constexpr int P = 32 / LG;
#pragma unroll
    for (int q = 0; q < 8; q++)
      *(u32x4 *)(buf + l * GROW + 4 * q) = u32x4{key[4 * q], key[4 * q + 1], key[4 * q + 2], key[4 * q + 3]};
    lds_wave_sync();
#pragma unroll
    for (int r = 0; r < 32; r++) key[r] = buf[(r / P) * GROW + (r % P) * LG + l];
#pragma unroll
    for (int b = M - 1; b >= 5; b--) {
      const int j = P << (b - 5), d = LAST ? 0 : P << (M - 5);
#pragma unroll
      for (int r = 0; r < 32; r++)
        if (!(r & j)) {
          if (r & d) cx_up(key[r | j], key[r]);
          else cx_up(key[r], key[r | j]);
        }
    }
#pragma unroll
    for (int r = 0; r < 32; r++) buf[(r / P) * GROW + (r % P) * LG + l] = key[r];
    lds_wave_sync();
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const u32x4 v = *(const u32x4 *)(buf + l * GROW + 4 * q);
      key[4 * q] = v.x; key[4 * q + 1] = v.y; key[4 * q + 2] = v.z; key[4 * q + 3] = v.w;
    }
    lds_wave_sync();
  }
  const uint32_t sel = dir ? 0xffffffffu : 0u;
#pragma unroll
  for (int j = 16; j >= 1; j /= 2)
#pragma unroll
    for (int r = 0; r < 32; r++)
      if (!(r & j)) {
        if constexpr (LAST) cx_up(key[r], key[r | j]);
        else cx_dir(key[r], key[r | j], sel);
      }
  if constexpr (!LAST) merge_wide<T, M + 1>(key, l, buf);
}

template <int T>
__global__ __launch_bounds__(256, 4) void k_group_sort(const uint32_t *keys, uint32_t *out, int64_t n) {
  constexpr int LG = T / 32, GPW = 64 / LG, GS = GroupLds<T>::GS;
  __shared__ __align__(16) uint32_t s_buf[4][GPW * GS];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l = lane % LG;
  uint32_t *buf = s_buf[wv] + (lane / LG) * GS;
  for (int64_t w0 = ((int64_t)blockIdx.x * 4 + wv) * 2048; w0 < n; w0 += (int64_t)gridDim.x * 8192) {
    const int64_t g0 = w0 + (lane / LG) * T + l * 4;  // the lane's vectors: g0 + 4 LG q
    const bool full = w0 + 2048 <= n;
    const int rem = g0 < n ? (n - g0 < 2048 ? (int)(n - g0) : 2048) : 0;  // keys from g0 on
    uint32_t key[32];
    if (full) {
#pragma unroll
      for (int q = 0; q < 8; q++) {
        const u32x4 v = ld_stream4(keys + g0 + 4 * LG * q);
        key[4 * q] = v.x; key[4 * q + 1] = v.y; key[4 * q + 2] = v.z; key[4 * q + 3] = v.w;
      }
    } else {
      // past n the maximum key; every load is valid and none waits for
      // another
      const uint32_t *src = g0 < n ? keys + g0 : keys;
#pragma unroll
      for (int r = 0; r < 32; r++) {
        const int o = 4 * LG * (r / 4) + r % 4;
        key[r] = src[o < rem ? o : rem > 0 ? rem - 1 : 0];
      }
#pragma unroll
      for (int r = 0; r < 32; r++)
        if (4 * LG * (r / 4) + r % 4 >= rem) key[r] = 0xffffffffu;
    }
    oem_sort_dir<0, 32>(key, l & 1 ? 0xffffffffu : 0u);
    merge_wide<T, 6>(key, l, buf);
    // through shared memory to vectors that are consecutive over the wave
#pragma unroll
    for (int q = 0; q < 8; q++)
      *(u32x4 *)(buf + l * GROW + 4 * q) = u32x4{key[4 * q], key[4 * q + 1], key[4 * q + 2], key[4 * q + 3]};
    lds_wave_sync();
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const int v = q * 64 + lane;  // vector of the wave's 2048 keys
      const u32x4 k4 = *(const u32x4 *)(s_buf[wv] + (v / (T / 4)) * GS + (v % (T / 4)) / 8 * GROW + v % 8 * 4);
      uint32_t *dst = out + w0 + 4 * v;
      if (full) {
        st_stream4(dst, k4.x, k4.y, k4.z, k4.w);
      } else {
        const int o = 4 * v, rw = (int)(n - w0);
        if (o < rw) dst[0] = k4.x;
        if (o + 1 < rw) dst[1] = k4.y;
        if (o + 2 < rw) dst[2] = k4.z;
        if (o + 3 < rw) dst[3] = k4.w;
      }
    }
    lds_wave_sync();  // buf is written again by the next round
  }
}

// Key-value form: the network runs on 64-bit composites (key << 32 |
// position in the group), so equal keys keep their original order (a
// stable sort, which makes the result unique) and every comparison is one
// 64-bit compare.  After the network each output takes its value from the
// group's original values at its position (the group's 128 bytes, loaded
// once).
template <int K, int PM, int LB>
__device__ __forceinline__ void cx_layer_kv(uint64_t (&c)[K], int g) {
  constexpr int RM = PM & (K - 1);
  constexpr int LM = PM / K;
  if constexpr (LM == 0) {
#pragma unroll
    for (int r = 0; r < K; r++) {
      const int r2 = r ^ RM;
      if (r < r2) {
        const uint64_t a = c[r], b = c[r2];
        c[r] = a < b ? a : b;
        c[r2] = a < b ? b : a;
      }
    }
  } else {
    uint64_t other[K];
#pragma unroll
    for (int r = 0; r < K; r++) {
      const uint64_t v = c[r ^ RM];
      const uint32_t lo = (uint32_t)xor_lane<LM>((int)(uint32_t)v);
      const uint32_t hi = (uint32_t)xor_lane<LM>((int)(uint32_t)(v >> 32));
      other[r] = ((uint64_t)hi << 32) | lo;
    }
    const bool upper = (g & (LB / K)) != 0;
#pragma unroll
    for (int r = 0; r < K; r++) {
      const bool less = other[r] < c[r];
      c[r] = (less != upper) ? other[r] : c[r];
    }
  }
}

template <int K, int K2, int J>
__device__ __forceinline__ void half_cleaners_kv(uint64_t (&c)[K], int g) {
  if constexpr (J >= 1) {
    cx_layer_kv<K, J, J>(c, g);
    half_cleaners_kv<K, K2, J / 2>(c, g);
  }
}

template <int K, int K2>
__device__ __forceinline__ void merge_stages_kv(uint64_t (&c)[K], int g) {
  if constexpr (K2 <= 32) {
    cx_layer_kv<K, K2 - 1, K2 / 2>(c, g);
    half_cleaners_kv<K, K2, K2 / 4>(c, g);
    merge_stages_kv<K, K2 * 2>(c, g);
  }
}

// same rounds and row layout as k_tile_sort; keys / out_keys may be the
// same buffer, vals / out_vals may not
template <int K>
__global__ __launch_bounds__(256) void k_tile_sort_kv(const uint32_t *keys, const uint32_t *__restrict__ vals,
                                                      uint32_t *out_keys, uint32_t *__restrict__ out_vals,
                                                      int64_t n) {
  constexpr int LG = 32 / K;
  constexpr int U = K >= 8 ? 1 : 8 / K > 4 ? 4 : 8 / K;
  const int g = (int)(threadIdx.x % LG);
  const int64_t nvec = (n + K - 1) / K;
  const int64_t per_round = (int64_t)gridDim.x * 256 * U;
  const int64_t rounds = (nvec + per_round - 1) / per_round;
  for (int64_t it = 0; it < rounds; it++) {
    const int64_t vbase = it * per_round + (int64_t)blockIdx.x * 256 * U + threadIdx.x;
    const bool full = (vbase - threadIdx.x + 256 * U) * K <= n;
    uint64_t c[U][K];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int64_t e0 = (vbase + 256 * u) * K;
      uint32_t key[K];
      if (full) {
        load_keys<K>(keys + e0, key);
      } else {
#pragma unroll
        for (int r = 0; r < K; r++) key[r] = e0 + r < n ? keys[e0 + r] : 0xffffffffu;
      }
#pragma unroll
      for (int r = 0; r < K; r++) c[u][r] = ((uint64_t)key[r] << 32) | (uint32_t)(g * K + r);
    }
#pragma unroll
    for (int u = 0; u < U; u++) merge_stages_kv<K, 2>(c[u], g);
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int64_t e0 = (vbase + 256 * u) * K;
      const int64_t gb = e0 & ~(int64_t)31;
      uint32_t key[K], val[K];
#pragma unroll
      for (int r = 0; r < K; r++) {
        key[r] = (uint32_t)(c[u][r] >> 32);
        const bool ok = full || e0 + r < n;
        val[r] = ok ? vals[gb + ((uint32_t)c[u][r] & 31u)] : 0u;
      }
      if (full) {
        store_keys<K>(out_keys + e0, key);
        store_keys<K>(out_vals + e0, val);
      } else {
#pragma unroll
        for (int r = 0; r < K; r++)
          if (e0 + r < n) {
            out_keys[e0 + r] = key[r];
            out_vals[e0 + r] = val[r];
          }
      }
    }
  }
}

using sort_fn = void (*)(const uint32_t *, uint32_t *, int64_t);
static sort_fn pick_sort(int k, int tile, bool wide) {
  if (tile == 32) {
    switch (k) {
    case 1: return k_tile_sort<1, 32>;
    case 2: return k_tile_sort<2, 32>;
    case 4: return k_tile_sort<4, 32>;
    case 8: return k_tile_sort<8, 32>;
    case 16: return k_tile_sort<16, 32>;
    }
  } else if (k == 1) {
    switch (tile) {
    case 64: return k_tile_sort<1, 64>;
    case 128: return k_tile_sort<1, 128>;
    case 256: return k_tile_sort<1, 256>;
    }
  } else if (k == 4) {
    switch (tile) {
    case 64: return k_tile_sort<4, 64>;
    case 128: return wide ? k_group_sort<128> : k_tile_sort<4, 128>;
    case 256: return wide ? k_group_sort<256> : k_tile_sort<4, 256>;
    case 512: return wide ? k_group_sort<512> : k_tile_sort<4, 512>;
    case 1024: return wide ? k_group_sort<1024> : k_tile_sort<4, 1024>;
    }
  }
  return nullptr;
}

using sort_kv_fn = void (*)(const uint32_t *, const uint32_t *, uint32_t *, uint32_t *, int64_t);
static sort_kv_fn pick_sort_kv(int k) {
  switch (k) {
  case 1: return k_tile_sort_kv<1>;
  case 2: return k_tile_sort_kv<2>;
  case 4: return k_tile_sort_kv<4>;
  case 8: return k_tile_sort_kv<8>;
  }
  return nullptr;
}

}  // namespace cox

using namespace cox;

// Keys past which k_group_sort takes groups of 128 .. 1024 keys at four keys a
// lane.  It has a quarter of k_tile_sort's waves, each with four times the work,
// so up to here its one round takes longer (us per call, k_tile_sort /
// k_group_sort: 65,536 keys in groups of 128 / 1024 4.7 and 5.5 / 7.3 and 8.7; 2^20
// 5.2 and 6.2 / 7.9 and 9.1; 2^21 in groups of 128 / 256 / 512 / 1024 6.4 and 6.6 /
// 7.2 and 7.5 / 8.6 and 8.4 / 10.2 and 9.4; 3 x 2^20 7.7 and 7.5 / 9.5 and 8.9).
static int64_t wide_min(int tile) { return tile <= 256 ? 1 << 21 : 1 << 20; }

extern "C" cox_status cox_tile_sort(const uint32_t *keys, uint32_t *out, int64_t n, int tile,
                                    const cox_cfg *cfg, void *stream) {
  if (n < 0 || tile < 32 || tile > 1024 || (tile & (tile - 1))) return COX_ERR_INVALID;
  const int k = (cfg && cfg->items_per_lane) ? cfg->items_per_lane : 4;
  if (cfg && cfg->grid_blocks < 0) return COX_ERR_INVALID;
  const bool wide = k == 4 && tile >= 128 && n > wide_min(tile);
  sort_fn fn = pick_sort(k, tile, wide);
  if (!fn) return k > 0 && k <= 32 && (k & (k - 1)) == 0 ? COX_ERR_UNSUPPORTED : COX_ERR_INVALID;
  if (n == 0) return COX_OK;
  if (!keys || !out) return COX_ERR_INVALID;
  if (!aligned16(keys) || !aligned16(out)) return COX_ERR_ALIGN;
  const int64_t nvec = (n + k - 1) / k;
  const int U = k >= 16 ? 1 : 16 / k > 4 ? 4 : 16 / k;
  const int32_t want = cfg ? cfg->grid_blocks : 0;
  if (wide) {
    // k_group_sort: a block per 8192 keys, all of them launched (2^26 keys
    // in 1024-key groups: 128 us, 137 with a grid that fills the device)
    const int64_t items = (n + 8191) / 8192, most = want ? want : 0x7fffffff;
    hipLaunchKernelGGL(fn, dim3((unsigned)(items < most ? items : most)), dim3(256), 0, (hipStream_t)stream, keys, out,
                       n);
    return launch_status();
  }
  // default blocks per compute unit (measured at 2^28 keys): two for
  // 32-key groups and for 64-key groups with several keys per lane; six
  // for 64 keys over a full wave (0.420 ms against 0.434 with eight); eight
  // for wider groups, whose longer networks need more waves in flight.  Where two would take more than one round and six do not, all
  // rounds are launched at once: 2^22 + 17 keys in 32-key groups 7.5 us
  // against 9.8, in 64-key groups 8.2 against 11.4 (past that, two: 2^23
  // keys 14.9 us against 15.3 with six, 2^28 355 against 380).
  const int64_t items = (nvec + 256 * U - 1) / (256 * U);
  const int two = items <= 6 * (int64_t)device_cus() ? 6 : 2;
  const int per_cu = tile == 32 || (k >= 2 && tile <= 64) ? two : tile == 64 ? 6 : 8;
  const int grid = persistent_grid((const void *)fn, 256, items, want, 0, per_cu);
  hipLaunchKernelGGL(fn, dim3(grid), dim3(256), 0, (hipStream_t)stream, keys, out, n);
  return launch_status();
}

extern "C" cox_status cox_tile_sort_kv(const uint32_t *keys, const uint32_t *vals, uint32_t *out_keys,
                                       uint32_t *out_vals, int64_t n, int tile, const cox_cfg *cfg, void *stream) {
  if (n < 0 || tile != 32) return COX_ERR_INVALID;
  const int k = (cfg && cfg->items_per_lane) ? cfg->items_per_lane : 4;
  if (cfg && cfg->grid_blocks < 0) return COX_ERR_INVALID;
  sort_kv_fn fn = pick_sort_kv(k);
  if (!fn) return k > 0 && k <= 32 && (k & (k - 1)) == 0 ? COX_ERR_UNSUPPORTED : COX_ERR_INVALID;
  if (n == 0) return COX_OK;
  if (!keys || !vals || !out_keys || !out_vals) return COX_ERR_INVALID;
  if (!aligned16(keys) || !aligned16(out_keys) || !aligned16(out_vals)) return COX_ERR_ALIGN;
  if (out_vals == vals) return COX_ERR_INVALID;
  const int64_t nvec = (n + k - 1) / k;
  const int U = k >= 8 ? 1 : 8 / k > 4 ? 4 : 8 / k;
  // default: four 256-thread blocks per compute unit (measured at 2^28
  // pairs: 0.82 ms against 1.21 ms with two)
  const int grid = persistent_grid((const void *)fn, 256, (nvec + 256 * U - 1) / (256 * U),
                                   cfg ? cfg->grid_blocks : 0, 0, 4);
  hipLaunchKernelGGL(fn, dim3(grid), dim3(256), 0, (hipStream_t)stream, keys, vals, out_keys, out_vals, n);
  return launch_status();
}
