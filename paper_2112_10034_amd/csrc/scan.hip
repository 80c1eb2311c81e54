// Single-pass int32 inclusive scan and ballot compaction.
//
// Chunk layout (schedule sigma = (k, W)): warp w of the block owns the 32k
// consecutive elements [c*S + 32kw, c*S + 32k(w+1)); in row i lane l holds
// the V consecutive elements at offset (32i + l) * V of that range, loaded
// as one 16-byte vector.
//
// Scan: per row, a lane-serial prefix over its V elements, a Kogge-Stone
// shfl_up scan of the lane totals (DPP row_shr:1,2,4,8 inside each 16-lane
// row, then row_bcast:15 carries row 0's total into row 1 -- never across
// lanes 31 -> 32), and the row total from logical lane 31; warp totals meet
// in shared memory, warp 0 scans them, and the chunk's exclusive prefix
// comes from a decoupled look-back (Merrill and Garland) over status words
// [tag | flag | value] published with device-scope atomics.
//
// Compaction: p = (x > 0); per row and vector slot v a ballot B_v; the
// rank of (l, v) inside the row is sum_v' popc(B_v' & lanemask_lt) plus the
// lane's own earlier slots (mbcnt over the wave's 64-bit ballots).  Kept
// elements are staged in the warp's own shared-memory region at their rank
// (the others in a trash slot, without branches), warp counts are scanned
// in shared memory, chunk offsets chained by the same look-back, and each
// warp then
// writes its run in 16-byte vectors aligned in global memory (the run's
// ragged first and last vectors element by element).
//
// Chunks are claimed from a ticket counter, so a chunk only ever waits for
// chunks that running blocks already hold.  Every block finally draws one
// ticket past the end; the block drawing the very last one (all others
// have finished) resets the counter and advances the epoch whose tag marks
// this call's status words, so the workspace needs no clearing between
// calls.  Every wait is bounded (MAX_SPIN); running out sets HDR_ERR.
//
// Short inputs under the default schedule take k_once instead (below).
#include <mutex>

#include "cox_internal.hpp"

namespace cox {

// 16-byte vectors at 4-byte aligned addresses (one dwordx4 access each)
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));

// inclusive scan of v over the 32 lanes of the logical warp (integers)
__device__ __forceinline__ uint32_t warp_incl_scan_u32(uint32_t v) {
  v += (uint32_t)dpp<DPP_ROW_SHR1>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_SHR2>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_SHR4>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_SHR8>(0, (int)v);
  v += (uint32_t)dpp<DPP_ROW_BCAST15, 0xa>(0, (int)v);
  return v;
}

__device__ __forceinline__ uint32_t warp_sum_u32(uint32_t v) {
  v += (uint32_t)xor_lane<16>((int)v);
  v += (uint32_t)xor_lane<8>((int)v);
  v += (uint32_t)xor_lane<4>((int)v);
  v += (uint32_t)xor_lane<2>((int)v);
  v += (uint32_t)xor_lane<1>((int)v);
  return v;
}

// Decoupled look-back, run by the lanes (64 or 32) of wave 0, in two halves so that
// other loads can be issued in between: lookback_begin publishes the chunk's
// aggregate and requests the status words of the 64 chunks before it (lane L
// chunk c - 1 - L; 32 for small chunks); lookback_end waits for them as far as the nearest
// inclusive prefix, walks further back if there is none, and publishes the
// chunk's inclusive prefix.  Returns the exclusive prefix (same in every lane).
//
// The look-back is the longest part of a compaction's chunk (9900 of 20500
// cycles at 2^28, and the next chunk's loads are back by half of it).  A request
// that comes before the words is paid for with another round trip and stands
// in the stores' way, so a wait comes first (units of 64 cycles; us at
// 2^28 for 0 / 8 / 14 / 20 / 28 / 36 / 48: compaction 306 / 304 / 304 / 300 /
// 295 / 291 / 292, scan 354 / 345 / 345 / 345 / 344 / 345 / 343).  64 words, 32
// before: compaction 319 and 306, scan 353 and 355; 128 / 256 words 321 / 338 and
// 368 / 388 without the wait.
// Less than 64 chunks, all under way at once, are not waited for (2000 elements
// 5.1 us, 5.6 with the wait); chunks below 16384 elements neither, and their
// windows stay at 32 words (2^24 with 1024 / 4096 a chunk: scan 242 / 81.9,
// with 64 words 254 / 84.3, and no wait gains it back).
__device__ __forceinline__ int lb_lanes(int64_t S) { return S < 16384 ? 32 : 64; }

__device__ __forceinline__ uint64_t lb_request(int64_t top, const uint64_t *__restrict__ status, int64_t sst,
                                               uint32_t tag) {
  const int64_t idx = top - (int)threadIdx.x;
  return idx >= 0 ? ld_dev(&status[idx * sst]) : st_pack(tag, ST_PREFIX, 0u);
}

__device__ __forceinline__ uint64_t lookback_begin(int64_t c, uint32_t agg, int64_t nch, int64_t S,
                                                   uint64_t *__restrict__ status, int64_t sst, uint32_t tag) {
  if (threadIdx.x == 0) st_dev(&status[c * sst], st_pack(tag, c == 0 ? ST_PREFIX : ST_AGG, agg));
  if (nch >= 64 && S >= 16384) __builtin_amdgcn_s_sleep(32);
  return lb_request(c - 1, status, sst, tag);
}

__device__ __forceinline__ uint32_t lookback_end(int64_t c, uint32_t agg, uint64_t s, int lanes,
                                                 uint64_t *__restrict__ status, int64_t sst, uint32_t tag,
                                                 uint32_t *__restrict__ hdr) {
  if (c == 0) return 0u;
  const int L = (int)threadIdx.x;
  uint32_t part = 0u, spins = 0u;  // this lane's words
  for (int64_t top = c - 1;;) {
    const bool ready = st_tag(s) == tag && st_flag(s) != 0u;
    const uint64_t pm = __builtin_amdgcn_ballot_w64(ready && st_flag(s) == ST_PREFIX);
    const uint64_t late = __builtin_amdgcn_ballot_w64(!ready);
    const uint64_t upto = pm ? pm ^ (pm - 1u) : ~0ull;  // lanes to the nearest prefix
    if (!(late & upto)) {
      part += (upto >> L & 1u) ? st_val(s) : 0u;
      if (pm) break;
      top -= lanes;
      s = lb_request(top, status, sst, tag);
      continue;
    }
    if (++spins >= MAX_SPIN || ((spins & 1023u) == 0u && ld_dev32(&hdr[HDR_ERR]) == tag)) {
      st_dev32(&hdr[HDR_ERR], tag);  // give up: result invalid, kernel still ends
      break;
    }
    __builtin_amdgcn_s_sleep(4);
    if (!ready) s = lb_request(top, status, sst, tag);
  }
  const uint32_t half = warp_sum_u32(part);
  uint32_t run = (uint32_t)__builtin_amdgcn_readlane((int)half, 0);
  if (lanes == 64) run += (uint32_t)__builtin_amdgcn_readlane((int)half, 32);
  if (L == 0) st_dev(&status[c * sst], st_pack(tag, ST_PREFIX, agg + run));
  return run;
}

// last exit ticket: reset the ticket counter, advance the epoch
__device__ __forceinline__ void finish_call(uint32_t *hdr, uint32_t ticket, uint32_t last, uint32_t epoch) {
  if (ticket == last) {
    st_dev32(&hdr[HDR_TICKET], 0u);
    st_dev32(&hdr[HDR_EPOCH], epoch + 1u);
  }
}

enum { MODE_SCAN = 0, MODE_COMPACT = 1 };

// One kernel for both look-back operations.  Per block: draw a ticket,
// then for every full chunk c: (1) row work on c's registers (scan: lane
// prefixes, warp scans, warp carry; compaction: ballots, ranks, warp
// count), (2) draw the next ticket and request its vectors into the other
// register buffer (a ticket past the full chunks reloads c, which is
// always valid, so the loads are unconditional), (3) warp 0 scans the warp
// values and runs the look-back, (4) outputs of c.  The partial last chunk
// is handled after the loop with element-wise bounds.
template <int K, int MODE>
__global__ __launch_bounds__(1024) void k_lookback(const int32_t *__restrict__ x, int32_t *__restrict__ out,
                                                   long long *__restrict__ count, int64_t n, int64_t nch,
                                                   uint64_t *__restrict__ status, int64_t sst,
                                                   uint32_t *__restrict__ hdr) {
  constexpr int V = K < 4 ? K : 4;
  constexpr int R = K / V;
  __shared__ uint32_t s_epoch, s_tk[2];
  __shared__ uint32_t s_w[32];
  extern __shared__ int32_t s_stage[];  // compaction: 32K elements per warp
  const int W = blockDim.x >> 5;
  const int w = threadIdx.x >> 5, l = threadIdx.x & 31;
  const int64_t S = (int64_t)blockDim.x * K;
  const int64_t nfull = n / S;
  const int lanes = lb_lanes(S);
  if (threadIdx.x == 0) {
    s_epoch = ld_epoch(hdr);
    s_tk[0] = add_dev32(&hdr[HDR_TICKET], 1u);
  }
  __syncthreads();
  const uint32_t epoch = s_epoch;
  const uint32_t tag = tag_of_epoch(epoch);
  const bool hi_half = lhalf() != 0;

  // vectors of chunk c; with dummy set every lane reads the array's first
  // vector instead (a ticket past the full chunks: keeps the loads
  // unconditional while fetching a single line)
  auto load_full = [&](int64_t c, uint32_t (&v)[R][V], bool dummy) {
    // one base pointer and one row stride per lane (not a select per load)
    const int32_t *src = x + (dummy ? 0 : c * S + (int64_t)w * 32 * K + l * V);
    const int rstride = dummy ? 0 : 32 * V;
#pragma unroll
    for (int i = 0; i < R; i++) {
      const int32_t *p = src + i * rstride;
      if constexpr (V == 4) {
        const u32x4 q = ld_stream4(p);
        v[i][0] = q.x; v[i][1] = q.y; v[i][2] = q.z; v[i][3] = q.w;
      } else if constexpr (V == 2) {
        const u32x2 q = ld_stream2(p);
        v[i][0] = q.x; v[i][1] = q.y;
      } else {
        v[i][0] = ld_stream1(p);
      }
    }
  };
  auto load_tail = [&](int64_t c, uint32_t (&v)[R][V]) {
    const int64_t wbase = c * S + (int64_t)w * 32 * K;
#pragma unroll
    for (int i = 0; i < R; i++)
#pragma unroll
      for (int j = 0; j < V; j++) {
        const int64_t e = wbase + (int64_t)(i * 32 + l) * V + j;
        v[i][j] = e < n ? ld_stream1(x + e) : 0u;
      }
  };

  // process chunk c held in cur; when `full`, prefetch the next ticket's
  // chunk into nxt.  Returns the next ticket.
  auto process = [&](int64_t c, uint32_t (&cur)[R][V], uint32_t (&nxt)[R][V], bool full) -> int64_t {
    uint32_t wval = 0u;  // warp carry (scan) or warp count (compaction)
    if constexpr (MODE == MODE_SCAN) {
#pragma unroll
      for (int i = 0; i < R; i++) {
#pragma unroll
        for (int j = 1; j < V; j++) cur[i][j] += cur[i][j - 1];
        const uint32_t r = cur[i][V - 1];
        const uint32_t incl = warp_incl_scan_u32(r);
        const uint32_t add = wval + (incl - r);
#pragma unroll
        for (int j = 0; j < V; j++) cur[i][j] += add;
        wval += (uint32_t)bcast31((int)incl);
      }
    } else {
      // ranks inside the warp from ballots: the wave's 64-bit ballot, lanes
      // below counted by mbcnt (an upper-half lane also counts the whole
      // lower half, subtracted once per row); kept elements go to the
      // warp's own shared-memory region at their rank, the others to the
      // lane's trash slot past the region (no branches).  The region is
      // written and later read by the same warp: no block barrier.
      int32_t *region = s_stage + w * (32 * K + 32);
      const uint32_t trash = 32 * K + l;
#pragma unroll
      for (int i = 0; i < R; i++) {
        uint32_t base = 0u, lo_cnt = 0u, hi_cnt = 0u;
#pragma unroll
        for (int j = 0; j < V; j++) {
          const uint64_t B = __builtin_amdgcn_ballot_w64((int32_t)cur[i][j] > 0);
          base = __builtin_amdgcn_mbcnt_hi((uint32_t)(B >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)B, base));
          lo_cnt += __builtin_popcount((uint32_t)B);
          hi_cnt += __builtin_popcount((uint32_t)(B >> 32));
        }
        if (hi_half) base -= lo_cnt;
        uint32_t pos = wval + base;
#pragma unroll
        for (int j = 0; j < V; j++) {
          const bool k = (int32_t)cur[i][j] > 0;
          region[k ? pos : trash] = (int32_t)cur[i][j];
          pos += k ? 1u : 0u;
        }
        wval += hi_half ? hi_cnt : lo_cnt;
      }
    }
    if (l == 0) s_w[w] = wval;
    if (threadIdx.x == 0) s_tk[1] = add_dev32(&hdr[HDR_TICKET], 1u);
    __syncthreads();
    const int64_t cn = s_tk[1];
    // warp 0: scan of the warp values, aggregate published, first window
    // of predecessor words requested -- before this block's prefetch, so
    // that waiting for the window does not also wait for the prefetch
    uint32_t wa = 0u, wincl = 0u, agg = 0u;
    uint64_t first = 0;
    if ((int)threadIdx.x < lanes) {
      wa = l < W ? s_w[l] : 0u;
      wincl = warp_incl_scan_u32(wa);
      agg = (uint32_t)bcast31((int)wincl);
      first = lookback_begin(c, agg, nch, S, status, sst, tag);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (full) load_full(cn, nxt, cn >= nfull);
    __builtin_amdgcn_sched_barrier(0);
    if ((int)threadIdx.x < lanes) {
      const uint32_t pre = lookback_end(c, agg, first, lanes, status, sst, tag, hdr);
      if (w == 0 && l < W) s_w[l] = pre + (wincl - wa);
      if constexpr (MODE == MODE_COMPACT)
        if (c == nch - 1 && threadIdx.x == 0) *count = (long long)pre + (long long)agg;
    }
    __syncthreads();
    const uint32_t off = s_w[w];
    const int64_t wbase = c * S + (int64_t)w * 32 * K;
    if constexpr (MODE == MODE_SCAN) {
      if (full) {
#pragma unroll
        for (int i = 0; i < R; i++) {
          const int64_t e = wbase + (int64_t)(i * 32 + l) * V;
          if constexpr (V == 4) {
            st_stream4(out + e, cur[i][0] + off, cur[i][1] + off, cur[i][2] + off, cur[i][3] + off);
          } else if constexpr (V == 2) {
            st_stream2(out + e, cur[i][0] + off, cur[i][1] + off);
          } else {
            st_stream1(out + e, cur[i][0] + off);
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < R; i++)
#pragma unroll
          for (int j = 0; j < V; j++) {
            const int64_t e = wbase + (int64_t)(i * 32 + l) * V + j;
            if (e < n) out[e] = (int32_t)(cur[i][j] + off);
          }
      }
    } else {
      // the warp writes its kept run [off, off + wval) from its region in
      // 16-byte vectors aligned in global memory: lane j takes positions
      // [A + 4j, A + 4j + 4) of each 128-position step, A = off rounded down
      // to a multiple of 4; the run's partial first and last vectors are
      // written element by element.  Offsets below are relative to A.
      const int32_t *region = s_stage + w * (32 * K + 32);
      const uint64_t A = (uint64_t)off & ~(uint64_t)3;
      const uint32_t head = (uint32_t)((uint64_t)off - A);  // 0..3 positions before the run
      uint32_t span = head + wval;
      // the bound on n only matters if a look-back wait gave up
      if (A + span > (uint64_t)n) span = A < (uint64_t)n ? (uint32_t)((uint64_t)n - A) : 0u;
      int32_t *dst = out + A;
      for (uint32_t t = 4u * (uint32_t)l; t < span; t += 128u) {
        if (t >= head && t + 4u <= span) {
          const u32x4u v = *(const u32x4u *)(region + (t - head));
          *(u32x4u *)(dst + t) = v;
        } else {
#pragma unroll
          for (uint32_t j = 0; j < 4u; j++)
            if (t + j >= head && t + j < span) dst[t + j] = region[t + j - head];
        }
      }
    }
    return cn;
  };

  int64_t c = s_tk[0];
  uint32_t A[R][V], B[R][V];
  if (c < nfull) {
    load_full(c, A, false);
    for (;;) {
      c = process(c, A, B, true);
      if (c >= nfull) break;
      c = process(c, B, A, true);
      if (c >= nfull) break;
    }
  }
  if (c < nch) {  // the partial last chunk
    load_tail(c, A);
    c = process(c, A, B, false);
  }
  if (threadIdx.x == 0) {
    if constexpr (MODE == MODE_COMPACT)
      if (nch == 0 && c == (int64_t)gridDim.x - 1) *count = 0;
    finish_call(hdr, (uint32_t)c, (uint32_t)(nch + gridDim.x - 1), epoch);
  }
}

// ---------------------------------------------------------------- short inputs
// One pass, one chunk per block, for inputs of at most ONCE_CHUNKS chunks
// (default schedule only; the result does not depend on it).  What bounds a
// short call of k_lookback is its chain of round trips: epoch, ticket (11.5
// ns each, one after another), loads, look-back windows of 32 chunks, and
// with chunks of 32768 elements most of the chip idle.  Here block b is chunk
// b, chunks are small enough to spread over the chip, and every block reads
// the aggregates of all chunks before it at once: one exchange instead of a
// chain.  Time per call in a graph of calls (empty kernel 2.5 us): scan of
// 1000 / 65,613 / 1,000,003 / 4,194,304 elements 3.2 / 4.4 / 4.8 / 6.4 us, with
// k_lookback 5.6 / 6.9 / 12.8 / 12.6 us; compaction 3.4 / 4.8 / 5.1 / 6.5
// us, 7.2 / 8.6 / 11.0 / 13.9.
//
// No ticket orders the blocks, so a block may wait for one that the device
// has not started.  After HAND_POLLS polls it therefore adds up the missing
// chunk from x itself (nothing writes x: the output lies apart), so every
// block ends whatever order the blocks start in, also beside other kernels.
// The last chunk's block advances the epoch once it has seen every other
// block's own word: each was published by a block that has read the epoch.
// If one is missing for too long it leaves that to the block that publishes
// last (HDR_HAND).  (Counting the started blocks with an atomic instead cost
// 2.4 us at 245 blocks.)
constexpr int ONCE_CHUNKS = 1024;

// inclusive scan of v over the 64 lanes of the wave
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
  v = warp_incl_scan_u32(v);
  // lane 31's value into lanes 32 .. 63 (rows 2 and 3)
  v += (uint32_t)dpp<0x143, 0xc>(0, (int)v);  // row_bcast:31
  return v;
}

// Ahead of the first reading of the aggregates: one that comes too early has
// to be repeated, a round trip later, and all blocks' early readings are in
// the way of the aggregates' stores.  By the number of chunks (units of 64
// cycles; us per scan / compaction without and with the wait): up to 16 none
// (20,000 elements 4.8 / 4.6, 4.9 / 4.7 with 12), then 14 (1,000,003: 6.0 / 6.3
// and 4.8 / 5.1; 2^22: 8.3 / 8.7 and 6.4 / 6.5), past 512 chunks 28 (2^23: scan
// 17.3 and 13.1; 2^24: compaction 26.7 and 24.3).
__device__ __forceinline__ void once_wait(int nch) {
  if (nch > 512) __builtin_amdgcn_s_sleep(28);
  else if (nch > 16) __builtin_amdgcn_s_sleep(14);
}

template <int K, int BT, int MODE>
__global__ __launch_bounds__(BT, BT == 1024 ? 8 : 1) void k_once(const int32_t *__restrict__ x, int32_t *__restrict__ out,
                                             long long *__restrict__ count, int64_t n, int nch,
                                             uint64_t *__restrict__ status, uint32_t *__restrict__ hdr,
                                             uint32_t polls, int away) {
  static_assert(K % 4 == 0, "rows of 16-byte vectors");
  constexpr int R = K / 4, NW = BT / 64, S = BT * K;
  __shared__ uint32_t s_w[NW], s_pre[NW], s_epoch, s_miss, s_late;
  __shared__ int32_t s_stage[MODE == MODE_COMPACT ? S + NW * 64 : 1];
  const int t = threadIdx.x, wv = t >> 6, lane = t & 63;
  const int c = blockIdx.x;
  if (c == away) stay_away();
  uint32_t e = 0u;
  if (t == 0 && nch > 1) {
    e = ld_epoch(hdr);
    s_miss = 0u;
  }
  // the wave's rows of 256 elements; past n every lane rereads the last one
  const int64_t wbase = (int64_t)c * S + wv * (64 * K);
  const bool full = (int64_t)(c + 1) * S <= n;
  uint32_t v[R][4];
  if (full) {
    const int32_t *src = x + wbase + lane * 4;
#pragma unroll
    for (int i = 0; i < R; i++) {
      const u32x4 q = ld_stream4(src + i * 256);
      v[i][0] = q.x; v[i][1] = q.y; v[i][2] = q.z; v[i][3] = q.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < R; i++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int64_t p = wbase + i * 256 + lane * 4 + j;
        v[i][j] = ld_stream1(x + (p < n ? p : n - 1));
      }
#pragma unroll
    for (int i = 0; i < R; i++)
#pragma unroll
      for (int j = 0; j < 4; j++)
        if (wbase + i * 256 + lane * 4 + j >= n) v[i][j] = 0u;
  }
  if (t == 0 && nch > 1) {
    s_epoch = e;
  }
  uint32_t wsum = 0u;  // wave-uniform: the rows before, then the wave's total
  int32_t *region = s_stage + (MODE == MODE_COMPACT ? wv * (64 * K + 64) : 0);
  if constexpr (MODE == MODE_SCAN) {
#pragma unroll
    for (int i = 0; i < R; i++) {
#pragma unroll
      for (int j = 1; j < 4; j++) v[i][j] += v[i][j - 1];
      const uint32_t r = v[i][3], incl = wave_incl_scan_u32(r), add = wsum + (incl - r);
#pragma unroll
      for (int j = 0; j < 4; j++) v[i][j] += add;
      wsum += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
  } else {
    // kept elements to their rank in the wave's region, the others to the
    // lane's trash slot after it
#pragma unroll
    for (int i = 0; i < R; i++) {
      uint32_t pos = wsum, cnt = 0u;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const uint64_t B = __builtin_amdgcn_ballot_w64((int32_t)v[i][j] > 0);
        pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(B >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)B, pos));
        cnt += (uint32_t)__builtin_popcountll(B);
      }
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const bool k = (int32_t)v[i][j] > 0;
        region[k ? pos : (uint32_t)(64 * K + lane)] = (int32_t)v[i][j];
        pos += k ? 1u : 0u;
      }
      wsum += cnt;
    }
  }
  if (lane == 0) s_w[wv] = wsum;
  __syncthreads();
  uint32_t off = 0u, agg = 0u;  // the waves before this one, the block's total
#pragma unroll
  for (int j = 0; j < NW; j++) {
    const uint32_t u = s_w[j];
    off += j < wv ? u : 0u;
    agg += u;
  }
  uint32_t pre = 0u, tag = 0u, hand = 0u;
  if (nch > 1) {
    tag = tag_of_epoch(s_epoch);
    if (t == 0) st_dev(&status[c], st_pack(tag, ST_AGG, agg));
    once_wait(nch);
    // thread t: the aggregates of chunks t, t + BT, .. below c
    constexpr int NP = (ONCE_CHUNKS + BT - 1) / BT;
    uint64_t w[NP];
#pragma unroll
    for (int k = 0; k < NP; k++) w[k] = t + k * BT < c ? ld_dev(&status[t + k * BT]) : st_pack(tag, ST_AGG, 0u);
    bool late = false;
#pragma unroll
    for (int k = 0; k < NP; k++) {
      uint32_t spins = 0;
      while (st_tag(w[k]) != tag && spins++ < polls) {
        __builtin_amdgcn_s_sleep(1);
        w[k] = ld_dev(&status[t + k * BT]);
      }
      late = late || st_tag(w[k]) != tag;
    }
    if (late) s_miss = 1u;
    auto sum_words = [&]() {
      uint32_t sum = 0u;
#pragma unroll
      for (int k = 0; k < NP; k++) sum += st_val(w[k]);
      sum = wave_incl_scan_u32(sum);
      if (lane == 63) s_pre[wv] = sum;
    };
    sum_words();
    __syncthreads();
    if (s_miss) {
      // some block before this one has not published: its chunk is added up
      // here, by the whole block (all chunks before c are full)
      for (int p = 0; p < c; p++) {
        const int k0 = p / BT;
        if (t == p % BT) {
          s_late = 0u;
#pragma unroll
          for (int k = 0; k < NP; k++)
            if (k == k0) s_late = st_tag(w[k]) != tag ? 1u : 0u;
        }
        __syncthreads();
        if (s_late) {  // uniform: written before the barrier, next after the one below
          uint32_t a = 0u;
          for (int i = t; i < S; i += BT) {
            const int32_t xv = x[(int64_t)p * S + i];
            a += MODE == MODE_SCAN ? (uint32_t)xv : (xv > 0 ? 1u : 0u);
          }
          a = wave_incl_scan_u32(a);
          if (lane == 63) s_w[wv] = a;
          __syncthreads();
          if (t == p % BT) {
            a = 0u;
            for (int j = 0; j < NW; j++) a += s_w[j];
#pragma unroll
            for (int k = 0; k < NP; k++)
              if (k == k0) w[k] = st_pack(tag, ST_AGG, a);
          }
        }
        __syncthreads();
      }
      sum_words();
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < NW; j++) pre += s_pre[j];
    if (c == nch - 1) {
      if (t == 0 && !s_miss) st_dev32(&hdr[HDR_EPOCH], s_epoch + 1u);
    } else if (t < 64) {
      wait_stores();  // the block's word; what was polled for came after it
      hand = ld_dev32(&hdr[HDR_HAND]);
    }
  }
  const uint32_t at = pre + off;
  if constexpr (MODE == MODE_SCAN) {
#pragma unroll
    for (int i = 0; i < R; i++) {
      const int64_t p = wbase + i * 256 + lane * 4;
      if (full) {
        st_stream4(out + p, v[i][0] + at, v[i][1] + at, v[i][2] + at, v[i][3] + at);
      } else {
#pragma unroll
        for (int j = 0; j < 4; j++)
          if (p + j < n) out[p + j] = (int32_t)(v[i][j] + at);
      }
    }
  } else {
    if (c == nch - 1 && t == 0) *count = (long long)pre + (long long)agg;
    // the wave's run in 16-byte vectors aligned in global memory, its ragged
    // first and last elements by lanes 0 .. 3 and 4 .. 7
    int32_t *dst = out + at;
    const uint32_t h0 = (uint32_t)(-(uintptr_t)dst >> 2) & 3u, hn = h0 < wsum ? h0 : wsum;
    const uint32_t nv = (wsum - hn) >> 2, tn = (wsum - hn) & 3u, l = (uint32_t)lane;
    for (uint32_t k = l; k < nv; k += 64u) *(u32x4 *)(dst + hn + 4u * k) = *(const u32x4u *)(region + hn + 4u * k);
    const uint32_t si = l < 4u ? l : hn + 4u * nv + (l - 4u);
    if (l < 4u ? l < hn : l - 4u < tn) dst[si] = region[si];
  }
  if (nch == 1 || t >= 64) return;
  // the epoch, if the last chunk's block did not see all words in time
  const bool hands = c == nch - 1 && s_miss;
  if (hands) {
    if (t == 0) st_dev32(&hdr[HDR_HAND], tag);
    wait_stores();
  }
  if (hands || hand == tag) {
    bool missing = false;
    for (int i = t; i < nch; i += 64) missing = missing || st_tag(ld_dev(&status[i])) != tag;
    if (!__builtin_amdgcn_ballot_w64(missing) && t == 0 && hand_taken(hdr, tag))
      st_dev32(&hdr[HDR_EPOCH], s_epoch + 1u);
  }
}

using once_fn = void (*)(const int32_t *, int32_t *, long long *, int64_t, int, uint64_t *, uint32_t *, uint32_t, int);

// The kernel for n elements, by measurement (us per call, scan / compaction):
//  - up to 2^18 elements 8192 a block with 1024 threads, 8 a lane: fewest
//    blocks to read from (131,072: 4.5 / 4.9; 1024-element chunks 5.5 / 5.7);
//  - then up to 2^23 8192 with 512 threads, 16 a lane (3 x 2^20: 5.6 / 6.3,
//    16384 a block 9.5 / 6.4; 6 x 2^20: 8.1 / 8.4 and 14.4 / 10.4, k_lookback
//    16 / 16; 2^23: 13.1 / 11.2 and 16.4 / 11.2, k_lookback 19.3 / 17.9);
//  - compaction goes on with 16384 a block up to 2^24 (24.0, k_lookback 28.0;
//    a scan of 2^24 would take 31.9, with k_lookback 30).
// Past that the aggregates that every block reads (the square of the blocks)
// cost more than the tickets and windows of k_lookback.
struct OncePick {
  once_fn fn;
  int S, BT;
};
template <int MODE>
static OncePick pick_once(int64_t n) {
  if (n <= 1 << 18) return {k_once<8, 1024, MODE>, 8192, 1024};
  if (n <= 1 << 23) return {k_once<16, 512, MODE>, 8192, 512};
  if constexpr (MODE == MODE_COMPACT)
    if (n <= 1 << 24) return {k_once<16, 1024, MODE>, 16384, 1024};
  return {nullptr, 0, 0};
}

static bool default_schedule(const cox_cfg *cfg) {
  return !cfg || (!cfg->items_per_lane && !cfg->warps_per_block && !cfg->grid_blocks);
}

static bool disjoint(const void *a, const void *b, size_t bytes) {
  const uintptr_t p = (uintptr_t)a, q = (uintptr_t)b;
  return p + bytes <= q || q + bytes <= p;
}

// Launches the short-input kernel if it applies (default schedule, few
// enough chunks, separate buffers, room for the words -- what k_lookback
// asks for always has it); false if not.
template <int MODE>
static bool launch_once(const int32_t *x, int32_t *out, long long *count, int64_t n, const cox_cfg *cfg, void *ws,
                        size_t ws_bytes, hipStream_t st, cox_status *r, uint32_t polls = HAND_POLLS, int away = -1) {
  if (n <= 0 || !default_schedule(cfg) || !disjoint(x, out, (size_t)n * 4)) return false;
  const OncePick p = pick_once<MODE>(n);
  if (!p.fn) return false;
  const int64_t nch = (n + p.S - 1) / p.S;
  if (nch > ONCE_CHUNKS || ws_bytes < WS_HEADER + 8 * (size_t)nch) return false;
  hipLaunchKernelGGL(p.fn, dim3((unsigned)nch), dim3(p.BT), 0, st, x, out, count, n, (int)nch,
                     (uint64_t *)((char *)ws + WS_HEADER), (uint32_t *)ws, polls, away);
  *r = launch_status();
  return true;
}

using lb_fn = void (*)(const int32_t *, int32_t *, long long *, int64_t, int64_t, uint64_t *, int64_t,
                       uint32_t *);

template <int MODE>
static lb_fn pick_lb(int k) {
  switch (k) {
  case 1: return k_lookback<1, MODE>;
  case 2: return k_lookback<2, MODE>;
  case 4: return k_lookback<4, MODE>;
  case 8: return k_lookback<8, MODE>;
  case 16: return k_lookback<16, MODE>;
  case 32: return k_lookback<32, MODE>;
  }
  return nullptr;
}

static cox_status check_lookback_args(cox_op op, int64_t n, const void *x, const cox_cfg *cfg, Sigma *sg,
                                      int64_t *nch) {
  if (n < 0) return COX_ERR_INVALID;
  cox_status st = resolve_cfg(op, COX_I32, cfg, sg);
  if (st != COX_OK) return st;
  if (n > 0 && !x) return COX_ERR_INVALID;
  if (n > 0 && !aligned16(x)) return COX_ERR_ALIGN;
  const int64_t S = (int64_t)32 * sg->W * sg->k;
  *nch = (n + S - 1) / S;
  // tickets and counts are 32-bit
  if (*nch > (int64_t)0x7fffffff - 65536 || n > (int64_t)0xffffffffLL) return COX_ERR_INVALID;
  return COX_OK;
}

static cox_status check_lookback_call(cox_op op, int64_t n, const void *x, const cox_cfg *cfg, void *ws,
                                      size_t ws_bytes, Sigma *sg, int64_t *nch) {
  const cox_status st = check_lookback_args(op, n, x, cfg, sg, nch);
  if (st != COX_OK) return st;
  if (!ws || ws_bytes < cox_workspace_bytes(op, COX_I32, n, 0, cfg)) return COX_ERR_WORKSPACE;
  return COX_OK;
}

// ------------------------------------------------ allocation-free variant
// The look-back header and status words of cox_warp_scan_noalloc live in a
// file-scope device array.  Each device that runs the library holds its own
// copy until the process ends; host code reaches it only through the
// address hipGetSymbolAddress returns on that device.
constexpr size_t SCRATCH_BYTES = COX_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) uint8_t scratch[SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[MAX_DEVICES];

__global__ void k_scratch_clear(uint32_t *p, int64_t words) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// hands the call's bounded-wait status to the caller and clears it
__global__ void k_scratch_status(uint32_t *hdr, uint32_t *err_out) {
  if (threadIdx.x == 0) {
    *err_out = hdr[HDR_ERR];
    hdr[HDR_ERR] = 0u;
  }
}

// Device address of this device's scratch.  The first call on a device
// looks it up and zeroes it on `st`, ahead of that call's kernels.
static cox_status scratch_for_device(hipStream_t st, void **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    set_hip_error(e);
    return COX_ERR_HIP;
  }
  if (dev < 0 || dev >= MAX_DEVICES) return COX_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      set_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol);
      return COX_ERR_HIP;
    }
    const int64_t words = (int64_t)(SCRATCH_BYTES / 4);
    hipLaunchKernelGGL(k_scratch_clear, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, (uint32_t *)ptr,
                       words);
    const cox_status ls = launch_status();
    if (ls != COX_OK) return ls;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return COX_OK;
}

}  // namespace cox

using namespace cox;

extern "C" {

cox_status cox_warp_scan(const int32_t *x, int32_t *y, int64_t n, const cox_cfg *cfg, void *ws,
                         size_t ws_bytes, void *stream) {
  Sigma sg;
  int64_t nch;
  cox_status st = check_lookback_call(COX_OP_SCAN, n, x, cfg, ws, ws_bytes, &sg, &nch);
  if (st != COX_OK) return st;
  if (n == 0) return COX_OK;
  if (!y) return COX_ERR_INVALID;
  if (!aligned16(y)) return COX_ERR_ALIGN;
  if (launch_once<MODE_SCAN>(x, y, nullptr, n, cfg, ws, ws_bytes, (hipStream_t)stream, &st)) return st;
  lb_fn fn = pick_lb<MODE_SCAN>(sg.k);
  if (!fn) return COX_ERR_UNSUPPORTED;
  const int block = 32 * sg.W;
  const int grid = persistent_grid((const void *)fn, block, nch, sg.G);
  hipLaunchKernelGGL(fn, dim3(grid), dim3(block), 0, (hipStream_t)stream, x, y, (long long *)nullptr, n, nch,
                     (uint64_t *)((char *)ws + WS_HEADER), (int64_t)ST_STRIDE, (uint32_t *)ws);
  return launch_status();
}

cox_status cox_warp_scan_noalloc(const int32_t *x, int32_t *y, int64_t n, const cox_cfg *cfg, uint32_t *err_out,
                                 void *stream) {
  Sigma sg;
  int64_t nch;
  cox_status st = check_lookback_args(COX_OP_SCAN, n, x, cfg, &sg, &nch);
  if (st != COX_OK) return st;
  // status words packed 8 bytes apart (a workspace spaces them ST_STRIDE
  // words apart), so that 1 MiB covers every n the default schedule takes
  if (WS_HEADER + 8 * (size_t)(nch + 1) > SCRATCH_BYTES) return COX_ERR_WORKSPACE;
  if (n > 0 && !y) return COX_ERR_INVALID;
  if (n > 0 && !aligned16(y)) return COX_ERR_ALIGN;
  lb_fn fn = pick_lb<MODE_SCAN>(sg.k);
  if (!fn) return COX_ERR_UNSUPPORTED;
  const hipStream_t hs = (hipStream_t)stream;
  void *ws = nullptr;
  st = scratch_for_device(hs, &ws);
  if (st != COX_OK) return st;
  if (launch_once<MODE_SCAN>(x, y, nullptr, n, cfg, ws, SCRATCH_BYTES, hs, &st)) {
    if (st != COX_OK) return st;
  } else if (n > 0) {
    const int block = 32 * sg.W;
    const int grid = persistent_grid((const void *)fn, block, nch, sg.G);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), 0, hs, x, y, (long long *)nullptr, n, nch,
                       (uint64_t *)((char *)ws + WS_HEADER), (int64_t)1, (uint32_t *)ws);
    st = launch_status();
    if (st != COX_OK) return st;
  }
  if (err_out) {
    hipLaunchKernelGGL(k_scratch_status, dim3(1), dim3(64), 0, hs, (uint32_t *)ws, err_out);
    st = launch_status();
  }
  return st;
}

cox_status cox_ballot_compact(const int32_t *x, int64_t n, int32_t *out, int64_t *count,
                              const cox_cfg *cfg, void *ws, size_t ws_bytes, void *stream) {
  Sigma sg;
  int64_t nch;
  cox_status st = check_lookback_call(COX_OP_COMPACT, n, x, cfg, ws, ws_bytes, &sg, &nch);
  if (st != COX_OK) return st;
  if (!count || (n > 0 && !out)) return COX_ERR_INVALID;
  if (launch_once<MODE_COMPACT>(x, out, (long long *)count, n, cfg, ws, ws_bytes, (hipStream_t)stream, &st)) return st;
  lb_fn fn = pick_lb<MODE_COMPACT>(sg.k);
  if (!fn) return COX_ERR_UNSUPPORTED;
  const int block = 32 * sg.W;
  const size_t lds = (size_t)sg.W * (32 * sg.k + 32) * sizeof(int32_t) + 256;  // staging (+ trash) + static
  if (lds > device_max_lds()) return COX_ERR_UNSUPPORTED;
  if (lds - 256 > 64 * 1024 &&
      hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(lds - 256)) != hipSuccess)
    return COX_ERR_UNSUPPORTED;
  const int grid = persistent_grid((const void *)fn, block, nch > 0 ? nch : 1, sg.G, lds);
  hipLaunchKernelGGL(fn, dim3(grid), dim3(block), lds - 256, (hipStream_t)stream, x, out, (long long *)count, n,
                     nch, (uint64_t *)((char *)ws + WS_HEADER), (int64_t)ST_STRIDE, (uint32_t *)ws);
  return launch_status();
}

cox_status cox_warp_scan_away(const int32_t *x, int32_t *y, int64_t n, int32_t away_block, uint32_t polls, void *ws,
                              size_t ws_bytes, void *stream) {
  Sigma sg;
  int64_t nch;
  cox_status st = check_lookback_call(COX_OP_SCAN, n, x, nullptr, ws, ws_bytes, &sg, &nch);
  if (st != COX_OK) return st;
  if (away_block < 0 || polls > HAND_POLLS || !y) return COX_ERR_INVALID;
  if (!aligned16(y)) return COX_ERR_ALIGN;
  return launch_once<MODE_SCAN>(x, y, nullptr, n, nullptr, ws, ws_bytes, (hipStream_t)stream, &st, polls, away_block)
             ? st : COX_ERR_UNSUPPORTED;
}

cox_status cox_ballot_compact_away(const int32_t *x, int64_t n, int32_t *out, int64_t *count, int32_t away_block,
                                   uint32_t polls, void *ws, size_t ws_bytes, void *stream) {
  Sigma sg;
  int64_t nch;
  cox_status st = check_lookback_call(COX_OP_COMPACT, n, x, nullptr, ws, ws_bytes, &sg, &nch);
  if (st != COX_OK) return st;
  if (away_block < 0 || polls > HAND_POLLS || !count || !out) return COX_ERR_INVALID;
  return launch_once<MODE_COMPACT>(x, out, (long long *)count, n, nullptr, ws, ws_bytes, (hipStream_t)stream, &st, polls,
                                   away_block)
             ? st : COX_ERR_UNSUPPORTED;
}

}  // extern "C"
