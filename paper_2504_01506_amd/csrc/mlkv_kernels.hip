// HIP kernels of libmlkv for gfx950 (MI355X): hash-index probe, row copy, row
// assignment of new keys, in-batch dedup by hash partition and LDS grouping (or
// a radix sort), and the fp64 sums with the row-wise Adagrad or SGD update.
//
// The kernels that move rows are templates over a row map. This file is
// compiled once for each map M with MLKV_MAP=M (that map's kernels and their
// launchers) and once without (the other kernels, and the choice of a map).
#include "mlkv_kernels.h"

#include <type_traits>

namespace mlkv {

// ===========================================================================
// Get: probe + gather (+ insert-on-miss), one key per lane.
// ===========================================================================
template <int VEC>
__device__ __forceinline__ typename VecT<VEC>::T load_vec(const float* p) {
  if constexpr (VEC == 4) {
    const Words4 v = *reinterpret_cast<const Words4*>(p);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
  } else {
    return *p;
  }
}

// As load_vec, for rows read once (kStream): around the caches.
template <int VEC, bool kStream>
__device__ __forceinline__ typename VecT<VEC>::T load_vec_once(const float* p) {
  if constexpr (VEC == 4 && kStream) {
    const Words4 v = __builtin_nontemporal_load(reinterpret_cast<const Words4*>(p));
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
  } else {
    return load_vec<VEC>(p);
  }
}

template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const typename VecT<VEC>::T& v) {
  if constexpr (VEC == 4) {
    *reinterpret_cast<Words4*>(p) =
        Words4{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
  } else {
    *p = v;
  }
}

template <int VEC>
__device__ __forceinline__ void store_vec_nt(float* p, const typename VecT<VEC>::T& v) {
  if constexpr (VEC == 4) {
    __builtin_nontemporal_store(
        Words4{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)},
        reinterpret_cast<Words4*>(p));
  } else {
    __builtin_nontemporal_store(v, p);
  }
}

template <int VEC>
__device__ __forceinline__ typename VecT<VEC>::T init_vec(uint64_t s0, int col) {
  typename VecT<VEC>::T v;
#pragma unroll
  for (int e = 0; e < VEC; ++e) VecT<VEC>::set(v, e, init_elem(s0, col + e));
  return v;
}

#ifndef MLKV_MAP
// Copies the rows of a wave's 64 positions (`first` on) into `out`, LPR lanes a
// row, every load of a lane in flight at once: row is the lane's own
// position's row, kPendingRow for a key new in the call (its row is generated
// from s0), kNoCopy for a position to leave alone. out's rows may start at any
// 4-byte boundary.
constexpr uint32_t kNoCopy = kPendingRow - 1;  // (no row's number: a capacity is at most 2^32 - 2)
template <int LPR, bool kStream>
__device__ __forceinline__ void copy_wave_rows(float* __restrict__ out, const RowStore& store, int64_t first,
                                               uint32_t row, uint64_t s0) {
  const int D = store.D, lane = threadIdx.x & 63;
  const int c = lane % LPR * 4;
  const bool on = c < D;
  const int col = c < D - 4 ? c : D - 4;  // the last lane of a row: its last four columns
  const int g = lane / LPR;
  float* const o = out + (size_t)first * (size_t)D + col;
  float4 v[LPR];
  uint32_t r[LPR];
#pragma unroll
  for (int u = 0; u < LPR; ++u) {
    r[u] = __shfl(row, u * (64 / LPR) + g, 64);
    if (on && r[u] < kNoCopy) v[u] = load_vec<4>(store.ptr(r[u]) + col);
  }
#pragma unroll
  for (int u = 0; u < LPR; ++u) {
    if (!on || r[u] >= kNoCopy) continue;
    float* p = o + (size_t)(u * (64 / LPR) + g) * (size_t)D;
    if constexpr (kStream) store_vec_nt<4>(p, v[u]);
    else store_vec<4>(p, v[u]);
  }
  if (__ballot(row == kPendingRow ? 1 : 0) == 0) return;
#pragma unroll 1
  for (int u = 0; u < LPR; ++u) {
    const int at = u * (64 / LPR) + g;
    const uint32_t x = __shfl(row, at, 64);
    const uint64_t s = __shfl((unsigned long long)s0, at, 64);
    if (on && x == kPendingRow) store_vec<4>(o + (size_t)at * (size_t)D, init_vec<4>(s, col));
  }
}

// Get, first kernel: each position's key is looked up (inserted if missing)
// and its row left in row[i] (kPendingRow: the key is new in the call). Rows of
// some widths and batch sizes are copied here too (LPR lanes a row, 1: by the
// key's own lane; VEC 0: none), the others by the second kernel, see
// copy_lanes. Bound by the latency of the dependent loads key -> bucket line (->
// row), so few registers and many waves.
// kPcIn: a position whose key equals pc_key[i] takes row[i] without
// probing (an instance of its own, so that other gets run unchanged)
template <int VEC, int LPR, bool kTrack, bool kPcIn, bool kStream>
__global__ __launch_bounds__(kGetTile) void k_get_probe(
    Bucket* __restrict__ idx, uint32_t nb_log2, const uint64_t* __restrict__ keys, int64_t n,
    float* __restrict__ out, const RowStore store, uint64_t seed, NewKey* __restrict__ newlist, uint32_t* __restrict__ tile_cnt, Ctrl* ctrl, uint64_t epoch,
    unsigned long long* __restrict__ clock, uint64_t cepoch, uint32_t bound, uint8_t* __restrict__ blocked,
    uint64_t* __restrict__ pc_key, uint32_t* __restrict__ rows, int tlen, const RangeLists rl,
    uint32_t nranges) {
  __shared__ uint32_t s_cnt;
  __shared__ uint64_t s_nkey[kGetTile];  // the tile's new keys and their slots
  __shared__ uint32_t s_nslot[kGetTile];
  __shared__ uint64_t s_cuts[kMaxRanges - 1];
  const int tid = threadIdx.x;
  // the block's tile: tlen (<= kGetTile) positions, so that every CU gets the
  // same number of positions
  const int64_t base = (int64_t)blockIdx.x * tlen;
  const int64_t end = min(n, base + tlen);
  const int64_t i = base + tid;
  if (tid == 0) s_cnt = 0;
  __syncthreads();
  uint64_t key = 0;
  Probe pr = {0, kPendingRow, P_NONE};
  bool recorded = false;  // the key and its row came from the row cache
  if (i < end) {
    key = keys[i];
    if (key == kEmptyKey) {
      pr.status = P_BAD;
      ctrl->bad_epoch = epoch;
    } else {
      if constexpr (kPcIn) {
        const uint64_t ck = pc_key[i];
        const uint32_t cr = rows[i];
        if (ck == key) {
          pr = {0u, cr, P_HIT};
          recorded = true;
        }
      }
      if (!recorded) {
        pr = probe_key(idx, nb_log2, key, true);
        if (pr.status == P_OVERFLOW) ctrl->overflow_epoch = epoch;
      }
    }
  }
  if (pr.status == P_NEW_MINE) {
    const uint32_t j = atomicAdd(&s_cnt, 1u);
    s_nkey[j] = key;
    s_nslot[j] = pr.slot;
    ctrl->new_epoch = epoch;
  }
  // a key present before the call, with its row, for a put of the same
  // batch: a key's row never changes once assigned, so the pair stays valid
  if (i < end && !recorded) {
    if (pc_key != nullptr) pc_key[i] = pr.status == P_HIT ? key : kEmptyKey;
    rows[i] = pr.row;
  }
  bool served = i < end;
  if (kTrack && i < end) {
    // bounded staleness: a present key is served while its count before the
    // call is at most the bound. Serving it stamps the word with the call's
    // epoch and that count plus one. Nothing else writes the word during the
    // call, so a position reads either the word from before the call or the
    // stamp; every position that reads the former stores the same stamp, and
    // a plain store suffices (hot keys would serialise atomics). The count
    // thus rises once per call, however often the key occurs.
    bool blk = false;
    if (pr.status == P_HIT) {
      unsigned long long* cw = clock + pr.row;
      const unsigned long long w = *cw;
      if ((w >> kClockBits) != cepoch) {
        if ((w & kClockCount) > bound) blk = true;
        else *cw = (cepoch << kClockBits) | ((w & kClockCount) + 1);
      }
    }
    blocked[i] = blk ? 1 : 0;
    served = !blk;
  }
  if constexpr (LPR > 1) {
    copy_wave_rows<LPR, kStream>(out, store, base + (tid & ~63),
                                 !served ? kNoCopy : pr.status == P_HIT ? pr.row : kPendingRow,
                                 splitmix_mix(key ^ seed));
  } else if constexpr (VEC > 0) {
    if (served)  // a row is one access
      store_vec<VEC>(out + (size_t)i * VEC, pr.status == P_HIT ? load_vec<VEC>(store.ptr(pr.row))
                                                               : init_vec<VEC>(splitmix_mix(key ^ seed), 0));
  }
  __syncthreads();
  // the tile's list of new keys, in ascending key order (each at its rank)
  const uint32_t c = s_cnt;
  if ((uint32_t)tid < c) {
    const uint64_t k = s_nkey[tid];
    uint32_t r = 0;
    for (uint32_t e = 0; e < c; ++e) r += s_nkey[e] < k ? 1u : 0u;
    newlist[base + r] = NewKey{k, s_nslot[tid], 0u};
  }
  if (tid == 0) tile_cnt[blockIdx.x] = c;
  // the same keys filed by key range, when the cut points are for this
  // call's number of ranges (block-uniform: c and the cut count)
  if (rl.list != nullptr && c > 0 && *rl.cuts_g == nranges) {
    for (uint32_t e = tid; e + 1 < nranges; e += kGetTile) s_cuts[e] = rl.cuts[e];
    __syncthreads();
    if ((uint32_t)tid < c) {
      const uint64_t k = s_nkey[tid];
      uint32_t q = 0;  // range q holds [cut q-1, cut q): q = cut points <= k
      for (uint32_t step = kMaxRanges / 2; step >= 1; step >>= 1)
        if (q + step < nranges && s_cuts[q + step - 1] <= k) q += step;
      const uint32_t at = atomicAdd(&rl.cnt[q], 1u);
      if (at < rl.cap) rl.list[(size_t)q * rl.cap + at] = NewKey{k, s_nslot[tid], 0u};
      else ctrl->rl_overflow_epoch = epoch;
    }
    if (tid == 0) ctrl->rl_epoch = epoch;
  }
}

#endif  // MLKV_MAP

// ===========================================================================
// Streaming every new key of the call through LDS (used to rank new keys).
// ===========================================================================
constexpr int kChunk = 2048;

// Calls body(s_chunk, cnt) for consecutive chunks of this call's new keys;
// the block's NT threads must all call it. s_pref: NT+1 words.
template <int NT, class Body>
__device__ __forceinline__ void for_each_new_key_chunk(const NewKey* __restrict__ newlist,
                                       const uint32_t* __restrict__ tile_cnt, int ntiles,
                                       int tile_size, uint32_t* s_pref, uint32_t* s_w,
                                       uint64_t* s_chunk, Body body) {
  constexpr int PER = kChunk / NT;
  for (int t0 = 0; t0 < ntiles; t0 += NT) {
    const int nt = min(NT, ntiles - t0);
    const uint32_t c = (int)threadIdx.x < nt ? tile_cnt[t0 + threadIdx.x] : 0u;
    uint32_t total;
    const uint32_t pre = block_exclusive_scan<NT>(c, s_w, &total);
    s_pref[threadIdx.x] = pre;
    __syncthreads();
    for (uint32_t k0 = 0; k0 < total; k0 += kChunk) {
      const uint32_t cnt = min((uint32_t)kChunk, total - k0);
      uint64_t v[PER];
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const uint32_t k = threadIdx.x + e * NT;
        v[e] = 0;
        if (k < cnt) {
          const uint32_t gk = k0 + k;
          int lo = 0, hi = nt - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_pref[mid] <= gk) lo = mid;
            else hi = mid - 1;
          }
          v[e] = newlist[(size_t)(t0 + lo) * tile_size + (gk - s_pref[lo])].key;
        }
      }
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const uint32_t k = threadIdx.x + e * NT;
        if (k < cnt) s_chunk[k] = v[e];
      }
      __syncthreads();
      body(s_chunk, cnt);
      __syncthreads();
    }
    __syncthreads();
  }
}

// Sum of the per-tile new-key counts, i.e. the number M of distinct keys the
// call inserts.
template <int NT>
__device__ __forceinline__ uint64_t count_new_keys(const uint32_t* __restrict__ tile_cnt, int ntiles,
                                                   unsigned long long* s_w64) {
  uint64_t m = 0;
  for (int t = threadIdx.x; t < ntiles; t += NT) m += tile_cnt[t];
  return block_sum_u64<NT>(m, s_w64);
}

// Decides whether the call fails, and publishes the size for the next call.
__device__ __forceinline__ int call_verdict(Ctrl* ctrl, uint64_t epoch, uint64_t size0, uint64_t M,
                                            int64_t capacity, uint64_t bad_epoch, uint64_t overflow_epoch,
                                            uint64_t absent_epoch = 0) {
  int err = 0;
  if (bad_epoch == epoch) err = -1;                                           // MLKV_EINVAL
  else if (absent_epoch == epoch) err = kErrAbsent;                          // MLKV_EINVAL, its own message
  else if (overflow_epoch == epoch || size0 + M > (uint64_t)capacity) err = -2;  // MLKV_EFULL
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctrl->size[(epoch + 1) & 1] = err ? size0 : size0 + M;
    if (err) atomicCAS(&ctrl->latched, 0, err);
  }
  return err;
}

// ===========================================================================
// Get, second kernel: the rows of the call's positions are copied out (if the
// first has not), then its first blocks assign rows to the call's new keys
// (ascending key order), write their initial rows and zero accumulators; or
// roll the call back. The copy reads only rows that were present before the
// call and generates those of new keys from their seed, so neither part waits
// for the other.
// ===========================================================================
constexpr int kAssignThreads = 512;
constexpr int kAssignMine = 2048;  // list entries a block ranks directly at a time
// With few new keys each block ranks its tiles' keys against all of them,
// streamed through LDS once per NT tiles of the call; with more, each block
// ranks the keys of a key range, which costs a put about 50 us to begin with
// (a sorted sample, a search of every tile's list). A put of 213k keys, 256
// tiles, that inserts 2,129 of them takes 47 us directly and 84 by range,
// with 10,649 64 and 89, with 31,948 111 and 102. A get's blocks take their
// range from range lists where a call of as many ranges came before, which
// beats the direct ranking sooner (213k keys, 2 times 512 tiles, 425 new: 33
// us directly, 28 by range; 4096 keys, 614 new: 27 directly, 49 with each
// tile's keys compared with all others, the earlier direct ranking). Limits
// in new keys x rounds of NT tiles.
template <int NT>
constexpr uint64_t kAssignDirectWork = NT >= 1024 ? 16384 : 768;
// Sample of the new keys that splits the key space among the blocks: the more
// of them, the fewer ranges outgrow kRangeCap, which are ranked in chunks. A
// put's blocks of 1024 threads sort 4096 as fast as a get's of 512 sort 2048 (a
// million rows loaded: 2.8 ms with 2048, 1.95 with 4096).
template <int NT>
constexpr int kRangeSamples = NT >= 1024 ? 4096 : 2048;
constexpr int kRangeCap = 3072;      // keys of a block's key range ranked in LDS at once

// Each tile's list of new keys is sorted (ascending key). For the key range
// [lo, hi) this returns the thread's share of the number of new keys below lo
// and calls emit(offset, n) for each tile run of the range's keys (offset
// into the lists, n > 0 entries). Threads take kSearchTiles tiles at a time
// and search both bounds in all of them together (branch-free binary search,
// each step one load per bound and tile in flight).
constexpr int kSearchTiles = 4;
template <int NT, int TM, class Emit>
__device__ __forceinline__ uint64_t search_tile_lists(const NewKey* __restrict__ newlist,
                                                      const uint32_t* __restrict__ tile_cnt, int ntiles,
                                                      int tile_size, uint64_t lo, uint64_t hi, Emit emit) {
  uint64_t below = 0;
  for (int t0 = threadIdx.x; t0 < ntiles; t0 += NT * kSearchTiles) {
    uint32_t c[kSearchTiles], a[kSearchTiles], b[kSearchTiles];
#pragma unroll
    for (int u = 0; u < kSearchTiles; ++u) {
      const int t = t0 + u * NT;
      c[u] = t < ntiles ? tile_cnt[t] : 0u;
      a[u] = 0;  // keys below lo
      b[u] = 0;  // keys below hi
    }
    // a tile holds at most TM (a power of two) keys
    for (uint32_t step = (uint32_t)TM; step >= 1; step >>= 1) {
#pragma unroll
      for (int u = 0; u < kSearchTiles; ++u) {
        const NewKey* l = newlist + (size_t)(t0 + u * NT) * tile_size;
        if (a[u] + step <= c[u] && l[a[u] + step - 1].key < lo) a[u] += step;
        if (b[u] + step <= c[u] && l[b[u] + step - 1].key < hi) b[u] += step;
      }
    }
#pragma unroll
    for (int u = 0; u < kSearchTiles; ++u) {
      below += a[u];
      if (b[u] > a[u]) emit((uint32_t)(t0 + u * NT) * (uint32_t)tile_size + a[u], b[u] - a[u]);
    }
  }
  return below;
}

// Ascending bitonic sort of NT * PT keys, thread t holding the elements PT t
// .. PT t + PT - 1 in v. Compare-exchanges whose partner lies in the same
// thread run in registers; the others exchange through LDS, alternating
// between buf0 and buf1 (NT * PT keys each), so one barrier per such stage
// suffices.
template <int NT, int PT>
__device__ __forceinline__ void sort_keys(uint64_t (&v)[PT], uint64_t* buf0, uint64_t* buf1) {
  static_assert(PT == 2 || PT == 4, "the stages within a thread");
  constexpr uint32_t N = (uint32_t)NT * PT;
  const uint32_t t = threadIdx.x;
  auto reg_stage = [&](auto J, uint32_t k) {
    constexpr uint32_t j = decltype(J)::value;
#pragma unroll
    for (uint32_t r = 0; r < PT; ++r) {
      if ((r & j) == 0) {
        const bool asc = ((t * PT + r) & k) == 0;
        const uint64_t a = v[r], b = v[r + j];
        if ((a > b) == asc) {
          v[r] = b;
          v[r + j] = a;
        }
      }
    }
  };
  bool second = false;
  for (uint32_t k = 2; k <= N; k <<= 1) {
    for (uint32_t j = k >> 1; j >= PT; j >>= 1) {
      uint64_t* b = second ? buf1 : buf0;
      second = !second;
#pragma unroll
      for (uint32_t r = 0; r < PT; ++r) b[r * NT + t] = v[r];
      lds_barrier();
      const uint32_t pt = t ^ (j / PT);
#pragma unroll
      for (uint32_t r = 0; r < PT; ++r) {
        const uint32_t i = t * PT + r;
        const uint64_t p = b[r * NT + pt];
        const bool asc = (i & k) == 0, low = (i & j) == 0;
        v[r] = (asc == low) ? (v[r] < p ? v[r] : p) : (v[r] > p ? v[r] : p);
      }
    }
    if constexpr (PT >= 4) {
      if (k >= 4) reg_stage(std::integral_constant<uint32_t, 2>{}, k);
    }
    reg_stage(std::integral_constant<uint32_t, 1>{}, k);
  }
}

// Staleness word of a row that a get inserts: served once by this call.
__device__ __forceinline__ unsigned long long new_row_clock(uint64_t cepoch) {
  return ((unsigned long long)cepoch << kClockBits) | 1ull;
}

// A failed get call gives back the counts it raised: every row stamped with
// its epoch loses one, and the stamp (needed only within the call) is cleared.
__device__ __forceinline__ void rollback_clocks(unsigned long long* __restrict__ clock, uint64_t nrows,
                                                uint64_t cepoch, uint32_t blocks) {
  const uint64_t stride = (uint64_t)blocks * blockDim.x;
  for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nrows; r += stride) {
    const unsigned long long w = clock[r];
    if ((w >> kClockBits) == cepoch) clock[r] = (w & kClockCount) - 1;
  }
}

// Initial rows of new keys ks[j] (j < m) at rows base + rk[j]: a wave per
// row, its lanes along the row, kInitRows rows of a wave at a time so that
// each lane has that many independent hash chains in flight (the 64-bit
// multiplies of one chain are serial).
constexpr int kInitRows = 4;
template <int NT, class KP, class RP>
__device__ __forceinline__ void write_init_rows(const KP ks, const RP rk, uint32_t m, uint64_t base,
                                                const RowStore& store, int D, uint64_t seed) {
  constexpr uint32_t NW = NT / 64;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t j0 = wave; j0 < m; j0 += NW * kInitRows) {
    float* w[kInitRows];
    uint64_t s0[kInitRows];
#pragma unroll
    for (int r = 0; r < kInitRows; ++r) {
      const uint32_t j = j0 + (uint32_t)r * NW;
      w[r] = nullptr;
      s0[r] = 0;
      if (j < m) {
        w[r] = store.wptr((uint32_t)(base + rk[j]));
        s0[r] = splitmix_mix(ks[j] ^ seed);
      }
    }
    for (int col = (int)lane; col < D; col += 64) {
#pragma unroll
      for (int r = 0; r < kInitRows; ++r)
        if (w[r] != nullptr) w[r][col] = init_elem(s0[r], col);
    }
  }
}

// The rows of an upsert's new keys, as write_init_rows: row base + rk[j] takes
// the value row of position ks[j].
template <int NT, class KP, class RP>
__device__ __forceinline__ void write_value_rows(const KP ks, const RP rk, uint32_t m, uint64_t base,
                                                 const RowStore& store, int D, const float* __restrict__ values) {
  constexpr uint32_t NW = NT / 64;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t j0 = wave; j0 < m; j0 += NW * kInitRows) {
    float* w[kInitRows];
    const float* v[kInitRows];
#pragma unroll
    for (int r = 0; r < kInitRows; ++r) {
      const uint32_t j = j0 + (uint32_t)r * NW;
      w[r] = nullptr;
      v[r] = nullptr;
      if (j < m) {
        w[r] = store.wptr((uint32_t)(base + rk[j]));
        v[r] = values + (size_t)ks[j] * (size_t)D;
      }
    }
    for (int col = (int)lane; col < D; col += 64) {
      float x[kInitRows];
#pragma unroll
      for (int r = 0; r < kInitRows; ++r)
        if (w[r] != nullptr) x[r] = v[r][col];
#pragma unroll
      for (int r = 0; r < kInitRows; ++r)
        if (w[r] != nullptr) w[r][col] = x[r];
    }
  }
}

// The last position of an upsert's new key, from the spare word of its index
// slot (see k_put_probe), which is put back.
__device__ __forceinline__ uint64_t take_position(Bucket* __restrict__ idx, uint32_t slot) {
  uint32_t* w = &idx[slot / kSlots].aux[slot % kSlots];
  const uint32_t pos = ~*w;
  *w = 0xFFFFFFFFu;
  return pos;
}

// Rows for the new keys ks[0, m) (index slots sl[...]) whose ranks among all
// new keys of the call are base + rk[...]: index row ids, zero accumulators,
// initial rows, or an upsert's value rows (written along rows).
template <int NT, class KP, class SP, class RP>
__device__ __forceinline__ void write_new_rows(KP ks, const SP sl, const RP rk, uint32_t m, uint64_t base,
                                               Bucket* __restrict__ idx, const RowStore& store,
                                               float* __restrict__ state, int D, uint64_t seed,
                                               unsigned long long* __restrict__ clock, uint64_t cepoch,
                                               const float* __restrict__ values) {
  for (uint32_t j = threadIdx.x; j < m; j += NT) {
    const uint32_t slot = sl[j];
    const uint32_t row = (uint32_t)(base + rk[j]);
    idx[slot / kSlots].row[slot % kSlots] = row;
    state[row] = 0.0f;
    if (clock != nullptr) clock[row] = new_row_clock(cepoch);
    if (values != nullptr) ks[j] = take_position(idx, slot);
  }
  if (values != nullptr) {
    __syncthreads();
    write_value_rows<NT>(ks, rk, m, base, store, D, values);
  } else {
    write_init_rows<NT>(ks, rk, m, base, store, D, seed);
  }
}

#ifndef MLKV_MAP
// Position, in the tiles' lists laid end to end, of sample k of S out of M
// new keys: a hashed place in the k-th of S equal shares. The lists are
// sorted, so evenly spaced positions take the same few quantiles of every
// tile's list when the tiles hold equally many new keys (a table being
// loaded); one range then holds nearly half of the keys.
__device__ __forceinline__ uint64_t sample_at(uint64_t k, uint64_t M, uint32_t S) {
  const uint64_t lo = k * M / S, width = (k + 1) * M / S - lo;
  uint32_t h = (uint32_t)k * 0x9E3779B1u;
  h = (h ^ (h >> 15)) * 0x85EBCA77u;
  h ^= h >> 13;
  return lo + (((uint64_t)h * width) >> 32);
}

// LDS of a block that assigns rows (NT threads).
template <int NT>
struct AssignLds {
  // 48 or 64 KiB; the two ranking methods lay it out differently
  static constexpr int kBuf = std::max(kChunk + 2 * kAssignMine, std::max(2 * kRangeSamples<NT>, kRangeCap * 14 / 8));
  uint64_t buf[kBuf];
  unsigned long long w64[NT / 64];
  uint64_t cut[2];
  __align__(16) uint32_t pref[NT + 1];
  uint32_t w[NT / 64];
  uint32_t nc;
};

// Rows for the call's M new keys, from size0 on in ascending key order (or,
// with `err`, their index entries emptied again), by the first a.blocks
// blocks of a kernel of NT threads. A probe tile lists at most TM new keys.
template <int NT, int TM>
__device__ __forceinline__ void assign_new(const AssignArgs& a, const RowStore& store, uint64_t seed, uint64_t size0,
                                           uint64_t M, int err, AssignLds<NT>& lds) {
  Bucket* __restrict__ const idx = a.idx;
  const NewKey* __restrict__ const newlist = a.newlist;
  const uint32_t* __restrict__ const tile_cnt = a.tile_cnt;
  const int ntiles = a.ntiles, tile_size = a.tile_size, D = store.D;
  float* __restrict__ const state = a.state;
  Ctrl* const ctrl = a.ctrl;
  const uint64_t epoch = a.epoch, cepoch = a.cepoch;
  uint64_t* __restrict__ const xkey = a.xkey;
  uint32_t* __restrict__ const xslot = a.xslot;
  unsigned long long* __restrict__ const clock = a.clock;
  const RangeLists& rl = a.rl;
  unsigned long long* const s_w64 = lds.w64;
  uint32_t* const s_w = lds.w;
  uint32_t* const s_pref = lds.pref;
  uint32_t& s_nc = lds.nc;
  uint64_t* const s_cut = lds.cut;
  uint64_t* const s_buf = lds.buf;
  constexpr int kSortPT = kRangeSamples<NT> / NT;
  static_assert(kRangeCap * 14 <= (int)sizeof(lds.buf) && kRangeSamples<NT> * 16 <= (int)sizeof(lds.buf), "LDS");
  static_assert(kRangeSamples<NT> == NT * kSortPT && kRangeCap <= 65536 && kRangeCap % NT == 0, "sample and range sizes");
  if (M == 0) return;

  if (err) {  // undo this call's insertions: the index returns to its state before the call
    for (int t = blockIdx.x; t < ntiles; t += a.blocks) {
      const uint32_t c = tile_cnt[t];
      for (uint32_t j = threadIdx.x; j < c; j += NT) {
        const uint32_t slot = newlist[(size_t)t * tile_size + j].slot;
        idx[slot / kSlots].key[slot % kSlots] = kEmptyKey;
        idx[slot / kSlots].aux[slot % kSlots] = 0xFFFFFFFFu;
      }
    }
    return;
  }

  // the probe kernel filed the new keys by range (RangeLists): ranking them
  // by range then costs little for any number of them
  const bool listed = rl.list != nullptr && ctrl->rl_epoch == epoch && ctrl->rl_overflow_epoch != epoch;
  if (listed || M * (uint64_t)((ntiles + NT - 1) / NT) > kAssignDirectWork<NT>) {
    // ---- many new keys: key ranges. Block g ranks the new keys of the g-th
    // key range among themselves, after the count of new keys below the
    // range. The probe kernel has filed the keys by range when cut points for
    // this many ranges were left (RangeLists): the range's keys are its list,
    // the keys below it the lists before. Otherwise every block takes the
    // same sample of the new keys (sample_at) and the same cut
    // points from it, which give block g the keys in [lo, hi); a binary
    // search of both bounds in every tile's sorted list of new keys counts
    // the keys below lo and finds the block's own. No block waits for another.
    const uint32_t g = blockIdx.x, G = a.blocks;
    uint64_t* s_key = s_buf;                                                 // [kRangeCap]
    uint32_t* s_sr = reinterpret_cast<uint32_t*>(s_buf + kRangeCap);        // [kRangeCap]
    uint16_t* s_ord = reinterpret_cast<uint16_t*>(s_sr + kRangeCap);        // [kRangeCap]
    const NewKey* my_list = listed ? rl.list + (size_t)g * rl.cap : nullptr;
    uint64_t below = 0, lo = 0, hi = kEmptyKey;
    uint32_t c = 0;
    if (listed) {
      uint64_t mine = 0;
      for (uint32_t r = threadIdx.x; r < g; r += NT) mine += rl.cnt[r];
      below = block_sum_u64<NT>(mine, s_w64);
      c = rl.cnt[g];
      if (c <= (uint32_t)kRangeCap)
        for (uint32_t j = threadIdx.x; j < c; j += NT) {
          const NewKey nk = my_list[j];
          s_key[j] = nk.key;
          s_sr[j] = nk.slot;
        }
      __syncthreads();
    } else {
      constexpr uint32_t S = kRangeSamples<NT>;
      uint32_t* s_sat = reinterpret_cast<uint32_t*>(s_buf + S);     // [S] offsets of the samples in the lists
      {
        const int tpt = (ntiles + NT - 1) / NT;  // consecutive tiles per thread
        const int tb = min(ntiles, (int)threadIdx.x * tpt), te = min(ntiles, tb + tpt);
        uint32_t mine = 0;
        for (int t = tb; t < te; ++t) mine += tile_cnt[t];
        uint32_t tot;
        uint64_t pre = block_exclusive_scan<NT>(mine, s_w, &tot);
        uint64_t k = pre * S / M;  // the sample of pre's share
        for (int t = tb; t < te && k < S; ++t) {
          const uint32_t c = tile_cnt[t];
          for (; k < S; ++k) {
            const uint64_t gk = sample_at(k, M, S);
            if (gk < pre) continue;
            if (gk >= pre + c) break;
            s_sat[k] = (uint32_t)t * (uint32_t)tile_size + (uint32_t)(gk - pre);
          }
          pre += c;
        }
      }
      __syncthreads();
      uint64_t v[kSortPT];
#pragma unroll
      for (uint32_t u = 0; u < kSortPT; ++u) v[u] = newlist[s_sat[threadIdx.x + u * NT]].key;
      // the cut points: the samples of rank g S / G and (g + 1) S / G of the
      // sorted sample (with fewer new keys than samples a key is sampled more
      // than once, and equal cut points give an empty range): at 512 ranges
      // eight sample gaps a range in a put, four in a get. The largest range is
      // two to three times the mean: of a put's ranges 41 to 46 of 512 hold more
      // than kRangeCap keys at 2^20 new ones, nearly all from 1.57M on
      sort_keys<NT, kSortPT>(v, s_buf, s_buf + S);
      {
        const uint32_t r1 = (uint32_t)((uint64_t)g * S / G), r2 = (uint32_t)((uint64_t)(g + 1) * S / G);
#pragma unroll
        for (uint32_t u = 0; u < kSortPT; ++u) {
          if (threadIdx.x * kSortPT + u == r1) s_cut[0] = v[u];
          if (threadIdx.x * kSortPT + u == r2) s_cut[1] = v[u];
        }
        if (threadIdx.x == 0) s_nc = 0;
      }
      __syncthreads();
      lo = g == 0 ? 0ull : s_cut[0];
      hi = g + 1 == G ? kEmptyKey : s_cut[1];
      // keys in [lo, hi) first go to LDS: key, slot (later the rank), and
      // their order by local sub-range
      below = search_tile_lists<NT, TM>(newlist, tile_cnt, ntiles, tile_size, lo, hi, [&](uint32_t off, uint32_t cnt) {
        const uint32_t at = atomicAdd(&s_nc, cnt);
        for (uint32_t e = 0; e < cnt && at + e < (uint32_t)kRangeCap; ++e) {
          s_key[at + e] = newlist[off + e].key;
          s_sr[at + e] = off + e;  // slot and position are read later
        }
      });
      below = block_sum_u64<NT>(below, s_w64);  // its barriers also publish s_nc and the gathered keys
      c = s_nc;
      if (c <= (uint32_t)kRangeCap) {
        // the slot of each gathered key, from its list entry
        for (uint32_t j = threadIdx.x; j < c; j += NT) s_sr[j] = newlist[s_sr[j]].slot;
      }
      __syncthreads();
    }
    const uint64_t base = size0 + below;
    // cut points for the next call: cut j is the key of global rank
    // floor(j M / G), so the keys of rank R give cuts j in [ceil(R G / M),
    // ceil((R + 1) G / M))
    auto leave_cuts = [&](uint64_t key, uint64_t R) {
      if (rl.list == nullptr) return;
      const uint64_t jb = (R * G + M - 1) / M, je = ((R + 1) * G + M - 1) / M;
      for (uint64_t j = jb < 1 ? 1 : jb; j < je && j < G; ++j) rl.cuts[j - 1] = key;
    };
    if (c <= (uint32_t)kRangeCap) {
      // rank among the range's keys, through kSub local sub-ranges cut at a
      // sample of the gathered keys: sub-range counts and their prefix, the
      // keys listed by sub-range, then each key ranked inside its sub-range
      constexpr int kSub = 32;
      uint64_t* s_lc = reinterpret_cast<uint64_t*>(s_pref);  // [kSub - 1] local cut points (s_pref is free)
      uint32_t* s_sc = s_pref + 2 * kSub;                      // [kSub + 1] counts, then prefix, then cursors
      const uint32_t nl = c < (uint32_t)(kSub * 4) ? 0u : (uint32_t)kSub - 1;  // small ranges: one sub-range
      if (threadIdx.x < nl) {  // local cut l: the rank-l key of an evenly spaced sample of the gathered keys
        const uint64_t x = s_key[(uint64_t)(threadIdx.x + 1) * c / kSub];
        uint32_t rr = 0;
        for (uint32_t l = 0; l < nl; ++l) rr += s_key[(uint64_t)(l + 1) * c / kSub] < x ? 1u : 0u;
        s_lc[rr] = x;
      }
      if (threadIdx.x <= (uint32_t)kSub) s_sc[threadIdx.x] = 0;
      __syncthreads();
      uint32_t sub[kRangeCap / NT];
#pragma unroll
      for (int u = 0; u < kRangeCap / NT; ++u) {
        const uint32_t j = threadIdx.x + u * NT;
        sub[u] = 0;
        if (j < c) {
          const uint64_t key = s_key[j];
          uint32_t l = 0;  // sub-range l holds keys in [cut l-1, cut l): l = cuts <= key
          if (nl) {
#pragma unroll
            for (uint32_t step = kSub / 2; step >= 1; step >>= 1)
              if (l + step <= nl && s_lc[l + step - 1] <= key) l += step;
          }
          sub[u] = l;
          atomicAdd(&s_sc[l], 1u);
        }
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (int l = 0; l <= kSub; ++l) {
          const uint32_t x = s_sc[l];
          s_sc[l] = acc;
          acc += x;
        }
      }
      __syncthreads();
      uint32_t sbeg[kRangeCap / NT];
#pragma unroll
      for (int u = 0; u < kRangeCap / NT; ++u) {
        const uint32_t j = threadIdx.x + u * NT;
        sbeg[u] = 0;
        if (j < c) sbeg[u] = s_sc[sub[u]];
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kRangeCap / NT; ++u) {
        const uint32_t j = threadIdx.x + u * NT;
        if (j < c) s_ord[atomicAdd(&s_sc[sub[u]], 1u)] = (uint16_t)j;
      }
      __syncthreads();
      // after the cursors ran, s_sc[l] is the end of sub-range l
      uint32_t rk[kRangeCap / NT];
#pragma unroll
      for (int u = 0; u < kRangeCap / NT; ++u) {
        const uint32_t j = threadIdx.x + u * NT;
        rk[u] = 0;
        if (j < c) {
          const uint64_t key = s_key[j];
          const uint32_t b0 = sbeg[u], e0 = s_sc[sub[u]];
          uint32_t r = b0, i = b0;
          for (; i + 4 <= e0; i += 4) {
            const uint32_t o0 = s_ord[i], o1 = s_ord[i + 1], o2 = s_ord[i + 2], o3 = s_ord[i + 3];
            r += (s_key[o0] < key ? 1u : 0u) + (s_key[o1] < key ? 1u : 0u) + (s_key[o2] < key ? 1u : 0u) +
                 (s_key[o3] < key ? 1u : 0u);
          }
          for (; i < e0; ++i) r += s_key[s_ord[i]] < key ? 1u : 0u;
          rk[u] = r;
          const uint32_t slot = s_sr[j];
          idx[slot / kSlots].row[slot % kSlots] = (uint32_t)(base + r);
          state[base + r] = 0.0f;
          if (clock != nullptr) clock[base + r] = new_row_clock(cepoch);
          leave_cuts(key, below + r);
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kRangeCap / NT; ++u) {
        const uint32_t j = threadIdx.x + u * NT;
        if (j < c) {
          if (a.values != nullptr) s_key[j] = take_position(idx, s_sr[j]);
          s_sr[j] = rk[u];
        }
      }
      __syncthreads();
      if (a.values != nullptr) write_value_rows<NT>(s_key, s_sr, c, base, store, D, a.values);
      else write_init_rows<NT>(s_key, s_sr, c, base, store, D, seed);
    } else {
      // more keys in the range than LDS holds: gather them in global scratch
      // at [below, below + c), which no other block's range overlaps, then
      // rank them in chunks streamed through LDS
      __syncthreads();
      if (threadIdx.x == 0) s_nc = 0;
      __syncthreads();
      if (listed) {
        for (uint32_t j = threadIdx.x; j < c; j += NT) {
          const NewKey nk = my_list[j];
          xkey[below + j] = nk.key;
          xslot[below + j] = nk.slot;
        }
      } else {
        search_tile_lists<NT, TM>(newlist, tile_cnt, ntiles, tile_size, lo, hi, [&](uint32_t off, uint32_t cnt) {
          const uint32_t at = atomicAdd(&s_nc, cnt);
          for (uint32_t e = 0; e < cnt; ++e) {
            const NewKey nk = newlist[off + e];
            xkey[below + at + e] = nk.key;
            xslot[below + at + e] = nk.slot;
          }
        });
      }
      __syncthreads();
      const uint64_t* rk_key = xkey + below;
      const uint32_t* rk_slot = xslot + below;
      uint64_t* s_cmp = s_buf;                                                    // [kChunk]
      uint64_t* s_mk = s_buf + kChunk;                                            // [kAssignMine]
      uint32_t* s_ms = reinterpret_cast<uint32_t*>(s_buf + kChunk + kAssignMine);  // [kAssignMine]
      uint32_t* s_mr = s_ms + kAssignMine;                                        // [kAssignMine]
      constexpr int PER = kAssignMine / NT;
      for (uint32_t j0 = 0; j0 < c; j0 += kAssignMine) {
        const uint32_t m = min((uint32_t)kAssignMine, c - j0);
        uint64_t mk[PER];
        uint32_t r[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const uint32_t j = threadIdx.x + u * NT;
          mk[u] = j < m ? rk_key[j0 + j] : 0ull;
          r[u] = 0;
        }
        for (uint32_t e0 = 0; e0 < c; e0 += kChunk) {
          const uint32_t cnt = min((uint32_t)kChunk, c - e0);
          for (uint32_t e = threadIdx.x; e < cnt; e += NT) s_cmp[e] = rk_key[e0 + e];
          __syncthreads();
          for (uint32_t e = 0; e < cnt; ++e) {
            const uint64_t v = s_cmp[e];
#pragma unroll
            for (int u = 0; u < PER; ++u) r[u] += v < mk[u] ? 1u : 0u;
          }
          __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const uint32_t j = threadIdx.x + u * NT;
          if (j < m) {
            s_mk[j] = mk[u];
            s_ms[j] = rk_slot[j0 + j];
            s_mr[j] = r[u];
            leave_cuts(mk[u], below + r[u]);
          }
        }
        __syncthreads();
        write_new_rows<NT>(s_mk, s_ms, s_mr, m, base, idx, store, state, D, seed, clock, cepoch, a.values);
        __syncthreads();
      }
    }
    if (rl.list != nullptr && g == 0 && threadIdx.x == 0) *rl.cuts_g = G;
    return;
  }

  // ---- few new keys: this block owns those of the tiles t = blockIdx.x (mod
  // a.blocks), whatever number of tiles that is. It sorts them, kAssignMine at
  // a time, and counts every new key of the call at the first of them above it
  // (a search in LDS); the prefix sums of the counts are their ranks.
  constexpr int PER = kAssignMine / NT;
  static_assert(kChunk >= kAssignMine && kAssignMine % NT == 0, "the own keys take the chunk's place");
  uint64_t* s_chunk = s_buf;                                                   // [kChunk], then the own keys
  uint64_t* s_sorted = s_buf + kChunk;                                        // [kAssignMine]
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_sorted + kAssignMine);      // [kAssignMine]
  uint32_t* s_rank = s_cnt + kAssignMine;                                     // [kAssignMine]
  const int g = (int)blockIdx.x, G = (int)a.blocks;
  const int own = g < ntiles ? (ntiles - 1 - g) / G + 1 : 0;
  for (int o0 = 0; o0 < own; o0 += NT) {
    const int no = min(NT, own - o0);
    for (uint32_t k0 = 0;; k0 += kAssignMine) {
      const uint32_t c = (int)threadIdx.x < no ? tile_cnt[g + (o0 + (int)threadIdx.x) * G] : 0u;
      uint32_t total;
      const uint32_t pre = block_exclusive_scan<NT>(c, s_w, &total);
      if (k0 >= total) break;  // (block-uniform)
      const uint32_t m = min((uint32_t)kAssignMine, total - k0);
      uint32_t P2 = 1;
      while (P2 < m) P2 <<= 1;
      s_pref[threadIdx.x] = pre;
      __syncthreads();
      uint64_t mk[PER];
      uint32_t ms[PER];
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const uint32_t j = threadIdx.x + u * NT;
        mk[u] = kEmptyKey;
        ms[u] = 0;
        if (j < m) {
          int lo = 0, hi = no - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_pref[mid] <= k0 + j) lo = mid;
            else hi = mid - 1;
          }
          const NewKey nk = newlist[(size_t)(g + (o0 + lo) * G) * tile_size + (k0 + j - s_pref[lo])];
          mk[u] = nk.key;
          ms[u] = nk.slot;
        }
        if (j < P2) s_sorted[j] = mk[u];
        s_cnt[j] = 0;
      }
      __syncthreads();
      block_bitonic_sort<NT>(s_sorted, P2);
      auto not_above = [&](uint64_t key) {  // own keys <= key
        uint32_t x = 0;
        for (uint32_t step = P2; step >= 1; step >>= 1)
          if (x + step <= m && s_sorted[x + step - 1] <= key) x += step;
        return x;
      };
      for_each_new_key_chunk<NT>(newlist, tile_cnt, ntiles, tile_size, s_pref, s_w, s_chunk,
                                 [&](const uint64_t* ck, uint32_t cnt) {
                                   for (uint32_t e = threadIdx.x; e < cnt; e += NT) {
                                     const uint32_t x = not_above(ck[e]);
                                     if (x < m) atomicAdd(&s_cnt[x], 1u);
                                   }
                                 });
      uint32_t v[PER], sum = 0, tot;
#pragma unroll
      for (int u = 0; u < PER; ++u) sum += v[u] = s_cnt[threadIdx.x * PER + u];
      uint32_t acc = block_exclusive_scan<NT>(sum, s_w, &tot);
#pragma unroll
      for (int u = 0; u < PER; ++u) s_cnt[threadIdx.x * PER + u] = acc += v[u];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const uint32_t j = threadIdx.x + u * NT;
        if (j >= m) continue;
        const uint32_t r = s_cnt[not_above(mk[u]) - 1];
        const uint32_t row = (uint32_t)(size0 + r);
        idx[ms[u] / kSlots].row[ms[u] % kSlots] = row;
        state[row] = 0.0f;
        if (clock != nullptr) clock[row] = new_row_clock(cepoch);
        s_chunk[j] = a.values != nullptr ? take_position(idx, ms[u]) : mk[u];
        s_rank[j] = r;
      }
      __syncthreads();
      if (a.values != nullptr) write_value_rows<NT>(s_chunk, s_rank, m, size0, store, D, a.values);
      else write_init_rows<NT>(s_chunk, s_rank, m, size0, store, D, seed);
      __syncthreads();
    }
  }
}

// Copies the block's share of the positions' rows into `out`: kCopyUnits
// units of 16 bytes per thread, consecutive threads on consecutive units of
// the output, whatever the width of a row, so that no lane idles on a row's
// end. Rows of keys present before the call are read from the table, rows of
// keys new in it are generated from their seed (they equal what the table
// will hold), rows of blocked positions are left alone (kTrack).
// Bound by HBM (copy_lanes says which gets copy their rows here). Two units a
// thread; four are 4 to 8 % slower at dims 128 and 400. An output of kStreamOut
// bytes does not stay in the 32 MB of L2 anyway and goes around it
// (non-temporal), which leaves the caches to the rows and to the kernels that
// follow: two DLRM steps 199 -> 186 us, two of dim 400 640 -> 595.
constexpr int kCopyThreads = kAssignThreads;
constexpr int kCopyUnits = 2;
constexpr uint64_t kStreamOut = 32ull << 20;
constexpr uint64_t kCopyBlocks = 1ull << 22;  // blocks at most (a launch holds fewer than 2^32 threads)
template <int VEC, bool kTrack, bool kStream>
__device__ __forceinline__ void copy_rows(const GetRowsArgs& a) {
  constexpr uint32_t PER = kCopyThreads * kCopyUnits;
  using V = typename VecT<VEC>::T;
  const int D = a.store.D;
  const uint32_t Q = VEC == 4 ? (uint32_t)(D + 3) / 4u : (uint32_t)D;  // units of a row
  const uint64_t total = (uint64_t)a.n * Q;
  for (uint64_t first = (uint64_t)blockIdx.x * PER; first < total; first += (uint64_t)gridDim.x * PER) {
    const uint64_t p0 = first / Q;  // (block-uniform)
    const uint32_t rem = (uint32_t)(first - p0 * Q);
    V v[kCopyUnits];
    uint64_t p[kCopyUnits];
    int col[kCopyUnits];
    uint32_t row[kCopyUnits];
    bool on[kCopyUnits];
#pragma unroll
    for (int u = 0; u < kCopyUnits; ++u) {
      const uint32_t e = rem + (uint32_t)u * kCopyThreads + threadIdx.x;  // < Q + PER
      // e / Q by magic = ceil(2^32 / Q): exact, since e * (magic * Q - 2^32) < (Q + PER) * Q < 2^32
      // (Q > 1: the probe kernel copies rows of one unit)
      const uint32_t d = (uint32_t)(((uint64_t)e * a.magic) >> 32);
      p[u] = p0 + d;
      const int c = (int)(e - d * Q) * VEC;
      col[u] = VEC == 1 || c < D - VEC ? c : D - VEC;  // the last unit of a row: its last four columns
      on[u] = p[u] < (uint64_t)a.n;
      row[u] = on[u] ? a.rows[p[u]] : kPendingRow;
      if constexpr (kTrack) on[u] = on[u] && a.blocked[p[u]] == 0;
    }
#pragma unroll
    for (int u = 0; u < kCopyUnits; ++u)
      if (row[u] != kPendingRow) v[u] = load_vec<VEC>(a.store.ptr(row[u]) + col[u]);
#pragma unroll
    for (int u = 0; u < kCopyUnits; ++u)
      if (on[u] && row[u] == kPendingRow) v[u] = init_vec<VEC>(splitmix_mix(a.keys[p[u]] ^ a.seed), col[u]);
#pragma unroll
    for (int u = 0; u < kCopyUnits; ++u) {
      if (!on[u]) continue;
      float* o = a.out + (size_t)p[u] * (size_t)D + col[u];
      if constexpr (kStream) store_vec_nt<VEC>(o, v[u]);
      else store_vec<VEC>(o, v[u]);
    }
  }
}

// At most 80 registers (six waves per SIMD): the copy needs the waves.
template <int VEC, bool kTrack, bool kStream>
__global__ __launch_bounds__(kAssignThreads, 6) void k_get_rows(const GetRowsArgs ra, const AssignArgs aa) {
  if (ra.out != nullptr) copy_rows<VEC, kTrack, kStream>(ra);
  if (blockIdx.x >= aa.blocks) return;
  __shared__ AssignLds<kAssignThreads> lds;
  Ctrl* const ctrl = aa.ctrl;
  // the next call's range counts start at zero (this call's are read by assign_new)
  if (aa.rl.list != nullptr && blockIdx.x == 0)
    for (int e = threadIdx.x; e < kMaxRanges; e += kAssignThreads) aa.rl.cnt_next[e] = 0u;
  const uint64_t size0 = ctrl->size[aa.epoch & 1];
  const uint64_t M =
      ctrl->new_epoch == aa.epoch ? count_new_keys<kAssignThreads>(aa.tile_cnt, aa.ntiles, lds.w64) : 0ull;
  const int err = call_verdict(ctrl, aa.epoch, size0, M, aa.capacity, ctrl->bad_epoch, ctrl->overflow_epoch);
  if (err && aa.clock != nullptr) rollback_clocks(aa.clock, size0, aa.cepoch, aa.blocks);
  assign_new<kAssignThreads, kGetTile>(aa, ra.store, ra.seed, size0, M, err, lds);
}
#endif  // MLKV_MAP

// ===========================================================================
// Put. The (key, position) pairs of a call flow through "items":
//   bit 63     1 if the key is inserted by this call (row not yet known)
//   bits 31-62 the key's row, or its index slot when bit 63 is set
//   bit 30     1 if the item stands for several positions of one tile whose
//              gradient rows were already summed (fp64) into partials[pos]
//   bits 0-29  the position of the key in the batch (the first one for a
//              summed item)
// Sorting items groups the positions of each key (single positions first,
// then summed tiles, each in ascending order) and puts new keys last.
// ===========================================================================
constexpr uint64_t kItemSummed = 1ull << 30;

__device__ __forceinline__ uint64_t make_item(bool fresh, uint32_t tag, uint32_t low31) {
  return ((uint64_t)(fresh ? 1u : 0u) << 63) | ((uint64_t)tag << 31) | (uint64_t)(low31 & 0x7FFFFFFFu);
}
__device__ __forceinline__ uint32_t item_pos(uint64_t it) { return (uint32_t)(it & 0x3FFFFFFFull); }
__device__ __forceinline__ uint32_t item_low31(uint64_t it) { return (uint32_t)(it & 0x7FFFFFFFull); }
__device__ __forceinline__ bool item_summed(uint64_t it) { return (it & kItemSummed) != 0; }
__device__ __forceinline__ uint32_t item_tag(uint64_t it) { return (uint32_t)(it >> 31); }
__device__ __forceinline__ bool item_fresh(uint64_t it) { return (it >> 63) != 0; }
__device__ __forceinline__ uint64_t item_group(uint64_t it) { return it >> 31; }

// Partition of a key's group: top bits of a hash of (fresh, row or slot).
__device__ __forceinline__ uint32_t group_partition(uint64_t group, int pb) {
  return pb ? (uint32_t)(index_hash(group) >> (64 - pb)) : 0u;
}

// ---------------------------------------------------------------------------
// Put, first kernel (one block per tile of kPutTile keys, kPutThreads
// threads): probe (+ insert) each key; find the keys that occur more than once
// in the tile with an LDS hash table and sum each one's gradient rows
// (positions ascending, fp64) into one partial; partition the resulting items
// by a hash of the key (one MSD radix digit).
// ---------------------------------------------------------------------------
constexpr int kTileHash = 2 * kPutTile;  // LDS hash slots per tile

// kAhead: the put's probe runs ahead of the kernels of the get whose epoch is
// one less, its other kernels after them (PutArgs::ahead): it looks keys up
// without inserting, and a key absent from the table fails the put.
template <class M, bool kAhead>
__global__ __launch_bounds__(kPutThreads) void k_put_probe(
    Bucket* __restrict__ idx, uint32_t nb_log2, const uint64_t* __restrict__ keys,
    const float* __restrict__ grads, int64_t n, int tlen, int D, int op, uint32_t dup_min, int pb, int ntiles,
    uint64_t* __restrict__ items,
    uint32_t* __restrict__ meta, double* __restrict__ partials, NewKey* __restrict__ newlist,
    uint32_t* __restrict__ tile_cnt, Ctrl* ctrl, uint64_t epoch, const uint64_t* __restrict__ pc_key,
    const uint32_t* __restrict__ pc_row) {
  constexpr int NT = kPutThreads;
  constexpr int KPT = kPutTile / kPutThreads;  // keys per thread
  constexpr int VEC = M::VEC, LPR = M::LPR, K = M::K, RPW = M::RPW;
  constexpr int NG = (NT / 64) * RPW;
  using V = typename VecT<VEC>::T;
  __shared__ uint32_t s_hist[kMaxParts];
  __shared__ unsigned long long s_hkey[kTileHash];  // key of each hash slot
  __shared__ uint32_t s_hcnt[kTileHash];            // occurrences of the key in the tile
  __shared__ uint32_t s_hfirst[kTileHash];          // first entry holding the key
  __shared__ uint32_t s_hcur[kTileHash];            // fill cursor of the key's entry list
  __shared__ uint16_t s_hdup[kTileHash];            // index of a repeated key
  __shared__ uint16_t s_lanes[kPutTile];            // entries of repeated keys, grouped
  __shared__ uint16_t s_doff[kPutTile / 2 + 1];     // start of each repeated key's entries
  __shared__ uint32_t s_w[NT / 64];
  __shared__ uint32_t s_cnt;
  const int NP = 1 << pb;
  const int tid = threadIdx.x;
  const int tile = blockIdx.x;
  const int64_t base = (int64_t)tile * tlen;        // batch position of the tile's entry 0
  const int64_t sbase = (int64_t)tile * kPutTile;   // the tile's slots in items / newlist
  if (tile == 0 && tid == 0) {
    ctrl->spill_next = 0;
    ctrl->unit_single = 0;
    ctrl->unit_multi = 0;
  }
  for (int d = tid; d < NP; d += NT) s_hist[d] = 0;
  for (int h = tid; h < kTileHash; h += NT) {
    s_hkey[h] = ~0ull;
    s_hcnt[h] = 0;
    s_hfirst[h] = 0xFFFFFFFFu;
    s_hcur[h] = 0;
  }
  if (tid == 0) s_cnt = 0;

  // entry e = kk * NT + tid of the tile is batch position base + e. The
  // index buckets of the tile's keys are loaded first; while they are in
  // flight the tile's keys are deduplicated in LDS (a key and its slot are
  // one to one), and the probe reads the buckets afterwards.
  // a key that the last get found present at the same position takes the
  // row it found there; the others load their home bucket
  uint64_t key[KPT];
  bool inb[KPT];
  uint64_t hb[KPT];
  BucketView bv[KPT];
  uint64_t ck[KPT];
  uint32_t crow[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    const int64_t i = base + kk * NT + tid;
    inb[kk] = kk * NT + tid < tlen && i < n;
    key[kk] = inb[kk] ? keys[i] : kEmptyKey;
    ck[kk] = inb[kk] ? pc_key[i] : kEmptyKey;
    crow[kk] = inb[kk] ? pc_row[i] : kPendingRow;
  }
  bool cached[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    cached[kk] = key[kk] != kEmptyKey && ck[kk] == key[kk];
    if (key[kk] != kEmptyKey && !cached[kk]) {
      hb[kk] = home_bucket(key[kk], nb_log2);
      bv[kk] = load_bucket(idx + hb[kk]);
    }
  }
  lds_barrier();  // the hash table is initialised

  uint32_t hs[KPT];
  bool valid[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    const int e = kk * NT + tid;
    valid[kk] = key[kk] != kEmptyKey;
    // count the tile's occurrences of every key
    hs[kk] = 0;
    if (valid[kk]) {
      uint32_t h = (uint32_t)index_hash(key[kk]) & (kTileHash - 1);
      while (true) {
        const unsigned long long old = atomicCAS(&s_hkey[h], ~0ull, (unsigned long long)key[kk]);
        if (old == ~0ull || old == key[kk]) break;
        h = (h + 1) & (kTileHash - 1);
      }
      hs[kk] = h;
      atomicAdd(&s_hcnt[h], 1u);
      atomicMin(&s_hfirst[h], (uint32_t)e);
    }
  }
  lds_barrier();
  // a key repeated in the tile ("dup") gets the sorted list of its entries;
  // one repeated at least dup_min times is merged into one item (an
  // assignment keeps the last position; a sum adds the key's gradient rows
  // here, in fp64), the entries of the others stay items of their own, which
  // the key's first entry emits together in position order
  uint32_t cnt[KPT];
  bool dup[KPT], merged[KPT], owner[KPT];
  uint32_t n_own = 0, l_own = 0;
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    const int e = kk * NT + tid;
    cnt[kk] = valid[kk] ? s_hcnt[hs[kk]] : 0u;
    dup[kk] = cnt[kk] >= 2;
    merged[kk] = cnt[kk] >= dup_min;
    owner[kk] = dup[kk] && s_hfirst[hs[kk]] == (uint32_t)e;
    n_own += owner[kk] ? 1u : 0u;
    l_own += owner[kk] ? cnt[kk] : 0u;
  }

  // repeated groups: index them, then list their entries contiguously. The
  // in-tile sums below take one work item per repeated key, or, for a key
  // with more than kSumChunk entries, one per chunk of kSumChunk entries.
  constexpr int UNR = (K * VEC >= 16) ? 2 : (K * VEC >= 8) ? 4 : 8;  // rows loaded together
  constexpr uint32_t kSumChunk = 2 * UNR;
  auto n_items = [](uint32_t c) { return c <= kSumChunk ? 1u : (c + kSumChunk - 1) / kSumChunk; };
  uint32_t w_own = 0;
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) w_own += owner[kk] && merged[kk] ? n_items(cnt[kk]) : 0u;
  // one scan for the three prefixes, packed 10 | 11 | 11 bits (a tile holds
  // at most 512 repeated keys and 1024 entries, so no field overflows)
  static_assert(kPutTile <= 1024, "packed prefix fields");
  uint32_t ptot;
  const uint32_t ppre = block_exclusive_scan<NT>(n_own | (l_own << 10) | (w_own << 21), s_w, &ptot);
  const uint32_t ndup = ptot & 0x3FFu, nlanes = (ptot >> 10) & 0x7FFu, nwork = ptot >> 21;
  uint32_t dpre = ppre & 0x3FFu, lpre = (ppre >> 10) & 0x7FFu, wpre = ppre >> 21;
  uint32_t my_d[KPT], my_w[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    my_d[kk] = dpre;
    my_w[kk] = wpre;
    if (owner[kk]) {
      s_hdup[hs[kk]] = (uint16_t)dpre;
      s_doff[dpre] = (uint16_t)lpre;
      ++dpre;
      lpre += cnt[kk];
      wpre += merged[kk] ? n_items(cnt[kk]) : 0u;
    }
  }
  if (tid == 0) s_doff[ndup] = (uint16_t)nlanes;
  lds_barrier();
  uint32_t my_off[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    my_off[kk] = 0;
    if (dup[kk]) {
      my_off[kk] = s_doff[s_hdup[hs[kk]]];
      s_lanes[my_off[kk] + atomicAdd(&s_hcur[hs[kk]], 1u)] = (uint16_t)(kk * NT + tid);
    }
  }
  lds_barrier();
  // first work item of each repeated key (the fill cursors are no longer needed)
  uint16_t* s_wfirst = reinterpret_cast<uint16_t*>(s_hcur);
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk)
    if (owner[kk]) s_wfirst[my_d[kk]] = (uint16_t)my_w[kk];
  if (tid == 0) s_wfirst[ndup] = (uint16_t)nwork;
  // sort each repeated group's entry list: an entry's rank is the number of
  // smaller entries in its group's list
  uint32_t rank[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    rank[kk] = 0;
    if (dup[kk]) {
      const uint32_t e = kk * NT + tid;
      for (uint32_t m = 0; m < cnt[kk]; ++m) rank[kk] += s_lanes[my_off[kk] + m] < e ? 1u : 0u;
    }
  }
  lds_barrier();
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk)
    if (dup[kk]) s_lanes[my_off[kk] + rank[kk]] = (uint16_t)(kk * NT + tid);
  lds_barrier();

  // each lane group sums the rows of repeated keys, positions ascending (an
  // assignment needs no sum: its item is the key's last position instead).
  // Work items are dealt to the groups in turn. A key of at most kSumChunk
  // entries leaves its fp64 sum over the partials row of its first entry; a
  // longer key's chunks leave partial sums over the rows of their own first
  // entries (the first chunk over the key's second entry), which are added
  // in chunk order at the end of the kernel.
  const int lane = tid & 63;
  const int g = lane / LPR;
  const int q = lane % LPR;
  const int gid = (tid >> 6) * RPW + g;
  // some merged key has more than kSumChunk entries
  bool my_chunked = false;
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) my_chunked |= owner[kk] && cnt[kk] > kSumChunk;
  const bool chunked = __syncthreads_or(my_chunked ? 1 : 0) != 0;
  double acc[K][VEC];
  auto store_row = [&](uint32_t entry) {
    double* dst = partials + (size_t)(base + s_lanes[entry]) * (size_t)D;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int col = M::col(k, q, D);
#pragma unroll
      for (int v = 0; v < VEC; ++v)
        if (M::on(k, q, D)) dst[col + v] = acc[k][v];
    }
  };
  if (op != kOpAssign) {
    for (uint32_t w = gid; w < nwork; w += NG) {
      // the key of item w: the last d with s_wfirst[d] <= w (keys that are
      // not merged have no work item and share the next key's first one)
      uint32_t d = 0, dh = ndup;
      while (d + 1 < dh) {
        const uint32_t mid = (d + dh) >> 1;
        if (s_wfirst[mid] <= w) d = mid;
        else dh = mid;
      }
      const uint32_t c = w - s_wfirst[d];
      const uint32_t kb = s_doff[d], kend = s_doff[d + 1];
      const bool whole = kend - kb <= kSumChunk;
      const uint32_t b = kb + c * kSumChunk, e = whole ? kend : min(b + kSumChunk, kend);
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[k][v] = 0.0;
      for (uint32_t j = b; j < e; j += UNR) {
        V gv[UNR][K];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          if (j + u < e) {
            const float* gr = grads + (size_t)(base + s_lanes[j + u]) * (size_t)D;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const int col = M::col(k, q, D);
              if (M::on(k, q, D)) gv[u][k] = load_vec<VEC>(gr + col);
            }
          }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          if (j + u < e) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
              if (M::on(k, q, D)) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[k][v] += (double)VecT<VEC>::get(gv[u][k], v);
              }
            }
          }
        }
      }
      store_row(whole ? kb : (c == 0 ? kb + 1 : b));
    }
  }

  // probe (and insert) each key now that its bucket has arrived
  Probe pr[KPT];
  // ahead of a get: the size word that get starts from (it writes the other)
  const uint64_t size_before = kAhead ? ctrl->size[(epoch + 1) & 1] : 0ull;
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    pr[kk] = {0, kPendingRow, inb[kk] ? P_BAD : P_NONE};
    if (cached[kk]) {
      pr[kk] = {0, crow[kk], P_HIT};
    } else if (key[kk] != kEmptyKey) {
      pr[kk] = probe_with(idx, nb_log2, key[kk], !kAhead, hb[kk], bv[kk]);
      if constexpr (kAhead) {
        if (pr[kk].status != P_HIT || pr[kk].row >= size_before) {
          pr[kk].status = P_ABSENT;
          ctrl->apput_absent_epoch = epoch;
        }
      } else {
        if (pr[kk].status == P_OVERFLOW) ctrl->overflow_epoch = epoch;
      }
    } else if (pr[kk].status == P_BAD) {
      if constexpr (kAhead) ctrl->apput_bad_epoch = epoch;
      else ctrl->bad_epoch = epoch;
    }
  }
  uint64_t x[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    const int e = kk * NT + tid;
    valid[kk] = pr[kk].status == P_HIT || pr[kk].status == P_NEW_MINE || pr[kk].status == P_NEW_OTHER;
    if (pr[kk].status == P_NEW_MINE) {
      const uint32_t j = atomicAdd(&s_cnt, 1u);
      s_hkey[j] = key[kk];  // (the tile's hash table is no longer read)
      s_hcnt[j] = pr[kk].slot;
      ctrl->new_epoch = epoch;
    }
    const bool fresh = pr[kk].status != P_HIT;
    uint32_t pos = (uint32_t)(base + e);
    if (op == kOpAssign && owner[kk]) pos = (uint32_t)(base + s_lanes[s_doff[s_hdup[hs[kk]] + 1] - 1]);
    x[kk] = valid[kk] ? make_item(fresh, fresh ? pr[kk].slot : pr[kk].row, pos) : ~0ull;
  }

  // emit single positions, one item per merged key, and the entries of each
  // other repeated key together, in position order, from its first entry
  bool emit[KPT];
  uint32_t d[KPT], r[KPT], ne[KPT];
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    emit[kk] = valid[kk] && (!dup[kk] || owner[kk]);
    ne[kk] = dup[kk] && !merged[kk] ? cnt[kk] : 1u;
    d[kk] = 0;
    r[kk] = 0;
    if (emit[kk]) {
      // an upsert's new key: its last position goes to the spare word of its
      // index slot (complemented: an unused word is all ones)
      if (!kAhead && op == kOpAssign && item_fresh(x[kk])) {
        const uint32_t slot = item_tag(x[kk]);
        atomicMin(&idx[slot / kSlots].aux[slot % kSlots], ~item_pos(x[kk]));
      }
      d[kk] = group_partition(item_group(x[kk]), pb);
      r[kk] = atomicAdd(&s_hist[d[kk]], ne[kk]);
    }
  }
  lds_barrier();
  constexpr int PER = kMaxParts / NT;
  uint32_t c[PER];
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int dd = tid * PER + j;
    c[j] = dd < NP ? s_hist[dd] : 0u;
    sum += c[j];
  }
  uint32_t tot;
  uint32_t off = block_exclusive_scan<NT>(sum, s_w, &tot);
  uint32_t offs[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int dd = tid * PER + j;
    offs[j] = off;
    if (dd < NP) meta[(size_t)dd * ntiles + tile] = off | (c[j] << 16);
    off += c[j];
  }
  lds_barrier();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int dd = tid * PER + j;
    if (dd < NP) s_hist[dd] = offs[j];
  }
  lds_barrier();
#pragma unroll
  for (int kk = 0; kk < KPT; ++kk) {
    if (!emit[kk]) continue;
    uint64_t* dst = items + (size_t)sbase + s_hist[d[kk]] + r[kk];
    if (dup[kk] && !merged[kk]) {
      const uint32_t kb = s_doff[s_hdup[hs[kk]]];
      for (uint32_t i = 0; i < cnt[kk]; ++i)
        dst[i] = (x[kk] & ~0x7FFFFFFFull) | (uint64_t)(uint32_t)(base + s_lanes[kb + i]);
    } else {
      dst[0] = merged[kk] && op != kOpAssign ? (x[kk] | kItemSummed) : x[kk];
    }
  }
  if constexpr (!kAhead) {  // ahead of a get, the lists and counts are the get's
    // the tile's list of new keys, in ascending key order (each at its rank)
    const uint32_t c = s_cnt;
    for (uint32_t j = tid; j < c; j += NT) {
      const uint64_t k = s_hkey[j];
      uint32_t at = 0;
      for (uint32_t e = 0; e < c; ++e) at += s_hkey[e] < k ? 1u : 0u;
      newlist[(size_t)sbase + at] = NewKey{k, s_hcnt[j], 0u};
    }
    if (tid == 0) tile_cnt[tile] = c;
  }
  // keys summed in chunks: add the chunks' partial sums in order
  if (op != kOpAssign && chunked) {
    __syncthreads();
    for (uint32_t d = gid; d < ndup; d += NG) {
      const uint32_t kb = s_doff[d], kend = s_doff[d + 1];
      if (kend - kb <= kSumChunk) continue;
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[k][v] = 0.0;
      for (uint32_t b = kb; b < kend; b += kSumChunk) {
        const double* src = partials + (size_t)(base + s_lanes[b == kb ? kb + 1 : b]) * (size_t)D;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const int col = M::col(k, q, D);
#pragma unroll
          for (int v = 0; v < VEC; ++v)
            if (M::on(k, q, D)) acc[k][v] += src[col + v];
        }
      }
      store_row(kb);
    }
  }
}

// ---------------------------------------------------------------------------
// Row updates
// ---------------------------------------------------------------------------

// Sum over the LPR lanes of a lane group (LPR a power of two, groups aligned);
// every lane of the group receives the same value. Steps within 16 lanes use
// DPP moves, wider steps lane shuffles.
template <int LPR>
__device__ __forceinline__ double group_sum(double x) {
  auto dpp = [](double v, auto ctrl_tag) {
    constexpr int ctrl = decltype(ctrl_tag)::value;
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
  };
  using Xor1 = std::integral_constant<int, 0xB1>;       // quad_perm [1,0,3,2]
  using Xor2 = std::integral_constant<int, 0x4E>;       // quad_perm [2,3,0,1]
  using HalfMirror = std::integral_constant<int, 0x141>;  // row_half_mirror
  using Mirror = std::integral_constant<int, 0x140>;      // row_mirror
  if constexpr (LPR >= 2) x += dpp(x, Xor1{});
  if constexpr (LPR >= 4) x += dpp(x, Xor2{});
  if constexpr (LPR >= 8) x += dpp(x, HalfMirror{});
  if constexpr (LPR >= 16) x += dpp(x, Mirror{});
  if constexpr (LPR >= 32) x += __shfl_xor(x, 16, 64);
  if constexpr (LPR >= 64) x += __shfl_xor(x, 32, 64);
  return x;
}

template <class M>
struct SegmentOps {
  static constexpr int VEC = M::VEC, LPR = M::LPR, K = M::K, RPW = M::RPW;
  using V = typename VecT<VEC>::T;

  // Row-wise Adagrad step of one row, given its summed gradient g (fp32):
  // m = fp32(sum g^2 / D) over the group's lanes; G' = G + m;
  // den = sqrt(G') + eps; w -= lr * (g / den); writes w and G'.
  static __device__ __forceinline__ void adagrad(const V (&g)[K], V (&w)[K], float G, float* __restrict__ wrow,
                                                 float* __restrict__ state, uint32_t row, int D, int q,
                                                 bool d_pow2, double inv_d, float lr, float eps) {
    double sq = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int x = 0; x < VEC; ++x) {
        const double gx = (double)VecT<VEC>::get(g[k], x);
        if (M::on(k, q, D) && x >= M::twice(k, q, D)) sq += gx * gx;
      }
    }
    sq = group_sum<LPR>(sq);
    // D a power of two: multiplying by 1/D is exact, hence equal to sq / D
    const float m = (float)(d_pow2 ? sq * inv_d : sq / (double)D);
    const float Gn = __fadd_rn(G, m);
    const float den = __fadd_rn(__builtin_sqrtf(Gn), eps);  // correctly rounded sqrt
    // g / den: a correctly rounded IEEE quotient per element, so that den = 0
    // (eps = 0 with an underflowing m), subnormal denominators and overflowing
    // quotients give the same infinities and NaNs as a plain fp32 division
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int col = M::col(k, q, D);
      if (M::on(k, q, D)) {
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
          const float gx = VecT<VEC>::get(g[k], x);
          const float qv = __fdiv_rn(gx, den);
          const float p = __fmul_rn(lr, qv);
          VecT<VEC>::set(w[k], x, __fsub_rn(VecT<VEC>::get(w[k], x), p));
        }
        store_vec<VEC>(wrow + col, w[k]);
      }
    }
    if (q == 0) state[row] = Gn;
  }

  // One SGD step: w -= lr * g (separate fp32 operations).
  static __device__ __forceinline__ void sgd(const V (&g)[K], V (&w)[K], float* __restrict__ wrow, int D, int q,
                                             float lr) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int col = M::col(k, q, D);
      if (M::on(k, q, D)) {
#pragma unroll
        for (int x = 0; x < VEC; ++x)
          VecT<VEC>::set(w[k], x, __fsub_rn(VecT<VEC>::get(w[k], x), __fmul_rn(lr, VecT<VEC>::get(g[k], x))));
        store_vec<VEC>(wrow + col, w[k]);
      }
    }
  }
};

// A put completes one served get on the row (bounded staleness, Sec.
// III-C1): its count drops by one, never below 0. One lane per row, from the
// low 32 bits of the word, loaded ahead with the row: they hold the count (a
// nonzero count drops without borrowing from the epoch bits above it, so only
// the low word is written).
static_assert(kClockBits < 32, "the count fits the low word of a staleness word");
__device__ __forceinline__ uint32_t clock_low(const unsigned long long* __restrict__ clock, uint32_t row) {
  return reinterpret_cast<const uint32_t*>(clock + row)[0];  // little-endian: the low word comes first
}
__device__ __forceinline__ void put_clock_low(unsigned long long* __restrict__ clock, uint32_t row, uint32_t lo) {
  if ((lo & (uint32_t)kClockCount) != 0u) reinterpret_cast<uint32_t*>(clock + row)[0] = lo - 1u;
}

// The row of a unit's key: its tag, or, for a key new in the call, the row
// its index slot holds by now.
__device__ __forceinline__ uint32_t unit_row(const Bucket* __restrict__ idx, uint32_t tag, bool fresh) {
  return fresh ? idx[tag / kSlots].row[tag % kSlots] : tag;
}

#ifndef MLKV_MAP
// ---------------------------------------------------------------------------
// Put, second kernel: one block per partition. It gathers the partition's
// items, groups them by key in LDS with each key's items in ascending
// position, and leaves the call's update as units, one per distinct key, in
// three lists of the whole call (PutUnits): keys with one gradient row
// (`single`, the item itself), keys whose items need a sum (`multi`: tag,
// number of items, where its items start in `mitem`) and those with more than
// long_over items (`lng`). Every unit is independent of the others, so the
// order of the lists, which depends on the blocks' timing, changes no result.
// The first blocks then assign rows to the keys the call inserted.
// An upsert (kUpsert) needs no units: the block writes the value row of each
// present key's last position itself, and the rows of new keys are written
// where they are assigned.
//
// Bound by the latency of LDS and of the barriers between its steps. Grouping
// and updating in one kernel of a block per CU (125 registers, 145 KB of LDS)
// left HBM idle while it grouped, and segments cut between its lane groups
// were added up by one of them in a serial chain (10 to 28 us at dims 10 to
// 16). Apart, this kernel runs two blocks per CU at 64 registers, and the
// update kernel below streams with every wave the chip holds. Both together
// against the one kernel, us: 213k lookups of dim 64 18 + 29 / 52, 131k of dim
// 32 16 + 14 / 42, 106k of dim 10 15 + 10 / 47, 4096 of dim 16 12 + 10 / 28, 150k
// of dim 400 16 + 132 / 184, 1M of dim 128 37 + 303 / 413.
// ---------------------------------------------------------------------------
constexpr size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }
constexpr int kGroupThreads = 1024;
// Units of more than kRankMask items are put in order through a bitmask of
// their items' places in the gathered list (at most kMaskUnits of them per
// partition; others compare their items pairwise).
constexpr uint32_t kRankMask = 32;
constexpr int kMaskUnits = 16;
constexpr int kMaskWords = kRedCap / 32;

// Dynamic LDS of a grouping block, in bytes (two blocks per CU).
struct GroupLds {
  static constexpr size_t it = 0;                                  // u64[kRedCap] gather order
  static constexpr size_t hidx = it + 8 * (size_t)kRedCap;         // u32[kRedHash] first item, then a fill cursor
  static constexpr size_t hcnt = hidx + 4 * (size_t)kRedHash;      // u32[kRedHash] items, then start | items << 16
  static constexpr size_t slot = hcnt + 4 * (size_t)kRedHash;      // u16[kRedCap] hash slot of each item
  static constexpr size_t ord = slot + 2 * (size_t)kRedCap;        // u16[kRedCap] items by unit
  static constexpr size_t lid = ord + 2 * (size_t)kRedCap;         // u8[kRedHash] mask of each unit
  static constexpr size_t mask = lid + (size_t)kRedHash;           // u32[kMaskUnits][kMaskWords]
  static constexpr size_t w64 = mask + 4 * (size_t)kMaskUnits * kMaskWords;  // u64[kGroupThreads / 64]
  static constexpr size_t w = w64 + 8 * (size_t)(kGroupThreads / 64);        // u32[kGroupThreads / 64]
  static constexpr size_t misc = align16(w + 4 * (size_t)(kGroupThreads / 64));  // u64[2], u32[8]
  static constexpr size_t grouping = misc + 48;
  static constexpr size_t total = grouping > sizeof(AssignLds<kGroupThreads>) ? align16(grouping)
                                                                             : align16(sizeof(AssignLds<kGroupThreads>));
  static constexpr size_t pref = hidx;  // u32[kGroupThreads], before the grouping
  static_assert(total <= 80 * 1024, "two blocks per CU");
};

// Units a block has counted: singles, multis, longs and items of multis and
// longs, 16 bits each (a block groups at most kRedCap < 2^16 items).
__device__ __forceinline__ uint64_t pack_unit(uint32_t single, uint32_t multi, uint32_t lng, uint32_t items) {
  return (uint64_t)single | ((uint64_t)multi << 16) | ((uint64_t)lng << 32) | ((uint64_t)items << 48);
}

// Exclusive prefix of v within the block's waves plus a base per wave taken
// from *s_tot (cleared before), so that every thread's share of the total is
// its own; the order of the waves is any. No barrier.
__device__ __forceinline__ uint64_t claim_u64(uint64_t v, unsigned long long* s_tot) {
  const int lane = threadIdx.x & 63;
  unsigned long long x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  unsigned long long base = 0;
  if (lane == 63) base = atomicAdd(s_tot, x);
  return __shfl(base, 63, 64) + x - v;
}

// Claims the block's entries in the call's lists: s_base[0..3] = first entry
// among singles, multis, longs and items. One thread; two additions per block,
// to different lines: additions to one line take about 10 ns each, whoever
// makes them (four counters in one line: 10 us more for 256 blocks).
__device__ __forceinline__ void claim_units(Ctrl* ctrl, uint64_t tot, uint32_t* s_base) {
  const uint64_t ns = tot & 0xFFFFu, nm = (tot >> 16) & 0xFFFFu, nl = (tot >> 32) & 0xFFFFu, ni = tot >> 48;
  const unsigned long long a = atomicAdd(&ctrl->unit_single, (unsigned long long)(ns | (ni << 32)));
  const unsigned long long b = nm | nl ? atomicAdd(&ctrl->unit_multi, (unsigned long long)(nm | (nl << 32))) : 0ull;
  s_base[0] = (uint32_t)a;
  s_base[1] = (uint32_t)b;
  s_base[2] = (uint32_t)(b >> 32);
  s_base[3] = (uint32_t)(a >> 32);
}

// Where a thread's next unit of each class goes.
struct UnitCursor {
  uint32_t c[4];
  __device__ __forceinline__ UnitCursor(uint64_t pre, const uint32_t* s_base) {
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = s_base[k] + ((uint32_t)(pre >> (16 * k)) & 0xFFFFu);
  }
};

// Writes the unit of the key of item x with n items (the first at c[3]).
__device__ __forceinline__ void emit_unit(const PutUnits& u, UnitCursor& at, uint64_t x, uint32_t n, bool single) {
  if (single) {
    u.single[at.c[0]++] = x;
    return;
  }
  const uint4 e = make_uint4(item_tag(x), n | (item_fresh(x) ? kUnitFresh : 0u), at.c[3], 0u);
  if (n > u.long_over) u.lng[at.c[2]++] = e;
  else u.multi[at.c[1]++] = e;
  at.c[3] += n;
}

// Groups the items it[0, mp) of a partition by key (see k_put_group) and
// writes their units. it: the partition's items in the order put_probe's tiles
// listed them: tiles ascending, and within a tile a key's items together in
// ascending position; so the items of each key appear in position order (an
// in-tile sum is one item at the first position it covers).
__device__ __forceinline__ void group_by_key(unsigned char* lds, uint32_t mp, const PutUnits& u, Ctrl* ctrl) {
  using L = GroupLds;
  constexpr int NT = kGroupThreads;
  constexpr int IPT = kRedCap / NT;
  constexpr int HPT = kRedHash / NT;
  static_assert(kRedCap % NT == 0 && HPT == 4 && kRedCap < kRedHash && kRedHash <= 65536, "grouping table sizes");
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  constexpr uint32_t kMask = kRedHash - 1;
  const uint64_t* it = reinterpret_cast<const uint64_t*>(lds + L::it);
  uint32_t* hidx = reinterpret_cast<uint32_t*>(lds + L::hidx);
  uint32_t* hcnt = reinterpret_cast<uint32_t*>(lds + L::hcnt);
  uint16_t* slot = reinterpret_cast<uint16_t*>(lds + L::slot);
  uint16_t* ord = reinterpret_cast<uint16_t*>(lds + L::ord);
  uint8_t* lid = lds + L::lid;
  uint32_t* mask = reinterpret_cast<uint32_t*>(lds + L::mask);
  unsigned long long* s_tot = reinterpret_cast<unsigned long long*>(lds + L::misc);
  uint32_t* s_base = reinterpret_cast<uint32_t*>(lds + L::misc + 16);
  uint32_t* s_masks = s_base + 4;
  const int tid = threadIdx.x;
  for (int h = tid; h < kRedHash / 4; h += NT) {
    reinterpret_cast<uint4*>(hidx)[h] = make_uint4(kNone, kNone, kNone, kNone);
    reinterpret_cast<uint4*>(hcnt)[h] = make_uint4(0u, 0u, 0u, 0u);
  }
  for (int w = tid; w < kMaskUnits * kMaskWords; w += NT) mask[w] = 0u;
  if (tid == 0) {
    *s_tot = 0ull;
    *s_masks = 0u;
  }
  lds_barrier();

  // 1. one slot per key (the first item to take it), and its item count
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const uint32_t j = tid + k * NT;
    if (j < mp) {
      const uint64_t gr = item_group(it[j]);
      uint32_t h = (uint32_t)index_hash(gr) & kMask;
      while (true) {
        const uint32_t old = atomicCAS(&hidx[h], kNone, j);
        if (old == kNone || item_group(it[old]) == gr) break;
        h = (h + 1) & kMask;
      }
      slot[j] = (uint16_t)h;
      atomicAdd(&hcnt[h], 1u);
    }
  }
  lds_barrier();

  // 2. the unit of each occupied slot, and where its items start
  uint64_t x[HPT];
  uint32_t n[HPT];
  bool one[HPT];
  uint64_t mine = 0;
  {
    const uint4 hi = reinterpret_cast<const uint4*>(hidx)[tid], hc = reinterpret_cast<const uint4*>(hcnt)[tid];
    const uint32_t j[HPT] = {hi.x, hi.y, hi.z, hi.w};
    const uint32_t c[HPT] = {hc.x, hc.y, hc.z, hc.w};
#pragma unroll
    for (int q = 0; q < HPT; ++q) {
      n[q] = j[q] != kNone ? c[q] : 0u;
      x[q] = j[q] != kNone ? it[j[q]] : 0ull;
      one[q] = n[q] == 1u && !item_summed(x[q]);
      if (n[q] == 0u) continue;
      mine += one[q] ? pack_unit(1, 0, 0, 0) : n[q] > u.long_over ? pack_unit(0, 0, 1, n[q]) : pack_unit(0, 1, 0, n[q]);
    }
  }
  const uint64_t pre = claim_u64(mine, s_tot);
  uint32_t off = (uint32_t)(pre >> 48);
#pragma unroll
  for (int q = 0; q < HPT; ++q) {
    const uint32_t h = (uint32_t)tid * HPT + q;
    hidx[h] = 0u;  // fill cursor
    if (n[q] == 0u) continue;
    hcnt[h] = one[q] ? 0u : off | (n[q] << 16);
    uint32_t l = 0xFFu;
    if (!one[q]) {
      off += n[q];
      if (n[q] > kRankMask) {
        l = atomicAdd(s_masks, 1u);  // which mask a unit gets does not matter
        if (l >= (uint32_t)kMaskUnits) l = 0xFFu;
      }
    }
    lid[h] = (uint8_t)l;
  }
  lds_barrier();  // every wave has claimed its share of *s_tot
  if (tid == 0) claim_units(ctrl, *s_tot, s_base);

  // 3. drop each item of a sum into its unit (any order within it); a long
  // unit also marks its items' places in its mask
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const uint32_t j = tid + k * NT;
    if (j < mp) {
      const uint32_t h = slot[j], v = hcnt[h];
      if (v != 0u) {
        ord[(v & 0xFFFFu) + atomicAdd(&hidx[h], 1u)] = (uint16_t)j;
        const uint32_t l = lid[h];
        if (l != 0xFFu) atomicOr(&mask[l * kMaskWords + (j >> 5)], 1u << (j & 31));
      }
    }
  }
  lds_barrier();
  // 4. units to the call's lists
  UnitCursor at(pre, s_base);
#pragma unroll
  for (int q = 0; q < HPT; ++q)
    if (n[q] != 0u) emit_unit(u, at, x[q], n[q], one[q]);
  // 5. each item of a sum at its rank within its unit: the number of the
  // unit's items at earlier places (the items of a key come in position order)
  const uint32_t mbase = s_base[3];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const uint32_t j = tid + k * NT;
    if (j < mp) {
      const uint32_t h = slot[j], v = hcnt[h];
      if (v == 0u) continue;
      const uint32_t b = v & 0xFFFFu, c = v >> 16;
      uint32_t r = 0;
      if (c > 1) {
        const uint32_t l = lid[h];
        if (l != 0xFFu) {
          const uint32_t* mw = mask + l * kMaskWords;
          const uint32_t wj = j >> 5;
          for (uint32_t w = 0; w < wj; ++w) r += __popc(mw[w]);
          r += __popc(mw[wj] & ((1u << (j & 31)) - 1u));
        } else {
          for (uint32_t i = b; i < b + c; ++i) r += ord[i] < j ? 1u : 0u;
        }
      }
      u.mitem[mbase + b + r] = item_low31(it[j]);
    }
  }
}

// Writes the value rows of an upsert's keys s < S: at(s) is the item of key
// s's last position (a fresh one is skipped). As the row copy of a get,
// consecutive threads move consecutive units of the keys' rows. S * units of a
// row < 2^20.
constexpr int kValueUnits = 4;
template <int NT, int VEC, bool kClk, class At>
__device__ __forceinline__ void write_values(uint32_t S, const PutGroupArgs& a, const RowStore& store, At at) {
  constexpr uint32_t U = kValueUnits;
  using V = typename VecT<VEC>::T;
  const int D = store.D;
  const uint32_t Q = VEC == 4 ? (uint32_t)(D + 3) / 4u : (uint32_t)D;  // units of a row
  const uint32_t total = S * Q;
  for (uint32_t e0 = threadIdx.x; e0 < total; e0 += NT * U) {
    V v[U];
    uint32_t row[U], cl[U];
    int col[U];
    bool on[U];
#pragma unroll
    for (uint32_t k = 0; k < U; ++k) {
      const uint32_t e = e0 + k * NT;
      // e / Q by magic = ceil(2^32 / Q): exact, since e * (magic * Q - 2^32) < 2^20 * Q <= 2^28 (Q <= 256)
      const uint32_t d = Q == 1 ? e : (uint32_t)(((uint64_t)e * a.magic) >> 32);
      const int c = (int)(e - d * Q) * VEC;
      col[k] = VEC == 1 || c < D - VEC ? c : D - VEC;  // the last unit of a row: its last four columns
      const uint64_t x = e < total ? at(d) : 0ull;
      on[k] = e < total && !item_fresh(x);
      row[k] = item_tag(x);
      cl[k] = 0;
      if (on[k]) {
        v[k] = load_vec<VEC>(a.values + (size_t)item_pos(x) * (size_t)D + col[k]);
        if (kClk && c == 0) cl[k] = clock_low(a.clock, row[k]);
      }
    }
#pragma unroll
    for (uint32_t k = 0; k < U; ++k) {
      if (!on[k]) continue;
      store_vec<VEC>(store.wptr(row[k]) + col[k], v[k]);
      if (kClk) put_clock_low(a.clock, row[k], cl[k]);  // (cl is 0 for all but a row's first unit)
    }
  }
}

// An upsert of the items it[0, mp) of a partition: an LDS hash table from key
// to its last position, then a row write per key.
template <int VEC, bool kClk>
__device__ __forceinline__ void upsert_last(unsigned char* lds, uint32_t mp, const PutGroupArgs& a,
                                            const RowStore& store) {
  using L = GroupLds;
  constexpr int NT = kGroupThreads;
  constexpr int IPT = kRedCap / NT;
  constexpr int HPT = kRedHash / NT;
  static_assert(kRedCap * 256 <= (1 << 20), "write_values");
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  constexpr uint32_t kMask = kRedHash - 1;
  uint64_t* it = reinterpret_cast<uint64_t*>(lds + L::it);
  uint32_t* hidx = reinterpret_cast<uint32_t*>(lds + L::hidx);
  uint32_t* hlast = reinterpret_cast<uint32_t*>(lds + L::hcnt);
  unsigned long long* s_tot = reinterpret_cast<unsigned long long*>(lds + L::misc);
  const int tid = threadIdx.x;
  for (int h = tid; h < kRedHash / 4; h += NT) {
    reinterpret_cast<uint4*>(hidx)[h] = make_uint4(kNone, kNone, kNone, kNone);
    reinterpret_cast<uint4*>(hlast)[h] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (tid == 0) *s_tot = 0ull;
  lds_barrier();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const uint32_t j = tid + k * NT;
    if (j < mp) {
      const uint64_t x = it[j];
      const uint64_t gr = item_group(x);
      uint32_t h = (uint32_t)index_hash(gr) & kMask;
      while (true) {
        const uint32_t old = atomicCAS(&hidx[h], kNone, j);
        if (old == kNone || item_group(it[old]) == gr) break;
        h = (h + 1) & kMask;
      }
      atomicMax(&hlast[h], item_pos(x) + 1u);
    }
  }
  lds_barrier();
  // the items of the keys' last positions, at the front of it (in any order)
  uint64_t x[HPT];
  uint32_t n = 0;
  {
    const uint4 hi = reinterpret_cast<const uint4*>(hidx)[tid], hl = reinterpret_cast<const uint4*>(hlast)[tid];
    const uint32_t j[HPT] = {hi.x, hi.y, hi.z, hi.w};
    const uint32_t l[HPT] = {hl.x, hl.y, hl.z, hl.w};
#pragma unroll
    for (int q = 0; q < HPT; ++q)
      if (j[q] != kNone) x[n++] = (it[j[q]] & ~0x7FFFFFFFull) | (uint64_t)(l[q] - 1u);
  }
  uint32_t to = (uint32_t)claim_u64(n, s_tot);
  lds_barrier();  // every item has been read, every share claimed
#pragma unroll
  for (uint32_t q = 0; q < (uint32_t)HPT; ++q)
    if (q < n) it[to + q] = x[q];
  lds_barrier();
  write_values<NT, VEC, kClk>((uint32_t)*s_tot, a, store, [&](uint32_t s) { return it[s]; });
}

// Run-length encodes items sorted by value: seg[s] = first item of segment s,
// seg[S] = mp; sid[j] = segment of item j. Returns S (block-uniform).
template <int NT, class IP, class SP, class QP>
__device__ __forceinline__ uint32_t encode_segments(IP it, uint32_t mp, SP seg, QP sid, uint32_t* s_w) {
  uint32_t S = 0;
  for (uint32_t b0 = 0; b0 < mp; b0 += NT) {
    const uint32_t j = b0 + threadIdx.x;
    const uint32_t head = (j < mp) && (j == 0 || item_group(it[j]) != item_group(it[j - 1])) ? 1u : 0u;
    uint32_t tot;
    const uint32_t pre = block_exclusive_scan<NT>(head, s_w, &tot);
    if (head) seg[S + pre] = j;
    if (j < mp) sid[j] = S + pre + head - 1u;
    S += tot;
  }
  if (threadIdx.x == 0) seg[S] = mp;
  __syncthreads();
  return S;
}

// The units of items sorted by key it[0, m), S segments starting at seg[s]
// (seg[S] = m), sid[j] the segment of item j; a segment's items keep their
// order. s_to: NT words. The items are written out by all threads: with one
// thread writing a hot key's items, one of every put tile, a radix put of 1M
// lookups (Zipf 1.1) took 421 us at dim 128 and 213 at dim 4, now 407 and 197.
template <int NT, class IP, class SP, class QP>
__device__ __forceinline__ void units_of_sorted(IP it, SP seg, QP sid, uint32_t S, const PutUnits& u, Ctrl* ctrl,
                                                unsigned long long* s_tot, uint32_t* s_base, uint32_t* s_to) {
  for (uint32_t s0 = 0; s0 < S; s0 += NT) {
    const uint32_t s = s0 + threadIdx.x;
    if (threadIdx.x == 0) *s_tot = 0ull;
    __syncthreads();
    uint32_t n = 0, b = 0;
    uint64_t x = 0;
    bool one = false;
    if (s < S) {
      b = seg[s];
      n = seg[s + 1] - b;
      x = it[b];
      one = n == 1 && !item_summed(x);
    }
    // the packed counts hold 2^16 items: a unit of many claims its items by itself
    constexpr uint32_t kBig = 64;
    static_assert(kBig * NT <= (1 << 16), "packed item counts");
    const bool big = !one && n >= kBig;
    uint64_t mine = 0;
    if (s < S)
      mine = one ? pack_unit(1, 0, 0, 0)
                 : n > u.long_over ? pack_unit(0, 0, 1, big ? 0u : n) : pack_unit(0, 1, 0, n);
    const uint64_t pre = claim_u64(mine, s_tot);
    __syncthreads();
    if (threadIdx.x == 0) claim_units(ctrl, *s_tot, s_base);
    __syncthreads();
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    uint32_t to = kNone;  // where the segment's items go, less its first item's place
    if (s < S) {
      UnitCursor at(pre, s_base);
      if (big) at.c[3] = (uint32_t)(atomicAdd(&ctrl->unit_single, (unsigned long long)n << 32) >> 32);
      if (!one) to = at.c[3];
      emit_unit(u, at, x, n, one);
    }
    s_to[threadIdx.x] = to;
    __syncthreads();
    const uint32_t jb = seg[s0], je = seg[min(S, s0 + NT)];
    for (uint32_t j = jb + threadIdx.x; j < je; j += NT) {
      const uint32_t y = sid[j], d = s_to[y - s0];
      if (d != kNone) u.mitem[d + (j - seg[y])] = item_low31(it[j]);
    }
    __syncthreads();
  }
}

// An upsert of items sorted by key, then position (see units_of_sorted).
template <int NT, int VEC, bool kClk, class IP, class SP>
__device__ __forceinline__ void upsert_sorted(IP it, SP seg, uint32_t S, const PutGroupArgs& a,
                                              const RowStore& store) {
  for (uint32_t s0 = 0; s0 < S; s0 += NT)
    write_values<NT, VEC, kClk>(min((uint32_t)NT, S - s0), a, store,
                                [&](uint32_t s) { return it[seg[s0 + s + 1] - 1]; });
}

// Partition of more items than the block groups in LDS (a few keys with an item
// in nearly every put tile): the items are sorted in place, in the block's LDS
// if kSortLds hold them, else in a global scratch area (a put of 1M lookups of
// 1024 keys, dim 64: 384 us with every sort in the scratch area, 243 so).
constexpr int kSortLds = 8192;
static_assert(8 * (kSortLds + kGroupThreads / 2) <= (int)GroupLds::w64, "the sorted items and s_to fit beside s_w and s_misc");
template <bool kUpsert, int VEC, bool kClk>
__device__ __forceinline__ void group_partition_global(const PutGroupArgs& a, const RowStore& store, uint32_t p, uint32_t mp, uint32_t* s_w,
                                                      uint64_t* s_misc, uint64_t* s_it) {
  constexpr int NT = kGroupThreads;
  uint32_t* s_to = reinterpret_cast<uint32_t*>(s_it + kSortLds);
  uint32_t P2 = 1;
  while (P2 < mp) P2 <<= 1;
  if (threadIdx.x == 0) {
    const uint64_t need = 2ull * P2 + 2;
    const uint64_t b = atomicAdd(&a.ctrl->spill_next, (unsigned long long)need);
    s_misc[0] = (b + need <= a.spill_words) ? b : ~0ull;
  }
  __syncthreads();
  const uint64_t base = s_misc[0];
  __syncthreads();
  if (base == ~0ull) {  // cannot happen when the spill area holds 4n words
    if (threadIdx.x == 0) atomicCAS(&a.ctrl->latched, 0, -4);
    return;
  }
  uint32_t* seg = reinterpret_cast<uint32_t*>(a.spill + base + P2);  // [mp + 1], then [mp] segments of the items
  uint32_t* sid = seg + mp + 1;
  auto group = [&](uint64_t* it) {
    uint32_t dst = 0;
    for (int t0 = 0; t0 < a.ntiles; t0 += NT) {
      const int t = t0 + (int)threadIdx.x;
      const uint32_t mt = t < a.ntiles ? a.meta[(size_t)p * a.ntiles + t] : 0u;
      const uint32_t off = mt & 0xFFFFu, cnt = mt >> 16;
      uint32_t tot;
      const uint32_t pre = block_exclusive_scan<NT>(cnt, s_w, &tot);
      for (uint32_t j = 0; j < cnt; ++j) it[dst + pre + j] = a.items[(size_t)t * kPutTile + off + j];
      dst += tot;
    }
    for (uint32_t j = mp + threadIdx.x; j < P2; j += NT) it[j] = ~0ull;
    __syncthreads();
    block_bitonic_sort<NT>(it, P2);
    const uint32_t S = encode_segments<NT>(it, mp, seg, sid, s_w);
    if constexpr (kUpsert) upsert_sorted<NT, VEC, kClk>(it, seg, S, a, store);
    else units_of_sorted<NT>(it, seg, sid, S, a.units, a.ctrl, reinterpret_cast<unsigned long long*>(s_misc),
                             reinterpret_cast<uint32_t*>(s_misc + 2), s_to);
  };
  if (P2 <= (uint32_t)kSortLds) group(s_it);
  else group(a.spill + base);
}

// The verdict of a put call (see call_verdict); a put whose probe ran ahead
// of a get marks its errors in fields of its own.
struct PutVerdict {
  uint64_t size0, M;
  int err;
};
template <int NT>
__device__ __forceinline__ PutVerdict put_verdict(Ctrl* ctrl, uint64_t epoch, int64_t capacity,
                                                  const uint32_t* tile_cnt, int ntiles, unsigned long long* s_w64) {
  PutVerdict v;
  v.size0 = ctrl->size[epoch & 1];
  const uint64_t new_e = ctrl->new_epoch, ovf_e = ctrl->overflow_epoch;
  const uint64_t bad_e = ctrl->apput_bad_epoch == epoch ? epoch : ctrl->bad_epoch;
  const uint64_t abs_e = ctrl->apput_absent_epoch;
  v.M = new_e == epoch ? count_new_keys<NT>(tile_cnt, ntiles, s_w64) : 0ull;
  v.err = call_verdict(ctrl, epoch, v.size0, v.M, capacity, bad_e, ovf_e, abs_e);
  return v;
}

template <bool kUpsert, int VEC, bool kClk>
__global__ __launch_bounds__(kGroupThreads, 8) void k_put_group(const PutGroupArgs a, const AssignArgs aa,
                                                                const RowStore store, uint64_t seed) {
  using L = GroupLds;
  constexpr int NT = kGroupThreads;
  constexpr int IPT = kRedCap / NT;
  extern __shared__ __align__(16) unsigned char s_raw[];
  uint64_t* s_it = reinterpret_cast<uint64_t*>(s_raw + L::it);
  uint32_t* s_pref = reinterpret_cast<uint32_t*>(s_raw + L::pref);
  uint32_t* s_w = reinterpret_cast<uint32_t*>(s_raw + L::w);
  unsigned long long* s_w64 = reinterpret_cast<unsigned long long*>(s_raw + L::w64);

  const uint32_t p = blockIdx.x;
  const int tid = threadIdx.x, ntiles = a.ntiles;
  const uint32_t* pm = a.meta + (size_t)p * ntiles;
  const bool one_chunk = ntiles <= NT;  // common case: one thread per tile
  const uint32_t mt0 = one_chunk && p < a.parts && tid < ntiles ? pm[tid] : 0u;

  // entries of this partition in every tile (blocks past the partitions only assign rows)
  uint32_t mp = 0, pre0 = 0;
  if (p >= a.parts) {
  } else if (one_chunk) {
    pre0 = block_exclusive_scan<NT>(mt0 >> 16, s_w, &mp);
  } else {
    uint64_t mp64 = 0;
    for (int t = tid; t < ntiles; t += NT) mp64 += pm[t] >> 16;
    mp = (uint32_t)block_sum_u64<NT>(mp64, s_w64);
  }
  const PutVerdict v = put_verdict<NT>(a.ctrl, a.epoch, a.capacity, aa.tile_cnt, ntiles, s_w64);

  if (!v.err && mp > (uint32_t)kRedCap) {
    group_partition_global<kUpsert, VEC, kClk>(a, store, p, mp, s_w, reinterpret_cast<uint64_t*>(s_raw + L::misc), s_it);
  } else if (!v.err && mp > 0) {
    // ---- gather the partition's items into LDS, tile order ----
    uint32_t dst = 0;
    for (int t0 = 0; t0 < ntiles; t0 += NT) {
      const int nt = min(NT, ntiles - t0);
      uint32_t mt = mt0, pre = pre0, tot = mp;
      if (!one_chunk) {
        mt = tid < nt ? pm[t0 + tid] : 0u;
        pre = block_exclusive_scan<NT>(mt >> 16, s_w, &tot);
      }
      s_pref[tid] = pre | (mt << 16);  // items before this tile | offset in the tile
      __syncthreads();
      uint64_t x[IPT];
#pragma unroll
      for (int e = 0; e < IPT; ++e) {
        const uint32_t k = tid + e * NT;
        x[e] = 0;
        if (k < tot) {
          int lo = 0, hi = nt - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if ((s_pref[mid] & 0xFFFFu) <= k) lo = mid;
            else hi = mid - 1;
          }
          const uint32_t pe = s_pref[lo];
          x[e] = a.items[(size_t)(t0 + lo) * kPutTile + (pe >> 16) + (k - (pe & 0xFFFFu))];
        }
      }
#pragma unroll
      for (int e = 0; e < IPT; ++e) {
        const uint32_t k = tid + e * NT;
        if (k < tot) s_it[dst + k] = x[e];
      }
      dst += tot;
      __syncthreads();
    }
    if constexpr (kUpsert) upsert_last<VEC, kClk>(s_raw, mp, a, store);
    else group_by_key(s_raw, mp, a.units, a.ctrl);
  }
  if (v.M != 0 && p < aa.blocks) {
    __syncthreads();  // the grouping's LDS is free
    assign_new<NT, kPutTile>(aa, store, seed, v.size0, v.M, v.err, *reinterpret_cast<AssignLds<NT>*>(s_raw));
  }
}

#endif  // MLKV_MAP

// One lane's VEC elements of a row, fp32 (a gradient row) or fp64 (an in-tile
// sum), as loaded.
template <int VEC>
struct RawRow;
template <>
struct RawRow<4> {
  Words4 lo, hi;
};
template <>
struct RawRow<1> {
  uint2 lo;
};

template <int VEC, bool kStream>
__device__ __forceinline__ void load_raw(RawRow<VEC>& r, const float* __restrict__ grads,
                                         const double* __restrict__ partials, size_t off, bool summed) {
  if constexpr (VEC == 4) {
    if (summed) {
      const Words4* p = reinterpret_cast<const Words4*>(partials + off);
      r.lo = p[0];
      r.hi = p[1];
    } else {
      const Words4* p = reinterpret_cast<const Words4*>(grads + off);
      if constexpr (kStream) r.lo = __builtin_nontemporal_load(p);
      else r.lo = *p;
    }
  } else {
    if (summed) r.lo = *reinterpret_cast<const uint2*>(partials + off);
    else r.lo.x = *reinterpret_cast<const uint32_t*>(grads + off);
  }
}

template <int VEC>
__device__ __forceinline__ void add_raw(double* acc, const RawRow<VEC>& r, bool summed) {
  if constexpr (VEC == 4) {
    if (summed) {
      acc[0] += __hiloint2double((int)r.lo.y, (int)r.lo.x);
      acc[1] += __hiloint2double((int)r.lo.w, (int)r.lo.z);
      acc[2] += __hiloint2double((int)r.hi.y, (int)r.hi.x);
      acc[3] += __hiloint2double((int)r.hi.w, (int)r.hi.z);
    } else {
      acc[0] += (double)__uint_as_float(r.lo.x);
      acc[1] += (double)__uint_as_float(r.lo.y);
      acc[2] += (double)__uint_as_float(r.lo.z);
      acc[3] += (double)__uint_as_float(r.lo.w);
    }
  } else {
    acc[0] += summed ? __hiloint2double((int)r.lo.y, (int)r.lo.x) : (double)__uint_as_float(r.lo.x);
  }
}

// ---------------------------------------------------------------------------
// Put, third kernel: the update of every unit (Adagrad or SGD). First the long
// units, a block each (see lane_max): its lane groups take the unit's items in turn, and
// their fp64 sums are added in a fixed order (across the wave's groups, then
// across waves). Then the other sums, a lane group each, items in order; then
// the keys seen once, a lane group each. Which block takes which unit changes
// no result.
// Bound by HBM: gradient rows and in-tile sums in, table rows in and out.
// ---------------------------------------------------------------------------
constexpr int kApplyThreads = 256;
template <class M>
struct ApplyCfg {
  static constexpr int B = (M::K * M::VEC >= 8) ? 2 : 4;       // rows of a sum a group has in flight
  // gradient rows of 256 bytes and more are read around the caches; shorter
  // ones share their lines with other keys' rows
  static constexpr bool kStream = M::LPR * M::VEC >= 64;
  // waves per SIMD. Six with a key seen once at a time: two at a time and five
  // waves took 99 us against 96.5 (a put of 213k uniform keys, dim 128), 603
  // against 584 (1M, dim 256); eight spill (113 us).
  static constexpr int WAVES = (M::K * M::VEC >= 16) ? 3 : (M::K * M::VEC >= 8) ? 4 : 6;
};

template <class M, bool kClk>
__global__ __launch_bounds__(kApplyThreads, ApplyCfg<M>::WAVES) void k_put_apply(const PutApplyArgs a,
                                                                                const RowStore store) {
  using Ops = SegmentOps<M>;
  constexpr int VEC = M::VEC, LPR = M::LPR, K = M::K, RPW = M::RPW;
  constexpr int NW = kApplyThreads / 64, NG = NW * RPW;
  constexpr int B = ApplyCfg<M>::B, DMAX = LPR * K * VEC;
  constexpr bool kStream = ApplyCfg<M>::kStream;
  using V = typename VecT<VEC>::T;
  __shared__ double s_sum[NW][DMAX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane % LPR;
  const int gid = wave * RPW + lane / LPR;
  const int D = store.D;
  const bool d_pow2 = (D & (D - 1)) == 0;
  const double inv_d = 1.0 / (double)D;
  const bool adagrad = a.op == kOpAdagrad;
  const bool clk = kClk && q == 0;

  // the row of a unit, loaded ahead of its update
  V w[K];
  float G = 0.0f;
  uint32_t cl = 0u;
  auto load_row = [&](uint32_t row, const float* wr) {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (M::on(k, q, D)) w[k] = load_vec<VEC>(wr + M::col(k, q, D));
    if (adagrad) G = a.state[row];
    if (clk) cl = clock_low(a.clock, row);
  };
  auto update = [&](const double (&acc)[K][VEC], uint32_t row, float* wr) {
    V g[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int x = 0; x < VEC; ++x) VecT<VEC>::set(g[k], x, (float)acc[k][x]);
    if (adagrad) Ops::adagrad(g, w, G, wr, a.state, row, D, q, d_pow2, inv_d, a.lr, a.eps);
    else Ops::sgd(g, w, wr, D, q, a.lr);
    if (clk) put_clock_low(a.clock, row, cl);
  };
  // adds items [j, end) by steps of `step` to acc, B of them in flight
  double acc[K][VEC];
  auto add_items = [&](const uint32_t* __restrict__ items, uint32_t j, uint32_t end, uint32_t step) {
    for (; j < end; j += B * step) {
      RawRow<VEC> raw[B][K];
      uint32_t x[B];
#pragma unroll
      for (int u = 0; u < B; ++u) x[u] = j + u * step < end ? items[j + u * step] : 0u;
#pragma unroll
      for (int u = 0; u < B; ++u) {
        if (j + u * step < end) {
          const size_t base = (size_t)(x[u] & 0x3FFFFFFFu) * (size_t)D;
#pragma unroll
          for (int k = 0; k < K; ++k)
            if (M::on(k, q, D))
              load_raw<VEC, kStream>(raw[u][k], a.grads, a.partials, base + M::col(k, q, D), (x[u] & (uint32_t)kItemSummed) != 0);
        }
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        if (j + u * step < end) {
#pragma unroll
          for (int k = 0; k < K; ++k)
            if (M::on(k, q, D)) add_raw<VEC>(acc[k], raw[u][k], (x[u] & (uint32_t)kItemSummed) != 0);
        }
      }
    }
  };
  auto zero = [&]() {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int x = 0; x < VEC; ++x) acc[k][x] = 0.0;
  };

  // ---- long units ----
  const uint32_t nl = (uint32_t)(a.ctrl->unit_multi >> 32);
  // Where there are more of them than blocks, lane groups take the shorter ones
  // with the other sums: a block each took 217 us for 1M lookups of 65,536 keys
  // (dim 4, about 16 items a key; with lane groups 123, the earlier single kernel
  // 134) and 69 for 213k of 16,384 (43, 34). Up to 64 items each against 32 is
  // 120 us and 141 for 1M of 32,768 keys, 59 and 51 for 213k of 4096.
  const uint32_t lane_max = nl > 8u * gridDim.x ? 64u : nl > gridDim.x ? 32u : 0u;
  for (uint32_t e = blockIdx.x; e < nl; e += gridDim.x) {
    const uint4 t = a.units.lng[e];
    const uint32_t n = t.y & ~kUnitFresh;
    if (n <= lane_max) continue;  // (block-uniform)
    uint32_t row = 0;
    float* wr = nullptr;
    if (gid == 0) {
      row = unit_row(a.idx, t.x, (t.y & kUnitFresh) != 0);
      wr = store.wptr(row);
      load_row(row, wr);
    }
    zero();
    add_items(a.units.mitem + t.z, gid, n, NG);
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int x = 0; x < VEC; ++x) {
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) acc[k][x] += __shfl_xor(acc[k][x], o, 64);
        if (lane < LPR) s_sum[wave][(k * LPR + q) * VEC + x] = acc[k][x];
      }
    }
    __syncthreads();
    if (gid == 0) {
#pragma unroll
      for (int o = 1; o < NW; ++o)
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
          for (int x = 0; x < VEC; ++x) acc[k][x] += s_sum[o][(k * LPR + q) * VEC + x];
      update(acc, row, wr);
    }
    __syncthreads();
  }

  // ---- other sums ----
  const uint32_t groups = gridDim.x * NG, g0 = blockIdx.x * NG + gid;
  const uint32_t nm = (uint32_t)a.ctrl->unit_multi;
  for (uint32_t e = g0; e < nm + (lane_max != 0u ? nl : 0u); e += groups) {
    const uint4 t = e < nm ? a.units.multi[e] : a.units.lng[e - nm];
    if (e >= nm && (t.y & ~kUnitFresh) > lane_max) continue;
    const uint32_t row = unit_row(a.idx, t.x, (t.y & kUnitFresh) != 0);
    float* wr = store.wptr(row);
    load_row(row, wr);
    zero();
    add_items(a.units.mitem + t.z, 0, t.y & ~kUnitFresh, 1);
    update(acc, row, wr);
  }

  // ---- keys seen once: g is the key's gradient row ----
  const uint32_t ns = (uint32_t)a.ctrl->unit_single;
  for (uint32_t e = g0; e < ns; e += groups) {
    const uint64_t x = a.units.single[e];
    const uint32_t row = unit_row(a.idx, item_tag(x), item_fresh(x));
    float* wr = store.wptr(row);
    const float* gr = a.grads + (size_t)item_pos(x) * (size_t)D;
    V g[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (M::on(k, q, D)) g[k] = load_vec_once<VEC, kStream>(gr + M::col(k, q, D));
    load_row(row, wr);
    if (adagrad) Ops::adagrad(g, w, G, wr, a.state, row, D, q, d_pow2, inv_d, a.lr, a.eps);
    else Ops::sgd(g, w, wr, D, q, a.lr);
    if (clk) put_clock_low(a.clock, row, cl);
  }
}

// ===========================================================================
// Put with dedup by radix sort (Dedup kDedupRadix), the alternative to the
// hash partition: put_probe with a single partition (its in-tile sums leave
// each key at most one item per put tile), then a stable LSD radix sort of
// all items by the key's row (rows below capacity, keys new in the call by
// capacity + index slot), in passes of at most kRsMaxBits bits, each a count
// kernel and a scatter kernel; then blocks that take even shares of the
// sorted items, each cut moved forward to the start of a key's run,
// run-length encode them in LDS and write the units that put_group writes.
// Stability keeps a key's items in put-tile order, which is position order.
// ===========================================================================
static_assert(kRsTile == 4 * kPutTile, "a radix tile is four put tiles");
constexpr int kRsThreads = 1024;
constexpr int kRsPer = kRsTile / kRsThreads;
constexpr int kRsDigits = 1 << kRsMaxBits;

__device__ __forceinline__ uint32_t rs_key(uint64_t x, uint32_t cap) {
  return item_fresh(x) ? cap + item_tag(x) : item_tag(x);
}

// Loads the tile's items: v[k] = item of element k * kRsThreads + tid, ok[k]
// whether it exists.
__device__ __forceinline__ void rs_load(const RsSrc& s, uint64_t (&v)[kRsPer], bool (&ok)[kRsPer]) {
  const int64_t base = (int64_t)blockIdx.x * kRsTile;
  const uint32_t T = s.meta == nullptr ? *s.total : 0u;
#pragma unroll
  for (int k = 0; k < kRsPer; ++k) {
    const int64_t i = base + k * kRsThreads + threadIdx.x;
    if (s.meta != nullptr) {
      const int pt = (int)(i / kPutTile);
      ok[k] = pt < s.ntiles && (uint32_t)(i % kPutTile) < (s.meta[pt] >> 16);
    } else {
      ok[k] = i < (int64_t)T;
    }
    v[k] = ok[k] ? s.src[i] : 0ull;
  }
}

#ifndef MLKV_MAP
// Digit counts of one radix tile: cnt[d * stride + tile], digit-major, so that
// a digit's counts over the tiles are contiguous (stride >= tiles, a multiple of 4).
__global__ __launch_bounds__(kRsThreads) void k_rsort_count(RsSrc s, uint32_t cap, int shift, int bits,
                                                            uint32_t* __restrict__ cnt, int stride) {
  __shared__ uint32_t h[kRsDigits];
  const int R = 1 << bits;
  for (int d = threadIdx.x; d < R; d += kRsThreads) h[d] = 0;
  uint64_t v[kRsPer];
  bool ok[kRsPer];
  rs_load(s, v, ok);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRsPer; ++k)
    if (ok[k]) atomicAdd(&h[(rs_key(v[k], cap) >> shift) & (uint32_t)(R - 1)], 1u);
  __syncthreads();
  for (int d = threadIdx.x; d < R; d += kRsThreads) cnt[(size_t)d * stride + blockIdx.x] = h[d];
}

// Stable scatter of one radix tile by digit. An item goes to: items of smaller
// digits in all tiles + items of its digit in earlier tiles + items of its
// digit before it in this tile. The last term comes from a multisplit per
// wave (lanes with the same digit found by one ballot per digit bit), waves
// and batches taken in element order.
__global__ __launch_bounds__(kRsThreads) void k_rsort_scatter(RsSrc s, uint32_t cap, int shift, int bits,
                                                              const uint32_t* __restrict__ cnt, int rtiles,
                                                              int stride, uint64_t* __restrict__ dst,
                                                              uint32_t* __restrict__ total_out) {
  constexpr int NT = kRsThreads, NW = NT / 64;
  __shared__ uint32_t s_wc[NW * kRsDigits];  // per wave and digit: items, then where they start
  __shared__ uint32_t s_run[kRsDigits];      // per digit: where the next batch's items start
  __shared__ uint32_t s_w[NW];
  const int R = 1 << bits;  // 16 .. kRsDigits
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = blockIdx.x;
  uint64_t v[kRsPer];
  bool ok[kRsPer];
  rs_load(s, v, ok);
  // the TPD threads of a digit (adjacent lanes) share the digit's counts
  // over the tiles, four at a time (a digit's row is 16-byte aligned; the
  // entries past the last tile are not counts)
  {
    const int TPD = NT / R;
    const int d = tid / TPD, part = tid % TPD;
    uint32_t all = 0, before = 0;
    const uint4* row = reinterpret_cast<const uint4*>(cnt + (size_t)d * stride);
    for (int u4 = part; u4 * 4 < rtiles; u4 += TPD) {
      const uint4 c = row[u4];
      const int u = u4 * 4;
      const uint32_t c0 = c.x, c1 = u + 1 < rtiles ? c.y : 0u, c2 = u + 2 < rtiles ? c.z : 0u,
                     c3 = u + 3 < rtiles ? c.w : 0u;
      all += c0 + c1 + c2 + c3;
      before += (u < t ? c0 : 0u) + (u + 1 < t ? c1 : 0u) + (u + 2 < t ? c2 : 0u) + (u + 3 < t ? c3 : 0u);
    }
    for (int o = 1; o < TPD; o <<= 1) {
      all += __shfl_xor(all, o, 64);
      before += __shfl_xor(before, o, 64);
    }
    uint32_t T;
    const uint32_t ex = block_exclusive_scan<NT>(part == 0 ? all : 0u, s_w, &T);
    if (part == 0) s_run[d] = ex + before;
    if (total_out != nullptr && t == 0 && tid == 0) *total_out = T;
  }
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int k = 0; k < kRsPer; ++k) {
    for (int e = tid; e < NW * R; e += NT) s_wc[e] = 0u;
    const uint32_t dg = ok[k] ? (rs_key(v[k], cap) >> shift) & (uint32_t)(R - 1) : 0u;
    uint64_t m = __ballot(ok[k] ? 1 : 0);
    for (int b = 0; b < bits; ++b) {
      const bool on = (dg >> b) & 1u;
      const uint64_t bb = __ballot(on ? 1 : 0);
      m &= on ? bb : ~bb;
    }
    const uint32_t rank = (uint32_t)__popcll(m & lt);
    __syncthreads();  // the table is cleared (and s_run written)
    if (ok[k] && rank == 0) s_wc[wave * R + dg] = (uint32_t)__popcll(m);
    __syncthreads();
    if (tid < R) {
      uint32_t run = s_run[tid];
      for (int w = 0; w < NW; ++w) {
        const uint32_t c = s_wc[w * R + tid];
        s_wc[w * R + tid] = run;
        run += c;
      }
      s_run[tid] = run;
    }
    __syncthreads();
    if (ok[k]) dst[s_wc[wave * R + dg] + rank] = v[k];
    __syncthreads();  // before the table is cleared again
  }
}
#endif  // MLKV_MAP

// Cut points of the sorted items at or after p[0] and p[1]: the first position
// q >= p where a key's run starts (q = T if none), both looked for at once.
template <int NT>
__device__ __forceinline__ void rs_cuts(const uint64_t* __restrict__ it, uint32_t T, uint32_t (&p)[2],
                                        uint32_t* s_min) {
  bool done[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    done[k] = p[k] == 0 || p[k] >= T;
    if (done[k]) p[k] = min(p[k], T);
  }
  while (!done[0] || !done[1]) {  // (block-uniform)
    if (threadIdx.x < 2) s_min[threadIdx.x] = T;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t q = p[k] + threadIdx.x;
      if (!done[k] && q < T && item_group(it[q]) != item_group(it[q - 1])) atomicMin(&s_min[k], q);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (done[k]) continue;
      const uint32_t f = s_min[k], next = p[k] + NT;
      done[k] = f < T || next >= T;
      p[k] = f < T ? f : min(next, T);
    }
    __syncthreads();
  }
}

#ifndef MLKV_MAP
template <bool kUpsert, int VEC, bool kClk>
__global__ __launch_bounds__(kGroupThreads) void k_rsort_group(const PutGroupArgs a,
                                                               const uint32_t* __restrict__ total, const AssignArgs aa,
                                                               const RowStore store, uint64_t seed) {
  using L = GroupLds;
  constexpr int NT = kGroupThreads;
  extern __shared__ __align__(16) unsigned char s_raw[];
  uint64_t* s_it = reinterpret_cast<uint64_t*>(s_raw + L::it);
  uint32_t* s_seg = reinterpret_cast<uint32_t*>(s_raw + L::hidx);  // [kRedCap + 1]
  uint16_t* s_sid = reinterpret_cast<uint16_t*>(s_raw + L::slot);  // [kRedCap]
  uint32_t* s_w = reinterpret_cast<uint32_t*>(s_raw + L::w);
  unsigned long long* s_w64 = reinterpret_cast<unsigned long long*>(s_raw + L::w64);
  unsigned long long* s_tot = reinterpret_cast<unsigned long long*>(s_raw + L::misc);
  uint32_t* s_base = reinterpret_cast<uint32_t*>(s_raw + L::misc + 16);
  static_assert(kRedHash >= kRedCap + 1, "run starts fit the hash region");

  const PutVerdict v = put_verdict<NT>(a.ctrl, a.epoch, a.capacity, aa.tile_cnt, a.ntiles, s_w64);
  const uint32_t T = *total;
  // the first nb blocks share the items, at least about NT each (in-tile sums
  // leave fewer than the call's keys): 65k keys of dim 64 80 -> 77.5 us. An
  // upsert's blocks also write the rows and all take part.
  const uint32_t nb = kUpsert ? gridDim.x : min(gridDim.x, max(1u, (T + NT - 1u) / NT)), b = blockIdx.x;
  uint32_t cut[2] = {(uint32_t)((uint64_t)T * min(b, nb) / nb), (uint32_t)((uint64_t)T * min(b + 1u, nb) / nb)};
  rs_cuts<NT>(a.items, T, cut, s_base);
  const uint32_t lo = cut[0], m = cut[1] - lo;
  if (!v.err && m > (uint32_t)kRedCap) {  // runs are at most one item per put tile; the host keeps this from happening
    if (threadIdx.x == 0) atomicCAS(&a.ctrl->latched, 0, -4);
  } else if (!v.err && m > 0) {
    for (uint32_t j = threadIdx.x; j < m; j += NT) s_it[j] = a.items[lo + j];
    __syncthreads();
    const uint32_t S = encode_segments<NT>(s_it, m, s_seg, s_sid, s_w);
    if constexpr (kUpsert) upsert_sorted<NT, VEC, kClk>(s_it, s_seg, S, a, store);
    else units_of_sorted<NT>(s_it, s_seg, s_sid, S, a.units, a.ctrl, s_tot, s_base,
                             reinterpret_cast<uint32_t*>(s_raw + L::hcnt));
  }
  if (v.M != 0 && b < aa.blocks) {
    __syncthreads();
    assign_new<NT, kPutTile>(aa, store, seed, v.size0, v.M, v.err, *reinterpret_cast<AssignLds<NT>*>(s_raw));
  }
}
#endif  // MLKV_MAP

#ifndef MLKV_MAP
// ===========================================================================
// Inspection kernels
// ===========================================================================
__global__ __launch_bounds__(256) void k_lookup(Bucket* __restrict__ idx, uint32_t nb_log2,
                                                const uint64_t* __restrict__ keys, int64_t n,
                                                int64_t* __restrict__ rows_out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint64_t key = keys[i];
  int64_t r = -1;
  if (key != kEmptyKey) {
    const Probe pr = probe_key(idx, nb_log2, key, false);
    if (pr.status == P_HIT) r = pr.row;
  }
  rows_out[i] = r;
}

__global__ __launch_bounds__(256) void k_export_slots(const Bucket* __restrict__ idx, uint64_t nslots,
                                                      uint64_t* __restrict__ keys_out,
                                                      uint32_t* __restrict__ rows_out) {
  const uint64_t s = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= nslots) return;
  const Bucket* B = idx + s / kSlots;
  if (keys_out) keys_out[s] = B->key[s % kSlots];
  if (rows_out) rows_out[s] = B->row[s % kSlots];
}

// Copies rows and accumulators by row id; ids outside [0, size) give NaN
// rows and latch MLKV_EINVAL (-1).
__global__ __launch_bounds__(256) void k_read_rows(const RowStore store, const float* __restrict__ state,
                                                   int D, const unsigned long long* size_now,
                                                   const int64_t* __restrict__ ids, int64_t n,
                                                   float* __restrict__ w_out, float* __restrict__ st_out,
                                                   Ctrl* ctrl) {
  const uint64_t size = *size_now;
  const uint64_t total = (uint64_t)n * (uint64_t)D;
  for (uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (uint64_t)gridDim.x * 256) {
    const uint64_t i = e / (uint64_t)D;
    const int c = (int)(e % (uint64_t)D);
    const int64_t r = ids[i];
    const bool ok = r >= 0 && (uint64_t)r < size;
    if (!ok && c == 0) atomicCAS(&ctrl->latched, 0, -1);
    if (w_out) w_out[e] = ok ? store.ptr((uint32_t)r)[c] : __builtin_nanf("");
    if (st_out && c == 0) st_out[i] = ok ? state[r] : __builtin_nanf("");
  }
}

// Staleness counts by row id; ids outside [0, size) give 0xFFFFFFFF and
// latch MLKV_EINVAL (-1).
__global__ __launch_bounds__(256) void k_read_clock(const unsigned long long* __restrict__ clock,
                                                    const unsigned long long* size_now,
                                                    const int64_t* __restrict__ ids, int64_t n,
                                                    uint32_t* __restrict__ out, Ctrl* ctrl) {
  const uint64_t size = *size_now;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < (uint64_t)n; i += (uint64_t)gridDim.x * 256) {
    const int64_t r = ids[i];
    const bool ok = r >= 0 && (uint64_t)r < size;
    if (!ok) atomicCAS(&ctrl->latched, 0, -1);
    out[i] = ok ? (uint32_t)(clock[r] & kClockCount) : 0xFFFFFFFFu;
  }
}
#endif  // MLKV_MAP

// ===========================================================================
// Launchers
// ===========================================================================
#ifndef MLKV_MAP
template <int VEC, int LPR, bool kStream>
static auto probe_kernel(const GetArgs& a) {
  return a.clock != nullptr ? k_get_probe<VEC, LPR, true, false, kStream>
         : a.pc_in          ? k_get_probe<VEC, LPR, false, true, kStream>
                            : k_get_probe<VEC, LPR, false, false, kStream>;
}

// Lanes a row with which the probe kernel copies rows of `units` accesses; 0:
// the second kernel copies them. Copied with the probe, other waves' lookups
// hide the row copy's latency and one launch has nothing to copy; apart, the
// probe has twice the waves in flight and the copy evens out its work. Times of
// one get in us, copied with the probe / apart, rows drawn uniformly:
//   dim      16k keys      131k          213k          426k          1M
//    16     10.2/10.4    15.2/16.1     20.6/23.5     33.4/36.5     68.0/70.4
//    32     11.0/10.4    17.5/19.2     23.9/26.5     39.8/42.0     84.8/86.4
//    64     12.8/10.7    23.0/26.2     34.9/36.1     70.6/61.3    149.3/143.3
// Rows of 5 accesses and more need more keys than one tile a CU, and those of
// 9 and more, whose kernel has 6 blocks of 256 lanes on a CU (78 registers), no
// more than these take at once. Wider rows are copied apart: 150k of dim 400 took
// 178 us with the probe and take 11 + 97, 1M of dim 128 274 and 46 + 189.
static int copy_lanes(uint64_t units, int64_t n, int cus) {
  if (units == 1) return 1;
  if (units <= 4) return 4;
  if (units > 16 || n <= (int64_t)kGetTile * cus) return 0;
  if (units <= 8) return 8;
  return n <= 6 * (int64_t)kGetTile * cus ? 16 : 0;
}

hipError_t launch_get(const GetArgs& a, hipStream_t st, const LaunchHook& hook) {
  const int tlen = get_tile_len(a.n, a.cus);
  const int64_t ntiles = (a.n + tlen - 1) / tlen;
  const uint32_t ranges = (uint32_t)std::min<int64_t>(ntiles, kMaxRanges);  // row assignment: a block per key range
  RangeLists rl = a.rl;
  if (rl.list != nullptr) rl.cap = (uint32_t)std::min<uint64_t>(rl.entries / ranges, 0xFFFFFFFFull);
  const int vec = a.D >= 4 ? 4 : 1;
  const uint64_t units = (uint64_t)(a.D + vec - 1) / vec;  // of a row
  const int lanes = a.out == nullptr || (vec == 1 && units > 1) ? 0 : copy_lanes(units, a.n, a.cus);
  const bool stream = (uint64_t)a.n * (uint64_t)a.D * sizeof(float) >= kStreamOut;
  hook(K_GET_PROBE, 0, st);
  auto kern = lanes == 0    ? probe_kernel<0, 0, false>(a)
              : lanes == 1  ? (vec == 4 ? probe_kernel<4, 1, false>(a) : probe_kernel<1, 1, false>(a))
              : lanes == 4  ? (stream ? probe_kernel<4, 4, true>(a) : probe_kernel<4, 4, false>(a))
              : lanes == 8  ? (stream ? probe_kernel<4, 8, true>(a) : probe_kernel<4, 8, false>(a))
                            : (stream ? probe_kernel<4, 16, true>(a) : probe_kernel<4, 16, false>(a));
  hipLaunchKernelGGL(kern, dim3((unsigned)ntiles), dim3(kGetTile), 0, st, a.idx, a.nb_log2, a.keys, a.n, a.out,
                     a.store, a.seed, a.newlist, a.tile_cnt, a.ctrl, a.epoch, a.clock, a.cepoch, a.bound, a.blocked,
                     a.pc_key, a.pos_row, tlen, rl, ranges);
  hook(K_GET_PROBE, 1, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const uint64_t per_block = (uint64_t)kCopyThreads * kCopyUnits;
  const bool copy = a.out != nullptr && lanes == 0;
  const uint64_t blocks =
      copy ? std::min<uint64_t>(((uint64_t)a.n * units + per_block - 1) / per_block, kCopyBlocks) : 0;
  GetRowsArgs r;
  r.out = copy ? a.out : nullptr;
  r.keys = a.keys;
  r.rows = a.pos_row;
  r.blocked = a.blocked;
  r.n = a.n;
  r.seed = a.seed;
  r.store = a.store;
  r.magic = units > 1 ? (uint32_t)((0x100000000ull + units - 1) / units) : 0u;
  AssignArgs s;
  s.idx = a.idx;
  s.newlist = a.newlist;
  s.tile_cnt = a.tile_cnt;
  s.ntiles = (int)ntiles;
  s.tile_size = tlen;
  s.state = a.state;
  s.capacity = a.capacity;
  s.ctrl = a.ctrl;
  s.epoch = a.epoch;
  s.xkey = a.xkey;
  s.xslot = a.xslot;
  s.clock = a.clock;
  s.cepoch = a.cepoch;
  s.rl = rl;
  s.values = nullptr;
  s.blocks = ranges;
  const unsigned grid = (unsigned)std::max<uint64_t>(blocks, ranges);
  const bool track = a.clock != nullptr;
  hook(K_GET_ROWS, 0, st);
  auto rows = vec != 4 ? (track ? k_get_rows<1, true, false> : k_get_rows<1, false, false>)
              : stream ? (track ? k_get_rows<4, true, true> : k_get_rows<4, false, true>)
                       : (track ? k_get_rows<4, true, false> : k_get_rows<4, false, false>);
  hipLaunchKernelGGL(rows, dim3(grid), dim3(kAssignThreads), 0, st, r, s);
  hook(K_GET_ROWS, 1, st);
  return hipGetLastError();
}

// One pass of the radix sort: counts, then the scatter by digit.
hipError_t launch_rsort_pass(const RsSrc& src, uint32_t cap, int shift, int bits, uint32_t* cnt, int rtiles,
                             int stride, uint64_t* dst, uint32_t* total_out, hipStream_t st,
                             const LaunchHook& hook) {
  hook(K_RSORT_COUNT, 0, st);
  hipLaunchKernelGGL(k_rsort_count, dim3((unsigned)rtiles), dim3(kRsThreads), 0, st, src, cap, shift, bits, cnt,
                     stride);
  hook(K_RSORT_COUNT, 1, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hook(K_RSORT_SCATTER, 0, st);
  hipLaunchKernelGGL(k_rsort_scatter, dim3((unsigned)rtiles), dim3(kRsThreads), 0, st, src, cap, shift, bits,
                     (const uint32_t*)cnt, rtiles, stride, dst, total_out);
  hook(K_RSORT_SCATTER, 1, st);
  return hipGetLastError();
}
#endif  // MLKV_MAP

// The probe kernel of a put, with 2^pb partitions.
template <class M>
hipError_t launch_put_probe_t(const PutArgs& a, int pb, hipStream_t st, const LaunchHook& hook) {
  const int64_t ntiles = (a.n + a.tlen - 1) / a.tlen;
  // an upsert keeps each key's last position; radix dedup has room for one item per key and tile
  const uint32_t dup_min =
      a.op == kOpAssign || a.dedup == kDedupRadix || a.D <= 32 ? 2u : (uint32_t)kPresumMinWide;
  auto kern = a.ahead ? k_put_probe<M, true> : k_put_probe<M, false>;
  hook(K_PUT_PROBE, 0, st);
  hipLaunchKernelGGL(kern, dim3((unsigned)ntiles), dim3(kPutThreads), 0, st, a.idx, a.nb_log2, a.keys, a.grads,
                     a.n, a.tlen, a.D, a.op, dup_min, pb, (int)ntiles, a.items, a.meta, a.partials, a.newlist, a.tile_cnt,
                     a.ctrl, a.epoch, a.pc_key, a.pc_row);
  hook(K_PUT_PROBE, 1, st);
  return hipGetLastError();
}

// The row updates of a put that sums gradients: about kApplyKeys keys a lane
// group, but up to kApplyBlocks blocks per CU for batches that have a key for
// each of their groups.
constexpr int64_t kApplyKeys = 4, kApplyBlocks = 8;
template <class M>
hipError_t launch_put_apply_t(const PutArgs& a, const PutApplyArgs& u, hipStream_t st) {
  constexpr int64_t NG = (kApplyThreads / 64) * M::RPW;
  const int64_t blocks = std::max<int64_t>(std::min<int64_t>(kApplyBlocks * a.cus, (a.n + NG - 1) / NG),
                                           (a.n + NG * kApplyKeys - 1) / (NG * kApplyKeys));
  auto kern = a.clock != nullptr ? k_put_apply<M, true> : k_put_apply<M, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kApplyThreads), 0, st, u, a.store);
  return hipGetLastError();
}

template <class M>
hipError_t load_map_code() {
  static std::atomic<uint64_t> on{0};
  return load_once(on, reinterpret_cast<const void*>(k_put_apply<M, false>));
}

#ifdef MLKV_MAP
template hipError_t load_map_code<MLKV_MAP>();
template hipError_t launch_put_probe_t<MLKV_MAP>(const PutArgs&, int, hipStream_t, const LaunchHook&);
template hipError_t launch_put_apply_t<MLKV_MAP>(const PutArgs&, const PutApplyArgs&, hipStream_t);
#else
#define MLKV_EXTERN(M)                                                                                   \
  extern template hipError_t load_map_code<M>();                                                         \
  extern template hipError_t launch_put_probe_t<M>(const PutArgs&, int, hipStream_t, const LaunchHook&); \
  extern template hipError_t launch_put_apply_t<M>(const PutArgs&, const PutApplyArgs&, hipStream_t);
MLKV_MAPS(MLKV_EXTERN)

template <class F>
static hipError_t dispatch_map(int D, F f) {
  if (D <= 3) return f(MapD3{});
  if (D <= 16) return f(MapD16{});
  if (D <= 32) return f(MapD32{});
  if (D <= 64) return f(MapD64{});
  if (D <= 128) return f(MapD128{});
  if (D <= 256) return f(MapD256{});
  if (D <= 512) return f(MapD512{});
  return f(MapD1024{});
}

hipError_t load_code(int D) {
  static std::atomic<uint64_t> on{0};
  const hipError_t e = load_once(on, reinterpret_cast<const void*>(k_lookup));
  return e != hipSuccess ? e : dispatch_map(D, [](auto m) { return load_map_code<decltype(m)>(); });
}

// Lets kernel `f` use `bytes` of dynamic LDS on the current device; `done`
// remembers the devices where that is set.
template <int kMaxDev>
static hipError_t lds_attr(const void* f, int bytes, bool (&done)[kMaxDev]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < kMaxDev && done[dev]) return hipSuccess;
  e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && dev >= 0 && dev < kMaxDev) done[dev] = true;
  return e;
}

// Launches grouping kernel `kern` (an instance, with `done` of its own) with its LDS.
template <class Kern, class... A>
static hipError_t launch_grouping(Kern kern, bool (&done)[64], unsigned blocks, hipStream_t st,
                                  const A&... args) {
  hipError_t e = lds_attr(reinterpret_cast<const void*>(kern), (int)GroupLds::total, done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(kGroupThreads), GroupLds::total, st, args...);
  return hipGetLastError();
}

template <bool kUpsert, int VEC, bool kClk>
static hipError_t launch_group_t(const PutGroupArgs& g, const uint32_t* total, const AssignArgs& s, const PutArgs& a,
                                 unsigned blocks, hipStream_t st) {
  static bool done[64] = {}, done_sorted[64] = {};
  if (total != nullptr)
    return launch_grouping(k_rsort_group<kUpsert, VEC, kClk>, done_sorted, blocks, st, g, total, s, a.store,
                           a.seed);
  return launch_grouping(k_put_group<kUpsert, VEC, kClk>, done, blocks, st, g, s, a.store, a.seed);
}

// The grouping kernel of a put: over the partitions, or over the sorted items
// (`total` of them).
static hipError_t launch_group(const PutGroupArgs& g, const uint32_t* total, const AssignArgs& s, const PutArgs& a,
                               unsigned blocks, hipStream_t st) {
  if (a.op != kOpAssign) return launch_group_t<false, 4, false>(g, total, s, a, blocks, st);
  const bool clk = a.clock != nullptr;
  if (a.D >= 4)
    return clk ? launch_group_t<true, 4, true>(g, total, s, a, blocks, st)
               : launch_group_t<true, 4, false>(g, total, s, a, blocks, st);
  return clk ? launch_group_t<true, 1, true>(g, total, s, a, blocks, st)
             : launch_group_t<true, 1, false>(g, total, s, a, blocks, st);
}

// The radix passes over put_probe's items (one partition): *sorted, *total.
static hipError_t launch_radix_sort(const PutArgs& a, hipStream_t st, const LaunchHook& hook, const uint64_t** sorted,
                                    const uint32_t** total_out) {
  const int64_t ntiles = (a.n + a.tlen - 1) / a.tlen;
  // passes of at most kRsMaxBits bits (at least 4: a sort key spans at least 4 bits)
  const int passes = (a.rs_bits + kRsMaxBits - 1) / kRsMaxBits;
  const int bits = (a.rs_bits + passes - 1) / passes;
  const int rtiles = (int)((ntiles + 3) / 4);
  const int stride = (rtiles + 3) / 4 * 4;  // a digit's row of counts, padded to 16 bytes
  uint32_t* cnt = a.rs_cnt;
  uint32_t* total = a.rs_cnt + (size_t)stride * (1u << bits);
  uint64_t* buf[2] = {a.rs_buf, a.rs_buf + a.n};
  for (int p = 0; p < passes; ++p) {
    RsSrc src;
    src.src = p == 0 ? a.items : buf[(p - 1) & 1];
    src.meta = p == 0 ? a.meta : nullptr;
    src.ntiles = (int)ntiles;
    src.total = total;
    hipError_t e = launch_rsort_pass(src, (uint32_t)a.capacity, p * bits, bits, cnt, rtiles, stride, buf[p & 1],
                                     p == 0 ? total : (uint32_t*)nullptr, st, hook);
    if (e != hipSuccess) return e;
  }
  *sorted = buf[(passes - 1) & 1];
  *total_out = total;
  return hipSuccess;
}

// Blocks of a hash put's grouping kernel at least, so that a few partitions'
// new keys are ranked and written by more.
constexpr int64_t kAssignBlocks = 32;

hipError_t launch_put(const PutArgs& a, hipStream_t st, const LaunchHook& hook, int phase) {
  const bool radix = a.dedup == kDedupRadix;
  const int64_t ntiles = (a.n + a.tlen - 1) / a.tlen;
  hipError_t e = hipSuccess;
  if (phase != kPutAfterProbe) {
    e = dispatch_map(a.D, [&](auto m) { return launch_put_probe_t<decltype(m)>(a, radix ? 0 : a.pb, st, hook); });
    if (e != hipSuccess) return e;
  }
  if (phase == kPutProbe) return hipSuccess;
  PutGroupArgs g;
  g.items = a.items;
  g.meta = a.meta;
  g.ntiles = (int)ntiles;
  const int vec = a.D >= 4 ? 4 : 1;
  const uint32_t row_units = (uint32_t)(a.D + vec - 1) / vec;
  g.magic = row_units > 1 ? (uint32_t)((0x100000000ull + row_units - 1) / row_units) : 0u;
  g.values = a.grads;
  g.clock = a.clock;
  g.units = a.units;
  g.ctrl = a.ctrl;
  g.epoch = a.epoch;
  g.capacity = a.capacity;
  g.spill = a.spill;
  g.spill_words = a.spill_words;
  AssignArgs s;  // rows for the keys the put inserts; their staleness counts start at 0
  s.idx = a.idx;
  s.newlist = a.newlist;
  s.tile_cnt = a.tile_cnt;
  s.ntiles = (int)ntiles;
  s.tile_size = kPutTile;
  s.state = a.state;
  s.capacity = a.capacity;
  s.ctrl = a.ctrl;
  s.epoch = a.epoch;
  s.xkey = a.xkey;
  s.xslot = a.xslot;
  s.clock = nullptr;
  s.cepoch = 0;
  s.rl = RangeLists{};
  s.values = a.op == kOpAssign ? a.grads : nullptr;
  const uint32_t* total = nullptr;
  // blocks: one per partition, or (radix) one per CU at least, at most kRsChunk
  // sorted items each before the cuts move
  const int64_t nb = radix ? std::max<int64_t>(a.cus, (a.n + kRsChunk - 1) / kRsChunk)
                           : std::max<int64_t>((int64_t)1 << a.pb, std::min<int64_t>(ntiles, kAssignBlocks));
  g.parts = 1u << a.pb;
  if (radix && (e = launch_radix_sort(a, st, hook, &g.items, &total)) != hipSuccess) return e;
  s.blocks = (uint32_t)std::min<int64_t>(nb, kMaxRanges);
  const int timed = radix ? K_RSORT_REDUCE : K_PUT_REDUCE;  // the grouping and the updates, timed as one
  hook(timed, 0, st);
  e = launch_group(g, total, s, a, (unsigned)nb, st);
  if (e != hipSuccess) return e;
  if (a.op == kOpAssign) {
    hook(timed, 1, st);
    return hipSuccess;
  }
  PutApplyArgs u;
  u.idx = a.idx;
  u.grads = a.grads;
  u.partials = a.partials;
  u.units = a.units;
  u.ctrl = a.ctrl;
  u.state = a.state;
  u.clock = a.clock;
  u.op = a.op;
  u.lr = a.lr;
  u.eps = a.eps;
  e = dispatch_map(a.D, [&](auto m) { return launch_put_apply_t<decltype(m)>(a, u, st); });
  hook(timed, 1, st);
  return e;
}

hipError_t launch_lookup(Bucket* idx, uint32_t nb_log2, const uint64_t* keys, int64_t n, int64_t* rows_out,
                         hipStream_t st) {
  const int64_t grid = (n + 255) / 256;
  hipLaunchKernelGGL(k_lookup, dim3((unsigned)grid), dim3(256), 0, st, idx, nb_log2, keys, n, rows_out);
  return hipGetLastError();
}

hipError_t launch_export_slots(const Bucket* idx, uint64_t nslots, uint64_t* keys_out, uint32_t* rows_out,
                               hipStream_t st) {
  const uint64_t grid = (nslots + 255) / 256;
  hipLaunchKernelGGL(k_export_slots, dim3((unsigned)grid), dim3(256), 0, st, idx, nslots, keys_out, rows_out);
  return hipGetLastError();
}

hipError_t launch_read_rows(const RowStore& store, const float* state, int D, const unsigned long long* size_now,
                            const int64_t* ids, int64_t n, float* w_out, float* st_out, Ctrl* ctrl,
                            hipStream_t st) {
  const uint64_t total = (uint64_t)n * (uint64_t)D;
  const uint64_t grid = std::min<uint64_t>((total + 255) / 256, 65536);
  hipLaunchKernelGGL(k_read_rows, dim3((unsigned)grid), dim3(256), 0, st, store, state, D, size_now, ids, n,
                     w_out, st_out, ctrl);
  return hipGetLastError();
}

// A long contiguous copy (rows 0 .. nrows-1 of a table in HBM), kFlatUnits
// accesses of 16 bytes a thread, around the caches: bound by HBM. One float a
// thread with a 64-bit division each (below, for tiered tables) took 238 us for
// 2M rows of dim 64.
constexpr int kFlatUnits = 4;
__global__ __launch_bounds__(256) void k_copy_flat(const float* __restrict__ src, float* __restrict__ dst,
                                                   uint64_t n) {
  const uint64_t b = (uint64_t)blockIdx.x * (256 * kFlatUnits) + threadIdx.x;
  const uint64_t n4 = n / 4;
  for (uint64_t base = b; base < n4; base += (uint64_t)gridDim.x * (256 * kFlatUnits)) {
    Words4 v[kFlatUnits];
#pragma unroll
    for (int u = 0; u < kFlatUnits; ++u)
      if (base + u * 256 < n4) v[u] = __builtin_nontemporal_load(reinterpret_cast<const Words4*>(src) + base + u * 256);
#pragma unroll
    for (int u = 0; u < kFlatUnits; ++u)
      if (base + u * 256 < n4) __builtin_nontemporal_store(v[u], reinterpret_cast<Words4*>(dst) + base + u * 256);
  }
  if (b < n - 4 * n4) dst[4 * n4 + b] = src[4 * n4 + b];
}

// Rows 0 .. nrows-1 in order, from wherever each lives.
__global__ __launch_bounds__(256) void k_export_rows(const RowStore store, int64_t nrows, int D,
                                                     float* __restrict__ out) {
  const uint64_t total = (uint64_t)nrows * (uint64_t)D;
  for (uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (uint64_t)gridDim.x * 256) {
    const uint64_t r = e / (uint64_t)D;
    out[e] = store.ptr((uint32_t)r)[e % (uint64_t)D];
  }
}

hipError_t launch_export_rows(const RowStore& store, int64_t nrows, int D, float* out, hipStream_t st) {
  const uint64_t total = (uint64_t)nrows * (uint64_t)D;
  if (total == 0) return hipSuccess;
  if (store.slot == nullptr) {
    const uint64_t blocks = std::min<uint64_t>((total / 4 + 256 * kFlatUnits - 1) / (256 * kFlatUnits), 1u << 22);
    hipLaunchKernelGGL(k_copy_flat, dim3((unsigned)std::max<uint64_t>(blocks, 1)), dim3(256), 0, st, store.rows, out,
                       total);
    return hipGetLastError();
  }
  const uint64_t grid = std::min<uint64_t>((total + 255) / 256, 65536);
  hipLaunchKernelGGL(k_export_rows, dim3((unsigned)grid), dim3(256), 0, st, store, nrows, D, out);
  return hipGetLastError();
}

hipError_t launch_read_clock(const unsigned long long* clock, const unsigned long long* size_now,
                             const int64_t* ids, int64_t n, uint32_t* out, Ctrl* ctrl, hipStream_t st) {
  const uint64_t grid = std::min<uint64_t>(((uint64_t)n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_read_clock, dim3((unsigned)grid), dim3(256), 0, st, clock, size_now, ids, n, out, ctrl);
  return hipGetLastError();
}

#endif  // MLKV_MAP

}  // namespace mlkv
