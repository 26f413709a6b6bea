// Steps a2-a4 of the path: keyed selection of every frontier node's neighbours (k_sample).
#pragma once
#include "a3_common.hpp"

namespace a3 {

// ---------------------------------------------------------------------------
// steps a2-a4: keyed selection
// ---------------------------------------------------------------------------
template <typename IdxT>
struct SampleArgs {
  const int64_t* indptr;
  const IdxT* indices;
  const uint32_t* cached_bits;  // bit u set: node u's row is in the device cache (weighted only)
  const IdxT* S;             // frontier: local id -> global id
  const int32_t* tile_offs;  // scanned tile offsets in global memory, or null: scan tile_sums here
  const int32_t* tile_sums;
  int64_t cap_tiles;         // the launch's bound on the tiles in use (at most the entries of tile_sums)
  int32_t tile_shift;        // log2 of the nodes per tile
  int32_t* blk_indptr;       // out: edge offsets of this hop
  IdxT* gid;                 // out: global id of each sampled neighbour
  int64_t* eids;             // out: CSR position of each sampled edge (may be null)
  int32_t* node_map;         // global id -> map_base + (first position / local id)
  int32_t map_base;
  DevState* st;
  NodeRec* bins[kNumBins];   // kWeightedFast sets `left` in the records that it leaves to the second launch
  const int32_t* bin_count;  // [kNumBins * kBinCountStride]
  uint32_t left_only;        // kWeightedFull as a second launch: only the records with `left` set
  int64_t num_nodes;
  int64_t cap_edges;         // entries in gid / eids (arena capacity of this hop)
  uint32_t hub_blocks;       // workgroups serving the hubs, the wide nodes (one wavefront each),
  uint32_t wide_blocks;      // and the lane groups (bins 0-7)
  uint32_t group_blocks;
  int32_t hop;
  int32_t fanout;
  uint32_t lambda;    // expected number of candidates kept by the draw threshold
  uint32_t group_lambda;  // the same for the 16-lane groups
  uint32_t cap;       // candidate buffer entries per wavefront (>= lambda)
  uint32_t xcap;      // challenger buffer entries (weighted only, multiple of 64, >= 128)
  uint32_t capb;      // second candidate list (weighted only; 0: rescan the row instead)
  uint32_t lds_per_wave;  // uint64 entries of LDS per wavefront
  uint32_t bias_q16;
  double inv_bias;    // 1.0 / bias_q16
  uint32_t seed_lo, seed_hi;
  uint32_t force_radix;
};

// Is node u's feature row in the device cache?  One bit per node (k_cached_bits): the lookups of
// a neighbourhood are random, and a bitmap of N / 8 bytes stays in the L2 where the 4 N bytes of
// the device map do not.  Ids outside the graph count as not cached (the emitter reports them).
template <typename IdxT>
__device__ __forceinline__ bool is_cached(const SampleArgs<IdxT>& a, int64_t u) {
  return u >= 0 && u < a.num_nodes && ((a.cached_bits[u >> 5] >> (u & 31)) & 1u);
}

// Writes sampled edge e of the hop: neighbour g, found at CSR position eid.
template <typename IdxT>
__device__ __forceinline__ void put_edge(const SampleArgs<IdxT>& a, int32_t n_dst, int32_t e, int64_t eid, IdxT g) {
  // a neighbour id outside the graph or an offset outside the arena is dropped, never written
  if (e < 0 || (int64_t)e >= a.cap_edges || (int64_t)g < 0 || (int64_t)g >= a.num_nodes) {
    atomicOr(&a.st->error, kErrEmit);
    return;
  }
  a.gid[e] = g;
  if (a.eids) a.eids[e] = eid;
  atomicMin(&a.node_map[(int64_t)g], a.map_base + n_dst + e);
}

// writes one sampled edge of a node, given its slot
template <typename IdxT>
struct Emitter {
  const SampleArgs<IdxT>& a;
  int64_t row;
  int32_t base;
  int32_t n_dst;
  __device__ __forceinline__ void operator()(uint32_t pos, uint32_t slot) const {
    const int64_t eid = row + slot;
    put_edge<IdxT>(a, n_dst, base + (int32_t)pos, eid, a.indices[eid]);
  }
};

// How a launch of k_sample treats the weights:
//   kUniform       all weights equal (no device map, or bias rate 1): the m largest draws;
//   kWeightedFast  two weights; a node of more than 32 neighbours is decided from the draws above the
//                  scan's threshold alone where that is enough (at least m of them cached: the usual
//                  case), and is marked for a second launch where it is not.  Keeps no second
//                  candidate list, no rescanning path and so far fewer registers;
//   kWeightedFull  two weights, every path: the second launch, which serves the marked nodes, or the
//                  only one of the hop.
constexpr int kUniform = 0, kWeightedFull = 1, kWeightedFast = 2;

// the lane's index as a value that the compiler cannot trace back: what is computed from it stays where
// it is used instead of being hoisted out of the node loop and held in registers for its whole length
__device__ __forceinline__ uint32_t local_lane_id() {
  uint32_t lane = lane_id();
  asm volatile("" : "+v"(lane));
  return lane;
}

constexpr double kInvOne = 1.0 / 65536.0;  // 1 / weight of an uncached neighbour (Q16.16)

__device__ __forceinline__ bool tuple_less(uint64_t K1, uint64_t k1, uint64_t K2, uint64_t k2) {
  return K1 < K2 || (K1 == K2 && k1 < k2);
}

// Rank R[0:nR) and X[0:nX) together under (K, draw-order key) and keep the best m in R, sorted.
__device__ __forceinline__ void merge_best(uint32_t m, uint32_t nR, uint32_t nX, uint64_t* RK,
                                           uint64_t* Rk, const uint64_t* XK, const uint64_t* Xk,
                                           uint64_t* NK, uint64_t* Nk) {
  const uint32_t lane = lane_id();
  const uint32_t total = nR + nX;
  for (uint32_t j = lane; j < total; j += kWave) {
    const uint64_t K = j < nR ? RK[j] : XK[j - nR];
    const uint64_t k = j < nR ? Rk[j] : Xk[j - nR];
    uint32_t r = 0;
    for (uint32_t t = 0; t < nR; ++t) r += tuple_less(RK[t], Rk[t], K, k) ? 1u : 0u;
    for (uint32_t t = 0; t < nX; ++t) r += tuple_less(XK[t], Xk[t], K, k) ? 1u : 0u;
    if (r < m) {
      NK[r] = K;
      Nk[r] = k;
    }
  }
  wave_sync();
  for (uint32_t j = lane; j < m; j += kWave) {
    RK[j] = NK[j];
    Rk[j] = Nk[j];
  }
  wave_sync();
}

// smallest draw x that a cached neighbour needs so that its key can still reach BK:
// K <= BK  <=>  -log2(u) in Q32 <= ((BK+1)*W - 1) >> 16.  Evaluated in double and lowered by a
// relative 2^-20 so that rounding can only let extra slots through, never drop one.
__device__ __forceinline__ uint32_t draw_floor_for_key(uint64_t BK, uint32_t w_q16) {
  const double bits = ((double)BK + 1.0) * (double)w_q16 * (1.0 / 65536.0) * (1.0 / 4294967296.0);
  if (bits >= 32.0) return 0u;
  const double xmin = exp2(32.0 - bits) * (1.0 - 1.0 / 1048576.0) - 2.0;
  if (xmin <= 0.0) return 0u;
  if (xmin >= 4294967295.0) return 0xFFFFFFFFu;
  return (uint32_t)xmin;
}

// the record that lane src_lane holds, in scalar registers: what is computed from it is computed
// once for the wavefront
__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, uint32_t src_lane);
__device__ __forceinline__ NodeRec readlane_rec(const NodeRec& r, uint32_t src_lane) {
  NodeRec one;
  one.v = (int64_t)readlane_u64((uint64_t)r.v, src_lane);
  one.row = (int64_t)readlane_u64((uint64_t)r.row, src_lane);
  one.deg = (uint32_t)__builtin_amdgcn_readlane((int32_t)r.deg, (int32_t)src_lane);
  one.i = __builtin_amdgcn_readlane(r.i, (int32_t)src_lane);
  one.local_off = __builtin_amdgcn_readlane(r.local_off, (int32_t)src_lane);
  one.left = 0;
  return one;
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, uint32_t src_lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)v, (int32_t)src_lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)(v >> 32), (int32_t)src_lane);
  return ((uint64_t)hi << 32) | lo;
}

// The m smallest of up to 64*NK keys held NK per lane in registers (key j lives in lane j % 64,
// register j / 64; keys are distinct).  Quickselect on wave-wide masks: a pivot is broadcast
// through the scalar unit, one comparison per lane and a ballot split the still undecided keys;
// about 2 ln(cnt) rounds of a dozen instructions, no LDS traffic.  The keys arrive in ascending
// slot order, so a chosen key's output position is the number of chosen keys before it.
// Calls on_selected(position, key) for each of the m chosen keys.
template <int NK, typename OnSelected>
__device__ __forceinline__ void select_in_registers(const uint64_t* cand, uint32_t cnt, uint32_t m,
                                                    OnSelected on_selected) {
  const uint32_t lane = lane_id();
  uint64_t mine[NK], active[NK], chosen[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const uint32_t idx = (uint32_t)k * kWave + lane;
    mine[k] = idx < cnt ? cand[idx] : ~0ull;
    const uint32_t n_k = cnt > (uint32_t)k * kWave ? min(cnt - (uint32_t)k * kWave, (uint32_t)kWave) : 0u;
    active[k] = n_k >= (uint32_t)kWave ? ~0ull : ((1ull << n_k) - 1ull);
    chosen[k] = 0;
  }
  uint32_t need = m, n_active = cnt;  // choose `need` of the n_active active keys; same in all lanes
  while (need > 0) {
    if (n_active == need) {
#pragma unroll
      for (int k = 0; k < NK; ++k) chosen[k] |= active[k];
      break;
    }
    // pivot: the first undecided key
    uint64_t pivot = 0;
    int pivot_reg = -1;
    uint64_t pivot_bit = 0;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      if (pivot_reg < 0 && active[k] != 0) {
        const uint32_t pl = (uint32_t)__ffsll((long long)active[k]) - 1u;
        pivot = readlane_u64(mine[k], pl);
        pivot_reg = k;
        pivot_bit = 1ull << pl;
      }
    }
    uint64_t less[NK];
    uint32_t n_less = 0;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      less[k] = __ballot(mine[k] < pivot) & active[k];
      n_less += (uint32_t)__popcll(less[k]);
    }
    if (n_less >= need) {  // all wanted keys are below the pivot
#pragma unroll
      for (int k = 0; k < NK; ++k) active[k] = less[k];
      n_active = n_less;
    } else {               // everything below the pivot and the pivot itself are in
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const uint64_t taken = less[k] | (k == pivot_reg ? pivot_bit : 0ull);
        chosen[k] |= taken;
        active[k] &= ~taken;
      }
      need -= n_less + 1;
      n_active -= n_less + 1;
    }
  }
  uint32_t before = 0;
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    if ((chosen[k] >> lane) & 1ull) on_selected(before + lanes_below(chosen[k]), mine[k]);
    before += (uint32_t)__popcll(chosen[k]);
  }
}

// Exhaustive selection for one wavefront: the m-th largest draw value is found bit by bit, the
// draws being recomputed in every pass; draws equal to it are taken in slot order.  Writes the m
// winners' draw-order keys to selk.  Used when the threshold kept too few or too many
// candidates (about one node in 10^5); kept out of line so that it costs the usual path no
// registers.
__device__ __noinline__ void radix_select(const PhiloxKey pk, uint32_t deg, uint32_t m, uint64_t* selk) {
  const uint32_t lane = lane_id();
  const uint32_t n_quads = (deg + 3) >> 2;
  {
    // exhaustive path: find the m-th largest draw value bit by bit, recomputing the draws
    uint32_t kth = 0;
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t trial = kth | (1u << bit);
      uint32_t c = 0;
      for (uint32_t q0 = 0; q0 < n_quads; q0 += kWave) {
        const uint32_t q = q0 + lane;
        uint32_t x[4];
        philox4x32_10(q, pk, x);
#pragma unroll
        for (int w = 0; w < 4; ++w) c += ((4u * q + w) < deg && x[w] >= trial) ? 1u : 0u;
      }
      c = wave_sum_u32(c);
      if (c >= m) kth = trial;
    }
    uint32_t n_gt = 0;
    for (uint32_t q0 = 0; q0 < n_quads; q0 += kWave) {
      const uint32_t q = q0 + lane;
      uint32_t x[4];
      philox4x32_10(q, pk, x);
#pragma unroll
      for (int w = 0; w < 4; ++w) n_gt += ((4u * q + w) < deg && x[w] > kth) ? 1u : 0u;
    }
    n_gt = wave_sum_u32(n_gt);
    const uint32_t need_eq = m - n_gt;  // draws equal to kth are taken in slot order
    uint32_t run_eq = 0, run_sel = 0;
    for (uint32_t q0 = 0; q0 < n_quads; q0 += kWave) {
      const uint32_t q = q0 + lane;
      uint32_t x[4];
      philox4x32_10(q, pk, x);
      uint32_t eqc = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) eqc += ((4u * q + w) < deg && x[w] == kth) ? 1u : 0u;
      uint32_t eq_before = run_eq + wave_excl_scan_u32(eqc);
      bool take[4];
      uint32_t selc = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const bool valid = (4u * q + w) < deg;
        const bool eq = valid && x[w] == kth;
        take[w] = (valid && x[w] > kth) || (eq && eq_before < need_eq);
        eq_before += eq ? 1u : 0u;
        selc += take[w] ? 1u : 0u;
      }
      uint32_t pos = run_sel + wave_excl_scan_u32(selc);
#pragma unroll
      for (int w = 0; w < 4; ++w)
        if (take[w]) selk[pos++] = draw_order_key(x[w], 4u * q + w);
      run_eq += wave_sum_u32(eqc);
      run_sel += wave_sum_u32(selc);
    }
    }
}

// ---- one wavefront, one node of any degree ------------------------------------------------------
// The m smallest of up to 64*NK (K, k) pairs held NK per lane in registers (pair j in lane j % 64,
// register j / 64; the k are distinct), by the same quickselect on wave-wide masks as
// select_in_registers, here on two-word keys.  The pairs come in no particular slot order, so a
// chosen pair's output position is counted: the number of chosen pairs with a smaller slot.
// Calls on_selected(position, k) for each of the m chosen pairs.
template <int NK, typename OnSelected>
__device__ __forceinline__ void select_pairs_in_registers(const uint64_t (&K)[NK], const uint64_t (&k)[NK],
                                                          uint32_t cnt, uint32_t m, OnSelected on_selected) {
  const uint32_t lane = lane_id();
  uint64_t active[NK], chosen[NK];
#pragma unroll
  for (int r = 0; r < NK; ++r) {
    const uint32_t n_r = cnt > (uint32_t)r * kWave ? min(cnt - (uint32_t)r * kWave, (uint32_t)kWave) : 0u;
    active[r] = n_r >= (uint32_t)kWave ? ~0ull : ((1ull << n_r) - 1ull);
    chosen[r] = 0;
  }
  uint32_t need = m, n_active = cnt;
  while (need > 0) {
    if (n_active == need) {
#pragma unroll
      for (int r = 0; r < NK; ++r) chosen[r] |= active[r];
      break;
    }
    uint64_t pK = 0, pk = 0, pivot_bit = 0;
    int pivot_reg = -1;
#pragma unroll
    for (int r = 0; r < NK; ++r) {
      if (pivot_reg < 0 && active[r] != 0) {
        const uint32_t pl = (uint32_t)__ffsll((long long)active[r]) - 1u;
        pK = readlane_u64(K[r], pl);
        pk = readlane_u64(k[r], pl);
        pivot_reg = r;
        pivot_bit = 1ull << pl;
      }
    }
    uint64_t less[NK];
    uint32_t n_less = 0;
#pragma unroll
    for (int r = 0; r < NK; ++r) {
      less[r] = __ballot(tuple_less(K[r], k[r], pK, pk)) & active[r];
      n_less += (uint32_t)__popcll(less[r]);
    }
    if (n_less >= need) {
#pragma unroll
      for (int r = 0; r < NK; ++r) active[r] = less[r];
      n_active = n_less;
    } else {
#pragma unroll
      for (int r = 0; r < NK; ++r) {
        const uint64_t taken = less[r] | (r == pivot_reg ? pivot_bit : 0ull);
        chosen[r] |= taken;
        active[r] &= ~taken;
      }
      need -= n_less + 1;
      n_active -= n_less + 1;
    }
  }
  uint32_t pos[NK];
#pragma unroll
  for (int r = 0; r < NK; ++r) pos[r] = 0;
#pragma unroll
  for (int r2 = 0; r2 < NK; ++r2) {
    uint64_t pending = chosen[r2];
    while (pending) {
      const uint32_t t = (uint32_t)__ffsll((long long)pending) - 1u;
      pending &= pending - 1;
      const uint32_t other_slot = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)k[r2], (int32_t)t);
#pragma unroll
      for (int r = 0; r < NK; ++r) pos[r] += other_slot < (uint32_t)k[r] ? 1u : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < NK; ++r)
    if ((chosen[r] >> lane) & 1ull) on_selected(pos[r], k[r]);
}

// Weighted selection from the two candidate lists (A: draws above the threshold, B: draws below it
// that could still matter as cached slots).  The answer lies among all of A and the cached
// members of B: an uncached slot outside the m largest draws loses to all of those, and a cached
// slot below B's floor has a key above that of the threshold draw taken as uncached, which every
// one of the m largest draws beats.  Inside one weight class the key K is monotone in the draw,
// so the answer also lies among the m largest draws of the uncached candidates and the m largest
// draws of the cached ones: only those 2 m slots get a key (the logarithm costs as much as
// scanning hundreds of slots), and with one class empty none does.
// All lookups are issued together, one memory round trip per node.  E [ecap] takes the two
// classes (uncached from the front, cached from the back; ecap >= both lists), T [2 m] their
// best.  Returns false (nothing written, the lists untouched) if the sizes do not fit the
// registers; the caller then rescans the row.
constexpr int kListPerLane = 8;  // list entries one lane looks up

// the m smallest of list [n] (all of them if n <= m), in any order, to out; n <= 256
__device__ __forceinline__ void smallest_to(const uint64_t* list, uint32_t n, uint32_t m, uint64_t* out) {
  auto put = [&](uint32_t pos, uint64_t key) { out[pos] = key; };
  if (n <= m) {
    for (uint32_t j = lane_id(); j < n; j += kWave) out[j] = list[j];
  } else if (n <= kWave) {
    select_in_registers<1>(list, n, m, put);
  } else if (n <= 2 * kWave) {
    select_in_registers<2>(list, n, m, put);
  } else {
    select_in_registers<4>(list, n, m, put);
  }
}

template <int NK, typename IdxT, typename Emit>
__device__ __forceinline__ void key_and_select(const SampleArgs<IdxT>& a, const uint64_t* T, uint32_t t_u,
                                               uint32_t t_c, uint32_t m, const Emit& emit) {
  const uint32_t lane = lane_id();
  const uint32_t n = t_u + t_c;
  uint64_t K[NK], k[NK];
#pragma unroll
  for (int r = 0; r < NK; ++r) {
    K[r] = ~0ull;
    k[r] = ~0ull;
    if ((uint32_t)r * kWave < n) {  // uniform: a dense round of keys
      const uint32_t j = (uint32_t)r * kWave + lane;
      if (j < n) {
        k[r] = j < t_u ? T[j] : T[m + (j - t_u)];
        K[r] = sample_key(~(uint32_t)(k[r] >> 32), j < t_u ? 65536u : a.bias_q16, j < t_u ? kInvOne : a.inv_bias);
      }
    }
  }
  select_pairs_in_registers<NK>(K, k, n, m, [&](uint32_t pos, uint64_t kk) { emit(pos, (uint32_t)kk); });
}

// The common case of the weighted selection needs the first list only.  If at least m of its
// slots are cached, no cached slot outside it can be chosen (the m best cached draws are all in
// it), and no uncached slot outside it ever can (it has m better draws against it), so the answer
// is the best m of the first list under (K, draw order): every entry gets its key in one pass over
// the lanes and one selection follows, all in registers.  With every candidate cached the keys
// are monotone in the draws and are not computed at all.  Returns false, with nothing written, if
// fewer than m candidates are cached (the second list is needed) or the list does not fit.
template <int NK, typename IdxT, typename Emit>
__device__ __forceinline__ bool weighted_from_first_list(const SampleArgs<IdxT>& a, int64_t row, const uint64_t* list_a,
                                                         uint32_t cnt_a, uint32_t m, const Emit& emit) {
  const uint32_t lane = lane_id();
  uint64_t k[NK], K[NK];
  bool cached[NK];
  uint32_t n_c = 0;  // same value in every lane
#pragma unroll
  for (int r = 0; r < NK; ++r) {
    k[r] = ~0ull;
    K[r] = ~0ull;
    cached[r] = false;
    if ((uint32_t)r * kWave < cnt_a) {  // uniform
      const uint32_t j = (uint32_t)r * kWave + lane;
      if (j < cnt_a) {
        k[r] = list_a[j];
        cached[r] = is_cached(a, (int64_t)a.indices[row + (uint32_t)k[r]]);
      }
      n_c += (uint32_t)__popcll(__ballot(cached[r]));
    }
  }
  if (n_c < m) return false;
  if (n_c == cnt_a) {  // one weight class among the candidates: the m largest draws, in slot order
    select_in_registers<NK>(list_a, cnt_a, m, [&](uint32_t pos, uint64_t key) { emit(pos, (uint32_t)key); });
    return true;
  }
#pragma unroll
  for (int r = 0; r < NK; ++r) {
    if ((uint32_t)r * kWave < cnt_a && (uint32_t)r * kWave + lane < cnt_a)
      K[r] = sample_key(~(uint32_t)(k[r] >> 32), cached[r] ? a.bias_q16 : 65536u, cached[r] ? a.inv_bias : kInvOne);
  }
  select_pairs_in_registers<NK>(K, k, cnt_a, m, [&](uint32_t pos, uint64_t kk) { emit(pos, (uint32_t)kk); });
  return true;
}

template <typename IdxT, typename Emit>
__device__ __forceinline__ bool weighted_from_lists(const SampleArgs<IdxT>& a, int64_t row, const uint64_t* list_a,
                                                    uint32_t cnt_a, const uint64_t* list_b, uint32_t cnt_b,
                                                    uint32_t m, uint64_t* E, uint32_t ecap, uint64_t* T,
                                                    const Emit& emit) {
  const uint32_t lane = lane_id();
  const uint32_t total = cnt_a + cnt_b;
  if (total > (uint32_t)kListPerLane * kWave || total > ecap || m > (uint32_t)kWave) return false;
  uint64_t key[kListPerLane];
  int64_t u[kListPerLane];
#pragma unroll
  for (int c = 0; c < kListPerLane; ++c) {
    key[c] = 0ull;
    u[c] = -1;
    if ((uint32_t)c * kWave < total) {  // uniform: rounds past the lists' end cost nothing
      const uint32_t j = (uint32_t)c * kWave + lane;
      if (j < total) {
        key[c] = j < cnt_a ? list_a[j] : list_b[j - cnt_a];
        u[c] = (int64_t)a.indices[row + (uint32_t)key[c]];
      }
    }
  }
  uint32_t n_u = 0, n_c = 0;  // same values in every lane
#pragma unroll
  for (int c = 0; c < kListPerLane; ++c) {
    if ((uint32_t)c * kWave < total) {
      const uint32_t j = (uint32_t)c * kWave + lane;
      const bool cached = j < total && is_cached(a, u[c]);
      const bool plain = j < cnt_a && !cached;
      const uint64_t mask_c = __ballot(cached), mask_u = __ballot(plain);
      if (cached) E[ecap - 1u - (n_c + lanes_below(mask_c))] = key[c];
      if (plain) E[n_u + lanes_below(mask_u)] = key[c];
      n_c += (uint32_t)__popcll(mask_c);
      n_u += (uint32_t)__popcll(mask_u);
    }
  }
  wave_sync();
  if (n_u > 4u * kWave || n_c > 4u * kWave) return false;
  const uint32_t t_u = min(n_u, m), t_c = min(n_c, m);
  smallest_to(E, n_u, m, T);
  smallest_to(E + (ecap - n_c), n_c, m, T + m);
  wave_sync();
  if (t_u == 0 || t_c == 0) {
    // one weight class: the m largest draws, in slot order
    const uint64_t* best = t_u ? T : T + m;  // exactly m entries (the lists hold at least m slots)
    for (uint32_t j = lane; j < m; j += kWave) {
      const uint32_t s = (uint32_t)best[j];
      uint32_t pos = 0;
      for (uint32_t t = 0; t < m; ++t) pos += (uint32_t)best[t] < s ? 1u : 0u;
      emit(pos, s);
    }
  } else if (t_u + t_c <= (uint32_t)kWave) {
    key_and_select<1>(a, T, t_u, t_c, m, emit);
  } else {
    key_and_select<2>(a, T, t_u, t_c, m, emit);
  }
  return true;
}

// Floor of the second list, known before anything is looked up.  With p = lambda / deg the
// threshold keeps draws with 1 - u <= p, and the worst key of the final reservoir is at most the
// key of the threshold draw taken as uncached.  A cached slot reaches that key only if
// u >= (1 - p)^gamma, and (1 - p)^gamma >= 1 - gamma p, so every such slot has 1 - u <= gamma p.
// keep = p * 2^32 as computed for the threshold; the relative and absolute margins (2^-10, and
// gamma * 2^-20 of the draw range) cover the float rounding here and the few units by which
// the fixed-point logarithm and the floor in the key differ from the exact values, all scaled
// by gamma.  A lower floor only lengthens the list.
__device__ __forceinline__ uint32_t second_list_floor(float keep, uint32_t bias_q16) {
  const float kb = (float)bias_q16 * (1.0f / 65536.0f) * (keep * (1.0f + 1.0f / 1024.0f) + 4096.0f);
  return kb >= 4294967040.0f ? 0u : 0u - (uint32_t)kb;
}

// kWeightedFast: the node goes to the second launch.  A mark in its own record and no shared
// list: a list needs a counter, and thousands of atomics on one word stall every wavefront
// that touches the counter's cache line (0.2 ms per hop with a few thousand nodes left over).
__device__ __forceinline__ void defer_node(int32_t* left) {
  if (lane_id() == 0) *left = 1;
}

// A wavefront, one node.  cand [cap] and rest [m (+ 3 m + 2 xcap + capb when weighted)] are its LDS buffers.
// With prefiltered set, cand already holds pre_cnt candidates in slot order (a workgroup scanned
// the row together; pre_cnt_b entries of the second list too) and the scan is skipped.
template <typename IdxT, int kMode>
__device__ __forceinline__ void sample_node_wave(const SampleArgs<IdxT>& a, const int32_t* tile_offs,
                                 const NodeRec& r, int32_t n_dst, uint64_t* cand, uint64_t* rest,
                                 bool prefiltered, uint32_t pre_cnt, uint32_t pre_cnt_b,
                                 bool both_classes, int32_t* left) {
  const uint32_t lane = local_lane_id();
  const int64_t v = r.v;
  const int64_t row = r.row;
  const int64_t i = r.i;
  const uint32_t deg = r.deg;
  const uint32_t f = (uint32_t)a.fanout;
  const int32_t base = tile_offs[i >> a.tile_shift] + r.local_off;
  if (lane == 0) a.blk_indptr[i] = base;
  const Emitter<IdxT> emit{a, row, base, n_dst};

  if (deg <= f) {  // keep every neighbour, no draw
    for (uint32_t s = lane; s < deg; s += kWave) emit(s, s);
    return;
  }
  const uint32_t m = f;
  const PhiloxKey pk{(uint32_t)(uint64_t)v, (uint32_t)((uint64_t)v >> 32), (uint32_t)a.hop,
                     a.seed_lo, a.seed_hi};
  const uint32_t n_quads = (deg + 3) >> 2;

  uint64_t* selk = rest;  // [m] draw-order keys of the m best draws

  // ---- the m largest draws (order: x descending, slot ascending) --------------------------
  // keep slots whose draw clears a threshold set so that about lambda survive, rank those
  // (any threshold gives the same result; this one only sets how many candidates survive)
  uint32_t X0 = 0;
  float keep = 4294967296.0f;
  if (deg > a.lambda) {
    keep = __fdividef((float)a.lambda, (float)deg) * 4294967296.0f;  // < 2^32
    X0 = 0u - (uint32_t)keep;
  }
  uint32_t cnt = pre_cnt;  // same value in every lane
  // weighted: a second list takes the slots below the threshold whose draw could still matter as
  // a cached slot, so that the row need not be scanned again
  uint64_t* list_b = rest + 4 * (size_t)m + 2 * (size_t)a.xcap;  // [capb]
  uint32_t cnt_b = pre_cnt_b;
  // with one weight class in the whole graph the weighted kernel takes the uniform path
  constexpr bool kWeighted = kMode != kUniform;
  constexpr bool kFast = kMode == kWeightedFast;
  const bool two_classes = kWeighted && both_classes;
  const bool want_b = !kFast && two_classes && a.capb > 0;
  uint32_t X1 = want_b ? second_list_floor(keep, a.bias_q16) : 0u;
  bool scan = !prefiltered;
  for (int attempt = 0;; ++attempt) {
  if (!a.force_radix && scan) {
    // One step: 64 quads = 256 slots.  Only the last step of a row can hold slots past its end,
    // so the steps before it run without the range test (tail = false): a lane's condition is
    // then one comparison, which is also its ballot.
    const uint32_t b_span = X0 - X1;  // second list: X1 <= x < X0, as one unsigned comparison
    auto step = [&](uint32_t q0, auto tail) {
      constexpr bool kTail = decltype(tail)::value;
      const uint32_t q = q0 + lane;
      uint32_t x[4];
      philox4x32_10(q, pk, x);
      bool pass[4];
      uint64_t mk[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        pass[w] = x[w] >= X0;
        if (kTail) pass[w] = pass[w] && (4u * q + (uint32_t)w < deg);
        mk[w] = __ballot(pass[w]);
      }
      if (mk[0] | mk[1] | mk[2] | mk[3]) {
        // append in slot order: all passing slots of lower lanes first, then the own words
        uint32_t idx = cnt + lanes_below(mk[0]) + lanes_below(mk[1]) + lanes_below(mk[2]) + lanes_below(mk[3]);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          if (pass[w]) {
            if (idx < a.cap) cand[idx] = draw_order_key(x[w], 4u * q + (uint32_t)w);
            ++idx;
          }
        }
        cnt += (uint32_t)(__popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]));
      }
      if (want_b) {
        bool pb[4];
        uint64_t mb[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          pb[w] = (x[w] - X1) < b_span;
          if (kTail) pb[w] = pb[w] && (4u * q + (uint32_t)w < deg);
          mb[w] = __ballot(pb[w]);
        }
        if (mb[0] | mb[1] | mb[2] | mb[3]) {
          uint32_t idx = cnt_b + lanes_below(mb[0]) + lanes_below(mb[1]) + lanes_below(mb[2]) + lanes_below(mb[3]);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            if (pb[w]) {
              if (idx < a.capb) list_b[idx] = draw_order_key(x[w], 4u * q + (uint32_t)w);
              ++idx;
            }
          }
          cnt_b += (uint32_t)(__popcll(mb[0]) + __popcll(mb[1]) + __popcll(mb[2]) + __popcll(mb[3]));
        }
      }
    };
    const uint32_t whole_steps_end = (deg >> 2) & ~(uint32_t)(kWave - 1);
    uint32_t q0 = 0;
    for (; q0 < whole_steps_end; q0 += kWave) step(q0, std::false_type{});
    for (; q0 < n_quads; q0 += kWave) step(q0, std::true_type{});
    wave_sync();
  }
  if (attempt == 1 || a.force_radix || cnt >= m) break;
  // Fewer than m draws cleared the threshold (about one node in 10^5).  The exhaustive path
  // would scan the row 34 times; one more scan by this wavefront, with a threshold that keeps
  // a number midway between m and the buffer's size, settles all but one in 10^10.
  const uint32_t more = (m + a.cap) >> 1;
  keep = 4294967296.0f;
  X0 = 0;
  if (deg > more) {
    keep = __fdividef((float)more, (float)deg) * 4294967296.0f;
    X0 = 0u - (uint32_t)keep;
  }
  X1 = want_b ? second_list_floor(keep, a.bias_q16) : 0u;
  cnt = 0;
  cnt_b = 0;
  scan = true;
  }
  // the first list alone decides most nodes (see weighted_from_first_list)
  if (two_classes && !a.force_radix && cnt >= m && cnt <= a.cap && cnt <= 2u * kWave && m <= (uint32_t)kWave) {
    const bool done = cnt <= (uint32_t)kWave ? weighted_from_first_list<1, IdxT>(a, row, cand, cnt, m, emit)
                                             : weighted_from_first_list<2, IdxT>(a, row, cand, cnt, m, emit);
    if (done) {
      wave_sync();  // the candidate buffer is reused by this wavefront's next node
      return;
    }
  }
  if (kFast && two_classes) {  // everything else is the second launch's business
    defer_node(left);
    wave_sync();
    return;
  }
  // the lists can replace the second scan if both are complete
  const bool lists_ok = want_b && !a.force_radix && cnt >= m && cnt <= a.cap && cnt_b <= a.capb;
  if (!kFast && two_classes && lists_ok) {
    uint64_t* E = rest + 4 * (size_t)m;  // [2 xcap], the challenger buffers of the rescanning path
    if (weighted_from_lists<IdxT>(a, row, cand, cnt, list_b, cnt_b, m, E, 2 * a.xcap, rest, emit)) {
      wave_sync();
      return;
    }
  }
  if (!a.force_radix && cnt >= m && cnt <= a.cap && cnt <= 4 * kWave) {
    // the usual case: few candidates, selected in registers.  With equal weights the winners
    // are final and are written out at once; otherwise they become the first reservoir.
    const bool final_now = !two_classes;
    auto take = [&](uint32_t pos, uint64_t key) {
      if (final_now)
        emit(pos, (uint32_t)key);
      else
        selk[pos] = key;
    };
    if (cnt <= kWave)
      select_in_registers<1>(cand, cnt, m, take);
    else if (cnt <= 2 * kWave)
      select_in_registers<2>(cand, cnt, m, take);
    else
      select_in_registers<4>(cand, cnt, m, take);
    if (final_now) {
      wave_sync();  // the candidate buffer is reused by this wavefront's next node
      return;
    }
  } else if (!a.force_radix && cnt >= m && cnt <= a.cap) {
    for (uint32_t j = lane; j < cnt; j += kWave) {
      const uint64_t mine = cand[j];
      uint32_t r = 0;
      for (uint32_t t = 0; t < cnt; ++t) r += cand[t] < mine ? 1u : 0u;
      if (r < m) selk[r] = mine;
    }
  } else {
    if (lane == 0) atomicAdd(&a.st->n_radix, 1);
    radix_select(pk, deg, m, selk);
  }
  wave_sync();

  if (!two_classes) {
    // all weights equal: the m largest draws are the answer; emit in slot order
    for (uint32_t j = lane; j < m; j += kWave) {
      const uint32_t s = (uint32_t)selk[j];
      uint32_t pos = 0;
      for (uint32_t t = 0; t < m; ++t) pos += (uint32_t)selk[t] < s ? 1u : 0u;
      emit(pos, s);
    }
    wave_sync();  // the buffers are reused by this wavefront's next node
    return;
  }

  if constexpr (kMode == kWeightedFull) {
  // ---- two weight classes (cached: gamma, others: 1) -----------------------------------------
  // T = the m largest draws is a first reservoir.  A slot outside T can only enter the answer if
  // it is cached (an uncached slot outside T loses to all of T).  So: key T, take its worst
  // member B as the bar, rescan, look up only slots whose draw could beat B as a cached slot,
  // and collect the challengers; merge whenever the buffer fills (this tightens B).
  uint64_t* RK = selk + m;   // [m] keys K of the reservoir
  uint64_t* Rk = selk;       // [m] draw-order keys of the reservoir (starts as T)
  uint64_t* NK = RK + m;     // [m] merge output
  uint64_t* Nk = NK + m;     // [m]
  uint64_t* XK = Nk + m;     // [xcap] challengers
  uint64_t* Xk = XK + a.xcap;
  uint64_t kT = 0;           // worst draw-order key inside T
  for (uint32_t j = lane; j < m; j += kWave) {
    const uint64_t k = selk[j];
    const uint32_t s = (uint32_t)k;
    const uint32_t x = ~(uint32_t)(k >> 32);
    const int64_t u = (int64_t)a.indices[row + s];
    const bool c = is_cached(a, u);
    RK[j] = sample_key(x, c ? a.bias_q16 : 65536u, c ? a.inv_bias : kInvOne);
    kT = k > kT ? k : kT;
  }
  kT = wave_max_u64(kT);
  wave_sync();
  merge_best(m, m, 0, RK, Rk, XK, Xk, NK, Nk);
  uint64_t BK = RK[m - 1], Bk = Rk[m - 1];
  uint32_t x_lo = draw_floor_for_key(BK, a.bias_q16);
  uint32_t nX = 0;  // same value in every lane
  // one slot per lane goes through lookup, key and comparison with the bar; challengers are
  // appended, and the buffer is folded into the reservoir when the next ballot might not fit
  auto challenge = [&](bool live, uint64_t k) {
    const uint32_t s = (uint32_t)k;
    const uint32_t x = ~(uint32_t)(k >> 32);
    bool challenger = false;
    uint64_t K = 0;
    if (live && x >= x_lo && k > kT) {
      const int64_t u = (int64_t)a.indices[row + s];
      if (is_cached(a, u)) {
        K = sample_key(x, a.bias_q16, a.inv_bias);
        challenger = tuple_less(K, k, BK, Bk);
      }
    }
    const uint64_t mask = __ballot(challenger);
    if (mask) {
      if (challenger) {
        const uint32_t idx = nX + lanes_below(mask);
        XK[idx] = K;
        Xk[idx] = k;
      }
      nX += (uint32_t)__popcll(mask);
      if (nX + kWave > a.xcap) {
        wave_sync();
        merge_best(m, m, nX, RK, Rk, XK, Xk, NK, Nk);
        nX = 0;
        BK = RK[m - 1];
        Bk = Rk[m - 1];
        x_lo = draw_floor_for_key(BK, a.bias_q16);
      }
    }
  };
  for (uint32_t q0 = 0; q0 < n_quads; q0 += kWave) {
    const uint32_t q = q0 + lane;
    uint32_t x[4];
    philox4x32_10(q, pk, x);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t s = 4u * q + (uint32_t)w;
      challenge(s < deg, draw_order_key(x[w], s));
    }
  }
  wave_sync();
  if (nX > 0) merge_best(m, m, nX, RK, Rk, XK, Xk, NK, Nk);
  for (uint32_t j = lane; j < m; j += kWave) {
    const uint32_t s = (uint32_t)Rk[j];
    uint32_t pos = 0;
    for (uint32_t t = 0; t < m; ++t) pos += (uint32_t)Rk[t] < s ? 1u : 0u;
    emit(pos, s);
  }
  wave_sync();
  }
}

// ---- reductions over a group of lanes, without LDS ------------------------------------------------
// the largest / smallest value of a group of G lanes, in each of them (after the first two steps a
// quad agrees, after the third a half row, so a mirror image serves as the exchange)
template <int G>
__device__ __forceinline__ uint32_t group_max_u32(uint32_t v) {
  v = max(v, dpp_u32<kDppXor1>(v));
  v = max(v, dpp_u32<kDppXor2>(v));
  if (G >= 8) v = max(v, dpp_u32<kDppHalfMirror>(v));
  return v;
}
// the same for the minimum; v must be active in all lanes of the row
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_min_u32(uint32_t v) {
  return min(v, dpp_u32<kCtrl>(v));
}
template <int G>
__device__ __forceinline__ uint32_t group_min_u32(uint32_t v) {
  v = dpp_min_u32<kDppXor1>(v);
  v = dpp_min_u32<kDppXor2>(v);
  if (G >= 8) v = dpp_min_u32<kDppHalfMirror>(v);
  if (G >= 16) v = dpp_min_u32<kDppMirror>(v);
  return v;
}
template <int kCtrl>
__device__ __forceinline__ uint64_t dpp_min_u64(uint64_t v) {
  const uint64_t other = ((uint64_t)dpp_u32<kCtrl>((uint32_t)(v >> 32)) << 32) | dpp_u32<kCtrl>((uint32_t)v);
  return other < v ? other : v;
}
template <int G>
__device__ __forceinline__ uint64_t group_min_u64(uint64_t v) {
  v = dpp_min_u64<kDppXor1>(v);
  v = dpp_min_u64<kDppXor2>(v);
  if (G >= 8) v = dpp_min_u64<kDppHalfMirror>(v);
  return v;
}

// The key -log2(u) / w in single precision, as bits that compare like the value (it is not negative).
// Against the exact key in Q32 it is off by at most 0.12 kKeyError (1 + key): the largest error over all
// 2^32 draws; dividing by the weight adds 2^-23 of the key.  Where the m-th best key and the next lie
// further apart than twice kKeyError each, the choice is the exact keys'.  Nearer ones are looked at
// again: the keys of cached neighbours, and with them their errors, are 1 / w of an uncached one's, so
// where no uncached neighbour is near the cut, a w-th of that distance is enough.  What is still open (one
// node in some hundreds, at any bias rate) the exact keys decide.  An exact key takes 32 dependent
// multiply-shift steps, 200 instructions; this one takes six (third hop of 237 k nodes: 174 -> 147 us;
// without the second look a call on 16 384 seeds with half of the nodes cached takes 650 us at bias rate
// 1 000 and 915 at 60 000, by exact keys alone 698 and 888, with it 581 and 608).
constexpr float kKeyError = 0x1p-20f;
__device__ __forceinline__ uint32_t approx_key(uint32_t x, float inv_w) {
  const float u = __builtin_fmaf((float)x, 0x1p-32f, 0x1p-32f);  // (x + 1) / 2^32
  return __float_as_uint(__builtin_fabsf(__builtin_amdgcn_logf(u)) * inv_w);
}
// may exact keys order these two the other way?  (next: ~0 for none)
__device__ __forceinline__ bool keys_too_close(uint32_t last, uint32_t next) {
  const float l = __uint_as_float(last);
  return next != ~0u && __uint_as_float(next) - l <= 4.0f * kKeyError * (1.0f + l);
}
// the same for two cached neighbours (2^-30: the exact keys end at 2^-32)
__device__ __forceinline__ bool cached_keys_too_close(uint32_t last, uint32_t next, float inv_w) {
  const float l = __uint_as_float(last);
  return __uint_as_float(next) - l <= 4.0f * kKeyError * (inv_w + l) + 0x1p-30f;
}
// may an uncached neighbour that drew x belong on the other side of a cut at `last`, whose next key is
// too close to it?
__device__ __forceinline__ bool uncached_near_cut(uint32_t x, uint32_t last) {
  const float l = __uint_as_float(last);
  return __builtin_fabsf(__uint_as_float(approx_key(x, 1.0f)) - l) <= 8.0f * kKeyError * (1.0f + l);
}

// ---- edges of the lane groups ---------------------------------------------------------------------
// A group's chosen slots stand in LDS, in order, k of them; consecutive lanes write consecutive edges.
// All neighbour ids of a group are asked for before the first is used; where one round of the lanes
// is enough the round is only begun here (`pending`) and written while the wavefront's next nodes are
// drawn, so that nothing waits for the ids.  ids: the ids themselves stand in LDS too (low words,
// then, kListIds further on, high words), or null.
constexpr uint32_t kListIds = 32;

template <typename IdxT>
struct PendingEdge {
  int64_t eid;
  IdxT g;
  int32_t e;
  bool on;
};

template <typename IdxT>
__device__ __forceinline__ void put_pending(const SampleArgs<IdxT>& a, int32_t n_dst, PendingEdge<IdxT>& p) {
  if (p.on) put_edge<IdxT>(a, n_dst, p.e, p.eid, p.g);
  p.on = false;
}

template <typename IdxT>
__device__ __forceinline__ IdxT listed_id(const uint32_t* ids, uint32_t j) {
  if (sizeof(IdxT) == 4) return (IdxT)ids[j];
  return (IdxT)(((uint64_t)ids[kListIds + j] << 32) | ids[j]);
}

template <typename IdxT, int G>
__device__ __forceinline__ void put_list(const SampleArgs<IdxT>& a, int64_t row, int32_t base, int32_t n_dst,
                                         uint32_t k, const uint32_t* list, const uint32_t* ids,
                                         PendingEdge<IdxT>& pending) {
  const uint32_t gl = local_lane_id() & (G - 1);
  if (__ballot(k > (uint32_t)G) == 0) {
    pending.on = gl < k;
    if (pending.on) {
      pending.eid = row + list[gl];
      pending.e = base + (int32_t)gl;
      pending.g = ids ? listed_id<IdxT>(ids, gl) : a.indices[pending.eid];
    }
    return;
  }
  int64_t eid[4];
  IdxT g[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t j = (uint32_t)(r * G) + gl;
    if (j < k) {
      eid[r] = row + list[j];
      g[r] = ids ? listed_id<IdxT>(ids, j) : a.indices[eid[r]];
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t j = (uint32_t)(r * G) + gl;
    if (j < k) put_edge<IdxT>(a, n_dst, base + (int32_t)j, eid[r], g[r]);
  }
}

// ---- a group of G lanes (4 or 8), one node of degree <= 4 G: four slots per lane -----------------
// The draws of a lane are one Philox block.  Selection is m rounds of "best remaining slot of the
// group" on 32-bit keys: lane-local minimum, reduction over the group, every slot that has the
// minimum is out.  Equal keys leave more than m chosen; then, and where single-precision keys leave the
// cut open, the choice is made again in full precision, one slot per round, all ties resolved.
template <typename IdxT, int G, int kMode>
__device__ __forceinline__ void sample_node_group(const SampleArgs<IdxT>& a, const int32_t* tile_offs,
                                                  const NodeRec& r, bool live, int32_t n_dst, uint32_t* lds,
                                                  bool both_classes, PendingEdge<IdxT>& pending) {
  constexpr uint32_t kStride = 4 * G + 4;  // groups start in other banks
  const uint32_t lane = local_lane_id();
  const uint32_t gl = lane & (G - 1);       // lane inside the group
  const uint32_t gshift = lane & ~(G - 1);  // first lane of the group inside the wavefront
  uint32_t* keys = lds + (lane / G) * kStride;
  const int64_t v = r.v;
  const int64_t row = r.row;
  const uint32_t deg = live ? r.deg : 0;  // <= 4 G by construction of the bins
  const uint32_t m = (uint32_t)a.fanout;
  const int32_t base = live ? tile_offs[r.i >> a.tile_shift] + r.local_off : 0;
  if (live && gl == 0) a.blk_indptr[r.i] = base;
  const bool draw = deg > m;  // else every neighbour is kept
  const PhiloxKey pk{(uint32_t)(uint64_t)v, (uint32_t)((uint64_t)v >> 32), (uint32_t)a.hop,
                     a.seed_lo, a.seed_hi};
  uint32_t chosen = 0;  // bit w: slot 4 gl + w
#pragma unroll
  for (int w = 0; w < 4; ++w) chosen |= (4u * gl + w < deg) ? (1u << w) : 0u;
  const uint64_t lower_lanes = ((1ull << gl) - 1ull) << gshift;  // of the group
  if (__ballot(draw)) {
    const uint32_t alive = draw ? chosen : 0u;
    uint32_t x[4];
    philox4x32_10(gl, pk, x);
    put_pending<IdxT>(a, n_dst, pending);
    const uint64_t group_lanes = ((1ull << G) - 1ull) << gshift;
    bool cached[4] = {false, false, false, false};
    bool mixed = false;
    if (kMode != kUniform && both_classes) {
      IdxT u[4];
#pragma unroll
      for (int w = 0; w < 4; ++w)
        if (alive & (1u << w)) u[w] = a.indices[row + 4u * gl + w];
      bool any_c = false, any_u = false;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (alive & (1u << w)) {
          cached[w] = is_cached(a, (int64_t)u[w]);
          any_c |= cached[w];
          any_u |= !cached[w];
        }
      }
      // keys are needed only when the group's neighbourhood mixes both classes (otherwise K is
      // monotone in x and the order is "larger draw first")
      const uint64_t mc = __ballot(any_c), mu = __ballot(any_u);
      mixed = (mc & group_lanes) != 0 && (mu & group_lanes) != 0;
    }
    uint32_t own[4];  // ascending is better; ~0 for no slot (a slot that drew 0 ranks with those)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      own[w] = ~0u;
      if (alive & (1u << w)) {
        own[w] = ~x[w];
        if (kMode != kUniform && mixed) own[w] = approx_key(x[w], cached[w] ? (float)a.inv_bias * 65536.0f : 1.0f);
      }
    }
    uint32_t last = 0;
#pragma unroll 1
    for (uint32_t it = 0; it < m; ++it) {
      last = group_min_u32<G>(min(min(own[0], own[1]), min(own[2], own[3])));
#pragma unroll
      for (int w = 0; w < 4; ++w) own[w] = own[w] == last ? ~0u : own[w];
    }
    bool close = false;
    if (kMode != kUniform && __ballot(mixed)) {
      const uint32_t next = group_min_u32<G>(min(min(own[0], own[1]), min(own[2], own[3])));
      close = mixed && keys_too_close(last, next);
      if (__ballot(close)) {
        bool near_cut = false;
#pragma unroll
        for (int w = 0; w < 4; ++w) near_cut |= (alive & (1u << w)) && !cached[w] && uncached_near_cut(x[w], last);
        close = close && ((__ballot(near_cut) & group_lanes) != 0 ||
                          cached_keys_too_close(last, next, (float)a.inv_bias * 65536.0f));
      }
    }
    uint32_t in_rounds = 0, n_chosen = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      in_rounds |= own[w] == ~0u ? (1u << w) : 0u;
      in_rounds &= alive;
      n_chosen += (uint32_t)__popcll(__ballot((in_rounds >> w) & 1u) & group_lanes);
    }
    if (draw) chosen = in_rounds;
    const bool tie = draw && (n_chosen != m || close);
    if (__ballot(tie)) {
      uint64_t K[4] = {0, 0, 0, 0};
      uint32_t rest = alive, picked = 0;
      if (kMode != kUniform && mixed) {
#pragma unroll
        for (int w = 0; w < 4; ++w)
          if (alive & (1u << w))
            K[w] = sample_key(x[w], cached[w] ? a.bias_q16 : 65536u, cached[w] ? a.inv_bias : kInvOne);
      }
#pragma unroll 1
      for (uint32_t it = 0; it < m; ++it) {
        // lane-local best remaining slot under (K ascending, x descending, word ascending)
        uint32_t best = 0, bx = 0;
        uint64_t bK = ~0ull;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          if ((rest & (1u << w)) && (best == 0 || K[w] < bK || (K[w] == bK && x[w] > bx))) {
            best = 1u << w;
            bK = K[w];
            bx = x[w];
          }
        }
        // group-wide best: smallest K, then largest x, then lowest lane (= lowest slot)
        const uint64_t gK = group_min_u64<G>(bK);
        const bool tied_K = best != 0 && bK == gK;
        const uint32_t gx = group_max_u32<G>(tied_K ? bx : 0u);
        const bool mine = tied_K && bx == gx;
        if (mine && (__ballot(mine) & lower_lanes) == 0) {
          rest &= ~best;
          picked |= best;
        }
      }
      if (tie) chosen = picked;
    }
    wave_sync();
  } else {
    put_pending<IdxT>(a, n_dst, pending);
  }
  // the chosen slots in slot order: those of lower lanes first, then lower words of the own lane
  uint32_t at = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) at += (uint32_t)__popcll(__ballot((chosen >> w) & 1u) & lower_lanes);
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if ((chosen >> w) & 1u) keys[at++] = 4u * gl + w;
  wave_sync();
  put_list<IdxT, G>(a, row, base, n_dst, min(deg, m), keys, nullptr, pending);
  wave_sync();  // the list is rewritten by the wavefront's next nodes
}

// ---- sixteen lanes, one node of 33 to kGroupDegree neighbours -----------------------------------
// Four nodes per wavefront.  A step draws 64 slots of each; slots whose draw clears the threshold go
// to the group's list in LDS, in slot order, as 32-bit keys (~draw: ascending is better) beside
// their slots.  With at most kListCap candidates a lane holds up to four of them in registers; the m
// smallest are taken out in m rounds of a minimum over the sixteen lanes (9 to 15 instructions a
// round for four nodes).  A chosen candidate's output position is a scan of the chosen ones before it.
// Equal keys leave more than m chosen (weighted: exact keys that agree in their upper 32 bits): such a
// node, and one whose list came out too short or too long, is left to the wavefront path (false).
// Weighted: the list decides as in weighted_from_first_list (at least m of it cached), or if it holds
// the whole neighbourhood; rows of up to 64 get a second attempt with exactly that.
// Where rows are short a node's fixed costs are what counts, and memory round trips: a wavefront per
// node spent some 350 vector instructions on a row of 65 to 512 neighbours and waited four fifths of its
// time.  Third hop of 616 k nodes (190 k of them above 64 neighbours), fanout 5: 303 -> 196 us, 98.7 M ->
// 65 M vector instructions; 337 k nodes on 100 M: 396 -> 269 us; 237 k nodes weighted: 262 -> 177 us.
constexpr uint32_t kListCap = 64;
constexpr uint32_t kListStride = kListCap + 4;  // one entry takes what does not fit; groups start in other banks
constexpr uint32_t kGroupLdsEntries = 4 * kListStride;  // uint64 entries per wavefront: keys, slots of four groups

// leaves the chosen slots in keys [m] (and, where the ids had to be looked up, the ids in slots)
template <typename IdxT, int kMode, int NK>
__device__ __forceinline__ bool finish_list(const SampleArgs<IdxT>& a, int64_t row, uint32_t deg, uint32_t m,
                                            uint32_t* keys, uint32_t* slots, uint32_t cnt, bool good, bool both_classes) {
  const uint32_t gl = local_lane_id() & 15u;
  uint32_t own[NK], slot[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const uint32_t at = (uint32_t)k * 16u + gl;
    own[k] = ~0u;
    if (good && at < cnt) own[k] = keys[at];  // below ~0: the threshold is at least 1
    slot[k] = slots[at];
  }
  bool decided = good, mixed = false;
  IdxT u[NK];
  bool cached[NK];
  if (kMode != kUniform && both_classes) {
#pragma unroll
    for (int k = 0; k < NK; ++k)
      if (own[k] != ~0u) u[k] = a.indices[row + slot[k]];
    uint32_t n_c = 0;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      cached[k] = own[k] != ~0u && is_cached(a, (int64_t)u[k]);
      n_c += cached[k] ? 1u : 0u;
    }
    n_c = row16_last(row16_incl_scan(n_c));
    decided = good && (n_c >= m || cnt == deg);
    mixed = decided && n_c != 0 && n_c != cnt;  // else the keys are monotone in the draws
#pragma unroll
    for (int k = 0; k < NK; ++k)
      if (mixed && own[k] != ~0u) own[k] = approx_key(~own[k], cached[k] ? (float)a.inv_bias * 65536.0f : 1.0f);
  }
  uint32_t mine = 0;  // a byte per k: the lane's candidate is chosen
  bool open = good;
  for (int pass = 0;; ++pass) {
    uint32_t best = 0;
#pragma unroll 1
    for (uint32_t it = 0; it < m; ++it) {
      best = own[0];
#pragma unroll
      for (int k = 1; k < NK; ++k) best = min(best, own[k]);
      best = group_min_u32<16>(best);
#pragma unroll
      for (int k = 0; k < NK; ++k) own[k] = own[k] == best ? ~0u : own[k];
    }
    uint32_t chosen = 0;
#pragma unroll
    for (int k = 0; k < NK; ++k)
      chosen |= ((uint32_t)k * 16u + gl < cnt && own[k] == ~0u) ? 1u << (8 * k) : 0u;
    if (open) mine = chosen;
    if (kMode == kUniform || pass != 0 || __ballot(mixed) == 0) break;
    // groups whose cut the single-precision keys leave open choose again, by the upper 32 bits of the
    // exact keys (K < 2^38)
    uint32_t next = own[0];
#pragma unroll
    for (int k = 1; k < NK; ++k) next = min(next, own[k]);
    next = group_min_u32<16>(next);
    const uint32_t n_chosen = (row16_last(row16_incl_scan(chosen)) * 0x01010101u) >> 24;
    open = mixed && (n_chosen != m || keys_too_close(best, next));
    if (__ballot(open) == 0) break;
    bool near_cut = false;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const uint32_t at = (uint32_t)k * 16u + gl;
      near_cut |= open && at < cnt && !cached[k] && uncached_near_cut(~keys[at], best);
    }
    const bool any_near = row16_last(row16_incl_scan(near_cut ? 1u : 0u)) != 0;
    open = open && (n_chosen != m || any_near || cached_keys_too_close(best, next, (float)a.inv_bias * 65536.0f));
    if (__ballot(open) == 0) break;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const uint32_t at = (uint32_t)k * 16u + gl;
      own[k] = ~0u;
      if (open && at < cnt)
        own[k] = (uint32_t)(sample_key(~keys[at], cached[k] ? a.bias_q16 : 65536u, cached[k] ? a.inv_bias : kInvOne) >> 6);
    }
  }
  const uint32_t incl = row16_incl_scan(mine);
  const uint32_t total = row16_last(incl);
  const bool done = decided && (total * 0x01010101u) >> 24 == m;  // the sum of the bytes
  const uint32_t pos = incl - mine + total * 0x01010100u;         // byte k: chosen ones before the lane's
  wave_sync();
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    if (done && ((mine >> (8 * k)) & 1u)) {
      const uint32_t at = (pos >> (8 * k)) & 255u;
      keys[at] = slot[k];
      if (kMode != kUniform && both_classes && m <= kListIds) {
        slots[at] = (uint32_t)(uint64_t)(int64_t)u[k];
        if (sizeof(IdxT) == 8) slots[kListIds + at] = (uint32_t)((uint64_t)(int64_t)u[k] >> 32);
      }
    }
  }
  return done;
}

template <typename IdxT, int kMode>
__device__ __forceinline__ bool sample_node_16(const SampleArgs<IdxT>& a, const int32_t* tile_offs, const NodeRec& r,
                                               bool live, int32_t n_dst, uint32_t* lds, bool both_classes,
                                               PendingEdge<IdxT>& pending) {
  const uint32_t lane = local_lane_id();
  const uint32_t gl = lane & 15u;
  uint32_t* keys = lds + (lane >> 4) * 2 * kListStride;
  uint32_t* slots = keys + kListStride;
  const uint32_t deg = live ? r.deg : 0;
  const uint32_t m = (uint32_t)a.fanout;
  const int32_t base = live ? tile_offs[r.i >> a.tile_shift] + r.local_off : 0;
  if (live && gl == 0) a.blk_indptr[r.i] = base;
  const bool whole = deg <= m;  // every neighbour is kept
  bool open = !whole;
  bool failed = false;
  const PhiloxKey pk{(uint32_t)(uint64_t)r.v, (uint32_t)((uint64_t)r.v >> 32), (uint32_t)a.hop, a.seed_lo, a.seed_hi};
  for (int attempt = 0;; ++attempt) {
    // at least 1: out-of-range slots take part as draws of 0 (and a slot that really drew 0 is the
    // worst of more than m)
    uint32_t X0 = 1;
    if (attempt == 0 && deg > a.group_lambda)
      X0 = 0u - (uint32_t)(__fdividef((float)a.group_lambda, (float)deg) * 4294967296.0f);
    const uint32_t n_slots = open ? deg : 0;
    uint32_t cnt = 0;  // same value in the lanes of a group
#pragma unroll 1
    for (uint32_t q = gl; __ballot(4u * q < n_slots) != 0; q += 16) {
      uint32_t x[4];
      philox4x32_10(q, pk, x);
      const int32_t left = (int32_t)n_slots - (int32_t)(4u * q);
      bool pass[4];
      uint32_t n = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        x[w] = left > w ? x[w] : 0u;
        pass[w] = x[w] >= X0;
        n += pass[w] ? 1u : 0u;
      }
      const uint32_t incl = row16_incl_scan(n);
      uint32_t at = cnt + incl - n;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (pass[w]) {
          const uint32_t to = min(at, kListCap);
          keys[to] = ~x[w];
          slots[to] = 4u * q + (uint32_t)w;
          ++at;
        }
      }
      cnt += row16_last(incl);
    }
    if (attempt == 0) put_pending<IdxT>(a, n_dst, pending);  // of the wavefront's previous nodes
    wave_sync();
    const bool good = open && cnt >= m && cnt <= kListCap;
    const uint32_t listed = good ? cnt : 0u;
    uint32_t max_cnt = 0;  // of the wavefront's four lists
#pragma unroll
    for (int g = 0; g < 4; ++g) max_cnt = max(max_cnt, (uint32_t)__builtin_amdgcn_readlane((int32_t)listed, 16 * g));
    bool done = false;
    if (max_cnt > 32)
      done = finish_list<IdxT, kMode, 4>(a, r.row, deg, m, keys, slots, cnt, good, both_classes);
    else if (max_cnt > 0)
      done = finish_list<IdxT, kMode, 2>(a, r.row, deg, m, keys, slots, cnt, good, both_classes);
    if (attempt == 0 && whole)
      for (uint32_t s = gl; s < deg; s += 16) keys[s] = s;
    wave_sync();
    const bool ids_known = kMode != kUniform && both_classes && m <= kListIds && __ballot(whole && live) == 0;
    const uint32_t k = done ? m : attempt == 0 && whole ? deg : 0u;
    if (__ballot(k != 0) != 0)
      put_list<IdxT, 16>(a, r.row, base, n_dst, k, keys, ids_known ? slots : nullptr, pending);
    wave_sync();  // the lists are rewritten
    open = open && !done;
    if (kMode == kUniform || attempt != 0) break;
    failed = open && deg > kListCap;
    open = open && !failed;
    if (__ballot(open) == 0) break;
    put_pending<IdxT>(a, n_dst, pending);  // the second attempt has edges of its own
  }
  return !(open || failed);
}

// ---- a workgroup, one hub ---------------------------------------------------------------------
// The wavefronts of the workgroup scan contiguous parts of the row, each collecting its
// candidates (in slot order) in its own LDS region; the regions are then laid end to end, which
// is slot order again, and wavefront 0 finishes the node as it would one it scanned alone.
constexpr uint32_t kHubRegion = 64;  // candidates one wavefront may contribute

template <typename IdxT, int kMode>
__device__ __forceinline__ void hub_scan(const SampleArgs<IdxT>& a, const NodeRec& r, uint64_t* lds,
                                         uint64_t*& joined_out, uint64_t*& rest_out, uint32_t& pre_cnt,
                                         uint32_t& pre_cnt_b, bool both_classes) {
  const uint32_t lane = local_lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const uint32_t n_waves = blockDim.x >> 6;
  uint64_t* region = lds + (size_t)wave * kHubRegion;         // [kHubRegion]
  uint64_t* joined = lds + (size_t)n_waves * kHubRegion;      // [cap]
  uint32_t* counts = (uint32_t*)(joined + a.cap);             // [n_waves] (<= 16 -> 8 entries)
  uint32_t* shared_cnt_b = (uint32_t*)(joined + a.cap + 8);   // one more entry
  uint64_t* rest = joined + a.cap + 9;
  const int64_t v = r.v;
  const uint32_t deg = r.deg;
  // the second candidate list of the weighted case is shared: wavefronts reserve space in it
  // with one LDS atomic per append (its order does not matter)
  uint64_t* list_b = rest + 4 * (size_t)a.fanout + 2 * (size_t)a.xcap;
  const bool want_b = kMode == kWeightedFull && a.capb > 0 && both_classes;
  if (want_b) {
    if (threadIdx.x == 0) *shared_cnt_b = 0;
    __syncthreads();
  }
  uint32_t mine = 0;
  if (deg > (uint32_t)a.fanout && !a.force_radix) {
    const PhiloxKey pk{(uint32_t)(uint64_t)v, (uint32_t)((uint64_t)v >> 32), (uint32_t)a.hop,
                       a.seed_lo, a.seed_hi};
    const uint32_t n_quads = (deg + 3) >> 2;
    uint32_t X0 = 0;
    float keep = 4294967296.0f;
    if (deg > a.lambda) {
      keep = __fdividef((float)a.lambda, (float)deg) * 4294967296.0f;
      X0 = 0u - (uint32_t)keep;
    }
    const uint32_t X1 = want_b ? second_list_floor(keep, a.bias_q16) : 0u;
    // contiguous share of the row per wavefront, a whole number of 64-quad steps
    const uint32_t share = (((n_quads + n_waves - 1) / n_waves) + kWave - 1) & ~(uint32_t)(kWave - 1);
    const uint32_t q_begin = wave * share;
    const uint32_t q_end = min(q_begin + share, n_quads);
    const uint32_t b_span = X0 - X1;
    auto step = [&](uint32_t q0, auto tail) {
      constexpr bool kTail = decltype(tail)::value;
      const uint32_t q = q0 + lane;
      uint32_t x[4];
      philox4x32_10(q, pk, x);
      bool pass[4];
      uint64_t mk[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        pass[w] = x[w] >= X0;
        if (kTail) pass[w] = pass[w] && (4u * q + (uint32_t)w < deg);
        mk[w] = __ballot(pass[w]);
      }
      if (mk[0] | mk[1] | mk[2] | mk[3]) {
        uint32_t idx = mine + lanes_below(mk[0]) + lanes_below(mk[1]) + lanes_below(mk[2]) + lanes_below(mk[3]);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          if (pass[w]) {
            if (idx < kHubRegion) region[idx] = draw_order_key(x[w], 4u * q + (uint32_t)w);
            ++idx;
          }
        }
        mine += (uint32_t)(__popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]));
      }
      if (want_b) {
        bool pb[4];
        uint64_t mb[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          pb[w] = (x[w] - X1) < b_span;
          if (kTail) pb[w] = pb[w] && (4u * q + (uint32_t)w < deg);
          mb[w] = __ballot(pb[w]);
        }
        if (mb[0] | mb[1] | mb[2] | mb[3]) {
          const uint32_t n_new = (uint32_t)(__popcll(mb[0]) + __popcll(mb[1]) + __popcll(mb[2]) + __popcll(mb[3]));
          uint32_t start = 0;
          if (lane == 0) start = atomicAdd(shared_cnt_b, n_new);
          start = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)start);
          uint32_t idx = start + lanes_below(mb[0]) + lanes_below(mb[1]) + lanes_below(mb[2]) + lanes_below(mb[3]);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            if (pb[w]) {
              if (idx < a.capb) list_b[idx] = draw_order_key(x[w], 4u * q + (uint32_t)w);
              ++idx;
            }
          }
        }
      }
    };
    // steps that lie wholly inside the row need no range test (see sample_node_wave)
    const uint32_t whole_steps_end = min(q_end, (deg >> 2) & ~(uint32_t)(kWave - 1));
    uint32_t q0 = q_begin;
    for (; q0 < whole_steps_end; q0 += kWave) step(q0, std::false_type{});
    for (; q0 < q_end; q0 += kWave) step(q0, std::true_type{});
  }
  if (lane == 0) counts[wave] = mine;
  __syncthreads();
  uint32_t offset = 0, total = 0;
  bool overflow = false;
  for (uint32_t w = 0; w < n_waves; ++w) {
    const uint32_t c = counts[w];
    offset += w < wave ? c : 0u;
    total += c;
    overflow |= c > kHubRegion;
  }
  overflow |= total > a.cap;
  if (!overflow)
    for (uint32_t j = lane; j < mine; j += kWave) joined[offset + j] = region[j];
  __syncthreads();
  // too few candidates, too many, or a forced exhaustive run: the finishing wavefront takes the
  // slow path
  joined_out = joined;
  rest_out = rest;
  pre_cnt = overflow ? a.cap + 1u : total;
  pre_cnt_b = want_b ? *shared_cnt_b : 0u;
}

constexpr int kSampleMaxThreads = 256;

// Workgroups take roles by index: hub_blocks serve the hubs (one workgroup each), wide_blocks the wide
// nodes (one wavefront each), group_blocks the nodes of bins 0-7 (a wavefront takes 4, 8 or 16
// nodes of one bin at a time).
template <typename IdxT, int kMode>
__global__ __launch_bounds__(kSampleMaxThreads) __attribute__((amdgpu_waves_per_eu(kMode == kUniform ? 5 : 4))) void k_sample(const SampleArgs<IdxT> a) {
  extern __shared__ uint64_t lds[];
  __shared__ int32_t fused_offs[kFuseTiles];
  __shared__ uint32_t fused_total;
  __shared__ uint32_t block_left;
  // Workgroups start in index order, so the roles whose workgroups run longest come first (hubs, then
  // the lane groups, which have a dozen nodes' chains each) and the single wide nodes fill the end
  // of the launch (wide nodes before the groups: hop 3 of a mini-batch 214 instead of 199 us at 616 k
  // nodes, 294 instead of 289 at 337 k).  In the only launch of a weighted hop the groups have rows of up
  // to 64 neighbours and every longer one is a wide node, scanned twice or three times: there the wide
  // nodes come first (16 384 seeds, three hops, one node in ten cached, bias rate 4: 1 095 us a call, with
  // the groups first 1 157; bias rate 1 000: 2 860 and 2 950).
  uint32_t b = blockIdx.x;
  const bool hub_role = b < a.hub_blocks;  // the same for the whole workgroup
  bool group_role = false;
  if (!hub_role) {
    b -= a.hub_blocks;
    if (kMode == kWeightedFull) {
      group_role = b >= a.wide_blocks;
      if (group_role) b -= a.wide_blocks;
    } else {
      group_role = b < a.group_blocks;
      if (!group_role) b -= a.group_blocks;
    }
  }
  // the wavefront's index inside the workgroup, held in a scalar register so that the node loops
  // below are uniform control flow for the whole wavefront
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const uint32_t n_waves = blockDim.x >> 6;
  const uint32_t lane = lane_id();
  uint32_t count[kNumBins];
#pragma unroll
  for (int k = 0; k < kNumBins; ++k) count[k] = (uint32_t)a.bin_count[k * kBinCountStride];
  const int64_t stride = hub_role ? (int64_t)a.hub_blocks
                                  : (int64_t)(group_role ? a.group_blocks : a.wide_blocks) * n_waves;
  const int64_t first = hub_role ? (int64_t)b : (int64_t)b * n_waves + wave;
  // Where item t of the role's list is.  Wide nodes and hubs: record t of the bin; as a second launch
  // the wide role goes through the records of the lane groups' bins too (those that hold marks).
  uint32_t n_items = hub_role ? count[kHubBin] : count[kWideBin];
  if (kMode == kWeightedFull && a.left_only && !hub_role) {
#pragma unroll
    for (int k = kWideBin - 1; k >= 3; --k) n_items += count[k];
    if (a.st->left_small) n_items += count[2];
  }
  auto wide_rec = [&](int64_t t) {
    if (hub_role) return bin_rec(a.bins, kHubBin, t);
    int bin = kWideBin;
    if (kMode == kWeightedFull) {
#pragma unroll
      for (int k = kWideBin; k > 2; --k)
        if (bin == k && t >= (int64_t)count[k]) {
          t -= (int64_t)count[k];
          bin = k - 1;
        }
    }
    return bin_rec(a.bins, bin, t);
  };
  // kWeightedFull as a second launch takes only the marked records, and most workgroups find none
  // and leave here, before anything else
  uint64_t round0 = 0;
  uint32_t n_left = 0;
  if constexpr (kMode == kWeightedFull) {
    if (a.left_only) {
      const int64_t tl = first + (int64_t)lane * stride;
      round0 = __ballot(tl < n_items && wide_rec(tl)->left != 0);
      if (threadIdx.x == 0) block_left = 0;
      if (!__syncthreads_or(round0 != 0 || first + 64 * stride < n_items)) return;
    }
  }
  const int32_t* tile_offs = a.tile_offs;
  TileSums sums = {};
  if (tile_offs == nullptr) sums = tile_sums_load(a.tile_sums, a.cap_tiles);  // does not wait for n_dst
  // items of the lane groups: wavefront loads of one bin, the longest rows first
  uint32_t end_of[kWideBin];  // items up to and including bin k
  if (group_role) {
    uint32_t run = 0;
#pragma unroll
    for (int k = kWideBin - 1; k >= 0; --k) {
      const uint32_t per_wave = k >= 2 ? 4 : k == 1 ? 8 : 16;
      run += (count[k] + per_wave - 1) / per_wave;
      end_of[k] = run;
    }
    n_items = run;
  }
  // A workgroup without work leaves once the counts are there, which it waits for no longer than for
  // the tile sums: thousands of them are surplus (the launch is sized for bounds), and their scans of
  // the tile sums held the others up.  Workgroup 0 stays, it publishes the hop's edge count.
  if (blockIdx.x != 0 && (hub_role ? (int64_t)b : (int64_t)b * n_waves) >= (int64_t)n_items) return;
  const int32_t n_dst = a.st->n_dst[a.hop];
  const bool both_classes = kMode != kUniform && a.st->class_mix == 3;  // read once, not per node
  if (tile_offs == nullptr) {  // few tiles: scan the tile sums here, publish the hop's edge count
    const uint32_t total = tile_prefix_from(sums, a.cap_tiles, ((int64_t)n_dst + (1 << a.tile_shift) - 1) >> a.tile_shift,
                                            fused_offs, &fused_total);
    tile_offs = fused_offs;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.st->n_edges[a.hop] = (int32_t)total;
      a.blk_indptr[n_dst] = (int32_t)total;
    }
  }
  uint64_t* my_lds = lds + (size_t)wave * a.lds_per_wave;
  // Every role ends in the same loop, so that the selection of one wavefront for one node exists once
  // in the kernel: `cur` holds a record per lane, `todo` says whose are to be sampled.
  PendingEdge<IdxT> pending = {};
  // item t of the lane groups: its bin, the lane's record (null: none)
  auto group_rec = [&](int64_t t, int& bin) -> NodeRec* {
    bin = kWideBin - 1;
    uint32_t begin = 0;
#pragma unroll
    for (int k = kWideBin - 1; k > 0; --k)
      if (t >= (int64_t)end_of[k]) {
        bin = k - 1;
        begin = end_of[k];
      }
    const uint32_t in_bin = (uint32_t)a.bin_count[bin * kBinCountStride];
    const uint32_t shift = bin >= 2 ? 4 : bin == 1 ? 3 : 2;  // log2 of the lanes per node
    const uint32_t pos = (((uint32_t)t - begin) << (6 - shift)) + (lane >> shift);
    return t < (int64_t)n_items && pos < in_bin ? bin_rec(a.bins, bin, pos) : nullptr;
  };
  int bin_ahead = 0;
  NodeRec* where_ahead = nullptr;
  NodeRec ahead = {};
  if (group_role) {
    where_ahead = group_rec(first, bin_ahead);
    if (where_ahead) ahead = *where_ahead;
  }
  for (int64_t t0 = first; t0 < (int64_t)n_items; t0 += group_role ? stride : 64 * stride) {
    NodeRec cur = {};
    NodeRec* where = nullptr;  // of cur, where marks are left
    uint64_t todo = 0;
    if (group_role) {
      cur = ahead;
      where = where_ahead;
      const int bin = bin_ahead;
      const bool live = where && cur.i >= 0 && cur.i < n_dst;
      where_ahead = group_rec(t0 + stride, bin_ahead);  // in flight while cur is sampled
      if (where_ahead) ahead = *where_ahead;
      if (bin >= 2) {
        const bool ok = sample_node_16<IdxT, kMode>(a, tile_offs, cur, live, n_dst, (uint32_t*)my_lds, both_classes, pending);
        todo = __ballot(!ok) & 0x0001000100010001ull;  // one lane of each group
        if (kMode == kWeightedFast && bin == 2 && todo != 0 && lane == 0) atomicOr(&a.st->left_small, 1);
      } else if (bin == 1) {
        sample_node_group<IdxT, 8, kMode>(a, tile_offs, cur, live, n_dst, (uint32_t*)my_lds, both_classes, pending);
      } else {
        sample_node_group<IdxT, 4, kMode>(a, tile_offs, cur, live, n_dst, (uint32_t*)my_lds, both_classes, pending);
      }
    } else {
      const int64_t tl = t0 + (int64_t)lane * stride;
      bool take = tl < (int64_t)n_items;
      if (take) where = wide_rec(tl);
      if (kMode == kWeightedFull && a.left_only) take = t0 == first ? (round0 >> lane) & 1u : take && where->left != 0;
      if (take) {
        cur = *where;
        take = cur.i >= 0 && cur.i < n_dst;
      }
      todo = __ballot(take);
      n_left += (uint32_t)__popcll(todo);
    }
    while (todo) {
      const uint32_t l = (uint32_t)__builtin_ctzll(todo);
      todo &= todo - 1;
      const NodeRec one = readlane_rec(cur, l);
      int32_t* left = nullptr;
      if (kMode == kWeightedFast) left = &reinterpret_cast<NodeRec*>(readlane_u64((uint64_t)(uintptr_t)where, l))->left;
      uint64_t* cand = my_lds;
      uint64_t* rest = my_lds + a.cap;
      uint32_t pre_cnt = 0, pre_cnt_b = 0;
      if (hub_role) hub_scan<IdxT, kMode>(a, one, lds, cand, rest, pre_cnt, pre_cnt_b, both_classes);
      if (!hub_role || wave == 0)
        sample_node_wave<IdxT, kMode>(a, tile_offs, one, n_dst, cand, rest, hub_role, pre_cnt, pre_cnt_b,
                                      both_classes, left);
      if (hub_role) __syncthreads();  // the regions are reused for the workgroup's next hub
    }
  }
  put_pending<IdxT>(a, n_dst, pending);
  if constexpr (kMode == kWeightedFull) {
    if (a.left_only) {  // the call's count of nodes that needed this launch: one atomic per workgroup
      if (lane == 0 && n_left != 0 && (!hub_role || wave == 0)) atomicAdd(&block_left, n_left);
      __syncthreads();
      if (threadIdx.x == 0 && block_left != 0) atomicAdd(&a.st->n_deferred[hub_role ? 1 : 0], (int32_t)block_left);
    }
  }
}

}  // namespace a3
