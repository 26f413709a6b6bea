// Step a1 of the path: the frontier's degrees, edge offsets and degree bins (k_frontier), and
// for weighted calls the bitmap of cached nodes (k_cached_bits).
#pragma once
#include "a3_common.hpp"

namespace a3 {

// ---------------------------------------------------------------------------
// step a1: frontier degrees -> edge offsets, degree bins
// ---------------------------------------------------------------------------
// One bit per node from the device map: bit u of the bitmap = (cache_map[u] >= 0).  A wavefront
// turns 64 consecutive entries into one 64-bit word with a ballot.  Each workgroup also notes
// whether it met cached nodes (bit 0) and uncached ones (bit 1); the first workgroup of hop 0's
// k_frontier folds the notes: with one class only (everything or nothing cached) all weights are
// equal and the sampler takes the uniform path whatever the bias rate.
__global__ __launch_bounds__(kTileThreads) void k_cached_bits(const int32_t* __restrict__ cache_map,
                                                             int64_t num_nodes, uint64_t* __restrict__ bits,
                                                             int32_t* __restrict__ block_seen) {
  __shared__ uint32_t seen_lds[kTileThreads / kWave];
  const int64_t n_words = (num_nodes + 63) >> 6;
  const int64_t n_waves = (int64_t)gridDim.x * (kTileThreads / kWave);
  const uint32_t lane = lane_id();
  uint32_t seen = 0;  // same value in every lane of the wavefront
  for (int64_t w0 = ((int64_t)blockIdx.x * kTileThreads + threadIdx.x) >> 6; w0 < n_words; w0 += 4 * n_waves) {
    int32_t c[4];
    bool valid[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t u = ((w0 + k * n_waves) << 6) + lane;
      valid[k] = u < num_nodes;
      c[k] = valid[k] ? cache_map[u] : -1;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t word = __ballot(c[k] >= 0);
      const uint64_t in_range = __ballot(valid[k]);
      seen |= (word ? 1u : 0u) | ((in_range & ~word) ? 2u : 0u);
      if (lane == 0 && w0 + k * n_waves < n_words) bits[w0 + k * n_waves] = word;
    }
  }
  if (lane == 0) seen_lds[threadIdx.x >> 6] = seen;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t all = 0;
    for (int w = 0; w < kTileThreads / kWave; ++w) all |= seen_lds[w];
    block_seen[blockIdx.x] = (int32_t)all;
  }
}

template <typename IdxT>
struct FrontierArgs {
  const IdxT* seeds;   // read only where from_seeds is set (may be null for an empty batch)
  int32_t from_seeds;  // hop 0 without validation: the frontier is the seed list itself
  int64_t num_seeds;
  const int32_t* cache_map;  // device map, or null: entries of the seeds go to S_slot
  int32_t* S_slot;
  IdxT* S;
  int32_t* node_map;
  int32_t map_base;  // the call's offset into the relabel map's value range
  const int64_t* indptr;
  DevState* st;
  int32_t hop;
  int32_t fanout;
  int32_t* tile_sums;
  int64_t num_nodes;
  NodeRec* bins[kNumBins];   // first record of every degree bin (see bin_rec)
  int32_t* bin_count;        // [kNumBins * kBinCountStride], zero between hops and between calls
  int32_t groups;            // bins 3-7 are in use
  uint32_t hub_degree;       // rows longer than this are hubs
  // hop 0 of a weighted call: where the weight classes of its map are kept; block_seen null where the
  // call reuses the bitmap of cached nodes, else the notes of k_cached_bits
  int32_t* class_mix_kept;
  const int32_t* block_seen;
  int32_t n_seen;
};

__device__ __forceinline__ int degree_bin(uint32_t deg, bool groups, uint32_t hub_degree) {
  if (deg <= 16) return 0;
  if (deg > hub_degree) return kHubBin;
  if (deg > kGroupDegree || (deg > 64 && !groups)) return kWideBin;
  return 28 - __clz((int)(deg - 1));  // 17..32: 1, 33..64: 2, ... 1025..2048: 7
}

// The launch is sized for a bound on the frontier; workgroups past its real size leave at once.
// One thread per node of the tile: with four nodes per thread the single workgroup of a small
// frontier, one wavefront per SIMD, went through four times the instructions one after the other
// (256 nodes 6.7 -> 3.9 us, 1 024 nodes 13.3 -> 11.5, 20 k nodes 10.4 -> 7.3).
// Two sizes of tile: small frontiers are cut into tiles of 256 nodes, since a node's random accesses
// (row bounds, relabel map, device map) miss the L1 and one CU gets through some hundred of them
// per microsecond (1 024 seeds: 11.5 us as one tile, 6.1 as four; 4 096 seeds 11.3 and 7.8).
template <typename IdxT, int kThreads>
__global__ __launch_bounds__(kThreads) void k_frontier(const FrontierArgs<IdxT> a) {
  __shared__ uint32_t lds[kThreads / kWave];
  __shared__ uint32_t bin_n[16];
  __shared__ uint32_t bin_base[kNumBins];
  __shared__ uint32_t seen_lds;
  const bool from_seeds = a.from_seeds != 0;
  if (threadIdx.x < 16) bin_n[threadIdx.x] = 0;
  if (threadIdx.x == 0) seen_lds = 0;
  __syncthreads();
  if (a.class_mix_kept && blockIdx.x == 0) {
    if (a.block_seen) {
      uint32_t seen = 0;
      for (int b = threadIdx.x; b < a.n_seen; b += kThreads) seen |= (uint32_t)a.block_seen[b];
      const uint32_t wave_seen = (__ballot(seen & 1u) ? 1u : 0u) | (__ballot(seen & 2u) ? 2u : 0u);
      if (lane_id() == 0 && wave_seen) atomicOr(&seen_lds, wave_seen);
      __syncthreads();
      if (threadIdx.x == 0) a.st->class_mix = *a.class_mix_kept = (int32_t)seen_lds;
    } else if (threadIdx.x == 0) {
      a.st->class_mix = *a.class_mix_kept;
    }
  }
  if (from_seeds && blockIdx.x == 0 && threadIdx.x == 0) a.st->n_dst[0] = (int32_t)a.num_seeds;
  const int64_t n = from_seeds ? a.num_seeds : (int64_t)a.st->n_dst[a.hop];
  if ((int64_t)blockIdx.x * kThreads >= n) return;
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  uint32_t cnt = 0, bin = 15;  // 15: no node
  NodeRec rec = {};
  if (i < n) {
    const int64_t v = from_seeds ? (int64_t)a.seeds[i] : (int64_t)a.S[i];
    const bool in_graph = v >= 0 && v < a.num_nodes;
    int64_t row = 0, end = 0;
    if (in_graph) {
      row = a.indptr[v];
      end = a.indptr[v + 1];
    } else {
      atomicOr(&a.st->error, kErrFrontierId);
    }
    if (from_seeds) {
      a.S[i] = (IdxT)v;
      if (in_graph) {
        a.node_map[v] = a.map_base + (int32_t)i;
        if (a.cache_map) a.S_slot[i] = a.cache_map[v];
      }
    }
    int64_t deg = end - row;
    if (deg < 0 || deg > 0x7FFFFFFF) {  // not a CSR this library can sample: the call fails,
      atomicOr(&a.st->error, kErrHugeRow);  // and the row is not touched
      deg = 0;
    }
    cnt = deg < (int64_t)a.fanout ? (uint32_t)deg : (uint32_t)a.fanout;
    bin = (uint32_t)degree_bin((uint32_t)deg, a.groups != 0, a.hub_degree);
    rec.v = v;
    rec.row = row;
    rec.deg = (uint32_t)deg;
    rec.i = (int32_t)i;
  }
  // rank of every node inside its bin and workgroup: the lanes of a wavefront that share a bin find
  // each other by ballots on the bin's four bits, and one of them reserves their places with an LDS
  // atomic (frontiers are lopsided, most nodes of a tile fall into one bin, and an atomic per node on
  // one LDS word would serialise)
  uint64_t same = ~0ull;
#pragma unroll
  for (int bit = 0; bit < 4; ++bit) {
    const bool set = (bin >> bit) & 1u;
    const uint64_t mask = __ballot(set);
    same &= set ? mask : ~mask;
  }
  const uint32_t in_wave = lanes_below(same);
  uint32_t reserved = 0;
  if (in_wave == 0) reserved = atomicAdd(&bin_n[bin], (uint32_t)__popcll(same));
  const uint32_t rank = (uint32_t)__shfl((int)reserved, __ffsll((long long)same) - 1, kWave) + in_wave;
  uint32_t total;
  const uint32_t local_off = block_excl_scan<kThreads>(cnt, lds, &total);
  // one global reservation per bin and block, then scatter the node records
  if (threadIdx.x < kNumBins)
    bin_base[threadIdx.x] = bin_n[threadIdx.x]
                                ? (uint32_t)atomicAdd(&a.bin_count[threadIdx.x * kBinCountStride], (int32_t)bin_n[threadIdx.x])
                                : 0u;
  __syncthreads();
  rec.local_off = (int32_t)local_off;
  if (bin < (uint32_t)kNumBins) *bin_rec(a.bins, (int)bin, (int64_t)bin_base[bin] + rank) = rec;
  if (threadIdx.x == 0) a.tile_sums[blockIdx.x] = (int32_t)total;
}

}  // namespace a3
