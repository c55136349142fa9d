// Selection of the kept blocks by one workgroup, for the kernels that retrieve for themselves.
#pragma once

#include "svf_device.h"

namespace svf {

constexpr int kSelectThreads = 512;
constexpr int kSelectWaves = kSelectThreads / 64;
constexpr int kMaxSelectBlocks = 2 * kSelectThreads;   // blocks per sequence: two keys per thread

// Top-cnt of keys[0 .. nb) by the whole workgroup (Sec. 3.1 top-N rule; equal keys: lowest index
// first).  nb <= kMaxSelectBlocks = 2 * kSelectThreads, so a thread holds keys tid and tid + kSelectThreads.
// Four 8-bit radix passes find the key of the weakest kept block: LDS histogram (one per pass,
// zeroed by the caller), one barrier, then every wavefront scans the 256 bins for itself (four
// bins per lane, wavefront prefix sum), so no second barrier is needed to share the outcome.
// The final placement needs one more barrier: position of a kept block = blocks above the
// threshold before it + min(equal blocks before it, equal blocks wanted).  sel[0 .. cnt) ends up
// ascending.  Requires 1 <= cnt <= nb; all threads of the workgroup must call.
// first_counted: the caller has already counted every key's top digit into hist[0] and passed a
// barrier since (the keys were counted as they came in): the first pass starts at its scan.
struct SelectScratch {
  uint32_t hist[4][256];
  uint32_t seg[2 * kSelectWaves][2];     // per (key slot, wavefront): blocks above / equal to the threshold
};
__device__ __forceinline__ void workgroup_select(const uint32_t* keys, SelectScratch* sc, int nb, int cnt,
                                                 int32_t* sel, int tid, int lane, int wave, bool first_counted) {
  const bool has0 = tid < nb, has1 = tid + kSelectThreads < nb;
  const uint32_t k0 = has0 ? keys[tid] : 0u, k1 = has1 ? keys[tid + kSelectThreads] : 0u;
  uint32_t prefix = 0, need = (uint32_t)cnt;
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const uint32_t hi_mask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
    if (!(pass == 0 && first_counted)) {             // (uniform)
      if (has0 && (k0 & hi_mask) == prefix) atomicAdd(&sc->hist[pass][(k0 >> shift) & 0xff], 1u);
      if (has1 && (k1 & hi_mask) == prefix) atomicAdd(&sc->hist[pass][(k1 >> shift) & 0xff], 1u);
      __syncthreads();
    }
    // lane l owns bins 255 - 4l (in .w) down to 252 - 4l (in .x): higher bins in lower lanes
    const uint4 hq = *reinterpret_cast<const uint4*>(&sc->hist[pass][252 - 4 * lane]);
    const uint32_t own = hq.x + hq.y + hq.z + hq.w;
    const uint32_t incl = wave_inclusive_sum(own);
    uint32_t run = incl - own;                      // keys in bins above this lane's
    const bool cross = incl >= need && run < need;  // exactly one lane
    uint32_t bin = 255u - 4u * (uint32_t)lane, in_bin = hq.w;
    if (run + hq.w < need) {
      run += hq.w; --bin; in_bin = hq.z;
      if (run + hq.z < need) {
        run += hq.z; --bin; in_bin = hq.y;
        if (run + hq.y < need) { run += hq.y; --bin; in_bin = hq.x; }
      }
    }
    const int src = __builtin_ctzll(__ballot(cross));
    prefix |= (uint32_t)__builtin_amdgcn_readlane((int)bin, src) << shift;
    need -= (uint32_t)__builtin_amdgcn_readlane((int)run, src);   // still wanted from inside that bin
    // every key of that bin is wanted: no need to look at the lower digits (the threshold is the
    // bin's smallest possible key, and every key equal to it is kept)
    if (need == (uint32_t)__builtin_amdgcn_readlane((int)in_bin, src)) {
      need = 0xffffffffu;
      break;
    }
  }
  const uint32_t tau = prefix;
  const uint64_t below = (1ull << lane) - 1ull;
  const uint64_t gt0 = __ballot(has0 && k0 > tau), eq0 = __ballot(has0 && k0 == tau);
  const uint64_t gt1 = __ballot(has1 && k1 > tau), eq1 = __ballot(has1 && k1 == tau);
  if (lane == 0) {
    sc->seg[wave][0] = (uint32_t)__popcll(gt0);
    sc->seg[wave][1] = (uint32_t)__popcll(eq0);
    sc->seg[kSelectWaves + wave][0] = (uint32_t)__popcll(gt1);
    sc->seg[kSelectWaves + wave][1] = (uint32_t)__popcll(eq1);
  }
  __syncthreads();
  // Counts over the segments in front of a wavefront's keys: lane s of every wavefront reads
  // segment s (both counts in one word: neither sum exceeds 1024), a prefix sum over the sixteen
  // lanes, and the wavefront picks the entries in front of its own two segments - one LDS round
  // trip instead of one per segment.
  uint32_t packed = 0;
  if (lane < 2 * kSelectWaves) {
    const uint2 sg = *reinterpret_cast<const uint2*>(&sc->seg[lane][0]);
    packed = sg.x | (sg.y << 16);
  }
  packed += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)packed, 0x111, 0xf, 0xf, true);   // row_shr:1
  packed += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)packed, 0x112, 0xf, 0xf, true);   // row_shr:2
  packed += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)packed, 0x114, 0xf, 0xf, true);   // row_shr:4
  packed += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)packed, 0x118, 0xf, 0xf, true);   // row_shr:8
  static_assert(2 * kSelectWaves == 16, "one row of sixteen lanes holds the segments");
  const uint32_t before0 = wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)packed, wave - 1) : 0u;
  uint32_t gt_before = before0 & 0xffffu, eq_before = before0 >> 16;
  {
    const uint32_t e = eq_before + (uint32_t)__popcll(eq0 & below);
    const bool is_gt = (gt0 >> lane) & 1ull, is_eq = (eq0 >> lane) & 1ull;
    if (is_gt || (is_eq && e < need)) sel[gt_before + (uint32_t)__popcll(gt0 & below) + min(e, need)] = tid;
  }
  if (nb > kSelectThreads) {
    const uint32_t before1 = (uint32_t)__builtin_amdgcn_readlane((int)packed, kSelectWaves + wave - 1);
    gt_before = before1 & 0xffffu;
    eq_before = before1 >> 16;
    const uint32_t e = eq_before + (uint32_t)__popcll(eq1 & below);
    const bool is_gt = (gt1 >> lane) & 1ull, is_eq = (eq1 >> lane) & 1ull;
    if (is_gt || (is_eq && e < need)) sel[gt_before + (uint32_t)__popcll(gt1 & below) + min(e, need)] = tid + kSelectThreads;
  }
}

// The same for up to 128 keys, two per lane, by every wavefront for itself: no barrier between the last key and the first
// address.  sel is valid for the wavefront that has called (all write the same).  Two histograms, counted as the keys come
// in with a barrier since, give the first fourteen bits of the weakest kept key, an interval of 1 / 32 of its scores; where that
// holds more keys than are wanted, its other bits are found one by one, by counting the keys that reach a trial value, until
// exactly cnt of them do.
// (us per anchor launch of the fp32 kernel: 64 blocks 8.5 -> 7.9, 94 blocks 16.5 -> 16.3, 125 blocks 18.6 -> 18.3; with eight or twelve bits of histogram no
// faster than the workgroup.  250 blocks 9.6 -> 9.6 and 13.5 -> 13.9: what the workgroup shares out, each of its eight wavefronts then does.)
constexpr int kWaveSelectBlocks = 128;
struct WaveSelectScratch {
  uint32_t coarse[256];                  // keys by their first eight bits,
  uint32_t fine[1 << 13];                // and by their first fourteen: two counts per word
};
__device__ __forceinline__ void clear_counts(WaveSelectScratch* sc, int tid) {
  uint4* const at = reinterpret_cast<uint4*>(sc);
  constexpr int n = (int)(sizeof(WaveSelectScratch) / 16);
#pragma unroll
  for (int u = 0; u < (n + kSelectThreads - 1) / kSelectThreads; ++u)
    if (tid + u * kSelectThreads < n) at[tid + u * kSelectThreads] = make_uint4(0u, 0u, 0u, 0u);
}
__device__ __forceinline__ void count_key(WaveSelectScratch* sc, uint32_t key) {
  atomicAdd(&sc->coarse[key >> 24], 1u);
  atomicAdd(&sc->fine[key >> 19], 1u << ((key >> 14) & 16u));
}
// keys: kWaveSelectBlocks words of LDS, of which nb are set
__device__ __forceinline__ void wave_select(const uint32_t* keys, const WaveSelectScratch* sc, int nb, int cnt, int32_t* sel, int lane) {
  constexpr int SEGS = kWaveSelectBlocks / 64;
  uint32_t key[SEGS];
#pragma unroll
  for (int s = 0; s < SEGS; ++s) key[s] = keys[64 * s + lane];       // (garbage past the last key)
  uint32_t need = (uint32_t)cnt, tau;
  bool all;                                            // every key from tau on is kept
  {
    // lane l owns bins 255 - 4l (in .w) down to 252 - 4l (in .x): higher bins in lower lanes
    const uint4 hq = *reinterpret_cast<const uint4*>(&sc->coarse[252 - 4 * lane]);
    const uint32_t own = hq.x + hq.y + hq.z + hq.w;
    const uint32_t incl = wave_inclusive_sum(own);
    uint32_t run = incl - own;                         // keys in bins above this lane's
    const uint64_t cross = __ballot(incl >= need && run < need);       // exactly one lane
    uint32_t bin = 255u - 4u * (uint32_t)lane, in_bin = hq.w;
    if (run + hq.w < need) {
      run += hq.w; --bin; in_bin = hq.z;
      if (run + hq.z < need) {
        run += hq.z; --bin; in_bin = hq.y;
        if (run + hq.y < need) { run += hq.y; --bin; in_bin = hq.x; }
      }
    }
    const int src = __builtin_ctzll(cross);
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)bin, src);
    need -= (uint32_t)__builtin_amdgcn_readlane((int)run, src);        // still wanted from inside that bin
    tau = first << 24;
    all = need == (uint32_t)__builtin_amdgcn_readlane((int)in_bin, src);
    if (!all) {
      // lane l: the 63 - l-th of the bin's 64 parts
      const uint32_t part = first * 64u + 63u - (uint32_t)lane;
      const uint32_t n = (sc->fine[part >> 1] >> ((part & 1u) * 16u)) & 0xffffu;
      const uint32_t upto = wave_inclusive_sum(n);
      const int at = __builtin_ctzll(__ballot(upto >= need && upto - n < need));
      const uint32_t of = (uint32_t)__builtin_amdgcn_readlane((int)n, at);
      need -= (uint32_t)__builtin_amdgcn_readlane((int)(upto - n), at);
      tau = (first * 64u + 63u - (uint32_t)at) << 18;
      all = need == of;
    }
  }
  for (uint32_t bit = 1u << 17; !all && bit != 0u; bit >>= 1) {
    const uint32_t trial = tau | bit;
    int reach = 0;
#pragma unroll
    for (int s = 0; s < SEGS; ++s)
      if (64 * s < nb) reach += __popcll(__ballot(64 * s + lane < nb && key[s] >= trial));
    if (reach >= cnt) tau = trial;
    all = reach == cnt;
  }
  // (otherwise the weakest kept key is tau and occurs more often than it is wanted)
  int wanted = kWaveSelectBlocks;
  if (!all) {
    wanted = cnt;
#pragma unroll
    for (int s = 0; s < SEGS; ++s)
      if (64 * s < nb) wanted -= __popcll(__ballot(64 * s + lane < nb && key[s] > tau));
  }
  int at = 0;                                          // kept so far
#pragma unroll
  for (int s = 0; s < SEGS; ++s) {
    if (64 * s >= nb) break;                           // (uniform)
    const bool in = 64 * s + lane < nb, equal = in && key[s] == tau;
    const uint64_t e = __ballot(equal);
    const bool keep = (in && key[s] > tau) ||
                      (equal && (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(e >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)e, 0u)) < wanted);
    const uint64_t m = __ballot(keep);
    if (keep) sel[__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)at))] = 64 * s + lane;
    at += __popcll(m);
    wanted -= min(wanted, __popcll(e));
  }
  // (what the lanes have written is read by other lanes of the wavefront)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace svf
