// Sparse feed-forward verification (Sec. 3.4, Eq. 10-14) for the M draft tokens of a step.
//
// Weight-bandwidth-bound: M <= 64 tokens against three [d_ff][d_model] bf16 matrices.  The
// matrix cores do the arithmetic (32x32x16 bf16, tokens padded to 32 or 64 columns; they idle
// most of the time), the work is organising the reads: every weight row is read at most once,
// in long contiguous runs, and the rows of W_up / W_down of hidden channels that are inactive
// for all M tokens are not read at all.
//
//   gate/up kernels one workgroup of four wavefronts per tile (pair of tiles) of hidden channels.
//                   Joint walk (default): the gate and the up matrix together, then
//                   h = act(W_gate x + b_gate), the active bits |h| >= tau per (channel, token),
//                   and h * up, masked per token, out as bf16 to the workspace; x is fetched once
//                   for both matrices and nothing waits between them, but every row of W_up is
//                   read.  Gate first: the gate walk, the active bits, then the same walk over
//                   W_up where a row that no token needs is replaced by a row that is read anyway;
//                   the wavefronts split the model dimension in chunks of 128, a chunk of the tile
//                   (32 rows x 256 bytes) goes to the wavefront's own LDS stage (two stages), the
//                   matching piece of x comes through registers.
//   down kernel     y^T = W_down^T-rows times h_up: one workgroup of eight wavefronts per
//                   (128 output columns, slice of the hidden channels).  The weight rows are
//                   contiguous along the output dimension while the matrix core wants its
//                   operand contiguous along the reduction; each lane therefore loads four
//                   output columns of eight channels and byte-permutes them into operands
//                   (row i of sub-product nt = output column 4 i + nt).  Rows of channels
//                   nobody needs are skipped.  Wavefront results are added in wavefront order
//                   through LDS (one barrier); the slices' partial sums are added, with b_down, by a third
//                   small kernel (fixed order: the result does not depend on scheduling).
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>

#include "svf_ffn_device.h"

namespace svf {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float floatx2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

#define FFN_GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define FFN_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int kTileRows = 32;                          // hidden channels per gate/up workgroup
constexpr int kChunkK = 128;                           // model dimensions per chunk
constexpr int kRowBytes = kChunkK * 2;                 // 256
constexpr int kChunkBytes = kTileRows * kRowBytes;     // 8 KB
constexpr int kGuWaves = 4;
constexpr int kGuThreads = kGuWaves * 64;
constexpr int kStages = 2;

// s_waitcnt with only the vector-memory counter constrained
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
  asm volatile("" ::: "memory");
}
// LDS read issued by hand (a compiler-issued one would first wait for every direct-to-LDS load
// in flight); valid once lds_wait has been given the registers
__device__ __forceinline__ u32x4 lds_read16(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr) : "memory");
  return v;
}
__device__ __forceinline__ void lds_wait(u32x4 (&r)[8]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7])
               :
               : "memory");
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const floatx2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));   // round to nearest even
}

__device__ __forceinline__ float activate(float z, int act) {
  if (act == SVF_ACT_SILU) return z / (1.0f + __expf(-z));
  return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}

// h * up of token m and hidden channel c in the workspace: [d_ff / 16][32 NT tokens][16 channels], so that
// what a step of the down projection reads (16 channels of all tokens) is contiguous.
template <int NT>
__device__ __forceinline__ char* h_up_at(const FfnParams& p, int m, int c) {
  return static_cast<char*>(p.h_up) + (((int64_t)(c >> 4) * (32 * NT) + m) * 16 + (c & 15)) * 2;
}

// One walk of a wavefront over its chunks of a 32-row tile of NMAT matrices at once (the same
// rows of each): acc[mat][t] += W_mat_tile(chunk) x^T(chunk).
//   w_rows[mat]: address of row 0 of the tile in matrix mat; row_of(r): which tile row to read
//   for row r (a row nobody needs is redirected, its products are thrown away); stage: the
//   wavefront's two LDS stages of NMAT chunks each.
//   The workgroup's n_waves wavefronts take the chunks wave, wave + n_waves, ...
template <int NT, int NMAT, typename RowOf>
__device__ __forceinline__ void walk_tile(const FfnParams& p, const char* const (&w_rows)[NMAT], RowOf row_of,
                                          const char* x, unsigned char* stage, int wave, int n_waves, int lane,
                                          floatx16 (&acc)[NMAT][NT]) {
  constexpr int kStageBytes = NMAT * kChunkBytes;
  const int l32 = lane & 31, g = lane >> 5;
  const int n_chunks = p.d_model / kChunkK;
  const int64_t row_bytes = (int64_t)p.d_model * 2;
  // direct-to-LDS loads: instruction n brings rows 4n .. 4n+3, 16 lanes per row; the 16-byte
  // piece at position c of row r holds piece c ^ (r mod 16) of the chunk (bank spreading)
  const int lrow = lane >> 4, lcol = lane & 15;
  int64_t src_off[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const int r = 4 * n + lrow;
    src_off[n] = (int64_t)row_of(r) * row_bytes + ((lcol ^ (r & 15)) << 4);
  }
  // x rows of this lane's token(s): eight 16-byte pieces per chunk (k-step ks, lane half g)
  const char* xrow[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) xrow[t] = x + (int64_t)min(l32 + 32 * t, p.M - 1) * row_bytes + g * 16;

  auto issue = [&](int kc, unsigned char* dst) {
#pragma unroll
    for (int mat = 0; mat < NMAT; ++mat)
#pragma unroll
      for (int n = 0; n < 8; ++n)
        __builtin_amdgcn_global_load_lds(FFN_GLOBAL_PTR(w_rows[mat] + src_off[n] + (int64_t)kc * kRowBytes),
                                         FFN_LDS_PTR(dst + mat * kChunkBytes + n * 1024), 16, 0, 2);
  };
  u32x4 xr[NT][8];
  auto load_x = [&](int kc) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
        xr[t][ks] = *reinterpret_cast<const u32x4*>(xrow[t] + (int64_t)kc * kRowBytes + ks * 32);
  };
  auto compute = [&](const unsigned char* src) {
    const uint32_t kx = (uint32_t)((g ^ (l32 & 15)) << 4);
#pragma unroll
    for (int mat = 0; mat < NMAT; ++mat) {
      const uint32_t base = (uint32_t)(uintptr_t)FFN_LDS_PTR(src + mat * kChunkBytes) + l32 * kRowBytes;
      u32x4 wf[8];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) wf[ks] = lds_read16(base + (kx ^ (uint32_t)(ks << 5)));
      lds_wait(wf);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[mat][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[ks]),
                                                                __builtin_bit_cast(bf16x8, xr[t][ks]), acc[mat][t], 0,
                                                                0, 0);
    }
  };

  // The weight chunk after this one is on its way into the other
  // stage while this one is multiplied; the x pieces of the next chunk are loaded right after
  // the multiply (one register set), long before that chunk's weights can have arrived.  Loads
  // retire in order, so "all but the 8 NMAT just issued" is one fixed wait count.
  int kc = wave;
  if (kc >= n_chunks) return;
  issue(kc, stage);
  load_x(kc);
  int cur = 0;
  while (true) {
    const int kn = kc + n_waves;
    if (kn >= n_chunks) {
      wait_vmcnt<0>();
      compute(stage + cur * kStageBytes);
      break;
    }
    issue(kn, stage + (cur ^ 1) * kStageBytes);
    wait_vmcnt<8 * NMAT>();
    compute(stage + cur * kStageBytes);
    load_x(kn);
    kc = kn;
    cur ^= 1;
  }
}

// grid: (d_ff / 32); block: 256
template <int NT>
__global__ __launch_bounds__(kGuThreads) void ffn_gate_up_kernel(FfnParams p) {
  constexpr int RS = 32 * NT + 1;                        // row stride of the [channel][token] tiles in LDS
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kGuWaves * kStages * kChunkBytes];
  __shared__ float s_h[kTileRows * RS];
  __shared__ uint64_t s_act[kTileRows];
  static_assert(kTileRows * RS * 4 <= kStages * kChunkBytes, "a wavefront's partial tile fits its own stages");

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31, g = lane >> 5;
  const int c0 = blockIdx.x * kTileRows;
  unsigned char* stage = smem + wave * (kStages * kChunkBytes);
  float* red = reinterpret_cast<float*>(stage);         // this wavefront's partial [channel][token]
  const char* x = static_cast<const char*>(p.x);
  const int64_t row_bytes = (int64_t)p.d_model * 2;

  auto put_partial = [&](const floatx16 (&acc)[NT]) {
    // value v of a lane is channel 8 (v / 4) + 4 g + v % 4, token l32 (+ 32 t)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[(8 * (v >> 2) + 4 * g + (v & 3)) * RS + l32 + 32 * t] = acc[t][v];
  };
  auto sum_partials = [&](int c, int m) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kGuWaves; ++w)
      s += reinterpret_cast<const float*>(smem + w * (kStages * kChunkBytes))[c * RS + m];
    return s;
  };

  // ---- gate: h = act(W_gate x + b_gate), active bits (Eq. 10, 12) ----
  floatx16 acc[1][NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][t][v] = 0.f;
  {
    const char* const rows[1] = {static_cast<const char*>(p.w_gate) + (int64_t)c0 * row_bytes};
    walk_tile<NT, 1>(p, rows, [](int r) { return r; }, x, stage, wave, kGuWaves, lane, acc);
  }
  put_partial(acc[0]);
  __syncthreads();
  {
    // thread: channel tid / 8, tokens (tid % 8) * 4 NT ... + 4 NT
    const int c = tid >> 3, m0 = (tid & 7) * 4 * NT;
    const float bg = p.b_gate ? p.b_gate[c0 + c] : 0.f;
    uint64_t bits = 0;
#pragma unroll
    for (int i = 0; i < 4 * NT; ++i) {
      const int m = m0 + i;
      const float h = activate(sum_partials(c, m) + bg, p.act);
      s_h[c * RS + m] = h;
      if (m < p.M && !(fabsf(h) < p.tau)) bits |= 1ull << m;
    }
    // the eight threads of a channel are neighbours in a wavefront
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      const uint32_t lo = __shfl_xor((uint32_t)bits, o, 64), hi = __shfl_xor((uint32_t)(bits >> 32), o, 64);
      bits |= (uint64_t)lo | ((uint64_t)hi << 32);
    }
    if ((tid & 7) == 0) {
      s_act[c] = bits;
      p.rowany[c0 + c] = bits != 0 ? 1 : 0;
      if (p.active) p.active[c0 + c] = bits;
    }
  }
  __syncthreads();                                        // partials read, s_h / s_act written

  // ---- up: only rows some token needs are read; h * up per token (Eq. 13) ----
  const uint64_t my_bits = s_act[l32];
  const uint32_t rowmask = (uint32_t)__ballot(my_bits != 0 && lane < 32);
  bf16x8 zero8;
#pragma unroll
  for (int i = 0; i < 8; ++i) zero8[i] = 0;
  // thread: token tid / 4, channels (tid % 4) * 8 ... + 8 (16 bytes of h_up)
  const int om = tid >> 2, oc = (tid & 3) * 8;
  char* out = h_up_at<NT>(p, om, c0 + oc);
  if (rowmask == 0) {                                     // uniform: nothing of this tile is used
    if (om < 32 * NT) *reinterpret_cast<bf16x8*>(out) = zero8;
    return;
  }
  const int first = __builtin_ctz(rowmask);
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][t][v] = 0.f;
  {
    const char* const rows[1] = {static_cast<const char*>(p.w_up) + (int64_t)c0 * row_bytes};
    walk_tile<NT, 1>(p, rows, [=](int r) { return ((rowmask >> r) & 1u) ? r : first; }, x, stage, wave, kGuWaves, lane,
                     acc);
  }
  put_partial(acc[0]);
  __syncthreads();
  if (om < 32 * NT) {
    u32x4 w;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float hu[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int c = oc + 2 * j + e;
        const float up = sum_partials(c, om) + (p.b_up ? p.b_up[c0 + c] : 0.f);
        hu[e] = ((s_act[c] >> om) & 1ull) ? s_h[c * RS + om] * up : 0.f;
      }
      w[j] = pack_bf16(hu[0], hu[1]);
    }
    *reinterpret_cast<u32x4*>(out) = w;
  }
}

// Four channels ch .. ch + 3 of all tokens: activation, active bits, h * up (Eq. 10, 12, 13).  A lane is a
// token (two groups of channels side by side where 32 lanes hold all tokens): the active bits of a channel
// are one ballot, and the four channels of h * up leave in one store.  gate(j, m), up(j, m): the sums of
// channel j of the four, with their biases; here: whether this lane's four channels are to be
// written.  All lanes must call.
template <int NT> constexpr int kSide = NT == 1 ? 2 : 1;
template <int NT, typename Gate, typename Up>
__device__ __forceinline__ void finish_channels(const FfnParams& p, int lane, int ch, bool here, Gate&& gate, Up&& up) {
  const int m = NT == 1 ? lane & 31 : lane;
  float hu[4];
  uint64_t bits[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float h = activate(gate(j, m), p.act);
    const bool on = here && m < p.M && !(fabsf(h) < p.tau);
    bits[j] = __ballot(on);
    if (NT == 1) bits[j] = lane >= 32 ? bits[j] >> 32 : bits[j] & 0xffffffffull;
    hu[j] = on ? h * up(j, m) : 0.f;
  }
  if (here) {
    *reinterpret_cast<u32x2*>(h_up_at<NT>(p, m, ch)) = u32x2{pack_bf16(hu[0], hu[1]), pack_bf16(hu[2], hu[3])};
    if (m < 4) {
      const uint64_t mine = m == 0 ? bits[0] : m == 1 ? bits[1] : m == 2 ? bits[2] : bits[3];
      p.rowany[ch + m] = mine != 0 ? 1 : 0;
      if (p.active) p.active[ch + m] = mine;
    }
  }
}

// The biases of a workgroup's channels go to LDS in front of the first stage ([gate, up][64], wavefronts 0 and
// 1).  Loaded where they are added, they were one trip to memory after the other behind the walk, and the
// branches around them kept the quads' sums apart also where there are none.  Whole layer, with what
// ffn_reduce_kernel saves: 20 tokens, 2048 x 4128, biases 22.2 -> 21.5 us; 60 tokens, 4096 x 14336, biases
// 72.8 -> 71.9, without 71.9 -> 71.3.
// channel: this lane's.  They have landed when a later stage has (wavefronts 0 and 1 wait for one at least); the
// caller's barriers show them to everybody.
__device__ __forceinline__ void request_biases(const FfnParams& p, int wave, int channel, float* s_bias) {
  const float* const b = wave == 0 ? p.b_gate : p.b_up;
  if (wave < 2 && b)
    __builtin_amdgcn_global_load_lds(FFN_GLOBAL_PTR(b + channel), FFN_LDS_PTR(s_bias + 64 * wave), 4, 0, 0);
}

// The same result with the gate and the up matrix walked together: the workgroup's memory pipeline does
// not run dry between a gate and an up walk; the price is that every row of W_up is read, needed or not.
//
// Bound by HBM, and that by the bytes a compute unit keeps in flight: a workgroup is four wavefronts, one
// per (matrix, channel tile) of two tiles, that walk the model dimension together in chunks of 64.
// A chunk of all four (32 rows x 128 bytes each) and of x goes straight to LDS; 6 (more than 32 tokens)
// or 7 chunks' stages form a ring of which all but one are on their way, 80 - 96 KB of weights per compute
// unit.  One barrier per chunk: behind it the chunk has landed for everybody, and everybody has left
// the one before, whose stage takes the next request.  x is shared by the four wavefronts, and a
// wavefront has its tile's whole sum: nothing is added up afterwards.
// (Wavefronts that split the model dimension with two private stages of 128 each kept 64 KB in flight at
// most, fetched x from L2 into registers and added four partial tiles at the end.  14336 x 4096: 40.6 -> 39.0 us,
// 6.0 TB/s, for 8 tokens; 51.4 -> 43.0 us for 60, where the order of the chunks matters, see `first`.)
//   One workgroup per compute unit, so the tile height tile_rows <= 32 is chosen such that the
//   workgroups fill whole rounds; the rows of the 32-row matrix-core tile past it repeat its last
//   row, and a tile that would reach past d_ff is moved back to end there (the channels it shares with
//   the tile before it are that tile's to write: workgroups add in different orders).
constexpr int kWalkK = 64;                               // model dimensions per chunk
constexpr int kWalkRow = kWalkK * 2;                     // 128 bytes
constexpr int kWalkTile = kTileRows * kWalkRow;          // 4 KB: one wavefront's rows, or 32 tokens of x
// XT: 32-token pieces of x in a stage, NT per chunk
template <int XT> constexpr int kWalkStage = (kGuWaves + XT) * kWalkTile;
template <int XT> constexpr int kWalkStages = XT == 1 ? 7 : 6;
template <int XT> constexpr int kWalkLoads = 4 + XT;     // load instructions of a wavefront per stage

// Waits until this wavefront's loads of all but `stages` (0 .. 5) stages have landed.
template <int XT>
__device__ __forceinline__ void wait_walk(int stages) {
  switch (stages) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<kWalkLoads<XT>>(); break;
    case 2: wait_vmcnt<2 * kWalkLoads<XT>>(); break;
    case 3: wait_vmcnt<3 * kWalkLoads<XT>>(); break;
    case 4: wait_vmcnt<4 * kWalkLoads<XT>>(); break;
    default: wait_vmcnt<5 * kWalkLoads<XT>>(); break;
  }
}

// Four reads of a 32-row piece of a stage (row l32, k-steps 0 .. 3): piece c of row r sits at position
// c ^ ((r / 2) mod 8), so that sixteen neighbouring rows hit different banks.
__device__ __forceinline__ void read_fragments(u32x4 (&f)[4], uint32_t row, uint32_t kx) {
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) f[ks] = lds_read16(row + (kx ^ (uint32_t)(ks << 5)));
}
__device__ __forceinline__ void fragments_wait(u32x4 (&f)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]) : : "memory");
}

// TILES = 2 as above.  TILES = 1 (up to 32 tokens): one channel tile per workgroup, for hidden sizes whose
// pairs of tiles fill their rounds badly; a stage then holds two chunks, wavefronts 0 and 1 walk the
// even ones and 2 and 3 the odd ones (d_model is a multiple of two chunks), and the two sums are added last.
// grid: (ceil(ceil(d_ff / tile_rows) / TILES)); block: 256
template <int NT, int TILES>
__global__ __launch_bounds__(kGuThreads) void ffn_gate_up_fused_kernel(FfnParams p) {
  constexpr int KP = 2 / TILES;                          // chunks per stage
  constexpr int XT = NT * KP;
  constexpr int RS = 32 * NT + 1;                        // row stride of the [wavefront][channel][token] sums
  constexpr int S = kWalkStages<XT>;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S * kWalkStage<XT>];
  __shared__ float s_bias[2 * 64];                       // [gate, up][32 tile + channel]
  static_assert(kGuWaves * kTileRows * RS * 4 <= S * kWalkStage<XT>, "the sums fit the stages");
  static_assert(S - 2 <= 5, "wait_walk");

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31, g = lane >> 5;
  const int R = p.walk.tile_rows;
  const int n_steps = p.d_model / (kWalkK * KP);         // stages to walk
  // wavefront w: gate (even) or up (odd) matrix; tile w / 2 of the workgroup's two, or chunk w / 2 of a stage
  const int half = wave >> 1;
  const int c0 = min((blockIdx.x * TILES + (TILES == 2 ? half : 0)) * R, p.d_ff - R);
  // (a tile's and x's offsets fit 32 bits: at most 64 rows of 2 MB)
  const uint32_t row_bytes = (uint32_t)p.d_model * 2u;
  const char* const w_tile = static_cast<const char*>((wave & 1) ? p.w_up : p.w_gate) + (int64_t)c0 * row_bytes;
  // load n of a tile brings rows 8n .. 8n + 7, eight lanes per row
  uint32_t w_off[4], x_off[XT];
  const int lrow = lane >> 3, lcol = lane & 7;
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int r = 8 * n + lrow;
    w_off[n] = (uint32_t)min(r, R - 1) * row_bytes + (uint32_t)((lcol ^ ((r >> 1) & 7)) << 4);
  }
  // x: wavefront w brings loads w XT .. w XT + XT - 1 of the stage's 4 XT, those of chunk w / 2 where there
  // are two (tokens past the last repeat it)
#pragma unroll
  for (int t = 0; t < XT; ++t) {
    const int r = 8 * ((wave * XT + t) % (4 * NT)) + lrow;
    x_off[t] = (uint32_t)min(r, p.M - 1) * row_bytes + (uint32_t)((lcol ^ ((r >> 1) & 7)) << 4);
  }
  // Workgroups start at different chunks: a chunk of x lies in rows d_model apart, a power of two as a
  // rule, which is few memory channels, and the 32 compute units of an XCD would all ask them at once.
  const int first = (int)((blockIdx.x / 8) % 32 * (uint32_t)n_steps / 32);
  auto request = [&](int i, unsigned char* st) {
    const int k = i + first;
    uint32_t koff = (uint32_t)((k >= n_steps ? k - n_steps : k) * KP + (TILES == 1 ? half : 0)) * kWalkRow;
    asm volatile("" : "+s"(koff));                       // (a scalar of its own: no per-lane pointers advanced in every round)
    const char* wb = w_tile + koff;
    const char* xb = static_cast<const char*>(p.x) + koff;
#pragma unroll
    for (int n = 0; n < 4; ++n)
      __builtin_amdgcn_global_load_lds(FFN_GLOBAL_PTR(wb + w_off[n]), FFN_LDS_PTR(st + wave * kWalkTile + n * 1024), 16, 0, 2);
#pragma unroll
    for (int t = 0; t < XT; ++t)
      __builtin_amdgcn_global_load_lds(FFN_GLOBAL_PTR(xb + x_off[t]),
                                       FFN_LDS_PTR(st + kGuWaves * kWalkTile + (wave * XT + t) * 1024), 16, 0, 0);
  };

  floatx16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

  const uint32_t lds = (uint32_t)(uintptr_t)FFN_LDS_PTR(smem);
  const uint32_t kx = (uint32_t)((g ^ ((l32 >> 1) & 7)) << 4);
  const uint32_t frag = lds + (uint32_t)l32 * kWalkRow;
  request_biases(p, wave, min((blockIdx.x * TILES + (TILES == 2 ? g : 0)) * R, p.d_ff - R) + min(l32, R - 1), s_bias);
  const uint32_t x_piece = (uint32_t)(kGuWaves + (TILES == 1 ? half : 0)) * kWalkTile;
  for (int i = 0; i < min(S - 1, n_steps); ++i) request(i, smem + i * kWalkStage<XT>);
  int st = 0;                                            // stage of step i
  for (int i = 0; i < n_steps; ++i) {
    wait_walk<XT>(min(S - 2, n_steps - 1 - i));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int prev = st == 0 ? S - 1 : st - 1;
    if (i + S - 1 < n_steps) request(i + S - 1, smem + prev * kWalkStage<XT>);
    uint32_t base = frag + (uint32_t)st * kWalkStage<XT>;
    u32x4 wf[4], xf[NT][4];
    read_fragments(wf, base + (uint32_t)wave * kWalkTile, kx);
#pragma unroll
    for (int t = 0; t < NT; ++t) read_fragments(xf[t], base + x_piece + (uint32_t)t * kWalkTile, kx);
    fragments_wait(wf);
#pragma unroll
    for (int t = 0; t < NT; ++t) fragments_wait(xf[t]);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[ks]),
                                                         __builtin_bit_cast(bf16x8, xf[t][ks]), acc[t], 0, 0, 0);
    st = st == S - 1 ? 0 : st + 1;
  }
  __syncthreads();                                       // everybody has left the last stages
  // value v of a lane is channel 8 (v / 4) + 4 g + v % 4, token l32 (+ 32 t)
  float* sums = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      sums[(wave * kTileRows + 8 * (v >> 2) + 4 * g + (v & 3)) * RS + l32 + 32 * t] = acc[t][v];
  __syncthreads();
  const int quads = R / 4;                               // groups of four channels per tile
  for (int q0 = wave * kSide<NT>; q0 < TILES * quads; q0 += kGuWaves * kSide<NT>) {
    const int q = q0 + (NT == 1 ? g : 0);
    const int tile = TILES == 2 && q >= quads ? 1 : 0, c = q < TILES * quads ? 4 * (q - tile * quads) : 0;
    const int nominal = (blockIdx.x * TILES + tile) * R;
    const int ch = min(nominal, p.d_ff - R) + c;
    const float* zg = sums + (2 * tile * kTileRows + c) * RS;
    auto sum = [&](int row, int m) {                     // (TILES = 1: the even and the odd chunks')
      float z = zg[row * RS + m];
      if (TILES == 1) z += zg[(2 * kTileRows + row) * RS + m];
      return z;
    };
    const float* bias = s_bias + kTileRows * tile + c;
    finish_channels<NT>(p, lane, ch, q < TILES * quads && ch >= nominal,
                        [&](int j, int m) { return sum(j, m) + (p.b_gate ? bias[j] : 0.f); },
                        [&](int j, int m) { return sum(kTileRows + j, m) + (p.b_up ? bias[64 + j] : 0.f); });
  }
}

// The same for few hidden channels, where the walk above would leave compute units idle: a workgroup takes
// RC channels only (16, or 8), gate and up rows in one 32-row matrix-core tile, and its four
// wavefronts split the model dimension (wavefront w: chunks w, w + 4, ...), each with a ring of
// stages of its own, so that nothing but the final addition needs a barrier.  Bound by the chain of trips to
// memory: a quarter as long as the walk above's, with everything that fits LDS on its way.  x takes
// XR kilobytes of a stage (eight tokens each: few tokens leave room for more stages).
// (Whole layer, all three launches: 4096 x 2048, 4 tokens 22.5 -> 18.0 us; 4096 x 1024, 60 tokens 52 ->
// 25.7 us; 5120 x 3072, 64 tokens 66 -> 39 us.)
// grid: (d_ff / RC); block: 256
template <int RC, int XR> constexpr int kSplitStage = RC * 2 * kWalkRow + XR * 8 * kWalkRow;
template <int RC, int XR> constexpr int kSplitStages = 36 * 1024 / kSplitStage<RC, XR> < 8 ? 36 * 1024 / kSplitStage<RC, XR> : 8;
template <int RC, int XR>
__device__ __forceinline__ void wait_split(int chunks) {   // all but `chunks` (0 .. 7) chunks have landed
  constexpr int LPC = RC / 4 + XR;                       // load instructions of a chunk
  switch (chunks) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<LPC>(); break;
    case 2: wait_vmcnt<2 * LPC>(); break;
    case 3: wait_vmcnt<3 * LPC>(); break;
    case 4: wait_vmcnt<4 * LPC < 64 ? 4 * LPC : 63>(); break;
    case 5: wait_vmcnt<5 * LPC < 64 ? 5 * LPC : 63>(); break;
    case 6: wait_vmcnt<6 * LPC < 64 ? 6 * LPC : 63>(); break;
    default: wait_vmcnt<7 * LPC < 64 ? 7 * LPC : 63>(); break;
  }
}
template <int RC, int XR>
__global__ __launch_bounds__(kGuThreads) void ffn_gate_up_split_kernel(FfnParams p) {
  constexpr int NT = XR == 8 ? 2 : 1;
  constexpr int RS = 32 * NT + 1;
  constexpr int S = kSplitStages<RC, XR>, SB = kSplitStage<RC, XR>;
  static_assert((S - 1) * (RC / 4 + XR) < 64, "the wait counts of a full ring are exact");
  constexpr int kSums = kGuWaves * kTileRows * RS * 4;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kGuWaves * S * SB > kSums ? kGuWaves * S * SB : kSums];
  __shared__ float s_bias[2 * 64];                       // [gate, up][channel]

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31, g = lane >> 5;
  const int c0 = blockIdx.x * RC;
  const int n_chunks = p.d_model / kWalkK;
  const int n = (n_chunks - wave + kGuWaves - 1) / kGuWaves;              // of this wavefront (may be 0)
  const uint32_t row_bytes = (uint32_t)p.d_model * 2u;
  const char* const wg = static_cast<const char*>(p.w_gate) + (int64_t)c0 * row_bytes;
  const char* const wu = static_cast<const char*>(p.w_up) + (int64_t)c0 * row_bytes;
  unsigned char* const ring = smem + wave * (S * SB);
  // load j brings rows 8j .. 8j + 7 (eight lanes per row) of: RC gate rows, RC up rows, 8 XR tokens
  const int lrow = lane >> 3, lcol = lane & 7;
  auto swizzled = [&](int r) { return (uint32_t)((lcol ^ ((r >> 1) & 7)) << 4); };
  uint32_t w_off[RC / 8], x_off[XR];
#pragma unroll
  for (int j = 0; j < RC / 8; ++j) w_off[j] = (uint32_t)(8 * j + lrow) * row_bytes + swizzled(8 * j + lrow);
#pragma unroll
  for (int j = 0; j < XR; ++j) x_off[j] = (uint32_t)min(8 * j + lrow, p.M - 1) * row_bytes + swizzled(8 * j + lrow);
  // (workgroups start at different chunks, see above)
  const int first = (int)((blockIdx.x / 8) % 32 * (uint32_t)n / 32);
  auto request = [&](int i, unsigned char* st) {
    const int k = i + first;
    uint32_t koff = (uint32_t)(wave + kGuWaves * (k >= n ? k - n : k)) * kWalkRow;
    asm volatile("" : "+s"(koff));
#pragma unroll
    for (int j = 0; j < RC / 8; ++j) {
      __builtin_amdgcn_global_load_lds(FFN_GLOBAL_PTR(wg + koff + w_off[j]), FFN_LDS_PTR(st + j * 1024), 16, 0, 2);
      __builtin_amdgcn_global_load_lds(FFN_GLOBAL_PTR(wu + koff + w_off[j]), FFN_LDS_PTR(st + (RC / 8 + j) * 1024), 16, 0, 2);
    }
#pragma unroll
    for (int j = 0; j < XR; ++j)
      __builtin_amdgcn_global_load_lds(FFN_GLOBAL_PTR(static_cast<const char*>(p.x) + koff + x_off[j]),
                                       FFN_LDS_PTR(st + (RC / 4 + j) * 1024), 16, 0, 0);
  };

  floatx16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

  // Matrix-core row l32: gate channel l32 (< 16) or up channel l32 - 16; at RC = 8 the upper eight of either repeat
  // the lower, and tokens past the staged ones repeat them (their results are not looked at).
  const int wr = (l32 & (RC - 1)) + (l32 >> 4) * RC;      // (swizzled by the row within its matrix)
  const uint32_t lds = (uint32_t)(uintptr_t)FFN_LDS_PTR(ring);
  const uint32_t w_row = lds + (uint32_t)wr * kWalkRow, w_kx = (uint32_t)((g ^ (((wr & (RC - 1)) >> 1) & 7)) << 4);
  uint32_t x_row[NT], x_kx[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int r = (l32 + 32 * t) & (8 * XR - 1);
    x_row[t] = lds + (uint32_t)(RC * 2 + r) * kWalkRow;
    x_kx[t] = (uint32_t)((g ^ ((r >> 1) & 7)) << 4);
  }
  request_biases(p, wave, c0 + (lane & (RC - 1)), s_bias);
  for (int i = 0; i < min(S, n); ++i) request(i, ring + i * SB);
  int st = 0;
  for (int i = 0; i < n; ++i) {
    wait_split<RC, XR>(min(S, n - i) - 1);
    const uint32_t at = (uint32_t)st * SB;
    u32x4 wf[4], xf[NT][4];
    read_fragments(wf, w_row + at, w_kx);
#pragma unroll
    for (int t = 0; t < NT; ++t) read_fragments(xf[t], x_row[t] + at, x_kx[t]);
    fragments_wait(wf);
#pragma unroll
    for (int t = 0; t < NT; ++t) fragments_wait(xf[t]);
    if (i + S < n) request(i + S, ring + st * SB);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[ks]),
                                                         __builtin_bit_cast(bf16x8, xf[t][ks]), acc[t], 0, 0, 0);
    st = st == S - 1 ? 0 : st + 1;
  }
  __syncthreads();                                       // everybody has left the rings
  float* sums = reinterpret_cast<float*>(smem);          // [wavefront][row][token]
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      sums[(wave * kTileRows + 8 * (v >> 2) + 4 * g + (v & 3)) * RS + l32 + 32 * t] = acc[t][v];
  __syncthreads();
  auto total = [&](int row, int m) {
    float z = 0.f;
#pragma unroll
    for (int w = 0; w < kGuWaves; ++w) z += sums[(w * kTileRows + row) * RS + m];
    return z;
  };
  constexpr int kQuads = RC / 4;
  for (int q0 = wave * kSide<NT>; q0 < kQuads; q0 += kGuWaves * kSide<NT>) {
    const int q = q0 + (NT == 1 ? g : 0);
    const int c = q < kQuads ? 4 * q : 0;
    finish_channels<NT>(p, lane, c0 + c, q < kQuads,
                        [&](int j, int m) { return total(c + j, m) + (p.b_gate ? s_bias[c + j] : 0.f); },
                        [&](int j, int m) { return total(16 + c + j, m) + (p.b_up ? s_bias[64 + c + j] : 0.f); });
  }
}

// ---- down projection ---------------------------------------------------------------------------
constexpr int kDnWaves = 8;
constexpr int kDnThreads = kDnWaves * 64;
constexpr int kDnCols = 128;                             // output columns per workgroup
constexpr int kDepth = 2;                                // k-steps of 16 channels loaded ahead

template <int NT>
struct DownLoads {
  u32x2 w[8];                                            // four output columns of eight channels
  u32x4 h[NT];                                           // h_up of this lane's token(s) for its eight channels
  uint32_t bits;                                         // which of the step's 16 channels are needed
};

// grid: (k_splits * d_model / 128), slices fastest: workgroups are dealt to the eight XCDs in turn, so with
// eight slices an XCD reads whole rows of the weights and one slice of h * up.  (Column tiles fastest, an
// XCD read every eighth 256-byte piece of all rows, d_model apart: a few of its L2's channels.  14336 x
// 4096, 80 % of the rows: 20.2 -> 19.0 us for 8 tokens; 31.5 -> 26.0 us for 60, whose h * up was 32 rows
// d_ff apart per load.)
// block: 512
template <int NT>
__global__ __launch_bounds__(kDnThreads) void ffn_down_kernel(FfnParams p) {
  constexpr int kRedStride = kDnCols + 4;                // floats per token row: keeps rows off each other's banks
  __shared__ __attribute__((aligned(16))) float s_red[kDnWaves][32 * kRedStride];        // [wavefront][token][column]

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31, g = lane >> 5;
  const int slice = blockIdx.x % p.k_splits;
  const int n0 = blockIdx.x / p.k_splits * kDnCols;
  const int n_steps = p.d_ff / 16;
  const int stride = kDnWaves * p.k_splits;
  const int first = slice * kDnWaves + wave;
  const int64_t row_bytes = (int64_t)p.d_model * 2;
  const char* wd = static_cast<const char*>(p.w_down_t) + (int64_t)(n0 + 4 * l32) * 2;

  floatx16 acc[NT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][nt][v] = 0.f;

  // k-slot e of lane half g in step s is channel 16 s + 8 g + e
  auto load_step = [&](int s, DownLoads<NT>& d) {
    d.bits = 0;
    if (s < n_steps) {                                                            // uniform
      const u32x4 any = *reinterpret_cast<const u32x4*>(p.rowany + 16 * s);     // one byte per channel
#pragma unroll
      for (int i = 0; i < 16; ++i) d.bits |= ((any[i >> 2] >> (8 * (i & 3))) & 0xffu) ? (1u << i) : 0u;
    }
    const uint32_t mine = (d.bits >> (8 * g)) & 0xffu;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      u32x2 v = {0u, 0u};
      if ((mine >> e) & 1u)
        v = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(wd + (int64_t)(16 * s + 8 * g + e) * row_bytes));
      d.w[e] = v;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (d.bits != 0) v = *reinterpret_cast<const u32x4*>(h_up_at<NT>(p, l32 + 32 * t, 16 * s + 8 * g));
      d.h[t] = v;
    }
  };
  auto compute_step = [&](const DownLoads<NT>& d) {
    if (d.bits == 0) return;                              // uniform: no channel of the step is needed
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      u32x4 w;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t a = nt < 2 ? d.w[2 * j][0] : d.w[2 * j][1];
        const uint32_t b = nt < 2 ? d.w[2 * j + 1][0] : d.w[2 * j + 1][1];
        w[j] = __builtin_amdgcn_perm(b, a, (nt & 1) ? 0x07060302u : 0x05040100u);
      }
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w),
                                                             __builtin_bit_cast(bf16x8, d.h[t]), acc[t][nt], 0, 0, 0);
    }
  };

  // software pipeline, kDepth steps ahead (register sets rotate by full unrolling)
  DownLoads<NT> ring[kDepth + 1];
#pragma unroll
  for (int i = 0; i < kDepth; ++i) load_step(first + i * stride, ring[i]);
  for (int s = first; s < n_steps; s += (kDepth + 1) * stride) {
#pragma unroll
    for (int i = 0; i <= kDepth; ++i) {
      load_step(s + (i + kDepth) * stride, ring[(i + kDepth) % (kDepth + 1)]);
      compute_step(ring[i]);
    }
  }

  // Every wavefront parks the rows of the real tokens (32 token columns at a time) in LDS; after
  // one barrier the 512 threads add the eight wavefronts' values in wavefront order and write
  // the slice's partial sums as whole rows.
  // value v of a lane: output column n0 + 4 (8 (v / 4) + 4 g + v % 4) + nt, token l32 (+ 32 t)
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t > 0) __syncthreads();                           // the round before has been read
    if (l32 + 32 * t < p.M) {
      float* row = &s_red[wave][l32 * kRedStride];
#pragma unroll
      for (int v = 0; v < 16; ++v)
        *reinterpret_cast<float4*>(row + 4 * (8 * (v >> 2) + 4 * g + (v & 3))) =
            make_float4(acc[t][0][v], acc[t][1][v], acc[t][2][v], acc[t][3][v]);
    }
    __syncthreads();
    const int rows = min(p.M - 32 * t, 32);
    for (int i = tid; i < rows * (kDnCols / 4); i += kDnThreads) {
      const int m = i / (kDnCols / 4), c4 = i - m * (kDnCols / 4);
      float4 sum = *reinterpret_cast<const float4*>(&s_red[0][m * kRedStride + 4 * c4]);
#pragma unroll
      for (int w = 1; w < kDnWaves; ++w) {
        const float4 o = *reinterpret_cast<const float4*>(&s_red[w][m * kRedStride + 4 * c4]);
        sum.x += o.x; sum.y += o.y; sum.z += o.z; sum.w += o.w;
      }
      *reinterpret_cast<float4*>(p.partial + ((int64_t)slice * p.M + 32 * t + m) * p.d_model + n0 + 4 * c4) = sum;
    }
  }
}

// y = bf16(sum over slices of partial + b_down); grid: (ceil(d_model / (4 * 64)), M).  A launch and one trip to
// memory: the bias is on its way with the partials, and a row per workgroup leaves no division in front of them.
__global__ __launch_bounds__(64) void ffn_reduce_kernel(FfnParams p) {
  const int n = (blockIdx.x * 64 + threadIdx.x) * 4;
  if (n >= p.d_model) return;
  const int64_t i4 = (int64_t)blockIdx.y * p.d_model + n;
  const int64_t total = (int64_t)p.M * p.d_model;
  float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
  if (p.b_down) b = *reinterpret_cast<const float4*>(p.b_down + n);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  // eight slices requested before the first is added (one after the other, every slice costs a
  // trip to memory); added in slice order
  for (int k0 = 0; k0 < p.k_splits; k0 += 8) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = *reinterpret_cast<const float4*>(p.partial + (int64_t)min(k0 + u, p.k_splits - 1) * total + i4);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (k0 + u < p.k_splits) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
  }
  if (p.b_down) { s.x += b.x; s.y += b.y; s.z += b.z; s.w += b.w; }
  u32x2 o = {pack_bf16(s.x, s.y), pack_bf16(s.z, s.w)};
  *reinterpret_cast<u32x2*>(static_cast<char*>(p.y) + i4 * 2) = o;
}

}  // namespace

namespace {
// (rounds of 256 workgroups, one per compute unit) x (channels per workgroup of `tiles` tiles of r rows): what the
// busiest compute unit reads
int64_t busiest_channels(int d_ff, int r, int tiles) {
  const int64_t wgs = ((d_ff + r - 1) / r + tiles - 1) / tiles;
  return (wgs + 255) / 256 * r * tiles;
}
}  // namespace

// Channels per tile (a multiple of four) and tiles per workgroup of the fused walk: the fewest channels on the
// busiest compute unit; of equals the larger tile, then two tiles, which share x.  One tile per workgroup for up
// to 32 tokens only (the stages have no room for two chunks of more).  Whole layer, d_model 2560, 8 tokens: 8192
// channels in single tiles of 32 33.2 us, in pairs of 16 36.8 us.
FfnWalk ffn_fused_walk(int d_ff, int M) {
  FfnWalk best = {kTileRows, 2};
  for (int tiles = 2; tiles >= (M <= 32 ? 1 : 2); --tiles)
    for (int r = kTileRows; r >= 16; r -= 4) {
      const int64_t cost = busiest_channels(d_ff, r, tiles), least = busiest_channels(d_ff, best.tile_rows, best.tiles);
      if (cost < least || (cost == least && r > best.tile_rows)) best = {r, tiles};
    }
  return best;
}

int ffn_k_splits(int d_model, int d_ff) {
  const int n_tiles = d_model / kDnCols;
  int ks = 256 / (n_tiles > 0 ? n_tiles : 1);                                     // one workgroup per compute unit
  const int max_ks = d_ff / (16 * kDnWaves) > 0 ? d_ff / (16 * kDnWaves) : 1;   // at least one step per wavefront
  if (ks > max_ks) ks = max_ks;
  return ks < 1 ? 1 : ks;
}

namespace {
// Channels per workgroup of the split kernel, or 0: the fused walk.  Eight where that is one round of 256
// workgroups at most.  Sixteen up to one round for up to 32 tokens: behind that a second one that is mostly
// idle is slower than the fused walk's single round of tiles of 20 - 32 channels (whole layer, d_model 4096,
// 8 / 32 tokens: 4608 channels 34.4 / 38.7 us split, 30.0 / 32.3 us fused; 6144: 37.8 / 42.9 and 34.8 / 37.1),
// and a full one hardly better (8192: 43.3 against 44.5 us; d_model 2560: 34.5 against 33.2).  Up to two
// rounds for more tokens, where the fused walk takes two tiles per workgroup (at 8192 channels 2 - 7 %
// faster than it, at 12000 9 % slower).
int split_channels(const FfnParams& p) {
  if (p.d_ff <= 2048) return 8;
  return p.d_ff <= (p.M <= 32 ? 4096 : 8192) ? 16 : 0;
}

template <int RC>
void launch_split(const FfnParams& p, hipStream_t st) {
  const dim3 grid(p.d_ff / RC);
  if (p.M <= 8) hipLaunchKernelGGL((ffn_gate_up_split_kernel<RC, 1>), grid, dim3(kGuThreads), 0, st, p);
  else if (p.M <= 16) hipLaunchKernelGGL((ffn_gate_up_split_kernel<RC, 2>), grid, dim3(kGuThreads), 0, st, p);
  else if (p.M <= 32) hipLaunchKernelGGL((ffn_gate_up_split_kernel<RC, 4>), grid, dim3(kGuThreads), 0, st, p);
  else hipLaunchKernelGGL((ffn_gate_up_split_kernel<RC, 8>), grid, dim3(kGuThreads), 0, st, p);
}
}  // namespace

hipError_t launch_sparse_ffn(const FfnParams& p, hipStream_t st) {
  const dim3 gu(p.d_ff / kTileRows);
  const int split = p.fused_walk ? split_channels(p) : 0;
  if (split) {
    if (split == 8) launch_split<8>(p, st);
    else launch_split<16>(p, st);
  } else if (p.fused_walk) {
    const int tiles = (p.d_ff + p.walk.tile_rows - 1) / p.walk.tile_rows;
    const dim3 grid((tiles + p.walk.tiles - 1) / p.walk.tiles);
    if (p.walk.tiles == 1) hipLaunchKernelGGL((ffn_gate_up_fused_kernel<1, 1>), grid, dim3(kGuThreads), 0, st, p);
    else if (p.M <= 32) hipLaunchKernelGGL((ffn_gate_up_fused_kernel<1, 2>), grid, dim3(kGuThreads), 0, st, p);
    else hipLaunchKernelGGL((ffn_gate_up_fused_kernel<2, 2>), grid, dim3(kGuThreads), 0, st, p);
  } else {
    if (p.M <= 32) hipLaunchKernelGGL(ffn_gate_up_kernel<1>, gu, dim3(kGuThreads), 0, st, p);
    else hipLaunchKernelGGL(ffn_gate_up_kernel<2>, gu, dim3(kGuThreads), 0, st, p);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 gd(p.d_model / kDnCols * p.k_splits);
  if (p.M <= 32) hipLaunchKernelGGL(ffn_down_kernel<1>, gd, dim3(kDnThreads), 0, st, p);
  else hipLaunchKernelGGL(ffn_down_kernel<2>, gd, dim3(kDnThreads), 0, st, p);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ffn_reduce_kernel, dim3((p.d_model / 4 + 63) / 64, p.M), dim3(64), 0, st, p);
  return hipGetLastError();
}

}  // namespace svf
