// Block representatives: the mean key of every retrieval block (Sec. 3.1; block term of Eq. 5),
// or, as a variant, the per-channel minimum and maximum of its keys (the block summary of Quest,
// which Sec. 3.1 names as its starting point); fp32 or bf16 output.
//
// HBM-bound streaming reduction: K is read exactly once with 16-byte loads, fp32 accumulation
// in a fixed (logical-token) order, fp32 representatives written once.  One workgroup per
// (sequence, block); a thread owns one 16-byte column chunk of one KV head and walks the
// block's tokens with a stride of TOK_PAR tokens, TOK_PAR thread groups cover the tokens in
// parallel and are combined through LDS in a fixed order, so the result does not depend on
// the physical page order.
#include <hip/hip_bf16.h>

#include "svf_device.h"

namespace svf {

namespace {

constexpr int kThreads = 256;

template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  static constexpr int N = 4;
  __device__ static void load(const float* p, float (&v)[4]) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  }
};
template <>
struct Vec16<__hip_bfloat16> {
  static constexpr int N = 8;
  __device__ static void load(const __hip_bfloat16* p, float (&v)[8]) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));   // read once
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

// Four consecutive values to the output's element type.
__device__ __forceinline__ void store4(float* o, float a, float b, float c, float d) {
  *reinterpret_cast<float4*>(o) = make_float4(a, b, c, d);
}
__device__ __forceinline__ void store4(__hip_bfloat16* o, float a, float b, float c, float d) {
  const __hip_bfloat16 h[4] = {__float2bfloat16(a), __float2bfloat16(b), __float2bfloat16(c), __float2bfloat16(d)};
  uint2 w;
  w.x = (uint32_t)__builtin_bit_cast(unsigned short, h[0]) | ((uint32_t)__builtin_bit_cast(unsigned short, h[1]) << 16);
  w.y = (uint32_t)__builtin_bit_cast(unsigned short, h[2]) | ((uint32_t)__builtin_bit_cast(unsigned short, h[3]) << 16);
  *reinterpret_cast<uint2*>(o) = w;
}

// grid: (blocks in range, B, column groups); block: kThreads.  MINMAX: acc holds the running
// minimum and acc2 the running maximum instead of the sum; OT: element type written.
template <typename T, bool MINMAX, typename OT>
__global__ __launch_bounds__(kThreads) void block_reps_kernel(RepsParams p, int cols, int cpb, int tok_par) {
  constexpr int N = Vec16<T>::N;
  __shared__ float red[kThreads * N * (MINMAX ? 2 : 1)];

  const int b = blockIdx.y;
  const int j = p.first_block + blockIdx.x;
  const int L = clamped_len(p.seq_lens, b, p.max_seq_len);
  const int t0 = j * p.block_size;
  if (t0 >= L) return;                                  // block does not exist in this sequence
  const int n_tok = min(p.block_size, L - t0);

  const int tid = threadIdx.x;
  const int tl = tid / cpb;                             // token lane
  const int col = blockIdx.z * cpb + (tid - tl * cpb);  // 16-byte column chunk over (head, channel)
  const bool active = tl < tok_par && col < cols;
  const int chunks_per_head = p.d / N;
  const int h = col / chunks_per_head;
  const int c = (col - h * chunks_per_head) * N;

  float acc[N], acc2[MINMAX ? N : 1];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    acc[i] = MINMAX ? __builtin_inff() : 0.f;
    if (MINMAX) acc2[i] = -__builtin_inff();
  }
  auto take = [&](const float (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (MINMAX) {
        acc[i] = fminf(acc[i], v[i]);
        acc2[i] = fmaxf(acc2[i], v[i]);
      } else {
        acc[i] += v[i];
      }
    }
  };

  if (active) {
    const T* K = static_cast<const T*>(p.K) + (int64_t)h * p.kv.stride_head + c;
    int t = tl;
    // four independent loads in flight per iteration
    for (; t + 3 * tok_par < n_tok; t += 4 * tok_par) {
      float v[4][N];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        Vec16<T>::load(K + token_offset(p.kv, p.table, b, t0 + t + u * tok_par), v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) take(v[u]);
    }
    for (; t < n_tok; t += tok_par) {
      float v[N];
      Vec16<T>::load(K + token_offset(p.kv, p.table, b, t0 + t), v);
      take(v);
    }
  }

  if (tok_par > 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      red[tid * N + i] = acc[i];
      if (MINMAX) red[(kThreads + tid) * N + i] = acc2[i];
    }
    __syncthreads();
    if (active && tl == 0) {
      for (int u = 1; u < tok_par; ++u)
#pragma unroll
        for (int i = 0; i < N; ++i) {
          if (MINMAX) {
            acc[i] = fminf(acc[i], red[(u * cpb + tid) * N + i]);
            acc2[i] = fmaxf(acc2[i], red[(kThreads + u * cpb + tid) * N + i]);
          } else {
            acc[i] += red[(u * cpb + tid) * N + i];
          }
        }
    }
  }
  if (active && tl == 0) {
    const float inv = MINMAX ? 1.0f : 1.0f / (float)n_tok;
    OT* r = static_cast<OT*>(p.reps) + ((((int64_t)b * p.Hkv + h) * p.nb_max + j) * (MINMAX ? 2 : 1)) * p.d + c;
#pragma unroll
    for (int i = 0; i < N; i += 4) {
      store4(r + i, acc[i] * inv, acc[i + 1] * inv, acc[i + 2] * inv, acc[i + 3] * inv);
      if (MINMAX) store4(r + p.d + i, acc2[i], acc2[i + 1], acc2[i + 2], acc2[i + 3]);
    }
  }
}

// The same representatives, bit for bit, for a launch of few blocks (the last ones after a step's tokens were
// added to the cache), which is bound by the chain of one thread's loads and not by bandwidth: with all
// heads of a block in one workgroup a thread walks block_size / tok_par tokens four at a time, eight round
// trips for 64 tokens of 8 heads.  Here a workgroup has one head of a block, all of its loads (at most
// kFewBytes, eight per thread) are in flight at once into LDS, and the sums are then taken from LDS in the
// order of the kernel above: item (tl, channel) adds tokens tl, tl + tok_par, ..., then the items of a
// channel are added in the order of tl.
// One block of 64 tokens, 8 heads of 128 channels, bf16: 6.1 - 8.4 -> 4.8 - 5.9 us for 1 to 16
// blocks with contiguous pages, 17.6 - 22.6 -> 5.4 - 7.5 us for 1 to 16 blocks of each of 4 sequences in
// pages of 16 tokens (keys out of memory).  Where it does not pay: few_is_faster.
// grid: (blocks in range, B, Hkv); block: kThreads
constexpr int kFewBytes = 32768;
constexpr int kFewWorkgroups = 512;
template <typename T, bool MINMAX, typename OT>
__global__ __launch_bounds__(kThreads) void block_reps_few_kernel(RepsParams p, int tok_par) {
  constexpr int N = Vec16<T>::N;
  constexpr int kLoads = kFewBytes / 16 / kThreads;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) T rows[kFewBytes / sizeof(T)];
  __shared__ float red[(MINMAX ? 2 : 1) * kThreads * 8];      // d * tok_par items (<= 8 kThreads, see the launcher)

  const int b = blockIdx.y, h = blockIdx.z;
  const int j = p.first_block + blockIdx.x;
  const int L = clamped_len(p.seq_lens, b, p.max_seq_len);
  const int t0 = j * p.block_size;
  if (t0 >= L) return;
  const int n_tok = min(p.block_size, L - t0);
  const int tid = threadIdx.x;
  const int chunks = p.d / N;                                 // 16-byte chunks of a row
  const T* K = static_cast<const T*>(p.K) + (int64_t)h * p.kv.stride_head;

  u32x4 v[kLoads];
#pragma unroll
  for (int u = 0; u < kLoads; ++u) {
    const int e = tid + u * kThreads, t = e / chunks;
    if (t < n_tok)
      v[u] = *reinterpret_cast<const u32x4*>(K + token_offset(p.kv, p.table, b, t0 + t) + (e - t * chunks) * N);
  }
#pragma unroll
  for (int u = 0; u < kLoads; ++u) {
    const int e = tid + u * kThreads;
    if (e / chunks < n_tok) reinterpret_cast<u32x4*>(rows)[e] = v[u];
  }
  __syncthreads();

  const int items = p.d * tok_par;
  for (int i = tid; i < items; i += kThreads) {
    const int tl = i / p.d, c = i - tl * p.d;
    float a = MINMAX ? __builtin_inff() : 0.f, a2 = -__builtin_inff();
#pragma unroll 8
    for (int t = tl; t < n_tok; t += tok_par) {
      const float x = (float)rows[t * p.d + c];
      if (MINMAX) {
        a = fminf(a, x);
        a2 = fmaxf(a2, x);
      } else {
        a += x;
      }
    }
    red[i] = a;
    if (MINMAX) red[items + i] = a2;
  }
  __syncthreads();
  if (tid * 4 < p.d) {
    const float inv = MINMAX ? 1.0f : 1.0f / (float)n_tok;
    float o[4], o2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[i] = red[tid * 4 + i];
      if (MINMAX) o2[i] = red[items + tid * 4 + i];
    }
    for (int u = 1; u < tok_par; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = red[u * p.d + tid * 4 + i];
        if (MINMAX) {
          o[i] = fminf(o[i], x);
          o2[i] = fmaxf(o2[i], red[items + u * p.d + tid * 4 + i]);
        } else {
          o[i] += x;
        }
      }
    OT* r = static_cast<OT*>(p.reps) + ((((int64_t)b * p.Hkv + h) * p.nb_max + j) * (MINMAX ? 2 : 1)) * p.d + tid * 4;
    store4(r, o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
    if (MINMAX) store4(r + p.d, o2[0], o2[1], o2[2], o2[3]);
  }
}

template <typename T>
void launch_few(const RepsParams& p, dim3 grid, int tok_par, hipStream_t st) {
  if (p.minmax) {
    if (p.out_bf16) hipLaunchKernelGGL((block_reps_few_kernel<T, true, __hip_bfloat16>), grid, dim3(kThreads), 0, st, p, tok_par);
    else hipLaunchKernelGGL((block_reps_few_kernel<T, true, float>), grid, dim3(kThreads), 0, st, p, tok_par);
  } else {
    if (p.out_bf16) hipLaunchKernelGGL((block_reps_few_kernel<T, false, __hip_bfloat16>), grid, dim3(kThreads), 0, st, p, tok_par);
    else hipLaunchKernelGGL((block_reps_few_kernel<T, false, float>), grid, dim3(kThreads), 0, st, p, tok_par);
  }
}

template <typename T>
void launch_for(const RepsParams& p, dim3 grid, int cols, int cpb, int tok_par, hipStream_t st) {
  if (p.minmax) {
    if (p.out_bf16) hipLaunchKernelGGL((block_reps_kernel<T, true, __hip_bfloat16>), grid, dim3(kThreads), 0, st, p, cols, cpb, tok_par);
    else hipLaunchKernelGGL((block_reps_kernel<T, true, float>), grid, dim3(kThreads), 0, st, p, cols, cpb, tok_par);
  } else {
    if (p.out_bf16) hipLaunchKernelGGL((block_reps_kernel<T, false, __hip_bfloat16>), grid, dim3(kThreads), 0, st, p, cols, cpb, tok_par);
    else hipLaunchKernelGGL((block_reps_kernel<T, false, float>), grid, dim3(kThreads), 0, st, p, cols, cpb, tok_par);
  }
}

}  // namespace

namespace {
// Is the launch of few blocks (one workgroup per head) the faster one?  It must fit: at most two workgroups per
// compute unit, one head's keys of a block within the stage (d * tok_par items stay within red[]: cols = Hkv d / N
// >= d / 8, so tok_par <= 2048 / d).  Then it depends on what each is bound by (both measured over 850 shapes:
// 1 - 16 heads, blocks of 16 - 256 tokens, both types, one or four sequences, keys out of memory).  The wide kernel
// takes 3 us and a trip to memory per four tokens of a thread, 0.75 us, or 2.4 with a page table
// (the key's address is a trip of its own); this one 3.6 us (paged 5), its stage filled and summed from
// LDS, 0.4 us per KB of bf16 (0.35 of fp32), and up to 1 us more with two workgroups per compute unit.
// In tenths of a microsecond; the constants are such that no shape is slower than with the wide kernel (which
// takes 4.5 us for 128 tokens of one head of 128 channels, this one 11) and at most 11 % of what can be had is left.
bool few_is_faster(const RepsParams& p, int dtype, int B, int tok_par) {
  const int64_t workgroups = (int64_t)p.n_blocks * B * p.Hkv, channels = (int64_t)p.block_size * p.d;
  if (workgroups > kFewWorkgroups || channels * (dtype == SVF_F32 ? 4 : 2) > kFewBytes) return false;
  const int64_t trips = (p.block_size + 4 * tok_par - 1) / (4 * tok_par);
  const int64_t wide = p.kv.page_size > 0 ? 22 * trips - 24 : 8 * trips - 12;      // beyond what both take
  return wide > channels * (dtype == SVF_F32 ? 7 : 4) / 1024 + workgroups / 51;
}
}  // namespace

hipError_t launch_block_reps(const RepsParams& p, int dtype, int B, hipStream_t st) {
  if (p.n_blocks <= 0) return hipSuccess;
  const int N = dtype == SVF_F32 ? 4 : 8;
  const int cols = p.Hkv * p.d / N;
  const int cpb = cols < kThreads ? cols : kThreads;
  const int tok_par = kThreads / cpb;
  if (few_is_faster(p, dtype, B, tok_par)) {
    const dim3 few(p.n_blocks, B, p.Hkv);
    if (dtype == SVF_F32) launch_few<float>(p, few, tok_par, st);
    else launch_few<__hip_bfloat16>(p, few, tok_par, st);
    return hipGetLastError();
  }
  dim3 grid(p.n_blocks, B, (cols + cpb - 1) / cpb);
  if (dtype == SVF_F32) launch_for<float>(p, grid, cols, cpb, tok_par, st);
  else launch_for<__hip_bfloat16>(p, grid, cols, cpb, tok_par, st);
  return hipGetLastError();
}

}  // namespace svf
