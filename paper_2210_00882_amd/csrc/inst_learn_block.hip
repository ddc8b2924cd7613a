// one-kernel gradient of the learner: packing of the weights, choice of the instance
#include "learn_block.h"
#include "learn_block_bf16.h"

namespace msrl {

namespace {
__global__ __launch_bounds__(256) void block_pack_kernel(BlockPackJobs jobs) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.y == 0)
    for (int k = idx; k < jobs.n_clear; k += gridDim.x * 256) jobs.clear[k] = 0.0f;
  const BlockPackJob& j = jobs.job[blockIdx.y];
  if (idx >= j.tiles * j.kt * 64) return;
  const int lane = idx & 63, kt = (idx >> 6) % j.kt, t = (idx >> 6) / j.kt;
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int k = j.form == 0 ? 8 * kt + 2 * e + lane / 32 : 16 * kt + 4 * e + lane / 16;
    const int n = j.form == 0 ? 32 * t + lane % 32 : 16 * t + lane % 16;
    v[e] = k < j.nk && n < j.nn ? j.src[(int64_t)k * j.sk + (int64_t)n * j.sn] : 0.0f;
  }
  j.dst[idx] = v;
}

__global__ __launch_bounds__(256) void block_pack_bf16_kernel(BlockPackJobsB jobs) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.y == 0)
    for (int k = idx; k < jobs.n_clear; k += gridDim.x * 256) jobs.clear[k] = 0.0f;
  const BlockPackJobB& j = jobs.job[blockIdx.y];
  if (idx >= j.tiles * j.kt * 64) return;
  const int lane = idx & 63, kt = (idx >> 6) % j.kt, t = (idx >> 6) / j.kt;
  const int h = lane / 32, n = 32 * t + lane % 32;
  f32x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = 16 * kt + (j.linear ? 8 * h + e : 8 * (e >> 2) + 4 * h + (e & 3));
    v[e] = 0.0f;
    if (n < j.nn) {
      if (k < j.nk) {
        v[e] = j.src[(int64_t)k * j.sk + (int64_t)n * j.sn];
      } else if (j.bias && k < j.nk + 2) {
        const float b = j.bias[n], hi = (float)(__bf16)b;
        v[e] = k == j.nk ? hi : b - hi;
      }
    }
  }
  j.dst[idx] = __builtin_bit_cast(u32x4, __builtin_convertvector(v, bf16x8));  // round to nearest even
}
}  // namespace

hipError_t launch_block_pack_bf16(const BlockPackJobsB& jobs, int max_items, hipStream_t s) {
  hipLaunchKernelGGL(block_pack_bf16_kernel, dim3((unsigned)((max_items + 255) / 256), (unsigned)jobs.n), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_ppo_block_bf16_h64(int in_dim, const BlockArgsB& a, dim3 grid, hipStream_t s);
hipError_t launch_ppo_block_bf16_h128(int in_dim, const BlockArgsB& a, dim3 grid, hipStream_t s);
hipError_t launch_ppo_block_bf16_h256(int in_dim, const BlockArgsB& a, dim3 grid, hipStream_t s);

hipError_t launch_ppo_block_bf16(int hidden, int in_dim, const BlockArgsB& a, dim3 grid, hipStream_t s) {
  return hidden == 64 ? launch_ppo_block_bf16_h64(in_dim, a, grid, s)
       : hidden == 128 ? launch_ppo_block_bf16_h128(in_dim, a, grid, s) : launch_ppo_block_bf16_h256(in_dim, a, grid, s);
}

hipError_t launch_block_pack(const BlockPackJobs& jobs, int max_items, hipStream_t s) {
  hipLaunchKernelGGL(block_pack_kernel, dim3((unsigned)((max_items + 255) / 256), (unsigned)jobs.n), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_ppo_block_h64(int in_dim, int out_dim, const BlockArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_ppo_block_h128(int in_dim, int out_dim, const BlockArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_ppo_block_h256(int in_dim, int out_dim, const BlockArgs& a, dim3 grid, hipStream_t s);

hipError_t launch_ppo_block(int hidden, int in_dim, int out_dim, const BlockArgs& a, unsigned slices, unsigned nets, hipStream_t s) {
  const dim3 grid(slices, nets);
  return hidden == 64 ? launch_ppo_block_h64(in_dim, out_dim, a, grid, s)
       : hidden == 128 ? launch_ppo_block_h128(in_dim, out_dim, a, grid, s)
                       : launch_ppo_block_h256(in_dim, out_dim, a, grid, s);
}

}  // namespace msrl
