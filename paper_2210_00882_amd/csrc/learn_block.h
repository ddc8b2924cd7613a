// Learner's gradient pass for fp32 networks of two hidden layers, in one kernel: forward pass, per-row loss, backward
// pass and weight gradients of a slice of the rows, with nothing but the observations read from memory and one copy of
// the gradient per slice written.
//
// A workgroup has one wave per 32 hidden units and takes 32 RT rows at a time; wave w computes units 32 w .. 32 w + 31
// of every layer for all of the rows.  The rows' activations live in LDS, where every wave reads those of all units;
// the weights come from memory (L2) as operand tiles, each read by one wave only and used for RT products.  The
// weight gradients stay in registers for the whole slice: wave w holds rows 32 w .. of dL/dW2 (H / 32 tiles of 16
// registers), the columns of its units of dL/dW1 and the rows of its units of dL/dW3.
//
// What bounds it: the fp32 matrix pipe (32x32x2: 64 cycles for 4096 flops; 157 TFLOP/s).  With the weights streamed
// past resident activations nothing else comes near it: per 64 rows and wave of 256 units some 900 MFMAs = 57 k
// cycles stand against 66 KiB of weights and 340 KiB of LDS reads.  Kept apart as one kernel per layer, the same
// work wrote and read back 7 KiB per row and ran at a fifth of the matrix rate.  One gradient of 32,768 rows, 256 units:
// 1.03 ms by layers (35 launches), 0.30-0.32 ms here (3 or 4; counters: 171 k cycles per 64-row tile, the store of the
// gradient included, of which the MFMAs of its two waves per SIMD take 111 k and the VALU, tanhf above all, 32 k); 64 units
// 0.37 -> 0.06 ms, 1000 rows of 64 units 0.35 -> 0.025 ms.  256 units with more than 32 inputs or 16 outputs spill 18 to 46
// registers (2 otherwise, with two copies to a slice).
//
// The products of a layer and, inside a slice, of a weight gradient are added in the order of the layer kernels
// (learn_kernels.h): inputs and rows ascending in one accumulator each (an fp32 MFMA adds its products one after the other,
// rounded each time, whatever its shape).  With BlockArgs::bsum the bias gradients are summed in those kernels' order
// too, and given their slices the whole gradient is theirs bit for bit; without, the sums over 32 rows are added up in a
// register.
#pragma once
#include "dev_common.h"
#include "row_sel.h"

namespace msrl {

struct BlockNet {
  // operand tiles [unit tile][k tile][lane][4]: lane (i, h) holds inputs 8 kt + 2 j + h, j = 0 .. 3, of unit 32 t + i;
  // w3 in the form of the 16x16x4 product, [output tile][k tile][lane][4]: inputs 16 kt + 4 e + lane / 16 of output
  // 16 t + lane % 16
  const f32x4 *w1, *w2, *w3;
  const f32x4 *w3t, *w2t;      // the transposes, for the backward pass
  const float *b1, *b2, *b3;   // biases, in the parameter vector
  float* dyt;                  // [out][ldt] dL/dy unit-major (with bsum), for the output layer's bias gradient
  int32_t oW1, ob1, oW2, ob2, oW3, ob3;  // offsets in the gradient vector
  int out;                     // outputs in use
  int policy;                  // 1: policy network, 0: value network
  int bsum;                    // offset of this network's columns in a row of BlockArgs::bsum
};
struct BlockArgs {
  BlockNet net[2];             // blockIdx.y picks one
  const float* obs;            // [., D]
  const void* actions;         // int32 or float [., out / 2]
  const float *logp_old, *adv, *ret;
  RowSel sel;
  int64_t R, ldt;
  int64_t rows_per_slice;      // a multiple of 32
  int D, dist;
  float clip, vf_coef, ent_coef, inv_R;
  float* part;                 // [slice][part_stride] copies of the gradient, or (split > 0, 256 units) two to a slice, of its
  int split;                   //   rows before and from row `split`, a multiple of the rows taken at a time
  int64_t part_stride;
  float* bsum;                 // [R / 32][bsum_stride] sums of dL/dz2 and dL/dz1 over 32 rows each; null: the bias
  int bsum_stride;             //   gradients of a slice go to `part` like the others
  float* stats;                // bins as in LossArgs
  int stat_bins;
};

// position of unit (or input) u inside a row of LDS: the even ones of a group of eight first, so that the four inputs
// a lane multiplies (8 kt + 2 j + h) are 16 consecutive bytes
__host__ __device__ constexpr int block_pos(int u) { return (u & ~7) | ((u & 1) << 2) | ((u >> 1) & 3); }

// LDS of a workgroup, in floats.  Row pitches are 4 more than a multiple of 64 or 32: a lane's 16 bytes then lie 4
// banks from its neighbour row's.
template <int H, int RT, int XT> struct BlockShape {
  static constexpr int NW = H / 32, THREADS = 64 * NW, ROWS = 32 * RT;
  static constexpr int HP = H + 4, XP = 32 * XT + 4, YP = 36, AP = 16;
  static constexpr int TPR = THREADS / ROWS;  // threads per row when the observations are copied
  static constexpr int XN = 32 * XT / TPR;    // ... and inputs per thread
  static constexpr int AN = 16 / TPR;         // ... and actions of a Gaussian policy
  static constexpr int LOSS_ITERS = (4 * ROWS + THREADS - 1) / THREADS;  // four threads take the loss of a row
};

// acc[rt] = sum over k of act[row][k] w[k][unit]: kn k tiles.  act: row i of the lane, at 4 h; w: the wave's first
// tile.  Weights are fetched DEPTH - 1 k tiles ahead, activations one.
template <int RT, int DEPTH>
__device__ __forceinline__ void block_layer(f32x16 (&acc)[RT], const float* act, int pitch, const f32x4* w, unsigned lane, int kn) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[rt][r] = 0.0f;
  f32x4 ring[DEPTH], a[2][RT];
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d) ring[d] = (w + min(d, kn - 1) * 64)[lane];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) a[0][rt] = *(const f32x4*)(act + 32 * rt * pitch);
  static_assert(DEPTH % 2 == 0, "the two activation buffers take turns inside a round");
#pragma unroll 1
  for (int k0 = 0; k0 < kn; k0 += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int k = k0 + d;
      if (k < kn) {  // uniform
        ring[(d + DEPTH - 1) % DEPTH] = (w + min(k + DEPTH - 1, kn - 1) * 64)[lane];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) a[(d + 1) % 2][rt] = *(const f32x4*)(act + 32 * rt * pitch + 8 * min(k + 1, kn - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[rt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[d % 2][rt][j], ring[d][j], acc[rt], 0, 0, 0);
      }
    }
  }
}

// acc[t] += sum over the rows of a[row][.] b[row][32 t + .]: a, b point at row h and this lane's column; PA, PB: floats
// from row to row.  The operands of a row pair are read while the products of the pair before run.
template <int NT, int ROWS, int PA, int PB>
__device__ __forceinline__ void block_outer(f32x16* acc, const float* a, const float* b) {
  float av[2], bv[2][NT];
  av[0] = a[0];
#pragma unroll
  for (int t = 0; t < NT; ++t) bv[0][t] = b[32 * t];
#pragma unroll 2
  for (int s = 0; s < ROWS / 2; ++s) {
    const int n = min(s + 1, ROWS / 2 - 1), c = s % 2;
    av[1 - c] = a[2 * n * PA];
#pragma unroll
    for (int t = 0; t < NT; ++t) bv[1 - c][t] = b[2 * n * PB + 32 * t];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[c], bv[c][t], acc[t], 0, 0, 0);
  }
}

// acc[mt][ct] += sum over the rows of a[row][16 mt + .] b[row][16 ct + .], 16x16x4 products (for few columns): a, b
// point at row lane / 16 and the first column
template <int NC, int ROWS, int PA, int PB>
__device__ __forceinline__ void block_outer16(f32x4 (&acc)[2][NC], const float* a, const float* b, const int (&pa)[2], const int (&pb)[NC]) {
#pragma unroll 4
  for (int s = 0; s < ROWS / 4; ++s) {
    float av[2], bv[NC];
#pragma unroll
    for (int m = 0; m < 2; ++m) av[m] = a[4 * s * PA + pa[m]];
#pragma unroll
    for (int c = 0; c < NC; ++c) bv[c] = b[4 * s * PB + pb[c]];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[m][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[m], bv[c], acc[m][c], 0, 0, 0);
  }
}

// The loss of a row (the arithmetic of loss_kernel, in its order) by four neighbouring lanes, lane q taking outputs q,
// q + 4, ...: y is the row's outputs in LDS, output k at block_pos(k), and is overwritten by dL/dy.  Returns the row's
// statistics: policy term, entropy, clipped, logp_old - logp, or the value term.
struct BlockRow {
  int act;
  float lpo, adv, ret;
};
// v of lane q of the four
template <int Q> __device__ __forceinline__ float quad_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), Q * 0x55, 0xF, 0xF, true));
}
// f(v of lane 0), f(v of lane 1), ... for the first `n` of the four
template <class F> __device__ __forceinline__ void quad_each(float v, int n, F&& f) {
  const float v0 = quad_lane<0>(v), v1 = quad_lane<1>(v), v2 = quad_lane<2>(v), v3 = quad_lane<3>(v);
  f(v0);
  if (n > 1) f(v1);
  if (n > 2) f(v2);
  if (n > 3) f(v3);
}
__device__ __forceinline__ f32x4 block_loss_row(const BlockArgs& a, int O, bool policy, float* y, const float* actions,
                                                const BlockRow& in, int q) {
#pragma clang fp contract(off)
  f32x4 st = {0.0f, 0.0f, 0.0f, 0.0f};
  if (!policy) {
    const float err = y[0] - in.ret;
    if (q == 0) y[0] = a.vf_coef * 2.0f * err * a.inv_R;
    st[0] = err * err;
    return st;
  }
  float logp = 0.0f, ent = 0.0f, lse = 0.0f;
  const int K = O / 2;
  if (a.dist == 0) {
    float mx = y[0];
    for (int k = 0; k < O; k += 4) quad_each(y[block_pos(k + q)], O - k, [&](float v) { mx = fmaxf(mx, v); });
    float z = 0.0f;
    for (int k = 0; k < O; k += 4) quad_each(expf(y[block_pos(k + q)] - mx), O - k, [&](float v) { z += v; });
    lse = mx + logf(z);
    for (int k = 0; k < O; k += 4) {
      const float lp = y[block_pos(k + q)] - lse;
      quad_each(expf(lp) * lp, O - k, [&](float v) { ent -= v; });
    }
    logp = y[block_pos(min(max(in.act, 0), 31))] - lse;
    if (in.act < 0 || in.act >= 32) logp = 0.0f;
  } else {
    for (int d = 0; d < K; d += 4) {
      const int dq = min(d + q, K - 1);
      const float ls = y[block_pos(K + dq)], e = (actions[dq] - y[block_pos(dq)]) / expf(ls);
      quad_each(__builtin_fmaf(-0.5f * e, e, -ls) - 0.9189385332046727f, K - d, [&](float v) { logp += v; });
      quad_each(ls + 1.4189385332046727f, K - d, [&](float v) { ent += v; });
    }
  }
  const float rho = expf(logp - in.lpo), A = in.adv;
  const float rc = fminf(fmaxf(rho, 1.0f - a.clip), 1.0f + a.clip);
  const float un = rho * A, cl = rc * A;
  const bool clipped = cl < un;
  const float gl = clipped ? 0.0f : -A * rho;
  if (a.dist == 0) {
    for (int k = q; k < O; k += 4) {
      const float lp = y[block_pos(k)] - lse, pk = expf(lp);
      const float dlp = (k == in.act ? 1.0f : 0.0f) - pk, dH = -pk * (lp + ent);
      y[block_pos(k)] = __builtin_fmaf(gl, dlp, -(a.ent_coef * dH)) * a.inv_R;
    }
  } else {
    for (int d = q; d < K; d += 4) {
      const float sg = expf(y[block_pos(K + d)]), e = (actions[d] - y[block_pos(d)]) / sg;
      y[block_pos(d)] = gl * (e / sg) * a.inv_R;
      y[block_pos(K + d)] = __builtin_fmaf(gl, __builtin_fmaf(e, e, -1.0f), -a.ent_coef) * a.inv_R;
    }
  }
  st[0] = -(clipped ? cl : un);
  st[1] = ent;
  st[2] = clipped ? 1.0f : 0.0f;
  st[3] = in.lpo - logp;
  return st;
}

// HALVES: with BlockArgs::split (an instance of its own: in one with the others it costs small minibatches 1 to 2 %)
template <int H, int RT, int XT, int OT, bool HALVES = false>
__global__ __launch_bounds__(2 * H) void ppo_block_kernel(BlockArgs a) {
  typedef BlockShape<H, RT, XT> S;
  constexpr int NW = S::NW, ROWS = S::ROWS, HP = S::HP, XP = S::XP, YP = S::YP, AP = S::AP, KH = H / 8;
  __shared__ __attribute__((aligned(16))) float s_h1[ROWS * HP];  // h1; a wave's own columns later hold dL/dz1
  __shared__ __attribute__((aligned(16))) float s_h2[ROWS * HP];  // h2, then dL/dz2
  __shared__ __attribute__((aligned(16))) float s_x[ROWS * XP];
  __shared__ __attribute__((aligned(16))) float s_y[ROWS * YP];   // outputs, then dL/dy
  __shared__ float s_act[ROWS * AP];                              // actions of a Gaussian policy
  const BlockNet& nt = a.net[blockIdx.y];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int lane = threadIdx.x & 63, i = lane & 31, h = lane >> 5;
  const int O = nt.out, kx = (a.D + 7) / 8, ky = (O + 7) / 8;
  const bool policy = nt.policy != 0, gauss = policy && a.dist != 0;
  const int64_t r_begin = (int64_t)blockIdx.x * a.rows_per_slice;  // this slice's first row
  const int n_rows = (int)min(a.R - r_begin, a.rows_per_slice);

  const int u0 = 32 * wave;      // this wave's first unit
  int cu = u0 + block_pos(i);    // the place of this lane's unit in a row
  const f32x4 *w1 = nt.w1 + (size_t)wave * kx * 64, *w2 = nt.w2 + (size_t)wave * KH * 64;
  const f32x4 *w3t = nt.w3t + (size_t)wave * ky * 64, *w2t = nt.w2t + (size_t)wave * KH * 64;

  f32x16 gW1[XT], gW2[NW];
  f32x4 gW3[2][OT];
  // bsum == null: sums of dL/dz1, dL/dz2 of this lane's unit over its half of the rows; in the last wave, of dL/dy
  float run1, run2, run3;

  // observations: thread -> row tx / TPR, inputs tx % TPR + TPR q; a row beyond the slice reads as zero
  int xr = threadIdx.x / S::TPR, xc = threadIdx.x % S::TPR;
  float xv[S::XN], xa[S::AN];
  auto fetch_x = [&](int t0) {
    const bool ok = t0 + xr < n_rows;
    const int64_t p = ok ? a.sel.at(r_begin + t0 + xr) : 0;
    const float* src = a.obs + p * a.D;
    if (gauss) {
      const float* act = (const float*)a.actions + p * (O / 2);
#pragma unroll
      for (int q = 0; q < S::AN; ++q) {
        const int d = xc + S::TPR * q;
        xa[q] = ok && d < O / 2 ? act[d] : 0.0f;
      }
    }
#pragma unroll
    for (int q = 0; q < S::XN; ++q) {
      const int c = xc + S::TPR * q;
      xv[q] = ok && c < a.D ? src[c] : 0.0f;
    }
  };
  for (int idx = threadIdx.x; idx < ROWS * YP; idx += S::THREADS) s_y[idx] = 0.0f;  // (columns from O on stay zero)
  fetch_x(0);
  // tanh(acc + bias) into this lane's column of s, zero for rows beyond the slice
  auto activate = [&](const f32x16 (&acc)[RT], float bias, float* s, int live) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[(32 * rt + 8 * (r / 4) + 4 * h + r % 4) * HP + cu] = tanhf(acc[rt][r] + bias);
        if (r % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // (32 of them side by side would not fit the registers)
      }
    if (live < ROWS)
      for (int row = live + h; row < ROWS; row += 2) s[row * HP + cu] = 0.0f;
  };
  // s <- acc (1 - s^2) in this lane's column
  auto derive = [&](const f32x16 (&acc)[RT], float* s) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float* p = s + (32 * rt + 8 * (r / 4) + 4 * h + r % 4) * HP + cu;
        const float hv = *p;
        *p = acc[rt][r] * (1.0f - hv * hv);
        if (r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
      }
  };

  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
#pragma unroll
      for (int t = 0; t < XT; ++t) gW1[t][r] = 0.0f;
#pragma unroll
      for (int t = 0; t < NW; ++t) gW2[t][r] = 0.0f;
    }
#pragma unroll
    for (int c = 0; c < OT; ++c) gW3[0][c] = gW3[1][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    run1 = run2 = run3 = 0.0f;
  };
  // a copy of the gradient: register r of lane (i, h) <-> row 8 (r / 4) + 4 h + r % 4 of a tile, column i
  auto store = [&](float* part) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = 8 * (r / 4) + 4 * h + r % 4;
#pragma unroll
      for (int t = 0; t < XT; ++t)
        if (32 * t + m < a.D) part[nt.oW1 + (32 * t + m) * H + u0 + i] = gW1[t][r];
#pragma unroll
      for (int t = 0; t < NW; ++t) part[nt.oW2 + (u0 + m) * H + 32 * t + i] = gW2[t][r];
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int c = 0; c < OT; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {  // register r of lane l <-> row 4 (l / 16) + r, column l % 16
          const int o = 16 * c + (lane & 15);
          if (o < O) part[nt.oW3 + (u0 + 16 * m + 4 * (lane >> 4) + r) * O + o] = gW3[m][c][r];
        }
    if (!a.bsum) {
      if (RT > 1) {
        run1 += __shfl_xor(run1, 32);
        run2 += __shfl_xor(run2, 32);
      }
      if (h == 0) {
        part[nt.ob1 + u0 + i] = run1;
        part[nt.ob2 + u0 + i] = run2;
      }
      run3 += __shfl_xor(run3, 32);
      if (wave == NW - 1 && h == 0 && i < O) part[nt.ob3 + i] = run3;
    }
  };
  float* part = a.part + (int64_t)(HALVES ? 2 * blockIdx.x : blockIdx.x) * a.part_stride;
  clear();

#pragma unroll 1
  for (int t0 = 0; t0 < n_rows; t0 += ROWS) {
    if (HALVES && t0 == a.split) {
      store(part);
      part += a.part_stride;
      clear();
    }
    const int live = min(ROWS, n_rows - t0);
    // (hidden from the compiler once per tile: the LDS addresses formed from them are cheap, and kept across tiles
    // they would be spilled)
    asm volatile("" : "+v"(lane), "+v"(i), "+v"(h), "+v"(cu), "+v"(xr), "+v"(xc));
    __syncthreads();  // the tile before is done with the observations
#pragma unroll
    for (int q = 0; q < S::XN; ++q) s_x[xr * XP + block_pos(xc + S::TPR * q)] = xv[q];
    if (gauss) {
#pragma unroll
      for (int q = 0; q < S::AN; ++q) s_act[xr * AP + xc + S::TPR * q] = xa[q];
    }
    __syncthreads();
    f32x16 acc[RT];
    // accumulator: register r of lane (i, h) <-> row 8 (r / 4) + 4 h + r % 4, unit i of the wave's
    const float bias1 = nt.b1[u0 + i];
    block_layer<RT, 2>(acc, s_x + i * XP + 4 * h, XP, w1, lane, kx);
    activate(acc, bias1, s_h1, live);
    __syncthreads();
    const float bias2 = nt.b2[u0 + i];
    // (of the two waves that share a SIMD one goes first, so that its tanh meets the other one's MFMAs)
    if (NW > 4 && wave < 4) __builtin_amdgcn_s_setprio(1);
    block_layer<RT, 4>(acc, s_h1 + i * HP + 4 * h, HP, w2, lane, KH);
    activate(acc, bias2, s_h2, live);
    if (NW > 4 && wave < 4) __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    BlockRow in[S::LOSS_ITERS];  // what the loss reads of this thread's rows
#pragma unroll
    for (int it = 0; it < S::LOSS_ITERS; ++it) {
      const int row = it * (S::THREADS / 4) + wave * 16 + (lane >> 2);
      in[it] = {0, 0.0f, 0.0f, 0.0f};
      if (row < live) {
        const int64_t p = a.sel.at(r_begin + t0 + row);
        if (policy) {
          if (!gauss) in[it].act = ((const int32_t*)a.actions)[p];
          in[it].lpo = a.logp_old[p];
          in[it].adv = a.adv[p];
        } else {
          in[it].ret = a.ret[p];
        }
      }
    }
    // output layer: 16 x 16 tiles, one per wave at a time
    {
      const int p = lane & 15, q = lane >> 4, nct = (O + 15) / 16;
#pragma unroll 1
      for (int job = wave; job < 2 * RT * nct; job += NW) {
        const int mt = job % (2 * RT), ct = job / (2 * RT);
        const float* arow = s_h2 + (16 * mt + p) * HP;
        const f32x4* wt = nt.w3 + (size_t)ct * (H / 16) * 64;
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
        constexpr int KT = H / 16;
        f32x4 ring[4];
        float av[2][4];
#pragma unroll
        for (int kt = 0; kt < 3; ++kt) ring[kt] = (wt + kt * 64)[lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) av[0][e] = arow[block_pos(4 * e + q)];
#pragma unroll 4
        for (int kt = 0; kt < KT; ++kt) {
          ring[(kt + 3) % 4] = (wt + min(kt + 3, KT - 1) * 64)[lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) av[(kt + 1) % 2][e] = arow[16 * min(kt + 1, KT - 1) + block_pos(4 * e + q)];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < 4; ++e) o = __builtin_amdgcn_mfma_f32_16x16x4f32(av[kt % 2][e], ring[kt % 4][e], o, 0, 0, 0);
        }
        const int c = 16 * ct + p;
        const float b3 = c < O ? nt.b3[c] : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) s_y[(16 * mt + 4 * q + r) * YP + block_pos(c)] = o[r] + b3;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < S::LOSS_ITERS; ++it) {
      const int row = it * (S::THREADS / 4) + wave * 16 + (lane >> 2);
      if (row < ROWS) {
        float* y = s_y + row * YP;
        if (row < live) {
          const f32x4 st = block_loss_row(a, O, policy, y, s_act + row * AP, in[it], lane & 3);
          // (the statistics wait in the padding of the row for the end of the slice)
          if ((lane & 3) == 0) *(f32x4*)(y + 32) += st;
        } else {
          for (int k = lane & 3; k < O; k += 4) y[block_pos(k)] = 0.0f;
        }
        for (int k = lane & 3; a.bsum && k < O && row < live; k += 4)
          nt.dyt[(int64_t)k * a.ldt + r_begin + t0 + row] = y[block_pos(k)];
      }
    }
    __syncthreads();
    // dL/dW3 += h2^T dL/dy (the wave's own units), then dL/dz2 in place of h2
    {
      const int p = lane & 15, q = lane >> 4;
      int pu[2], po[OT];
#pragma unroll
      for (int m = 0; m < 2; ++m) pu[m] = u0 + block_pos(16 * m + p);
#pragma unroll
      for (int c = 0; c < OT; ++c) po[c] = block_pos(16 * c + p);
      block_outer16<OT, ROWS, HP, YP>(gW3, s_h2 + q * HP, s_y + q * YP, pu, po);
    }
    if (!a.bsum && wave == NW - 1) {
      const float* col = s_y + h * (ROWS / 2) * YP + block_pos(i);
      float v = 0.0f;
#pragma unroll 8
      for (int r = 0; r < ROWS / 2; ++r) v += col[r * YP];
      run3 += v;
    }
    block_layer<RT, 2>(acc, s_y + i * YP + 4 * h, YP, w3t, lane, ky);
    derive(acc, s_h2);
    // sums over 32 rows, in row order: lane (i, h) takes row group h
    auto column_sum = [&](const float* s, float& run, int at, int32_t ob) {
      const float* col = s + (RT > 1 ? h * 32 * HP : 0) + cu;
      float v = 0.0f;
#pragma unroll 8
      for (int r = 0; r < 32; ++r) v += col[r * HP];
      run += v;  // (a chain over all of the slice's rows would be two to four times as far from the exact sum)
      const int g0 = t0 + (RT > 1 ? 32 * h : 0);
      if (a.bsum && g0 < n_rows && (RT > 1 || h == 0))
        a.bsum[((r_begin + g0) / 32) * a.bsum_stride + nt.bsum + at + u0 + i] = v;
    };
    __syncthreads();
    // (the two waves of a SIMD take the sums at different times, so that one of them has MFMAs to run)
    if (wave < 4) column_sum(s_h2, run2, H, nt.ob2);
    // dL/dW2 += h1^T dL/dz2, dL/dz1 = dL/dz2 W2^T times the derivative, in place of h1's own columns (which no other
    // wave reads any more)
    block_outer<NW, ROWS, HP, HP>(gW2, s_h1 + h * HP + cu, s_h2 + h * HP + block_pos(i));
    if (wave >= 4) column_sum(s_h2, run2, H, nt.ob2);
    block_layer<RT, 4>(acc, s_h2 + i * HP + 4 * h, HP, w2t, lane, KH);
    derive(acc, s_h1);
    fetch_x(t0 + ROWS);
    wave_lds_sync();
    column_sum(s_h1, run1, 0, nt.ob1);
    // dL/dW1 += x^T dL/dz1 (the wave's own units)
#pragma unroll
    for (int t = 0; t < XT; ++t)
      block_outer<1, ROWS, XP, HP>(&gW1[t], s_x + h * XP + 32 * t + block_pos(i), s_h1 + h * HP + cu);
  }

  if (wave == 0) {
    f32x4 st = {0.0f, 0.0f, 0.0f, 0.0f};
    if (lane < ROWS) st = *(const f32x4*)(s_y + lane * YP + 32);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int q = 0; q < 4; ++q) st[q] += __shfl_xor(st[q], o);
    const int bin = blockIdx.x % a.stat_bins;
    if (lane == 0 && policy) {
      atomicAdd(a.stats + 8 + bin, st[0]);
#pragma unroll
      for (int q = 1; q < 4; ++q) atomicAdd(a.stats + 8 + (q + 1) * a.stat_bins + bin, st[q]);
    } else if (lane == 0) {
      atomicAdd(a.stats + 8 + a.stat_bins + bin, st[0]);
    }
  }
  store(part);
  if (HALVES && n_rows <= a.split) {  // (the last slice: no second half)
    part += a.part_stride;
    for (int k = threadIdx.x; k < nt.ob3 + O - nt.oW1; k += S::THREADS) part[nt.oW1 + k] = 0.0f;
  }
}

// ---------------------------------------------------------------- packing
// dst[t][kt][lane][4] <- src[k * sk + n * sn] (zero from nk, nn on): form 0 (32x32x2): k = 8 kt + 2 e + lane / 32,
// n = 32 t + lane % 32; form 1 (16x16x4): k = 16 kt + 4 e + lane / 16, n = 16 t + lane % 16
struct BlockPackJob {
  const float* src;
  f32x4* dst;
  int sk, sn, nk, nn;
  int tiles, kt, form;
};
struct BlockPackJobs {
  BlockPackJob job[10];
  int n;
  float* clear;  // floats [0, n_clear) are set to zero (the statistics bins of the pass)
  int n_clear;
};
hipError_t launch_block_pack(const BlockPackJobs& jobs, int max_items, hipStream_t s);
hipError_t launch_ppo_block(int hidden, int in_dim, int out_dim, const BlockArgs& a, unsigned slices, unsigned nets, hipStream_t s);

// 32-row tiles a workgroup takes at a time, and workgroups that share a compute unit (by their LDS and registers)
constexpr int block_row_tiles(int H) { return H <= 128 ? 1 : 2; }
constexpr int block_per_cu(int H) { return H <= 64 ? 4 : H <= 128 ? 2 : 1; }
constexpr bool block_halves(int H) { return H > 128; }  // two copies to a slice (narrower networks have slices enough)

#define MSRL_BLOCK_LAUNCHER(HID)                                                                                          \
  hipError_t launch_ppo_block_h##HID(int in_dim, int out_dim, const BlockArgs& a, dim3 grid, hipStream_t s) {             \
    constexpr int RT = block_row_tiles(HID);                                                                              \
    constexpr bool HALVES = block_halves(HID);                                                                            \
    const dim3 threads(2 * HID);                                                                                          \
    const int one = in_dim <= 32, few = out_dim <= 16;                                                                    \
    if (a.split > 0 && !HALVES) return hipErrorInvalidValue;                                                              \
    if (a.split > 0 && one && few) hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 1, 1, HALVES>), grid, threads, 0, s, a); \
    else if (a.split > 0 && one) hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 1, 2, HALVES>), grid, threads, 0, s, a);   \
    else if (a.split > 0 && few) hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 2, 1, HALVES>), grid, threads, 0, s, a);   \
    else if (a.split > 0) hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 2, 2, HALVES>), grid, threads, 0, s, a);          \
    else if (one && few) hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 1, 1>), grid, threads, 0, s, a);                   \
    else if (one) hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 1, 2>), grid, threads, 0, s, a);                          \
    else if (few) hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 2, 1>), grid, threads, 0, s, a);                          \
    else hipLaunchKernelGGL((ppo_block_kernel<HID, RT, 2, 2>), grid, threads, 0, s, a);                                   \
    return hipGetLastError();                                                                                             \
  }

}  // namespace msrl
