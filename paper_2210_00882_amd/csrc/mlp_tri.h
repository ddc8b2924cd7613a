// fp32 policy / value networks on the 16-bit matrix pipe, one wave per 32 rows.
//
// Operands are taken apart into pieces (tri.h): three bf16 ones in layer 1, whose inputs have no bounds, two fp16 ones in the
// layers behind it.  What bounds it: the MFMAs of 128 and 256 units (the activation work beside them takes about a third of
// their time in those layers), the activation work of 64 units and of layer 1.  With three pieces in every layer, before and
// now: rollout of 16,384 x 6 rows, 128 units, 128 steps 6.80 -> 5.06 ms, of 32,768 linear-Gaussian rows, 256 units
// 5.98 -> 4.10; of 4096 x 3, 64 units 502 -> 453 us.
//
// Everything else is as in mlp.h: layers transposed, a layer's accumulators are the next layer's B operand (the
// bf16 "chained" input map), weights as A-operand tiles in LDS (packed.h: a k tile is three 1 KiB pieces), the tanh
// of a chunk beside the MFMAs of the next one.  The interleaving is spelled out: a wave issues in order and
// an MFMA keeps the pipe for 32 cycles, so between two MFMAs there is room for about seven vector instructions, and
// the work on the chunk before is cut into steps of two to ten instructions that are dealt out over those gaps
// (fp32 networks of 256 units run one wave per SIMD: nothing else would fill them).
#pragma once
#include <type_traits>

#include "mlp.h"
#include "tri.h"

namespace msrl {

// What is done with the accumulators of the chunk before beside the MFMAs of a chunk: nothing, tanh and split
// into operands of the next layer, tanh and the output layer on the VALU, tanh and split and the output layer of a
// Gaussian policy on the MFMA.
enum : int { TRI_NONE = 0, TRI_SPLIT = 1, TRI_OUT = 2, TRI_GAUSS = 3 };

// ... as a list of steps, two accumulator registers at a time.  SCALED: layers behind the first, whose accumulators want the
// units' factors and biases (sb) first.
template <int MODE, bool SCALED>
struct TriWork {
  static constexpr int PRE = SCALED ? 1 : 0;
  static constexpr int PER_PAIR = MODE == TRI_NONE ? 0 : PRE + (MODE == TRI_OUT ? 5 : MODE == TRI_SPLIT ? 7 : 8);
  static constexpr int STEPS = 8 * PER_PAIR;
  typedef std::conditional_t<MODE == TRI_GAUSS, Tri, Duo> Opd;
  f32x16 prev;        // pre-activations (times 2 log2(e), see fast_tanh_prescaled), or what SCALED makes them of
  float t[16];        // tanh chain, then remainders of the split
  Opd op[2];          // TRI_SPLIT / TRI_GAUSS: the chunk's 32 units as operands
  const float* w3h;   // TRI_OUT: this half-wave's output weights of the chunk (MlpTri::out_weights)
  f32x4 wg[8];
  const float* sb;    // this half-wave's factors of the chunk, biases 32 floats behind them; a group of four units ahead
  f32x4 sc[2], bi[2];
  __device__ __forceinline__ void fetch(int g) {
    sc[g & 1] = *(const f32x4*)(sb + 8 * g);
    bi[g & 1] = *(const f32x4*)(sb + 32 + 8 * g);
  }
  __device__ __forceinline__ void begin(const f32x16& acc, const float* factors) {
    prev = acc;
    sb = factors;
    if constexpr (SCALED) fetch(0);
  }
  template <int NOUT>
  __device__ __forceinline__ void step(int i, f32x16& out) {
    constexpr int P = PER_PAIR > 0 ? PER_PAIR : 1;
    const int r = 2 * (i / P), s = i % P - PRE, o = r / 8, w = r % 8 / 2;
    switch (s) {
      case -1:
        t[r] = __builtin_fmaf(prev[r], sc[r / 4 & 1][r % 4], bi[r / 4 & 1][r % 4]);
        t[r + 1] = __builtin_fmaf(prev[r + 1], sc[r / 4 & 1][r % 4 + 1], bi[r / 4 & 1][r % 4 + 1]);
        if (r % 4 == 0 && r < 12) fetch(r / 4 + 1);
        break;
      case 0:
        t[r] = __builtin_amdgcn_exp2f(SCALED ? t[r] : prev[r]);
        t[r + 1] = __builtin_amdgcn_exp2f(SCALED ? t[r + 1] : prev[r + 1]);
        if constexpr (MODE == TRI_OUT) {
          if (r % 4 == 0) {
#pragma unroll
            for (int k = 0; k < NOUT; ++k) wg[k] = *(const f32x4*)(w3h + (r / 4) * 64 + k * 4);
          }
        }
        break;
      case 1:
        t[r] += 1.0f;
        t[r + 1] += 1.0f;
        break;
      case 2:
        t[r] = __builtin_amdgcn_rcpf(t[r]);
        t[r + 1] = __builtin_amdgcn_rcpf(t[r + 1]);
        break;
      case 3:
        t[r] = 1.0f - 2.0f * t[r];
        t[r + 1] = 1.0f - 2.0f * t[r + 1];
        break;
      case 4:
        if constexpr (MODE == TRI_OUT) {
#pragma unroll
          for (int k = 0; k < NOUT; ++k) out[k] = __builtin_fmaf(t[r], wg[k][r % 4], out[k]);
#pragma unroll
          for (int k = 0; k < NOUT; ++k) out[k] = __builtin_fmaf(t[r + 1], wg[k][r % 4 + 1], out[k]);
        } else {
          op[o].p[0][w] = MODE == TRI_GAUSS ? bf16_pair(t[r], t[r + 1]) : f16_pair(t[r], t[r + 1]);
        }
        break;
      case 5:
        t[r] = MODE == TRI_GAUSS ? minus_low(t[r], op[o].p[0][w]) : minus_low_f16(t[r], op[o].p[0][w]);
        t[r + 1] = MODE == TRI_GAUSS ? minus_high(t[r + 1], op[o].p[0][w]) : minus_high_f16(t[r + 1], op[o].p[0][w]);
        break;
      case 6:
        op[o].p[1][w] = MODE == TRI_GAUSS ? bf16_pair(t[r], t[r + 1]) : f16_pair(t[r], t[r + 1]);
        break;
      default:
        if constexpr (MODE == TRI_GAUSS)
          op[o].p[2][w] = bf16_pair(minus_low(t[r], op[o].p[1][w]), minus_high(t[r + 1], op[o].p[1][w]));
    }
  }
};

// One chunk's MFMAs: layer 1 (P = 3 pieces of an operand, bf16) or a layer behind it (P = 2, fp16)
template <int P> struct Pieces;
template <> struct Pieces<3> {
  typedef Tri Opd;
  static constexpr int N = 6;
  static constexpr int w(int m) { return TRI_W[m]; }
  static constexpr int x(int m) { return TRI_X[m]; }
  static __device__ __forceinline__ f32x16 mma(const u32x4& a, const u32x4& b, f32x16 c) { return mma_piece(a, b, c); }
};
template <> struct Pieces<2> {
  typedef Duo Opd;
  static constexpr int N = 3;
  static constexpr int w(int m) { return DUO_W[m]; }
  static constexpr int x(int m) { return DUO_X[m]; }
  static __device__ __forceinline__ f32x16 mma(const u32x4& a, const u32x4& b, f32x16 c) { return mma_f16_piece(a, b, c); }
};

// GAUSS: the policy's output layer is that of a Gaussian policy (2 K <= 16 outputs, OUT_GAUSS), multiplied by the
// MFMA; otherwise both output layers have at most 8 outputs and run on the VALU.
template <int H, int KT1, bool GAUSS = false>
struct MlpTri {
  typedef Tri Op;                                     // layer 1's operands
  typedef Duo Act;                                    // those of the layers behind it
  static constexpr int PT = 1, PC = 2;                // operands per k tile; made from one 32-unit accumulator
  static constexpr int NUC = H / 32, KT2 = H / 16;
  // sizes in 1 KiB tiles (packed.h): layer 1; a chunk block = layer-2 tiles, the units' factors and biases, output layer
  // of chunk c-1, of chunk c
  static constexpr int L1_TILES = NUC * KT1 * 3;
  static constexpr int L3T = GAUSS ? 4 : 1;
  static constexpr int BIAS = 2 * KT2, L3_PREV = BIAS + 1, L3_OWN = L3_PREV + L3T;
  static constexpr int CHUNK_TILES = tri_chunk_tiles(KT2, L3T);
  static constexpr int L1_STAGES = tri_layer1_stages(H, KT1, CHUNK_TILES);  // where they come through the window
  static constexpr int G1 = 2, G2 = 4;  // LDS reads run this many k tiles (twelve MFMAs) ahead of the MFMAs

  template <uint32_t OUTS>
  static constexpr bool on_mfma() { return __builtin_popcount(OUTS) > 8; }
  // this half-wave's output weights in the L3 tile `at` of the chunk block at `tiles` (this lane's slot of tile 0):
  // weight of unit 8 i + 4 h + j, output o at float i * 64 + h * 32 + o * 4 + j
  __device__ static __forceinline__ const float* out_weights(const u32x4* tiles, int at, int h) {
    return (const float*)(tiles + at * 64 - lane_id()) + 32 * h;
  }
  __device__ static __forceinline__ int lane_id() {
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  }

  // this half-wave's factors (biases 32 floats behind them) of the chunk whose block is at `tiles`, or of the chunk before it
  __device__ static __forceinline__ const float* factors(const u32x4* tiles, bool before, int h) {
    return (const float*)(tiles + BIAS * 64 - lane_id()) + (before ? 64 : 0) + 4 * h;
  }

  // One chunk of NT k tiles: acc <- W b, the steps of wk dealt out over the gaps behind the MFMAs.  Tile `k` of the
  // stream of TOTAL tiles that this chunk belongs to lies (k / NT) STRIDE + P (k % NT) KiB behind `tiles`; `first` is
  // the chunk's first, whose pieces are in the ring with the G - 1 tiles behind it.  `lead` steps come before the
  // first MFMA (they cover the latency of the first LDS reads).  extra[]: the 1 KiB tiles at `xt`, fetched during the
  // last k tiles for what follows the chunk.  tick(kt) once per tile.
  template <int NT, int TOTAL, int STRIDE, int NOUT, int P, int G, int NX, class Work, class Tick>
  __device__ static __forceinline__ void chunk(const u32x4* tiles, int first, u32x4 (&ring)[G][P],
                                               const typename Pieces<P>::Opd* b, f32x16& acc, Work& wk, f32x16& out, int lead,
                                               const u32x4* xt, u32x4 (&extra)[NX], Tick&& tick) {
    typedef Pieces<P> Pc;
    constexpr int NM = Pc::N, GAPS = NM * NT, STEPS = Work::STEPS;
    acc = zero16();
#pragma unroll
    for (int i = 0; i < STEPS; ++i)
      if (i < lead) wk.template step<NOUT>(i, out);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) {
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const int k = first + kt, g = NM * kt + m, w = Pc::w(m);
        acc = Pc::mma(ring[k % G][w], b[kt].p[Pc::x(m)], acc);
        if ((m == NM - 1 || Pc::w(m + 1 < NM ? m + 1 : NM - 1) != w) && k + G < TOTAL)
          ring[k % G][w] = tiles[(((k + G) / NT) * STRIDE + P * ((k + G) % NT) + w) * 64];
#pragma unroll
        for (int i = 0; i < NX; ++i)
          if (xt && g == GAPS - 12 + 2 * i) extra[i] = xt[i * 64];
        if (m == NM - 1) tick(kt);
        __builtin_amdgcn_sched_barrier(0);
        const int left = STEPS - lead;
#pragma unroll
        for (int i = 0; i < STEPS; ++i)
          if (i >= lead + g * left / GAPS && i < lead + (g + 1) * left / GAPS) wk.template step<NOUT>(i, out);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  template <int NT, int TOTAL, int STRIDE, int P, int G>
  __device__ static __forceinline__ void fill_ring(const u32x4* tiles, u32x4 (&ring)[G][P]) {
#pragma unroll
    for (int k = 0; k < G && k < TOTAL; ++k)
#pragma unroll
      for (int w = P - 1; w >= 0; --w) ring[k][w] = tiles[((k / NT) * STRIDE + P * (k % NT) + w) * 64];
  }
  // the steps with no MFMAs to hide behind (behind a layer's last chunk)
  template <int NOUT, class Work>
  __device__ static __forceinline__ void drain(Work& wk, f32x16& out) {
#pragma unroll
    for (int g = 0; g < 4; ++g)  // (a group of four registers shares its output weights)
#pragma unroll
      for (int s = 0; s < Work::PER_PAIR; ++s)
#pragma unroll
        for (int q = 2 * g; q < 2 * g + 2; ++q) wk.template step<NOUT>(q * Work::PER_PAIR + s, out);
  }

  // Layer 1, chunks U0 .. U1 - 1.  tiles: this lane's slot of chunk U0's first tile in LDS; x holds the observation with
  // the constant 1 at input in_dim (its bias); acc carries the last chunk's pre-activations from part to part.  tick(i), i = 0
  // .. (U1 - U0) KT1 - 1, once per k tile.
  template <int U0, int U1, class Tick>
  __device__ static __forceinline__ void layer1_part(const u32x4* tiles, const Op (&x)[1][KT1], Act (&h1)[1][KT2], f32x16& acc,
                                                     Tick&& tick) {
    constexpr int TOTAL = (U1 - U0) * KT1;
    u32x4 ring[G1][3];
    fill_ring<KT1, TOTAL, 3 * KT1>(tiles, ring);
    f32x16 none;
    u32x4 no_tiles[1];
    TriWork<TRI_NONE, false> w0;
    TriWork<TRI_SPLIT, false> wk;
#pragma unroll
    for (int uc = U0; uc <= U1; ++uc) {
      if (uc == U1 && U1 < NUC) break;
      const int first = (uc - U0) * KT1;
      auto tk = [&](int kt) { tick(first + kt); };
      if (uc == 0) {
        chunk<KT1, TOTAL, 3 * KT1, 0>(tiles, first, ring, x[0], acc, w0, none, 0, nullptr, no_tiles, tk);
        continue;
      }
      wk.begin(acc, nullptr);
      if (uc < U1)
        chunk<KT1, TOTAL, 3 * KT1, 0>(tiles, first, ring, x[0], acc, wk, none, 0, nullptr, no_tiles, tk);
      else
        drain<0>(wk, none);
      h1[0][2 * uc - 2] = wk.op[0];
      h1[0][2 * uc - 1] = wk.op[1];
    }
  }
  __device__ static __forceinline__ void layer1(const u32x4* tiles, const Op (&x)[1][KT1], Act (&h1)[1][KT2]) {
    f32x16 acc;
    layer1_part<0, NUC>(tiles, x, h1, acc, [](int) {});
  }

  // start value of the output accumulators: the bias (MFMA), or zero (VALU: the bias comes in out_finish)
  template <uint32_t OUTS>
  __device__ static __forceinline__ f32x16 out_init(const float* lds_bias, int h) {
    if constexpr (on_mfma<OUTS>()) return bias_init(lds_bias, h);
    else return zero16();
  }
  // output layer of a Gaussian policy (w: its tiles): tile 0 of a k tile has the leading pieces of the weights in
  // output rows 0 .. 15 and the middle ones in rows 16 .. 31, tile 1 the last pieces in rows 0 .. 15; out_finish adds
  // the two row ranges
  __device__ static __forceinline__ void gauss_out(const u32x4* w, const Tri (&h2)[2], f32x16& out) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      out = mma_piece(w[2 * i + 1], h2[i].p[0], out);
#pragma unroll
      for (int m = 0; m < 3; ++m) out = mma_piece(w[2 * i], h2[i].p[m], out);
    }
  }
  // behind the last chunk: the outputs in accumulator layout (register r of lane (n, h): output 8 (r / 4) + 4 h + r % 4)
  template <uint32_t OUTS, bool SWAP>
  __device__ static __forceinline__ void out_finish(f32x16 (&out)[1], const float* lds_bias, int h) {
    f32x16 res;
    if constexpr (on_mfma<OUTS>()) {
#pragma unroll
      for (int r = 0; r < 16; ++r) res[r] = r < 8 ? out[0][r] + out[0][r + 8] : 0.0f;
    } else {
      // partial sums of the two lanes of a row, and the bias
      float tot[8];
#pragma unroll
      for (int o = 0; o < 8; ++o) tot[o] = (OUTS >> o) & 1u ? sum_of_32<SWAP>(out[0][o]) + lds_bias[o] : 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) res[r] = r < 4 ? (h ? tot[r + 4] : tot[r]) : 0.0f;
    }
    out[0] = res;
  }

  // The CPS chunk blocks of a stage (consecutive in the LDS buffer) as one stream of tiles.  On entry `acc` holds the
  // sums of the chunk before (PIPE0), which get tanh and feed the output layer meanwhile.
  // nout: outputs in use (a constant where the caller's loop over the networks is unrolled).  tick(c, kt) once per k tile.
  template <bool PIPE0, int CPS, uint32_t OUTS, class Tick>
  __device__ static __forceinline__ void layer2_chunks(const u32x4* tiles, const Act (&h1)[1][KT2], f32x16 (&acc)[1],
                                                       f32x16 (&out)[1], int h, int nout, Tick&& tick) {
    constexpr int MODE = on_mfma<OUTS>() ? TRI_GAUSS : TRI_OUT;
    constexpr int TOTAL = CPS * KT2;
    u32x4 ring[G2][2];
    fill_ring<KT2, TOTAL, CHUNK_TILES>(tiles, ring);
    f32x16 none;
#pragma unroll
    for (int c = 0; c < CPS; ++c) {
      auto tk = [&](int kt) { tick(c, kt); };
      const u32x4* block = tiles + c * CHUNK_TILES * 64;
      if (PIPE0 || c > 0) {
        TriWork<MODE, true> wk;
        wk.begin(acc[0], factors(block, true, h));
        if constexpr (MODE == TRI_OUT) wk.w3h = out_weights(block, L3_PREV, h);
        // (two pairs' chains ahead of the first MFMA of a stage: they cover the latency of its first LDS reads)
        const int lead = c == 0 ? 2 * wk.PER_PAIR : 0;
        constexpr int ALL = __builtin_popcount(OUTS);
        u32x4 extra[MODE == TRI_GAUSS ? L3T : 1];  // output layer of the chunk before
        const u32x4* xt = MODE == TRI_GAUSS ? block + L3_PREV * 64 : nullptr;
        if (ALL > 1 && nout == 1)
          chunk<KT2, TOTAL, CHUNK_TILES, 1>(tiles, c * KT2, ring, h1[0], acc[0], wk, out[0], lead, xt, extra, tk);
        else
          chunk<KT2, TOTAL, CHUNK_TILES, (MODE == TRI_OUT ? ALL : 0)>(tiles, c * KT2, ring, h1[0], acc[0], wk, out[0], lead,
                                                                      xt, extra, tk);
        if constexpr (MODE == TRI_GAUSS) gauss_out(extra, wk.op, out[0]);
      } else {
        TriWork<TRI_NONE, true> w0;
        u32x4 extra[1];
        chunk<KT2, TOTAL, CHUNK_TILES, 0>(tiles, c * KT2, ring, h1[0], acc[0], w0, none, 0, nullptr, extra, tk);
      }
    }
  }
  template <bool PIPE, uint32_t OUTS, class Tick>
  __device__ static __forceinline__ void layer2_chunk(const u32x4* tiles, const Act (&h1)[1][KT2], f32x16 (&acc)[1],
                                                      f32x16 (&out)[1], int h, int nout, Tick&& tick) {
    layer2_chunks<PIPE, 1, OUTS>(tiles, h1, acc, out, h, nout, [&](int, int kt) { tick(kt); });
  }
  // behind the last chunk block (tiles: that block): its tanh and share of the output layer
  template <uint32_t OUTS>
  __device__ static __forceinline__ void layer2_drain(const u32x4* tiles, const f32x16 (&acc)[1], f32x16 (&out)[1], int h,
                                                      int nout) {
    constexpr int MODE = on_mfma<OUTS>() ? TRI_GAUSS : TRI_OUT;
    TriWork<MODE, true> wk;
    wk.begin(acc[0], factors(tiles, false, h));
    u32x4 w3[L3T];
    if constexpr (MODE == TRI_OUT) {
      wk.w3h = out_weights(tiles, L3_OWN, h);
    } else {
#pragma unroll
      for (int i = 0; i < L3T; ++i) w3[i] = tiles[(L3_OWN + i) * 64];
    }
    constexpr int ALL = __builtin_popcount(OUTS);
    if (ALL > 1 && nout == 1)
      drain<1>(wk, out[0]);
    else
      drain<(MODE == TRI_OUT ? ALL : 0)>(wk, out[0]);
    if constexpr (MODE == TRI_GAUSS) gauss_out(w3, wk.op, out[0]);
  }

  // A chunk block of a hidden layer that is not the last one: acc <- sums of the chunk; if PIPE, those of
  // the chunk before, in `acc` on entry, are returned activated as operands in hprev.
  template <bool PIPE, class Tick>
  __device__ static __forceinline__ void hidden_chunk(const u32x4* tiles, const Act (&hin)[1][KT2], f32x16 (&acc)[1],
                                                      Act (&hprev)[1][PC], int h, Tick&& tick) {
    u32x4 ring[G2][2];
    fill_ring<KT2, KT2, CHUNK_TILES>(tiles, ring);
    f32x16 none;
    u32x4 no_tiles[1];
    if constexpr (PIPE) {
      TriWork<TRI_SPLIT, true> wk;
      wk.begin(acc[0], factors(tiles, true, h));
      chunk<KT2, KT2, CHUNK_TILES, 0>(tiles, 0, ring, hin[0], acc[0], wk, none, 2 * wk.PER_PAIR, nullptr, no_tiles, tick);
      hprev[0][0] = wk.op[0];
      hprev[0][1] = wk.op[1];
    } else {
      TriWork<TRI_NONE, true> w0;
      chunk<KT2, KT2, CHUNK_TILES, 0>(tiles, 0, ring, hin[0], acc[0], w0, none, 0, nullptr, no_tiles, tick);
    }
  }
  // behind the last chunk block of such a layer (tiles: that block)
  __device__ static __forceinline__ void hidden_drain(const u32x4* tiles, const f32x16 (&acc)[1], Act (&hlast)[1][PC], int h) {
    TriWork<TRI_SPLIT, true> wk;
    f32x16 none;
    wk.begin(acc[0], factors(tiles, false, h));
    drain<0>(wk, none);
    hlast[0][0] = wk.op[0];
    hlast[0][1] = wk.op[1];
  }
};

}  // namespace msrl
