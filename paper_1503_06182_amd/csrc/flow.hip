// flow.hip -- kernels and C ABI of the learned proposal (see flow.hpp).
//
// Training step on a batch of VEGAS-weighted events (y_i, w_i), loss
// L = -sum_i w_i log q(y_i) / sum_i w_i (importance-weighted forward KL), in four launches:
//   k_flow_wsum   sum w over the batch (a per-step bijection of the data indices)
//   k_flow_events each block takes 16 events through the six layers in the density
//                 direction and back (spline reverse sweeps, MLP backward on MFMA; the
//                 per-event loss seeds are dL/dlog q_i = -w_i / sum w)
//   k_flow_wgrad_part  weight gradients as MFMA contractions over the batch, all layers
//   k_flow_wgrad_sum   adds the parts; Adam on the FP32 master weights; BF16 copies
// Batches above kFusedBatch keep one layer's gradients at a time and run layer by layer
// (k_flow_layers, k_flow_layer_bwd), the same arithmetic.
// Sampling: z uniform (Philox) -> inverse layers 5..0 -> y, log q(y).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "device_common.hpp"
#include "flow.hpp"
#include "vegas.h"

namespace vg {

// ---------------------------------------------------------------------------
// FP32 master -> BF16 copies (transposed and natural), padded columns zero
// ---------------------------------------------------------------------------
__global__ void k_flow_prep(const float* __restrict__ master, uint16_t* __restrict__ wb) {
  const int l = blockIdx.y;
  const float* m = master + l * FL_LAYER;
  uint16_t* o = wb + static_cast<int64_t>(l) * FB_LAYER;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < FB_LAYER; i += gridDim.x * blockDim.x) {
    float v;
    if (i < FB_W3T) {  // W2t[out][in]
      const int out = i / FL_HID, in = i % FL_HID;
      v = m[FO_W2 + in * FL_HID + out];
    } else if (i < FB_W2N) {  // W3t[out][in], out < 192
      const int j = i - FB_W3T, out = j / FL_HID, in = j % FL_HID;
      v = out < FL_NOUT ? m[FO_W3 + in * FL_NOUT + out] : 0.f;
    } else if (i < FB_W3N) {  // W2n[in][out]
      v = m[FO_W2 + (i - FB_W2N)];
    } else {  // W3n[in][out], out < 192
      const int j = i - FB_W3N, in = j / FL_NOUTP, out = j % FL_NOUTP;
      v = out < FL_NOUT ? m[FO_W3 + in * FL_NOUT + out] : 0.f;
    }
    o[i] = f2bf(v);
  }
}

// He-uniform hidden layers from a Philox stream keyed by (seed, parameter index),
// zero output layer and biases: the initial flow is the identity (q = 1)
__global__ void k_flow_init(float* master, uint64_t seed) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < FL_NPARAMS; i += gridDim.x * blockDim.x) {
    const int off = i % FL_LAYER;
    float v = 0.f;
    if (off < FO_B1 || (off >= FO_W2 && off < FO_B2)) {
      const u32x4 r = philox4x32_10(u32x4{static_cast<uint32_t>(i), 0u, 0xF10Fu, 0u}, static_cast<uint32_t>(seed),
                                    static_cast<uint32_t>(seed >> 32));
      const float u = (static_cast<float>(r.x >> 8) + 0.5f) * (1.f / 16777216.f);
      const float bound = off < FO_B1 ? sqrtf(6.f / 4.f) : sqrtf(6.f / FL_HID);
      v = (2.f * u - 1.f) * bound;
    }
    master[i] = v;
  }
}

// ---------------------------------------------------------------------------
// MLP of one 32-event tile for the backward: cond (LDS [32][4]) -> h1, h2 (LDS bf16)
// -> spline parameters (LDS, binary32 holding the binary16-rounded values).  B comes
// from global memory; the MFMA sequence per output tile is the forward kernel's, so
// every value equals the forward's bit for bit.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void mlp_tile32(const float* __restrict__ m, const uint16_t* __restrict__ w,
                                           const float (*cond)[4], uint16_t* h1, uint16_t* h2, float* par) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  mlp_h1(load_h1_frag(m, wave, lane), cond, h1, FL_TILE);
  __syncthreads();
  // h2: 2 row blocks x 8 column blocks; wave w owns column blocks 2w, 2w+1
  for (int rb = 0; rb < 2; ++rb)
    for (int cc = 0; cc < 2; ++cc) {
      const int cb = 2 * wave + cc;
      const f32x4_t acc = mfma_rowcol(h1, FL_LDA, w + FB_W2T, FL_HID, rb * 16, cb * 16, FL_HID, lane);
      const int col = cb * 16 + (lane & 15);
      const float bias = m[FO_B2 + col];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = rb * 16 + 4 * (lane >> 4) + j;
        h2[row * FL_LDA + col] = f2bf(fmaxf(acc[j] + bias, 0.f));
      }
    }
  __syncthreads();
  // spline parameters: 2 row blocks x 12 column blocks; wave w owns column blocks 3w..3w+2
  for (int rb = 0; rb < 2; ++rb)
    for (int cc = 0; cc < 3; ++cc) {
      const int cb = 3 * wave + cc;
      const f32x4_t acc = mfma_rowcol(h2, FL_LDA, w + FB_W3T, FL_HID, rb * 16, cb * 16, FL_HID, lane);
      const int col = cb * 16 + (lane & 15);
      const float bias = col < FL_NOUT ? m[FO_B3 + col] : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = rb * 16 + 4 * (lane >> 4) + j;
        par[row * FL_LDP + col] = round_h(acc[j] + bias);
      }
    }
  __syncthreads();
}

// x of lane i ^ 1 (CTRL 0xB1) or i ^ 2 (0x4E) within each group of four lanes (DPP quad_perm)
template <int CTRL>
__device__ __forceinline__ float quad_xor(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}

// coupling layers s0 .. s1 - 1 of six over a batch; SAMPLE: inverse splines (z -> y, layers 5 .. 0), else
// forward (y -> z, layers 0 .. 5).  Step s reads what step s - 1 wrote (the first reads
// vfirst) and writes vbuf + s vstride, in place when vstride is 0; vfirst may be vbuf.
// logq[i] = sum of log s' of the transformed coordinates.  Tiles of 64 events; each wave
// keeps the weight fragments of its output units (W2: 2 blocks of 16, W3: 3) for all eight
// k-steps in registers for a layer.
//
// An event's layers need no other event, so a block can take its own tiles through all six
// with no launch between them: the blocks drift apart, and the last tiles of a layer (4.07 per
// block at 2e5 events) run beside the next layer's first.  A launch per layer cost 10 us
// beyond the tiles' time, six times, and the caller's copies and fills: log q of 2e5 points
// 200 -> 170 us, an iteration of 1e6 sampled events 701 -> 661.  (Loop-invariant addresses
// are spilled once per layer; the tile loop has no scratch access.)
template <bool SAMPLE>
__global__ __launch_bounds__(256, 3) void k_flow_layers(const float* __restrict__ master,
                                                         const uint16_t* __restrict__ wb, const float* vfirst,
                                                         float* vbuf, int64_t vstride, float* logq, int64_t B,
                                                         int s0, int s1) {
  // h1 is dead once the second layer has run (a barrier follows it), so the spline
  // parameters the third layer writes share its space: 52 KB per block, 3 blocks per CU
  static_assert(FL_TILE_F * FL_LDQ * sizeof(_Float16) >= FL_TILE_F * FL_LDA * sizeof(uint16_t), "h1 / par union");
  __shared__ float cond[FL_TILE_F][4];
  __shared__ __align__(16) _Float16 h1_par[FL_TILE_F * FL_LDQ];
  __shared__ __align__(16) uint16_t h2[FL_TILE_F * FL_LDA];
  uint16_t* const h1 = reinterpret_cast<uint16_t*>(h1_par);
  _Float16* const par = h1_par;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ __align__(16) float bias_s[FL_HID + FL_NOUTP];
  const int ri = lane & 15, kq = 4 * (lane >> 4), kq8 = 8 * (lane >> 4);
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  // thread (event e, slot c) of a tile: its conditioning input c goes to LDS, and it
  // transforms coordinate kFlowX[l][c] after the MLP.  Both inputs of the next tile are
  // loaded while the current one runs (tiles hold disjoint events, so an in-place
  // layer's stores never touch them).
  const int e = tid >> 2, c = tid & 3;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * FL_TILE_F;
#pragma unroll 1
  for (int s = s0; s < s1; ++s) {
    const int l = SAMPLE ? FL_NLAYER - 1 - s : s;
    const float* vin = s == 0 ? vfirst : vbuf + (s - 1) * vstride;
    float* vout = vbuf + s * vstride;
    const float* m = master + l * FL_LAYER;
    const uint16_t* w = wb + static_cast<int64_t>(l) * FB_LAYER;
    bf16x8_t b2[2][FL_HID / 32], b3[3][FL_HID / 32];
    // second layer: the units of the paired-tile order (the lanes of a group receive 8
    // consecutive units of an event)
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      const int row = pair_unit(wave, cc, lane & 15);
#pragma unroll
      for (int ks = 0; ks < FL_HID / 32; ++ks)
        b2[cc][ks] = *reinterpret_cast<const bf16x8_t*>(w + FB_W2T + row * FL_HID + ks * 32 + 8 * (lane >> 4));
    }
    // third layer: the 47 parameters of coordinate w (the 48th slot takes zero row 188 of the
    // padded copy), so that wave w's outputs are exactly the parameters of the spline of
    // coordinate w: tiles 0 and 1 give parameters 0 .. 31 in the paired-tile order,
    // tile 2 parameters 32 .. 47 in order
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      const int u = lane & 15;
      const int slot = cc < 2 ? 8 * (u >> 2) + 4 * cc + (u & 3) : 32 + u;
      const int row = slot < FL_NPAR ? wave * FL_NPAR + slot : FL_NOUT;
#pragma unroll
      for (int ks = 0; ks < FL_HID / 32; ++ks)
        b3[cc][ks] = *reinterpret_cast<const bf16x8_t*>(w + FB_W3T + row * FL_HID + ks * 32 + 8 * (lane >> 4));
    }
    // biases of the lane's four output rows (C^T = Bt^T A^T: the weights are the A operand, so
    // a lane receives four consecutive outputs of one event, eight over a pair of tiles,
    // stored in one 16-byte write), read from LDS (registers held through the splines would
    // spill): sampling starts the accumulators from them, the forward adds them after the
    // products, as the training kernels do, so that these agree bit for bit.  (The forward
    // with the activations as the A operand stored its outputs two bytes at a time:
    // 33.3 against 32.2 us per layer of 2e5 events.)
    for (int i = tid; i < FL_HID + FL_NOUTP; i += blockDim.x) {
      const int c = (i - FL_HID) / 48, slot = (i - FL_HID) % 48;
      bias_s[i] = i < FL_HID ? m[FO_B2 + i] : (slot < FL_NPAR ? m[FO_B3 + c * FL_NPAR + slot] : 0.f);
    }
    const H1Frag u1 = load_h1_frag(m, wave, lane);
    const int xc = kFlowX[l][c], cc_in = kFlowC[l][c];
    int64_t e0 = static_cast<int64_t>(blockIdx.x) * FL_TILE_F;
    float cn = 0.5f, vn = 0.f;
    if (e0 + e < B) {
      cn = vin[(e0 + e) * FL_NDIM + cc_in];
      vn = vin[(e0 + e) * FL_NDIM + xc];
    }
    for (; e0 < B; e0 += stride) {
      const int64_t ev = e0 + e;
      cond[e][c] = cn;
      const float vx = vn;
      if (ev + stride < B) {
        cn = vin[(ev + stride) * FL_NDIM + cc_in];
        vn = vin[(ev + stride) * FL_NDIM + xc];
      }
      __syncthreads();
      // the three products run at a raised wave priority and the splines at the base one:
      // a SIMD then issues the products of one block's waves ahead of another block's
      // spline work, which keeps the co-resident blocks in different phases, the matrix
      // cores busy beside the vector ALUs (measured 9 % faster than equal priorities, and
      // 5 % faster than the reverse order)
      __builtin_amdgcn_s_setprio(2);
      mlp_h1(u1, cond, h1, FL_TILE_F);
      __syncthreads();
      // the lane's slots' biases are read once per layer and tile; ReLU and the bfloat16
      // rounding on pairs (v_cvt_pk_bf16_f32, v_pk_max_i16)
      const f32x4_t bb2[2] = {*reinterpret_cast<const f32x4_t*>(bias_s + 32 * wave + 2 * kq),
                              *reinterpret_cast<const f32x4_t*>(bias_s + 32 * wave + 2 * kq + 4)};
#pragma unroll
      for (int rb = 0; rb < FL_TILE_F / 16; ++rb) {
        f32x4_t acc[2];
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          acc[cc] = SAMPLE ? bb2[cc] : zero;
#pragma unroll
          for (int ks = 0; ks < FL_HID / 32; ++ks) {
            const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(h1 + (rb * 16 + ri) * FL_LDA + ks * 32 + kq8);
            acc[cc] = mfma_step(b2[cc][ks], a, acc[cc]);
          }
          if (!SAMPLE) acc[cc] += bb2[cc];
        }
        *reinterpret_cast<uint4*>(h2 + (rb * 16 + ri) * FL_LDA + 32 * wave + 2 * kq) = pack_relu_bf16x8(acc[0], acc[1]);
      }
      __syncthreads();
      const f32x4_t bb3[3] = {*reinterpret_cast<const f32x4_t*>(bias_s + FL_HID + 48 * wave + 2 * kq),
                              *reinterpret_cast<const f32x4_t*>(bias_s + FL_HID + 48 * wave + 2 * kq + 4),
                              *reinterpret_cast<const f32x4_t*>(bias_s + FL_HID + 48 * wave + 32 + kq)};
#pragma unroll
      for (int rb = 0; rb < FL_TILE_F / 16; ++rb) {
        f32x4_t acc[3];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
          acc[cc] = SAMPLE ? bb3[cc] : zero;
#pragma unroll
          for (int ks = 0; ks < FL_HID / 32; ++ks) {
            const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(h2 + (rb * 16 + ri) * FL_LDA + ks * 32 + kq8);
            acc[cc] = mfma_step(b3[cc][ks], a, acc[cc]);
          }
          if (!SAMPLE) acc[cc] += bb3[cc];
        }
        _Float16* const q = par + (rb * 16 + ri) * FL_LDQ + wave * FL_SPS;
        *reinterpret_cast<uint4*>(q + 2 * kq) = make_uint4(pack_f16x2(acc[0][0], acc[0][1]), pack_f16x2(acc[0][2], acc[0][3]),
                                                           pack_f16x2(acc[1][0], acc[1][1]), pack_f16x2(acc[1][2], acc[1][3]));
        *reinterpret_cast<uint2*>(q + 32 + kq) = make_uint2(pack_f16x2(acc[2][0], acc[2][1]), pack_f16x2(acc[2][2], acc[2][3]));
      }
      __syncthreads();
      {
        __builtin_amdgcn_s_setprio(0);
        float ld = 0.f;
        if (ev < B) {
          const float o = spline_eval<SAMPLE>(par + e * FL_LDQ + c * FL_SPS, vx, ld);
          vout[ev * FL_NDIM + xc] = o;
          if (vout != vin) vout[ev * FL_NDIM + cc_in] = cond[e][c];
        }
        // the event's four log s' (lanes 4e .. 4e+3): sums over lane pairs, then pairs of pairs
        ld += quad_xor<0xB1>(ld);
        ld += quad_xor<0x4E>(ld);
        if (c == 0 && ev < B) logq[ev] = (s == 0 ? 0.f : logq[ev]) + ld;
      }
      __syncthreads();  // also: the tile's stores are seen by the block's next layer
    }
  }
}

// ---------------------------------------------------------------------------
// operands of the weight gradients: per layer and group of 32 events, feature-major --
// element (layer, event, feature) of an array with F features at
// ((layer groups + event / 32) F + feature) 32 + event % 32 -- so that the contractions over
// events read whole kilobytes and a tile of 16 or 32 events writes 32 or 64 bytes of a
// feature at once.  Rows past the batch (to a multiple of 32) carry zero gradients.
// ---------------------------------------------------------------------------
struct FlowBwdBufs {
  uint16_t *H1, *H2, *DRb, *DH2b;
  float *DRf, *DH2f, *DH1f, *COND;
  int64_t groups;  // groups of 32 events per layer
};

__device__ __forceinline__ int64_t bwd_at(const FlowBwdBufs& s, int slot, int64_t ev, int F, int feature) {
  return ((slot * s.groups + (ev >> 5)) * F + feature) * 32 + (ev & 31);
}

// ---------------------------------------------------------------------------
// backward of one layer over a batch (one 32-event tile per block iteration)
//   gout = dL/d(layer output) [B][8], glq = dL/d log q [B]  ->  gin = dL/d(layer input);
//   stores H1, H2, DR (bf16 and fp32), DH2 (bf16 and fp32), DH1 (fp32), COND in slot 0 of the
//   weight gradients' operands; every row of the last tile is written
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_flow_layer_bwd(const float* __restrict__ master,
                                                         const uint16_t* __restrict__ wb, int l,
                                                         const float* __restrict__ vin, const float* __restrict__ gout,
                                                         float* __restrict__ gin, const float* __restrict__ glq,
                                                         int64_t B, FlowBwdBufs s) {
  __shared__ float cond[FL_TILE][4];
  __shared__ __align__(16) uint16_t h1[FL_TILE * FL_LDA];
  __shared__ __align__(16) uint16_t h2[FL_TILE * FL_LDA];
  __shared__ __align__(16) float par[FL_TILE * FL_LDP];    // spline parameters, then their gradients, then dh1
  __shared__ __align__(16) uint16_t dpb[FL_TILE * FL_LDP];  // gradients of the spline parameters (bf16), then dh2 (bf16)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* m = master + l * FL_LAYER;
  const uint16_t* w = wb + static_cast<int64_t>(l) * FB_LAYER;
  for (int64_t e0 = static_cast<int64_t>(blockIdx.x) * FL_TILE; e0 < B; e0 += static_cast<int64_t>(gridDim.x) * FL_TILE) {
    if (tid < FL_TILE * 4) {
      const int e = tid >> 2, c = tid & 3;
      const int64_t ev = e0 + e;
      const float v = ev < B ? vin[ev * FL_NDIM + kFlowC[l][c]] : 0.5f;
      cond[e][c] = v;
      s.COND[bwd_at(s, 0, ev, 4, c)] = v;
    }
    __syncthreads();
    mlp_tile32(m, w, cond, h1, h2, par);
    // activations of the tile for the weight gradients
    for (int i = tid; i < FL_TILE * FL_HID; i += blockDim.x) {
      const int e = i % FL_TILE, j = i / FL_TILE;
      s.H1[bwd_at(s, 0, e0 + e, FL_HID, j)] = h1[e * FL_LDA + j];
      s.H2[bwd_at(s, 0, e0 + e, FL_HID, j)] = h2[e * FL_LDA + j];
    }
    // spline reverse sweep: thread (event, transformed coordinate)
    if (tid < FL_TILE * 4) {
      const int e = tid >> 2, j = tid & 3;
      const int64_t ev = e0 + e;
      float* p = &par[e * FL_LDP + j * FL_NPAR];
      if (ev < B) {
        const int d = kFlowX[l][j];
        gin[ev * FL_NDIM + d] = rqs_bwd(p, vin[ev * FL_NDIM + d], gout[ev * FL_NDIM + d], glq[ev], p);
      } else {
#pragma unroll
        for (int i = 0; i < FL_NPAR; ++i) p[i] = 0.f;
      }
      if (j == 3) {  // the 4 padded columns (188..191) of the event's row
#pragma unroll
        for (int i = 0; i < FL_NOUTP - FL_NOUT; ++i) p[FL_NPAR + i] = 0.f;
      }
    }
    __syncthreads();
    for (int i = tid; i < FL_TILE * FL_NOUTP; i += blockDim.x) {
      const int e = i % FL_TILE, c = i / FL_TILE;
      const float g = par[e * FL_LDP + c];
      dpb[e * FL_LDP + c] = f2bf(g);
      s.DRb[bwd_at(s, 0, e0 + e, FL_NOUTP, c)] = f2bf(g);
      s.DRf[bwd_at(s, 0, e0 + e, FL_NOUTP, c)] = g;
    }
    __syncthreads();
    // dh2 = dp W3^T (mask h2 > 0): A = dpb [32][192], Bt = W3n [128 in][192 out]
    float dh2v[2][2][4];
    for (int rb = 0; rb < 2; ++rb)
      for (int cc = 0; cc < 2; ++cc) {
        const int cb = 2 * wave + cc;
        const f32x4_t acc = mfma_rowcol(dpb, FL_LDP, w + FB_W3N, FL_NOUTP, rb * 16, cb * 16, FL_NOUTP, lane);
        const int col = cb * 16 + (lane & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = rb * 16 + 4 * (lane >> 4) + j;
          dh2v[rb][cc][j] = bf2f(h2[row * FL_LDA + col]) > 0.f ? acc[j] : 0.f;
        }
      }
    __syncthreads();  // dpb is read by every wave above; reuse it for dh2 (bf16) below
    for (int rb = 0; rb < 2; ++rb)
      for (int cc = 0; cc < 2; ++cc) {
        const int col = (2 * wave + cc) * 16 + (lane & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = rb * 16 + 4 * (lane >> 4) + j;
          const float g = dh2v[rb][cc][j];
          dpb[row * FL_LDA + col] = f2bf(g);
          s.DH2b[bwd_at(s, 0, e0 + row, FL_HID, col)] = f2bf(g);
          s.DH2f[bwd_at(s, 0, e0 + row, FL_HID, col)] = g;
        }
      }
    __syncthreads();
    // dh1 = dh2 W2^T (mask h1 > 0): A = dh2 [32][128] (in dpb, stride FL_LDA), Bt = W2n [128 in][128 out]
    for (int rb = 0; rb < 2; ++rb)
      for (int cc = 0; cc < 2; ++cc) {
        const int cb = 2 * wave + cc;
        const f32x4_t acc = mfma_rowcol(dpb, FL_LDA, w + FB_W2N, FL_HID, rb * 16, cb * 16, FL_HID, lane);
        const int col = cb * 16 + (lane & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = rb * 16 + 4 * (lane >> 4) + j;
          const float g = bf2f(h1[row * FL_LDA + col]) > 0.f ? acc[j] : 0.f;
          par[row * FL_LDP + col] = g;
          s.DH1f[bwd_at(s, 0, e0 + row, FL_HID, col)] = g;
        }
      }
    __syncthreads();
    // dcond = dh1 W1^T; gin of the conditioning coordinates = gout + dcond
    if (tid < FL_TILE * 4) {
      const int e = tid >> 2, c = tid & 3;
      const int64_t ev = e0 + e;
      if (ev < B) {
        float a = 0.f;
        for (int k = 0; k < FL_HID; ++k) a += par[e * FL_LDP + k] * m[FO_W1 + c * FL_HID + k];
        const int d = kFlowC[l][c];
        gin[ev * FL_NDIM + d] = gout[ev * FL_NDIM + d] + a;
      }
    }
    __syncthreads();
  }
}

// the data index of batch position i: the whole data in order (n == 0), or the bijection
// j -> (a j + c) mod n of the epoch (a, j, c < n < 2^31: no overflow)
struct BatchIdx {
  uint64_t n, a, c, start, magic;  // magic = floor((2^64 - 1) / n)
};
// x mod n for x < 2^63: the quotient by the reciprocal is at most 2 short
__device__ __forceinline__ uint64_t mod_magic(uint64_t x, uint64_t n, uint64_t magic) {
  uint64_t r = x - __umul64hi(x, magic) * n;
  r = r >= n ? r - n : r;
  return r >= n ? r - n : r;
}
__device__ __forceinline__ int64_t batch_at(const BatchIdx& x, int64_t i) {
  if (x.n == 0) return i;
  const uint64_t j = mod_magic(x.start + static_cast<uint64_t>(i), x.n, x.magic);
  return static_cast<int64_t>(mod_magic(x.a * j + x.c, x.n, x.magic));
}

// ---------------------------------------------------------------------------
// the six layers of 16 events per block (4 waves) in the density direction, and with BWD
// the backward through them: activations stay in LDS (the spline parameters of all six
// layers, binary16) and registers (the ReLU masks), so nothing is recomputed and a step has
// no launch per layer.  Every value is formed by the operations of k_flow_layers<false> and
// k_flow_layer_bwd in their order: the same bits.
//
// Bound by latency: 16 events (the matrix instructions' tile) give a batch of 4096 one block
// per CU; a layer's splines run on one wave while the others store the weight gradients'
// operands, and each phase's weights are loaded before the spline or product that precedes
// it.  4096 events: 68 us for the twelve launches' 195 (and the copies, fills and gaps between
// them); a step of 32 launches took 366 us, its four launches take 112.
// ---------------------------------------------------------------------------
constexpr int kEvTile = 16;
constexpr int kWgSplit = 256;  // events per split of the weight gradients (more above kFusedBatch)
// batches of up to this many events keep the weight gradients' operands of all six layers (18 KB
// per event) and run in one launch; larger ones keep one layer's.  The one launch is the faster
// at every size measured (loss and gradient of 4096 events 94 us against 254 layer by layer,
// 16384 278 and 409, 65536 1023 and 1273), so the line is drawn by the memory: 240 MB more up
// to here, 970 MB up to 65536 for the last fifth
constexpr int64_t kFusedBatch = 16384;

template <int KS>
struct WFrags {  // two 16-column blocks of a wave, KS steps of 32
  bf16x8_t f[2][KS];
};
template <int KS>
__device__ __forceinline__ void load_wfrags(WFrags<KS>& o, const uint16_t* __restrict__ Bt, int ldb, int wave, int lane) {
#pragma unroll
  for (int cc = 0; cc < 2; ++cc)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) o.f[cc][ks] = load_bfrag(Bt, ldb, (2 * wave + cc) * 16, ks * 32, lane);
}

template <bool BWD>
__global__ __launch_bounds__(256) void k_flow_events(const float* __restrict__ master, const uint16_t* __restrict__ wb,
                                                     const float* __restrict__ y, const double* __restrict__ w,
                                                     BatchIdx bx, const double* __restrict__ scal, float* logq,
                                                     int64_t B, FlowBwdBufs s) {
  __shared__ float v[kEvTile][FL_NDIM], vin[BWD ? FL_NLAYER : 1][kEvTile][4];  // current point; transformed inputs
  __shared__ float cond[kEvTile][4];
  __shared__ float g[kEvTile][FL_NDIM];
  __shared__ __align__(16) _Float16 par[BWD ? FL_NLAYER : 1][kEvTile * FL_LDQ];
  __shared__ __align__(16) uint16_t h1[kEvTile * FL_LDA], h2[kEvTile * FL_LDA];
  __shared__ __align__(16) float gp[BWD ? kEvTile * FL_LDP : 1];      // gradients of the spline parameters, then dh1
  __shared__ __align__(16) uint16_t gb[BWD ? kEvTile * FL_LDP : 1];   // their bf16, then dh2's
  __shared__ __align__(16) float w1[BWD ? 4 * FL_HID : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ri = lane & 15, kq = 4 * (lane >> 4), kq8 = 8 * (lane >> 4);
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kEvTile;
  // thread (event, slot) of the splines: wave 0
  const int se = (tid >> 2) & (kEvTile - 1), sc = tid & 3;
  const int64_t sev = e0 + se;
  const bool spl = tid < 4 * kEvTile;
  double wev = 0.0;
  if (tid < kEvTile * FL_NDIM) {
    const int e = tid >> 3, d = tid & 7;
    v[e][d] = e0 + e < B ? y[batch_at(bx, e0 + e) * FL_NDIM + d] : 0.5f;
    if (BWD) g[e][d] = 0.f;
  }
  if (BWD && spl && sev < B) wev = w[batch_at(bx, sev)];
  float lq = 0.f;
  uint64_t m1 = 0, m2 = 0;  // ReLU masks of this lane's elements of dh1, dh2: bit 8 l + 4 cc + j
  for (int l = 0; l < FL_NLAYER; ++l) {
    const float* m = master + l * FL_LAYER;
    const uint16_t* wl = wb + static_cast<int64_t>(l) * FB_LAYER;
    WFrags<FL_HID / 32> b2;
    load_wfrags(b2, wl + FB_W2T, FL_HID, wave, lane);
    bf16x8_t b3[3][FL_HID / 32];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc)
#pragma unroll
      for (int ks = 0; ks < FL_HID / 32; ++ks)
        b3[cc][ks] = load_bfrag(wl + FB_W3T, FL_HID, 48 * wave + 16 * cc, ks * 32, lane);
    float bias2[2], bias3[3];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) bias2[cc] = m[FO_B2 + (2 * wave + cc) * 16 + ri];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      const int col = (3 * wave + cc) * 16 + ri;
      bias3[cc] = col < FL_NOUT ? m[FO_B3 + col] : 0.f;
    }
    const H1Frag u1 = load_h1_frag(m, wave, lane);
    __syncthreads();  // v of the previous layer
    if (spl) {
      const float c = v[se][kFlowC[l][sc]];
      cond[se][sc] = c;
      if constexpr (BWD) {
        vin[l][se][sc] = v[se][kFlowX[l][sc]];
        s.COND[bwd_at(s, l, sev, 4, sc)] = sev < B ? c : 0.5f;
      }
    }
    __syncthreads();
    mlp_h1(u1, cond, h1, kEvTile);
    __syncthreads();
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < FL_HID / 32; ++ks)
        acc = mfma_step(*reinterpret_cast<const bf16x8_t*>(h1 + ri * FL_LDA + ks * 32 + kq8), b2.f[cc][ks], acc);
      const int col = (2 * wave + cc) * 16 + ri;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint16_t h = f2bf(fmaxf(acc[j] + bias2[cc], 0.f));
        h2[(kq + j) * FL_LDA + col] = h;
        if constexpr (BWD) {
          const int bit = 8 * l + 4 * cc + j;
          m2 |= static_cast<uint64_t>(bf2f(h) > 0.f) << bit;
          m1 |= static_cast<uint64_t>(bf2f(h1[(kq + j) * FL_LDA + col]) > 0.f) << bit;
        }
      }
    }
    __syncthreads();
    _Float16* const pl = par[BWD ? l : 0];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < FL_HID / 32; ++ks)
        acc = mfma_step(*reinterpret_cast<const bf16x8_t*>(h2 + ri * FL_LDA + ks * 32 + kq8), b3[cc][ks], acc);
      const int col = (3 * wave + cc) * 16 + ri;  // parameter col % 47 of coordinate col / 47
      if (col < FL_NOUT) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          pl[(kq + j) * FL_LDQ + (col / FL_NPAR) * FL_SPS + col % FL_NPAR] = static_cast<_Float16>(acc[j] + bias3[cc]);
      }
    }
    __syncthreads();
    if (spl) {
      float ld = 0.f;
      const int d = kFlowX[l][sc];
      v[se][d] = spline_eval<false>(pl + se * FL_LDQ + sc * FL_SPS, v[se][d], ld);
      // the event's four log s' (lanes 4e .. 4e+3): sums over lane pairs, then pairs of pairs
      ld += quad_xor<0xB1>(ld);
      ld += quad_xor<0x4E>(ld);
      lq += ld;
    } else if constexpr (BWD) {
      // meanwhile the activations, 8 events of a feature at a time
      for (int i = tid - 64; i < 4 * FL_HID; i += 192) {
        const int j = i >> 2, half = i & 1;
        const uint16_t* h = (i & 2) ? h2 : h1;
        uint16_t t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = h[(8 * half + e) * FL_LDA + j];
        uint4 o;
        __builtin_memcpy(&o, t, sizeof(o));
        *reinterpret_cast<uint4*>(((i & 2) ? s.H2 : s.H1) + bwd_at(s, l, e0 + 8 * half, FL_HID, j)) = o;
      }
    }
  }
  if (spl && sc == 0 && sev < B) logq[sev] = lq;
  if constexpr (BWD) {
    const float glq = sev < B ? static_cast<float>(-wev / scal[0]) : 0.f;
    __syncthreads();
    for (int l = FL_NLAYER - 1; l >= 0; --l) {
      const float* m = master + l * FL_LAYER;
      const uint16_t* wl = wb + static_cast<int64_t>(l) * FB_LAYER;
      WFrags<FL_NOUTP / 32> n3;
      load_wfrags(n3, wl + FB_W3N, FL_NOUTP, wave, lane);
      WFrags<FL_HID / 32> n2;
      load_wfrags(n2, wl + FB_W2N, FL_HID, wave, lane);
      if (spl) {
        // spline reverse sweep: thread (event, transformed coordinate)
        const _Float16* p = par[l] + se * FL_LDQ + sc * FL_SPS;
        float* q = gp + se * FL_LDP + sc * FL_NPAR;
        if (sev < B) {
          const int d = kFlowX[l][sc];
          g[se][d] = rqs_bwd(p, vin[l][se][sc], g[se][d], glq, q);
        } else {
#pragma unroll
          for (int i = 0; i < FL_NPAR; ++i) q[i] = 0.f;
        }
        if (sc == 3) {  // the 4 padded columns (188..191) of the event's row
#pragma unroll
          for (int i = 0; i < FL_NOUTP - FL_NOUT; ++i) q[FL_NPAR + i] = 0.f;
        }
      } else {
        for (int i = tid - 64; i < 4 * FL_HID; i += 192) w1[i] = m[FO_W1 + i];
      }
      __syncthreads();
      for (int i = tid; i < 2 * FL_NOUTP; i += 256) {
        const int c = i >> 1, half = i & 1;
        float t[8];
        uint16_t b[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          t[e] = gp[(8 * half + e) * FL_LDP + c];
          b[e] = f2bf(t[e]);
          gb[(8 * half + e) * FL_LDP + c] = b[e];
        }
        uint4 o;
        __builtin_memcpy(&o, b, sizeof(o));
        *reinterpret_cast<uint4*>(s.DRb + bwd_at(s, l, e0 + 8 * half, FL_NOUTP, c)) = o;
        float4* f = reinterpret_cast<float4*>(s.DRf + bwd_at(s, l, e0 + 8 * half, FL_NOUTP, c));
        f[0] = make_float4(t[0], t[1], t[2], t[3]);
        f[1] = make_float4(t[4], t[5], t[6], t[7]);
      }
      __syncthreads();
      // dh2 = dp W3^T (mask h2 > 0)
      float dh[2][4];
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < FL_NOUTP / 32; ++ks)
          acc = mfma_step(*reinterpret_cast<const bf16x8_t*>(gb + ri * FL_LDP + ks * 32 + kq8), n3.f[cc][ks], acc);
#pragma unroll
        for (int j = 0; j < 4; ++j) dh[cc][j] = (m2 >> (8 * l + 4 * cc + j)) & 1 ? acc[j] : 0.f;
      }
      __syncthreads();  // gb is read by every wave above; reuse it for dh2 (bf16) below
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const int col = (2 * wave + cc) * 16 + ri;
        uint16_t b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          b[j] = f2bf(dh[cc][j]);
          gb[(kq + j) * FL_LDA + col] = b[j];
        }
        uint2 o;
        __builtin_memcpy(&o, b, sizeof(o));
        *reinterpret_cast<uint2*>(s.DH2b + bwd_at(s, l, e0 + kq, FL_HID, col)) = o;
        *reinterpret_cast<float4*>(s.DH2f + bwd_at(s, l, e0 + kq, FL_HID, col)) =
            make_float4(dh[cc][0], dh[cc][1], dh[cc][2], dh[cc][3]);
      }
      __syncthreads();
      // dh1 = dh2 W2^T (mask h1 > 0)
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < FL_HID / 32; ++ks)
          acc = mfma_step(*reinterpret_cast<const bf16x8_t*>(gb + ri * FL_LDA + ks * 32 + kq8), n2.f[cc][ks], acc);
        const int col = (2 * wave + cc) * 16 + ri;
        float t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          t[j] = (m1 >> (8 * l + 4 * cc + j)) & 1 ? acc[j] : 0.f;
          gp[(kq + j) * FL_LDP + col] = t[j];
        }
        *reinterpret_cast<float4*>(s.DH1f + bwd_at(s, l, e0 + kq, FL_HID, col)) = make_float4(t[0], t[1], t[2], t[3]);
      }
      __syncthreads();
      // dcond = dh1 W1^T; the conditioning coordinates' gradient = gout + dcond
      if (l > 0 && spl) {
        float a = 0.f;
        for (int k = 0; k < FL_HID; ++k) a += gp[se * FL_LDP + k] * w1[sc * FL_HID + k];
        g[se][kFlowC[l][sc]] += a;
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// weight gradients, split over the batch (split-K): split sp of a layer sums the
// events [sp kc, (sp + 1) kc) into its own partial row; a second kernel adds the
// rows in split order (deterministic).
//   dW3 = H2^T DR, dW2 = H1^T DH2 on MFMA (32 events per step);
//   dW1 = COND^T DH1, db1..db3 = column sums, on the VALU
// A wave takes 2 x 3 (dW3) or 2 x 2 (dW2) output tiles of 16 x 16, so that each operand it
// loads is used two or three times; each tile's sum is the same chain of steps as alone.
// ---------------------------------------------------------------------------
constexpr int kWgTiles = 96 + 64;                  // 16x16 output tiles: dW3 (8 x 12), dW2 (8 x 8)
constexpr int kWgValu = 512 + 128 + 128 + FL_NOUT;  // dW1, db1, db2, db3
constexpr int kWgPart = kWgTiles * 256 + kWgValu;   // floats per split
constexpr int kWgMaxSplit = 64;
constexpr int kWgMfmaBlocks = 8;       // 16 waves of dW3, 16 of dW2
constexpr int kWgD1Blocks = 4, kWgD2Blocks = 2, kWgDrBlocks = 3;  // column sums: 32, 64, 64 features a block
constexpr int kWgBlocksX = kWgMfmaBlocks + kWgD1Blocks + kWgD2Blocks + kWgDrBlocks;

// C(16x16 tiles at m0 + 16 i, n0 + 16 j) = sum_k A[m][k] B[k][n] over the events [k_lo, k_hi)
// (multiples of 32), A and B feature-major with MF and NF features: lane l supplies
// feature m0 + l%16 (n0 + l%16) of events k0 + 8(l/16) .. +7, one 16-byte load each
template <int MT, int NT>
__device__ __forceinline__ void wgrad_tiles(const uint16_t* __restrict__ Ht, int MF, const uint16_t* __restrict__ Dt,
                                            int NF, int m0, int n0, int64_t k_lo, int64_t k_hi, int lane, float* out,
                                            int tile0, int ldt) {
  f32x4_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const uint16_t* ap = Ht + (m0 + (lane & 15)) * 32 + 8 * (lane >> 4);
  const uint16_t* bp = Dt + (n0 + (lane & 15)) * 32 + 8 * (lane >> 4);
#pragma unroll 4
  for (int64_t k0 = k_lo; k0 < k_hi; k0 += 32) {
    bf16x8_t a[MT], b[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) a[i] = *reinterpret_cast<const bf16x8_t*>(ap + k0 * MF + 512 * i);
#pragma unroll
    for (int j = 0; j < NT; ++j) b[j] = *reinterpret_cast<const bf16x8_t*>(bp + k0 * NF + 512 * j);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = mfma_step(a[i], b[j], acc[i][j]);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(tile0 + (m0 / 16 + i) * ldt + n0 / 16 + j) * 256 + lane * 4 + r] = acc[i][j][r];
}

// column sums of NF features of x over the events [k_lo, k_hi), and with DOT also their
// products with the four features of c: out[feature], and dout[4][ldd].  Chunks of 256
// events: every thread forms the sums of 4 consecutive events for some (feature, quad) from
// 16-byte loads, all in flight together; then one thread per sum adds the chunk's 64 quads
// in order from LDS.  (One thread per sum reading its own run, a chain of loads, took
// most of 31 us for 4096 events x 6 layers.)
constexpr int kQuads = 64;  // per chunk
template <int NF, bool DOT>
__device__ __forceinline__ void column_sums(const float* __restrict__ x, int FX, int nf, const float* __restrict__ c,
                                            int64_t k_lo, int64_t k_hi, float* lds, float* out, float* dout, int ldd) {
  constexpr int NS = DOT ? 5 : 1;             // sums per feature
  constexpr int ROUNDS = NF * kQuads / 256;
  const int tid = threadIdx.x, q = tid & 7, g8 = (tid >> 3) & 7, f0 = tid >> 6;  // quad of a group, group, feature
  float a = 0.f;
  for (int64_t k0 = k_lo; k0 < k_hi; k0 += 4 * kQuads) {
    const int64_t ev = k0 + 32 * g8 + 4 * q;
    const bool in = ev < k_hi;
    float4 u[ROUNDS], v[DOT ? 4 : 1];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int f = f0 + 4 * r;
      u[r] = in && f < nf ? *reinterpret_cast<const float4*>(x + (k0 + 32 * g8) * FX + f * 32 + 4 * q)
                          : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if constexpr (DOT)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[j] = in ? *reinterpret_cast<const float4*>(c + (k0 + 32 * g8) * 4 + j * 32 + 4 * q)
                  : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();  // the chunk before this one has been added
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      float* o = lds + (f0 + 4 * r) * (kQuads + 1) + 8 * g8 + q;
      o[0] = u[r].x + u[r].y + u[r].z + u[r].w;
      if constexpr (DOT)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          o[(1 + j) * NF * (kQuads + 1)] = __fmaf_rn(
              u[r].w, v[j].w, __fmaf_rn(u[r].z, v[j].z, __fmaf_rn(u[r].x, v[j].x, u[r].y * v[j].y)));
    }
    __syncthreads();
    if (tid < NS * NF) {
      const float* o = lds + tid * (kQuads + 1);
      const int nq = static_cast<int>(k_hi - k0 < 4 * kQuads ? (k_hi - k0) / 4 : kQuads);
#pragma unroll 8
      for (int k = 0; k < nq; ++k) a += o[k];
    }
  }
  const int f = tid % NF, j = tid / NF;
  if (tid < NS * NF && f < nf) {
    if (j == 0) out[f] = a;
    else dout[(j - 1) * ldd + f] = a;
  }
}

// k_hi is the batch rounded up to 32 (the padded rows hold zero gradients).  Bound by the
// latency of its loads (170 MB at 4096 events x 6 layers, mostly from L2): 22 us for six layers, which
// took 6 x 17 one by one
__global__ __launch_bounds__(256) void k_flow_wgrad_part(int64_t Bp, int kc, FlowBwdBufs s, float* part) {
  __shared__ float lds[5 * 32 * (kQuads + 1)];
  const int lane = threadIdx.x & 63, slot = blockIdx.z;
  const int64_t k_lo = static_cast<int64_t>(blockIdx.y) * kc;
  const int64_t k_hi = k_lo + kc < Bp ? k_lo + kc : Bp;
  float* out = part + (static_cast<int64_t>(slot) * gridDim.y + blockIdx.y) * kWgPart;
  float* vout = out + kWgTiles * 256;  // dW1 [4][128], db1, db2, db3
  const int64_t g0 = slot * s.groups * 32;  // the layer's first event position
  int b = blockIdx.x;  // the column sums, a longer chain, first
  if (b < kWgD1Blocks) {
    column_sums<32, true>(s.DH1f + g0 * FL_HID + b * 32 * 32, FL_HID, 32, s.COND + g0 * 4, k_lo, k_hi, lds,
                          vout + 512 + 32 * b, vout + 32 * b, FL_HID);
    return;
  }
  b -= kWgD1Blocks;
  if (b < kWgD2Blocks) {
    column_sums<64, false>(s.DH2f + g0 * FL_HID + b * 64 * 32, FL_HID, 64, nullptr, k_lo, k_hi, lds, vout + 640 + 64 * b,
                           nullptr, 0);
    return;
  }
  b -= kWgD2Blocks;
  if (b < kWgDrBlocks) {
    column_sums<64, false>(s.DRf + g0 * FL_NOUTP + b * 64 * 32, FL_NOUTP, min(64, FL_NOUT - 64 * b), nullptr, k_lo, k_hi,
                           lds, vout + 768 + 64 * b, nullptr, 0);
    return;
  }
  const int wave_g = (b - kWgDrBlocks) * 4 + (threadIdx.x >> 6);
  if (wave_g < 16) {
    wgrad_tiles<2, 3>(s.H2 + g0 * FL_HID, FL_HID, s.DRb + g0 * FL_NOUTP, FL_NOUTP, 32 * (wave_g / 4), 48 * (wave_g % 4),
                      k_lo, k_hi, lane, out, 0, 12);
  } else {
    const int t = wave_g - 16;
    wgrad_tiles<2, 2>(s.H1 + g0 * FL_HID, FL_HID, s.DH2b + g0 * FL_HID, FL_HID, 32 * (t / 4), 32 * (t % 4), k_lo, k_hi,
                      lane, out, 96, 8);
  }
}

// Adam on the FP32 master weights (bias-corrected, step t >= 1), and the BF16 copies
struct AdamArgs {
  float *master, *m1, *m2;  // master == nullptr: the gradient only
  uint16_t* wb;
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const AdamArgs& p, int i, float g) {
  const float a = p.b1 * p.m1[i] + (1.f - p.b1) * g;
  const float v = p.b2 * p.m2[i] + (1.f - p.b2) * g * g;
  p.m1[i] = a;
  p.m2[i] = v;
  const float w = p.master[i] - p.lr * (a / p.c1) / (sqrtf(v / p.c2) + p.eps);
  p.master[i] = w;
  const int l = i / FL_LAYER, o = i % FL_LAYER;
  uint16_t* wl = p.wb + static_cast<int64_t>(l) * FB_LAYER;
  if (o >= FO_W2 && o < FO_B2) {
    const int q = o - FO_W2, in = q / FL_HID, out = q % FL_HID;
    const uint16_t b = f2bf(w);
    wl[FB_W2T + out * FL_HID + in] = b;
    wl[FB_W2N + q] = b;
  } else if (o >= FO_W3 && o < FO_B3) {
    const int q = o - FO_W3, in = q / FL_NOUT, out = q % FL_NOUT;
    const uint16_t b = f2bf(w);
    wl[FB_W3T + out * FL_HID + in] = b;
    wl[FB_W3N + in * FL_NOUTP + out] = b;
  }
}

// adds the splits' rows of layer layer0 + blockIdx.y in order; then the gradient goes to
// `grad`, or straight into Adam
__global__ __launch_bounds__(256) void k_flow_wgrad_sum(int nsplit, const float* __restrict__ part, int layer0,
                                                        float* grad, AdamArgs ad) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= kWgPart) return;
  const float* row = part + static_cast<int64_t>(blockIdx.y) * nsplit * kWgPart + idx;
  float a = 0.f;
  int sp = 0;
  for (; sp + 8 <= nsplit; sp += 8) {
    float t[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) t[k] = row[static_cast<int64_t>(sp + k) * kWgPart];
#pragma unroll
    for (int k = 0; k < 8; ++k) a += t[k];
  }
  for (; sp < nsplit; ++sp) a += row[static_cast<int64_t>(sp) * kWgPart];
  int o = -1;
  if (idx < kWgTiles * 256) {
    const int tile = idx / 256, r = idx % 256, lane = r / 4, j = r % 4;
    const int row16 = 4 * (lane >> 4) + j, col16 = lane & 15;
    if (tile < 96) {
      const int rw = (tile / 12) * 16 + row16, col = (tile % 12) * 16 + col16;
      if (col < FL_NOUT) o = FO_W3 + rw * FL_NOUT + col;
    } else {
      const int t = tile - 96;
      o = FO_W2 + ((t / 8) * 16 + row16) * FL_HID + (t % 8) * 16 + col16;
    }
  } else {
    const int t = idx - kWgTiles * 256;
    if (t < 512) o = FO_W1 + t;  // [c][n] with c = t / 128
    else if (t < 640) o = FO_B1 + t - 512;
    else if (t < 768) o = FO_B2 + t - 640;
    else o = FO_B3 + t - 768;
  }
  if (o < 0) return;
  const int i = (layer0 + blockIdx.y) * FL_LAYER + o;
  if (ad.master) adam_update(ad, i, a);
  else grad[i] = a;
}

// ---------------------------------------------------------------------------
// loss terms: W = sum w (one block, fixed order), glq_i = -w_i / W; loss = -sum w log q / W
// (formed only for a caller that reads it)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_flow_wsum(const double* __restrict__ w, BatchIdx bx, int64_t B, double* scal) {
  __shared__ double red[256];
  double s = 0.0;
  int64_t i = threadIdx.x;
  for (; i + 15 * 256 < B; i += 16 * 256) {  // sixteen loads in flight, added in order
    double t[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) t[k] = w[batch_at(bx, i + 256 * k)];
#pragma unroll
    for (int k = 0; k < 16; ++k) s += t[k];
  }
  for (; i < B; i += 256) s += w[batch_at(bx, i)];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) scal[0] = red[0];
}

__global__ void k_flow_seed(const double* __restrict__ w, int64_t B, float* glq, const double* scal) {
  const double W = scal[0];
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < B;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    glq[i] = static_cast<float>(-w[i] / W);
}

__global__ __launch_bounds__(256) void k_flow_loss(const double* __restrict__ w, BatchIdx bx,
                                                   const float* __restrict__ logq, int64_t B, double* scal) {
  __shared__ double red[256];
  double s = 0.0;
  int64_t i = threadIdx.x;
  for (; i + 15 * 256 < B; i += 16 * 256) {
    double t[16];
    float q[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      t[k] = w[batch_at(bx, i + 256 * k)];
      q[k] = logq[i + 256 * k];
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) s += t[k] * static_cast<double>(q[k]);
  }
  for (; i < B; i += 256) s += w[batch_at(bx, i)] * static_cast<double>(logq[i]);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) scal[1] = -red[0] / scal[0];
}

// the batch's points and weights in order (layer-by-layer path only)
__global__ void k_flow_gather(const float* __restrict__ y, const double* __restrict__ w, BatchIdx bx, int64_t B,
                              float* yb, double* wb) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < B;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t idx = batch_at(bx, i);
    for (int d = 0; d < FL_NDIM; ++d) yb[i * FL_NDIM + d] = y[idx * FL_NDIM + d];
    wb[i] = w[idx];
  }
}

__global__ void k_flow_zero(float* p, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = 0.f;
}

// base points of a flow-proposal iteration: z_i = the event's Philox uniforms (binary32)
__global__ void k_flow_zinit(uint64_t seed, uint32_t iter, int64_t n, float* z) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    double u[FL_NDIM];
    event_uniforms<FL_NDIM>(seed, iter, static_cast<uint64_t>(i), FL_NDIM, u);
#pragma unroll
    for (int d = 0; d < FL_NDIM; ++d) z[i * FL_NDIM + d] = static_cast<float>(u[d]);
  }
}

}  // namespace vg

// ===========================================================================
// host
// ===========================================================================
using namespace vg;

namespace vg {
void record_hip_error(const char* what, hipError_t e);  // the message vegas_strerror(VEGAS_EHIP) returns
}

struct vegas_flow_state {
  hipStream_t stream;
  int32_t max_batch;
  int64_t max_sample;
  void* mem;
  float *master, *grad, *m1, *m2;
  uint16_t* wb;
  float *V;     // [6][max_batch][8] outputs of the layers of the density direction
  float *G;     // [2][max_batch][8] gradients w.r.t. layer outputs / inputs
  float *logq;  // [max_batch]
  float *glq;   // [max_batch]
  float *yb;    // [max_batch][8] gathered batch
  double *wbat; // [max_batch]
  double *scal; // [4] sum w, loss
  FlowBwdBufs bw;
  float *zs, *lqs;  // sampling buffers [max_sample][8], [max_sample]
  float* wpart;     // [layers][splits][kWgPart] split-K partials of the weight gradients
  uint64_t adam_t;
  hipEvent_t ev_ready, ev_used;  // cross-stream ordering with a VEGAS handle's stream
};

#define VF_HIP(call)                                                       \
  do {                                                                     \
    hipError_t e_ = (call);                                                \
    if (e_ != hipSuccess) {                                                \
      record_hip_error(#call, e_);                                          \
      return VEGAS_EHIP;                                                   \
    }                                                                      \
  } while (0)

namespace {

size_t al(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

int flow_prep(vegas_flow_state* f) {
  hipLaunchKernelGGL(k_flow_prep, dim3(80, FL_NLAYER), dim3(256), 0, f->stream, f->master, f->wb);
  VF_HIP(hipGetLastError());
  return VEGAS_OK;
}

// densities of up to this many points take k_flow_events (16 points per block) instead of
// k_flow_layers (64 per block): two of its blocks per CU.  Its time grows by the round of 256
// blocks, 4096 points 21.7 us, 8192 33.2, 12288 48.5, 16384 64.5, where the layers, a tile or
// less for each CU, take 40.4 to 41.0 throughout (and the six launches of before took 50)
constexpr int64_t kFusedDensity = 2 * 256 * kEvTile;

// forward-kernel blocks: three resident per CU (LDS 52 KB, at most 168 VGPRs); more tiles
// per block amortise the per-launch load of the weights into registers
constexpr int kFwdBlocks = 3 * 256;

int64_t grid_for(int64_t n, int per_block, int cap) {
  int64_t g = (n + per_block - 1) / per_block;
  if (g > cap) g = cap;
  return g < 1 ? 1 : g;
}

// the layers over B events, vfirst -> vbuf (k_flow_layers), in one launch or one by one.
// One launch saves the launches' fixed cost, which fades with the batch, and loses at the
// largest ones, where blocks in different layers are slower than blocks in step (sampling
// through a trained-like proposal, one launch against six: 2e5 events 182 and 209 us, 1e6 611
// and 653, 3e6 1728 and 1770, 4e6 2317 and 2318, 6e6 3652 and 3440, 1e7 6260 and 5800)
constexpr int64_t kOneLaunch = 3000000;
template <bool SAMPLE>
int flow_layers(vegas_flow_state* f, hipStream_t st, const float* vfirst, float* vbuf, int64_t vstride, float* logq,
                int64_t B) {
  const int step = B <= kOneLaunch ? FL_NLAYER : 1;
  for (int s = 0; s < FL_NLAYER; s += step) {
    hipLaunchKernelGGL(k_flow_layers<SAMPLE>, dim3(grid_for(B, FL_TILE_F, kFwdBlocks)), dim3(256), 0, st, f->master, f->wb,
                       vfirst, vbuf, vstride, logq, B, s, s + step);
    VF_HIP(hipGetLastError());
  }
  return VEGAS_OK;
}

// loss and gradient of L = -sum w log q / sum w over the batch bx of (y, w): the gradient
// into f->grad, or (ad.master) through Adam into the parameters
int flow_gradient(vegas_flow_state* f, const float* y, const double* w, BatchIdx bx, int64_t B, const AdamArgs& ad,
                  double* loss_host) {
  const int64_t Bp = (B + 31) / 32 * 32;  // rows past B (written by the backward) hold zero gradients
  int kc = kWgSplit;
  if ((Bp + kc - 1) / kc > kWgMaxSplit) kc = static_cast<int>(((Bp + kWgMaxSplit - 1) / kWgMaxSplit + 31) / 32 * 32);
  const int nsplit = static_cast<int>((Bp + kc - 1) / kc);
  FlowBwdBufs bw = f->bw;
  bw.groups = Bp / 32;
  auto launch_wgrad = [&](int nl) {
    hipLaunchKernelGGL(k_flow_wgrad_part, dim3(kWgBlocksX, nsplit, nl), dim3(256), 0, f->stream, Bp, kc, bw, f->wpart);
  };
  hipLaunchKernelGGL(k_flow_wsum, dim3(1), dim3(256), 0, f->stream, w, bx, B, f->scal);
  VF_HIP(hipGetLastError());
  if (B <= kFusedBatch) {
    hipLaunchKernelGGL(k_flow_events<true>, dim3(static_cast<unsigned>(Bp / kEvTile)), dim3(256), 0, f->stream, f->master,
                       f->wb, y, w, bx, f->scal, f->logq, B, bw);
    VF_HIP(hipGetLastError());
    launch_wgrad(FL_NLAYER);
    VF_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_flow_wgrad_sum, dim3((kWgPart + 255) / 256, FL_NLAYER), dim3(256), 0, f->stream, nsplit, f->wpart,
                       0, f->grad, ad);
    VF_HIP(hipGetLastError());
  } else {
    const float* yb = y;
    const double* wbat = w;
    if (bx.n) {
      hipLaunchKernelGGL(k_flow_gather, dim3(grid_for(B, 256, 1024)), dim3(256), 0, f->stream, y, w, bx, B, f->yb, f->wbat);
      VF_HIP(hipGetLastError());
      yb = f->yb;
      wbat = f->wbat;
    }
    const int64_t stride = static_cast<int64_t>(f->max_batch) * FL_NDIM;
    const int rc = flow_layers<false>(f, f->stream, yb, f->V, stride, f->logq, B);
    if (rc != VEGAS_OK) return rc;
    hipLaunchKernelGGL(k_flow_seed, dim3(grid_for(B, 256, 1024)), dim3(256), 0, f->stream, wbat, B, f->glq, f->scal);
    VF_HIP(hipGetLastError());
    float* gout = f->G;           // dL/d z = 0 (uniform base density)
    float* gin = f->G + stride;
    hipLaunchKernelGGL(k_flow_zero, dim3(grid_for(B * FL_NDIM, 256, 1024)), dim3(256), 0, f->stream, gout, B * FL_NDIM);
    VF_HIP(hipGetLastError());
    for (int l = FL_NLAYER - 1; l >= 0; --l) {
      hipLaunchKernelGGL(k_flow_layer_bwd, dim3(grid_for(B, FL_TILE, 4096)), dim3(256), 0, f->stream, f->master, f->wb,
                         l, l == 0 ? yb : f->V + (l - 1) * stride, gout, gin, f->glq, B, bw);
      VF_HIP(hipGetLastError());
      launch_wgrad(1);
      VF_HIP(hipGetLastError());
      // the layers below still need this layer's weights unchanged only in their own
      // backward, which reads their own weights: Adam may follow each layer's gradient
      hipLaunchKernelGGL(k_flow_wgrad_sum, dim3((kWgPart + 255) / 256, 1), dim3(256), 0, f->stream, nsplit, f->wpart, l,
                         f->grad, ad);
      VF_HIP(hipGetLastError());
      float* t = gout;
      gout = gin;
      gin = t;
    }
  }
  if (loss_host) {
    hipLaunchKernelGGL(k_flow_loss, dim3(1), dim3(256), 0, f->stream, w, bx, f->logq, B, f->scal);
    VF_HIP(hipGetLastError());
    double sc[2];
    VF_HIP(hipMemcpyAsync(sc, f->scal, sizeof(sc), hipMemcpyDeviceToHost, f->stream));
    VF_HIP(hipStreamSynchronize(f->stream));
    *loss_host = sc[1];
  }
  return VEGAS_OK;
}

}  // namespace

extern "C" {

int vegas_flow_create(int32_t max_batch, int64_t max_sample, uint64_t seed, void* stream, vegas_flow* out) {
  if (!out || max_batch < 1 || max_batch > (1 << 22) || max_sample < 0 || max_sample >= (int64_t(1) << 31))
    return VEGAS_EINVAL;
  *out = nullptr;
  vegas_flow_state* f = new (std::nothrow) vegas_flow_state();
  if (!f) return VEGAS_ENOMEM;
  f->stream = static_cast<hipStream_t>(stream);
  f->max_batch = max_batch;
  f->max_sample = max_sample;
  const size_t P = FL_NPARAMS, Bm = static_cast<size_t>(max_batch), S = static_cast<size_t>(max_sample);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = al(off + bytes);
    return o;
  };
  const size_t o_master = take(4 * P), o_grad = take(4 * P), o_m1 = take(4 * P), o_m2 = take(4 * P);
  const size_t o_wb = take(2 * static_cast<size_t>(FB_LAYER) * FL_NLAYER);
  const size_t o_V = take(4 * 6 * Bm * FL_NDIM), o_G = take(4 * 2 * Bm * FL_NDIM);
  const size_t o_logq = take(4 * Bm), o_glq = take(4 * Bm), o_yb = take(4 * Bm * FL_NDIM), o_wbat = take(8 * Bm);
  const size_t o_scal = take(8 * 4);
  // the weight gradients' operands: six layers of a batch that runs in one launch, or one
  // layer of a larger one
  const size_t Bf = std::min<size_t>(Bm, kFusedBatch);
  const size_t Bl = std::max((Bf + 31) / 32 * 32 * FL_NLAYER, (Bm + 31) / 32 * 32);
  const size_t nsp = std::min<size_t>((Bm + 255) / 256, kWgMaxSplit);
  const size_t o_H1 = take(2 * Bl * FL_HID), o_H2 = take(2 * Bl * FL_HID), o_DRb = take(2 * Bl * FL_NOUTP);
  const size_t o_DH2b = take(2 * Bl * FL_HID), o_DRf = take(4 * Bl * FL_NOUTP), o_DH2f = take(4 * Bl * FL_HID);
  const size_t o_DH1f = take(4 * Bl * FL_HID), o_COND = take(4 * Bl * 4);
  const size_t o_zs = take(4 * S * FL_NDIM), o_lqs = take(4 * S);
  const size_t o_wpart = take(4 * FL_NLAYER * nsp * kWgPart);
  if (hipMalloc(&f->mem, off) != hipSuccess) {
    delete f;
    return VEGAS_ENOMEM;
  }
  char* b = static_cast<char*>(f->mem);
  f->master = reinterpret_cast<float*>(b + o_master);
  f->grad = reinterpret_cast<float*>(b + o_grad);
  f->m1 = reinterpret_cast<float*>(b + o_m1);
  f->m2 = reinterpret_cast<float*>(b + o_m2);
  f->wb = reinterpret_cast<uint16_t*>(b + o_wb);
  f->V = reinterpret_cast<float*>(b + o_V);
  f->G = reinterpret_cast<float*>(b + o_G);
  f->logq = reinterpret_cast<float*>(b + o_logq);
  f->glq = reinterpret_cast<float*>(b + o_glq);
  f->yb = reinterpret_cast<float*>(b + o_yb);
  f->wbat = reinterpret_cast<double*>(b + o_wbat);
  f->scal = reinterpret_cast<double*>(b + o_scal);
  f->bw.H1 = reinterpret_cast<uint16_t*>(b + o_H1);
  f->bw.H2 = reinterpret_cast<uint16_t*>(b + o_H2);
  f->bw.DRb = reinterpret_cast<uint16_t*>(b + o_DRb);
  f->bw.DH2b = reinterpret_cast<uint16_t*>(b + o_DH2b);
  f->bw.DRf = reinterpret_cast<float*>(b + o_DRf);
  f->bw.DH2f = reinterpret_cast<float*>(b + o_DH2f);
  f->bw.DH1f = reinterpret_cast<float*>(b + o_DH1f);
  f->bw.COND = reinterpret_cast<float*>(b + o_COND);
  f->bw.groups = 0;  // set per batch
  f->zs = reinterpret_cast<float*>(b + o_zs);
  f->lqs = reinterpret_cast<float*>(b + o_lqs);
  f->wpart = reinterpret_cast<float*>(b + o_wpart);
  if (hipEventCreateWithFlags(&f->ev_ready, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&f->ev_used, hipEventDisableTiming) != hipSuccess) {
    (void)hipFree(f->mem);
    delete f;
    return VEGAS_EHIP;
  }
  hipLaunchKernelGGL(k_flow_init, dim3(256), dim3(256), 0, f->stream, f->master, seed);
  hipLaunchKernelGGL(k_flow_zero, dim3(256), dim3(256), 0, f->stream, f->m1, static_cast<int64_t>(P));
  hipLaunchKernelGGL(k_flow_zero, dim3(256), dim3(256), 0, f->stream, f->m2, static_cast<int64_t>(P));
  if (hipGetLastError() != hipSuccess || flow_prep(f) != VEGAS_OK || hipStreamSynchronize(f->stream) != hipSuccess) {
    (void)hipFree(f->mem);
    (void)hipEventDestroy(f->ev_ready);
    (void)hipEventDestroy(f->ev_used);
    delete f;
    return VEGAS_EHIP;
  }
  *out = f;
  return VEGAS_OK;
}

int vegas_flow_destroy(vegas_flow f) {
  if (!f) return VEGAS_EINVAL;
  int rc = VEGAS_OK;
  if (hipStreamSynchronize(f->stream) != hipSuccess) rc = VEGAS_EHIP;
  if (hipFree(f->mem) != hipSuccess) rc = VEGAS_EHIP;
  (void)hipEventDestroy(f->ev_ready);
  (void)hipEventDestroy(f->ev_used);
  delete f;
  return rc;
}

int vegas_flow_get_params(vegas_flow f, float* dst_dev) {
  if (!f || !dst_dev) return VEGAS_EINVAL;
  VF_HIP(hipMemcpyAsync(dst_dev, f->master, sizeof(float) * FL_NPARAMS, hipMemcpyDeviceToDevice, f->stream));
  return VEGAS_OK;
}

int vegas_flow_set_params(vegas_flow f, const float* src_dev) {
  if (!f || !src_dev) return VEGAS_EINVAL;
  VF_HIP(hipMemcpyAsync(f->master, src_dev, sizeof(float) * FL_NPARAMS, hipMemcpyDeviceToDevice, f->stream));
  hipLaunchKernelGGL(k_flow_zero, dim3(256), dim3(256), 0, f->stream, f->m1, static_cast<int64_t>(FL_NPARAMS));
  hipLaunchKernelGGL(k_flow_zero, dim3(256), dim3(256), 0, f->stream, f->m2, static_cast<int64_t>(FL_NPARAMS));
  VF_HIP(hipGetLastError());
  f->adam_t = 0;
  return flow_prep(f);
}

int vegas_flow_density(vegas_flow f, const float* y_dev, int64_t B, float* logq_dev) {
  if (!f || !y_dev || !logq_dev || B < 1 || B > f->max_batch) return VEGAS_EINVAL;
  if (B <= kFusedDensity) {
    hipLaunchKernelGGL(k_flow_events<false>, dim3(grid_for(B, kEvTile, 1 << 20)), dim3(256), 0, f->stream, f->master, f->wb,
                       y_dev, nullptr, BatchIdx{}, nullptr, logq_dev, B, f->bw);
    VF_HIP(hipGetLastError());
    return VEGAS_OK;
  }
  return flow_layers<false>(f, f->stream, y_dev, f->V, 0, logq_dev, B);
}

int vegas_flow_loss_grad(vegas_flow f, const float* y_dev, const double* w_dev, int64_t B, float* grad_dev,
                         double* loss_host) {
  if (!f || !y_dev || !w_dev || B < 1 || B > f->max_batch) return VEGAS_EINVAL;
  const int rc = flow_gradient(f, y_dev, w_dev, BatchIdx{}, B, AdamArgs{}, loss_host);
  if (rc != VEGAS_OK) return rc;
  if (grad_dev) VF_HIP(hipMemcpyAsync(grad_dev, f->grad, sizeof(float) * FL_NPARAMS, hipMemcpyDeviceToDevice, f->stream));
  return VEGAS_OK;
}

int vegas_flow_train_step(vegas_flow f, const float* y_dev, const double* w_dev, int64_t n_data, int32_t batch,
                          uint64_t step, float lr, double* loss_host) {
  if (!f || !y_dev || !w_dev || n_data < 1 || n_data >= (int64_t(1) << 31) || batch < 1 || batch > f->max_batch ||
      !(lr > 0.f))
    return VEGAS_EINVAL;
  // per-epoch bijection i -> (a i + c) mod n with a coprime to n, from a Philox draw keyed by the epoch
  const uint64_t per_epoch = (static_cast<uint64_t>(n_data) + batch - 1) / batch;
  const uint64_t epoch = step / per_epoch;
  const int64_t start = static_cast<int64_t>((step % per_epoch) * batch);
  uint64_t a = 1, c = 0;
  {
    uint32_t s0 = static_cast<uint32_t>(epoch) * 0x9E3779B9u + 0x7F4A7C15u;
    uint32_t s1 = static_cast<uint32_t>(epoch >> 32) ^ 0x85EBCA6Bu;
    for (int r = 0; r < 3; ++r) {
      s0 ^= s1 * 0xC2B2AE35u + static_cast<uint32_t>(r);
      s1 ^= (s0 << 13) | (s0 >> 19);
    }
    const uint64_t n = static_cast<uint64_t>(n_data);
    a = (static_cast<uint64_t>(s0) | 1u) % n;
    if (a == 0) a = 1;
    auto gcd = [](uint64_t x, uint64_t y) {
      while (y) {
        const uint64_t t = x % y;
        x = y;
        y = t;
      }
      return x;
    };
    while (gcd(a, n) != 1) a = (a + 2) % n ? (a + 2) % n : 1;
    c = static_cast<uint64_t>(s1) % n;
  }
  const int64_t B = batch;
  f->adam_t++;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, static_cast<float>(f->adam_t));
  const float c2 = 1.f - std::pow(b2, static_cast<float>(f->adam_t));
  const int rc = flow_gradient(f, y_dev, w_dev, BatchIdx{static_cast<uint64_t>(n_data), a, c, static_cast<uint64_t>(start), ~uint64_t(0) / n_data}, B,
                               AdamArgs{f->master, f->m1, f->m2, f->wb, lr, b1, b2, 1e-8f, c1, c2}, loss_host);
  if (rc != VEGAS_OK) f->adam_t--;
  return rc;
}

int vegas_flow_sample(vegas_flow f, const float* z_dev, int64_t n, float* y_dev, float* logq_dev) {
  if (!f || !z_dev || !y_dev || !logq_dev || n < 1) return VEGAS_EINVAL;
  return flow_layers<true>(f, f->stream, z_dev, y_dev, 0, logq_dev, n);
}

}  // extern "C"

namespace vg {

// proposal points of a flow iteration on stream s (a VEGAS handle's): z from the
// stream keyed by (seed, iter, i), y = F^{-1}(z), log q(y); the flow's own stream
// is ordered before, and (via finish) after, the use on s
int flow_sample_events(vegas_flow f, hipStream_t s, uint64_t seed, uint32_t iter, int64_t n, const float** y,
                       const float** lq) {
  if (!f || n < 1 || n > f->max_sample) return VEGAS_EINVAL;
  if (s != f->stream) {
    VF_HIP(hipEventRecord(f->ev_ready, f->stream));
    VF_HIP(hipStreamWaitEvent(s, f->ev_ready, 0));
  }
  hipLaunchKernelGGL(k_flow_zinit, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, seed, iter, n, f->zs);
  VF_HIP(hipGetLastError());
  const int rc = flow_layers<true>(f, s, f->zs, f->zs, 0, f->lqs, n);
  if (rc != VEGAS_OK) return rc;
  *y = f->zs;
  *lq = f->lqs;
  return VEGAS_OK;
}

int flow_sample_finish(vegas_flow f, hipStream_t s) {
  if (s != f->stream) {
    VF_HIP(hipEventRecord(f->ev_used, s));
    VF_HIP(hipStreamWaitEvent(f->stream, f->ev_used, 0));
  }
  return VEGAS_OK;
}

}  // namespace vg
