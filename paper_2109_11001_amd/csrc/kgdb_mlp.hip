// Training and evaluation of the learned double-bridging proposal's network on gfx950.
//
// Forward passes run on the bf16 matrix cores (kgdb_mlp_dev.h: exact for the quantised
// network).  Training minimises the mean binary cross-entropy of the logits against the
// accept (1) / reject (0) labels of logged attempts.  Back-propagation treats each rounding
// as the identity (straight-through) and passes no gradient through a hidden unit that is
// cut by the ReLU or saturated at 255/16.  Deltas and weight gradients are FP64, on the FP64
// matrix cores; each workgroup sums its rows in a fixed order and the workgroups' partial sums
// are added in a fixed order, so a gradient is reproducible.  Adam (Kingma & Ba, 2015) updates
// FP32 master parameters.
#include "kgdb_dev.h"
#include "kgdb_kernels.h"
#include "kgdb_mlp_dev.h"

namespace kgdb {

__device__ __forceinline__ bool nn_is_bias(int p) {
  return (p >= NN_OFF_B1 && p < NN_OFF_W2) || (p >= NN_OFF_B2 && p < NN_OFF_W3) ||
         (p >= NN_OFF_B3 && p < NN_OFF_W4) || p == NN_OFF_B4;
}

// FP32 master parameters -> quantised network
__global__ __launch_bounds__(256) void k_mlp_quant(const float* __restrict__ P, NetQ* __restrict__ q) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < NN_H * NN_INP) {
    const int o = t / NN_INP, k = t - o * NN_INP;
    q->W1[o][k] = (__bf16)(k < NN_IN ? (float)q_weight(P[NN_OFF_W1 + o * NN_IN + k]) * 0.015625f : 0.0f);
  }
  if (t < NN_H * NN_H) {
    const int o = t / NN_H, k = t - o * NN_H;
    q->W2[o][k] = (__bf16)((float)q_weight(P[NN_OFF_W2 + t]) * 0.015625f);
    q->W3[o][k] = (__bf16)((float)q_weight(P[NN_OFF_W3 + t]) * 0.015625f);
  }
  if (t < NN_H) {
    q->w4[t] = (float)q_weight(P[NN_OFF_W4 + t]) * 0.015625f;
    q->b1[t] = P[NN_OFF_B1 + t];
    q->b2[t] = P[NN_OFF_B2 + t];
    q->b3[t] = P[NN_OFF_B3 + t];
  }
  if (t == 0) q->b4 = P[NN_OFF_B4];
}

// logits of n input rows [n][25]; one workgroup of 4 wavefronts per 64 rows
__global__ __launch_bounds__(256) void k_mlp_forward(const NetQ* __restrict__ net, const float* __restrict__ feat,
                                                     int64_t n, float* __restrict__ logit) {
  __shared__ NetTile t;
  const int64_t r0 = (int64_t)blockIdx.x * NN_TILE;
  if (threadIdx.x < NN_TILE) {
    const int64_t r = r0 + threadIdx.x;
    if (r < n) {
      float f[NN_IN];
#pragma unroll
      for (int k = 0; k < NN_IN; ++k) f[k] = feat[r * NN_IN + k];
      nn_set_input(t, threadIdx.x, f);
    } else {
      nn_zero_input(t, threadIdx.x);
    }
  }
  nn_forward_tile<4>(t, net);
  if (threadIdx.x < NN_TILE && r0 + threadIdx.x < n) logit[r0 + threadIdx.x] = t.logit[threadIdx.x];
}

// ---------------------------------------------------------------------------------------
// Training, forward half: 16 RB rows a workgroup of four wavefronts.  Leaves the rows' records,
// their output deltas gs = (sigmoid(logit) - label) / n and the workgroup's sum of losses.
// ---------------------------------------------------------------------------------------
template <int RB>
__global__ __launch_bounds__(256) void k_mlp_record(const NetQ* __restrict__ net, const float* __restrict__ feat,
                                                    const int32_t* __restrict__ label, int64_t n,
                                                    NetRecord* __restrict__ rec, double* __restrict__ gs,
                                                    double* __restrict__ lossp) {
  __shared__ NetTile t;
  __shared__ double s_loss[16 * RB];
  const int64_t r0 = (int64_t)blockIdx.x * (16 * RB);
  rec += (size_t)blockIdx.x * RB;
  constexpr int PER = 16 * RB * NN_INP / 256;
  float in[PER];
  const int k = threadIdx.x % NN_INP;
#pragma unroll
  for (int e = 0; e < PER; ++e) {  // (clamped addresses: no branch between the loads)
    const int64_t r = r0 + (threadIdx.x + e * 256) / NN_INP;
    in[e] = feat[min(r, n - 1) * NN_IN + min(k, NN_IN - 1)];
  }
  const int nrow = (int)min((int64_t)(16 * RB), n - r0);
  double y = 0.0;
  if ((int)threadIdx.x < nrow) y = (double)label[r0 + threadIdx.x];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int r = (threadIdx.x + e * 256) / NN_INP;
    t.a0[r][k] = (__bf16)(k < NN_IN && r < nrow ? (float)q_input(in[e]) * 0.015625f : 0.0f);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < RB * NN_INP * 4; e += 256) {
    const int b = e / (NN_INP * 4), c = (e >> 2) % NN_INP, q = e & 3;
    u16x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __builtin_bit_cast(uint16_t, t.a0[16 * b + 4 * q + i][c]);
    *(u16x4*)&rec[b].x[c][4 * q] = v;
  }
  NnFrag<NN_INP, 4> f1;
  f1.load(&net->W1[0][0], net->b1);
  nn_layer<NN_INP, 4, RB, 0>(&t.a0[0][0], NN_SA0, &t.a1[0][0], f1, rec);
  __syncthreads();
  NnFrag<NN_H, 4> f2;
  f2.load(&net->W2[0][0], net->b2);
  nn_layer<NN_H, 4, RB, 1>(&t.a1[0][0], NN_SA, &t.a2[0][0], f2, rec);
  __syncthreads();
  f2.load(&net->W3[0][0], net->b3);
  nn_layer<NN_H, 4, RB, 2>(&t.a2[0][0], NN_SA, &t.a1[0][0], f2, rec);
  __syncthreads();
  nn_output<4, RB>(t.a1, net, t.logit);
  __syncthreads();
  if (threadIdx.x < 16 * RB) {
    double g = 0.0, ls = 0.0;
    if ((int)threadIdx.x < nrow) {
      const double z = (double)t.logit[threadIdx.x];
      const double ez = exp(z >= 0.0 ? -z : z);
      g = ((z >= 0.0 ? 1.0 / (1.0 + ez) : ez / (1.0 + ez)) - y) / (double)n;
      ls = (z > 0.0 ? z : 0.0) + log1p(ez) - y * z;
    }
    gs[r0 + threadIdx.x] = g;  // (0 past the last row: the workspace holds whole row blocks)
    s_loss[threadIdx.x] = ls;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double v = 0.0;
    for (int q = 0; q < 16 * RB; ++q) v += s_loss[q];
    lossp[blockIdx.x] = v;
  }
}

// ---------------------------------------------------------------------------------------
// Training, backward half: a workgroup of four wavefronts takes a run of row blocks, 16 rows at a
// time: the deltas run back through the layers on v_mfma_f64_16x16x4_f64 and the three weight
// gradients accumulate in registers (wavefront w owns outputs 32 w .. 32 w + 31 of every layer: 36
// blocks of 16 x 16, 288 registers).  Nothing but the partial gradient leaves the workgroup.
//
// What bounds it: the FP64 products (139,264 flops a row: 102 us for 46,000 rows at the 62.8 TFLOP/s
// a large FP64 matrix product reaches; measured 162 us, the matrix cores busy for 53% of it, where the former
// per-thread loops took 1,650 us); the rest is waits, for LDS and at the top of a row block for its record.
// One wavefront per SIMD with 512 registers keeps the
// gradient blocks, the weights and the next operands in registers; two of 256, with the forward
// layers in the same kernel, had no room for operands ahead of their use and waited on LDS before
// each product.  Layout of the instruction (wave64): lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and receives D[4 i + l / 16][l % 16], i = 0 .. 3.  Which of the 16 rows a row or
// a step of a product stands for is free; here lane group kq = l / 16 always holds rows
// 4 kq .. 4 kq + 3, whose codes of a column are one 8-byte read of a record.
// ---------------------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int TR_WAVES = 4;
constexpr int TR_BLOCK = 64 * TR_WAVES;
constexpr int TR_SG = NN_H + 2;  // row stride of the deltas: rows are 4 banks apart, so that a read of
                                 // 16 rows by two columns touches every bank once
static_assert(TR_WAVES * 32 == NN_H, "a wavefront owns 32 outputs of a layer");

// the low or high bf16 of a register (weights and inputs are signed)
__device__ __forceinline__ double bf16_half(uint32_t v, int hi) {
  return (double)__uint_as_float(hi ? v & 0xffff0000u : v << 16);
}
// the same of two hidden codes, without the sign bit, which says that the unit passes gradient
__device__ __forceinline__ double code_half(uint32_t v, int hi) {
  return (double)__uint_as_float(hi ? v & 0x7fff0000u : (v & 0x7fffu) << 16);
}

__global__ __launch_bounds__(TR_BLOCK, 1) void k_mlp_back(const NetQ* __restrict__ net,
                                                          const NetRecord* __restrict__ rec,
                                                          const double* __restrict__ gs, int nblk, int per,
                                                          double* __restrict__ part) {
  __shared__ double G[3][NN_ROWBLOCK][TR_SG];  // deltas of layers 3, 2, 1 of the current 16 rows
  __shared__ double s_red[4][2][NN_H];
  __shared__ double s_tail[NN_ROWBLOCK];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int col = 32 * wv + r16;  // and col + 16
  const int b0 = (int)blockIdx.x * per, b1 = min(nblk, b0 + per);
  // this wavefront's columns of W3 and W2 as B operands (step j: row 4 j + kq), two bf16 a register
  uint32_t w3[2][NN_H / 8], w2[2][NN_H / 8];
  const uint16_t* __restrict__ W3 = (const uint16_t*)&net->W3[0][0];
  const uint16_t* __restrict__ W2 = (const uint16_t*)&net->W2[0][0];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int q = 0; q < NN_H / 8; ++q) {
      const int o = (8 * q + kq) * NN_H + col + 16 * c;
      w3[c][q] = (uint32_t)W3[o] | ((uint32_t)W3[o + 4 * NN_H] << 16);
      w2[c][q] = (uint32_t)W2[o] | ((uint32_t)W2[o + 4 * NN_H] << 16);
    }
  f64x4 d3[2][8], d2[2][8], d1[2][2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
#pragma unroll
    for (int b = 0; b < 8; ++b) d3[c][b] = d2[c][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    d1[c][0] = d1[c][1] = f64x4{0.0, 0.0, 0.0, 0.0};
  }
  // column sums: thread (unit u, group p) adds rows 8 p .. 8 p + 7 of each 16
  const int u = threadIdx.x & (NN_H - 1), p = threadIdx.x >> 7;
  const double w4u = (double)net->w4[u];
  double s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0, sb = 0.0;

#pragma unroll 1
  for (int blk = b0; blk < b1; ++blk) {
    const NetRecord& r = rec[blk];
    const double* __restrict__ gr = gs + (size_t)blk * NN_ROWBLOCK + 8 * p;
    // layer-3 deltas (read by the others only past the next barrier; the last block's were read
    // before its own last one)
    {
      const uint4 h = *(const uint4*)&r.h[2][u][8 * p];
      const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double g = gr[e];
        const uint32_t on = (hw[e >> 1] >> ((e & 1) * 16)) & 0x8000u;
        const double v = on ? g * w4u : 0.0;
        G[0][8 * p + e][u] = v;
        s3 += v;
        s4 += g * code_half(hw[e >> 1], e & 1);
      }
      if (threadIdx.x < NN_ROWBLOCK) sb += gs[(size_t)blk * NN_ROWBLOCK + threadIdx.x];
    }
    __syncthreads();
    // deltas of the layer below, G[lo] = mask (G[hi] W), and the gradient dW += G[hi]^T a
    auto layer = [&](int hi, uint32_t (*w)[NN_H / 8], f64x4 (*dw)[8]) {
      const uint16_t(*h)[NN_ROWBLOCK] = r.h[1 - hi];  // the layer below
      uint2 c4[8], m4[2];
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) c4[nb] = *(const uint2*)&h[16 * nb + r16][4 * kq];
#pragma unroll
      for (int c = 0; c < 2; ++c) m4[c] = *(const uint2*)&h[col + 16 * c][4 * kq];
      // (opaque to the compiler, which would otherwise keep the weights' FP64 forms over the loop)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < NN_H / 8; ++q) asm volatile("" : "+v"(w[c][q]));
      f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
      double gT[2][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        gT[0][q] = G[hi][4 * kq + q][col];
        gT[1][q] = G[hi][4 * kq + q][col + 16];
      }
      const double* gp = &G[hi][4 * (r16 & 3) + (r16 >> 2)][kq];
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = 4 * nb + q;
          const double g = gp[4 * j], b = code_half((q >> 1) ? c4[nb].y : c4[nb].x, q & 1);
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(g, bf16_half(w[c][j >> 1], j & 1), acc[c], 0, 0, 0);
            dw[c][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(gT[c][q], b, dw[c][nb], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const uint32_t m = ((i >> 1) ? m4[c].y : m4[c].x) >> ((i & 1) * 16);
          G[hi + 1][4 * kq + i][col + 16 * c] = (m & 0x8000u) ? acc[c][i] : 0.0;
        }
      __syncthreads();
    };
    layer(0, w3, d3);
#pragma unroll
    for (int e = 0; e < 8; ++e) s2 += G[1][8 * p + e][u];
    layer(1, w2, d2);
#pragma unroll
    for (int e = 0; e < 8; ++e) s1 += G[2][8 * p + e][u];
    uint2 x4[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) x4[b] = *(const uint2*)&r.x[16 * b + r16][4 * kq];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double g = G[2][4 * kq + q][col + 16 * c];
#pragma unroll
        for (int b = 0; b < 2; ++b)
          d1[c][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(g, bf16_half((q >> 1) ? x4[b].y : x4[b].x, q & 1), d1[c][b],
                                                          0, 0, 0);
      }
  }
  // the partial gradient
  double* __restrict__ out = part + (size_t)blockIdx.x * NN_NPARAM;
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = 32 * wv + 16 * c + 4 * i + kq;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        out[NN_OFF_W3 + o * NN_H + 16 * b + r16] = d3[c][b][i];
        out[NN_OFF_W2 + o * NN_H + 16 * b + r16] = d2[c][b][i];
      }
#pragma unroll
      for (int b = 0; b < 2; ++b)
        if (16 * b + r16 < NN_IN) out[NN_OFF_W1 + o * NN_IN + 16 * b + r16] = d1[c][b][i];
    }
  // the column sums of the two groups, and the output bias
  s_red[0][p][u] = s1;
  s_red[1][p][u] = s2;
  s_red[2][p][u] = s3;
  s_red[3][p][u] = s4;
  if (threadIdx.x < NN_ROWBLOCK) s_tail[threadIdx.x] = sb;
  __syncthreads();
#pragma unroll
  for (int q = p; q < 4; q += 2)  // b1, b2, b3, w4
    out[(q == 0 ? NN_OFF_B1 : q == 1 ? NN_OFF_B2 : q == 2 ? NN_OFF_B3 : NN_OFF_W4) + u] = s_red[q][0][u] + s_red[q][1][u];
  if (threadIdx.x == 0) {
    double v = 0.0;
    for (int q = 0; q < NN_ROWBLOCK; ++q) v += s_tail[q];
    out[NN_OFF_B4] = v;
  }
}

// One Adam step of a parameter: m <- b1 m + (1-b1) g, v <- b2 v + (1-b2) g^2,
// P <- P - lr mhat / (sqrt(vhat) + eps) with the bias corrections of step t; weights are
// clamped to the representable range +-255/64.  FP64 arithmetic, FP32 storage.
struct AdamArgs {
  float *P, *m, *v;
  double c1, c2, lr, b1, b2, eps;
};
__device__ __forceinline__ void adam_one(const AdamArgs& a, int p, double gg) {
  const double mm = a.b1 * (double)a.m[p] + (1.0 - a.b1) * gg;
  const double vv = a.b2 * (double)a.v[p] + (1.0 - a.b2) * gg * gg;
  double q = (double)a.P[p] - a.lr * (mm / a.c1) / (sqrt(vv / a.c2) + a.eps);
  if (!nn_is_bias(p)) {
    if (q > 255.0 / 64.0) q = 255.0 / 64.0;
    if (q < -255.0 / 64.0) q = -255.0 / 64.0;
  }
  a.P[p] = (float)q;
  a.m[p] = (float)mm;
  a.v[p] = (float)vv;
}
__global__ __launch_bounds__(256) void k_mlp_adam(AdamArgs a, const double* __restrict__ g) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NN_NPARAM) adam_one(a, p, g[p]);
}

// The gradient from the nparts partial sums, 64 parameters a workgroup: its four wavefronts take
// every fourth partial each (so that about eight loads a lane are in flight) and are added in
// order.  With ADAM the step is taken at once, without the gradient in memory.  Workgroup 0 also
// adds the loss.  Bound by reading the partials once (70 MB at 46,000 rows).
template <bool ADAM>
__global__ __launch_bounds__(256) void k_mlp_reduce(const double* __restrict__ part, int nparts,
                                                    double* __restrict__ grad, AdamArgs a,
                                                    const double* __restrict__ lossp, int nloss, int64_t n,
                                                    double* __restrict__ loss) {
  __shared__ double s_g[4][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  double acc = 0.0;
  if (p < NN_NPARAM) {
#pragma unroll 8
    for (int c = grp; c < nparts; c += 4) acc += part[(size_t)c * NN_NPARAM + p];
  }
  s_g[grp][lane] = acc;
  __syncthreads();
  if (grp == 0 && p < NN_NPARAM) {
    const double g = ((s_g[0][lane] + s_g[1][lane]) + s_g[2][lane]) + s_g[3][lane];
    if constexpr (ADAM) adam_one(a, p, g);
    else grad[p] = g;
  }
  if (blockIdx.x == 0) {
    __shared__ double s_l[256];
    double v = 0.0;
    for (int c = threadIdx.x; c < nloss; c += 256) v += lossp[c];
    s_l[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) s_l[threadIdx.x] += s_l[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) *loss = s_l[0] / (double)n;
  }
}

// ---------------------------------------------------------------------------------------
size_t netq_bytes() { return sizeof(NetQ); }

MlpWork mlp_work_layout(void* base, int64_t n) {
  MlpWork w;
  char* p = (char*)base;
  size_t o = 0;
  auto take = [&](size_t bytes) { char* q = p ? p + o : nullptr; o += nn_align256(bytes); return q; };
  w.net = (NetQ*)take(sizeof(NetQ));
  w.rec = (NetRecord*)take(sizeof(NetRecord) * nn_blocks(n));
  w.gs = (double*)take(sizeof(double) * NN_ROWBLOCK * nn_blocks(n));
  w.lossp = (double*)take(sizeof(double) * nn_blocks(n));
  w.part = (double*)take(sizeof(double) * NN_NPARAM * (size_t)(nn_parts_cap(n) > 0 ? nn_parts_cap(n) : 1));
  w.grad = (double*)take(sizeof(double) * NN_NPARAM);
  w.loss = (double*)take(sizeof(double));
  w.bytes = o;
  return w;
}

void launch_mlp_quant(const float* P, NetQ* q, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_quant, dim3((NN_H * NN_H + 255) / 256), dim3(256), 0, s, P, q);
}

void launch_mlp_forward(const NetQ* net, const float* feat, int64_t n, float* logit, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)((n + NN_TILE - 1) / NN_TILE)), dim3(256), 0, s, net, feat, n,
                     logit);
}

// Partial gradients of n rows: their number, and that of the loss sums.  The forward half takes 64
// rows a workgroup (one read of the weights for them) once that fills the CUs, 16 below.
struct TrainParts { int parts, losses; };
static TrainParts launch_mlp_train(const MlpWork& w, const float* feat, const int32_t* label, int64_t n,
                                   hipStream_t s) {
  const int nblk = (int)((n + NN_ROWBLOCK - 1) / NN_ROWBLOCK);
  const int losses = n >= 64 * 256 ? (nblk + 3) / 4 : nblk;
  if (n >= 64 * 256)
    hipLaunchKernelGGL(k_mlp_record<4>, dim3(losses), dim3(256), 0, s, w.net, feat, label, n, w.rec, w.gs, w.lossp);
  else
    hipLaunchKernelGGL(k_mlp_record<1>, dim3(losses), dim3(256), 0, s, w.net, feat, label, n, w.rec, w.gs, w.lossp);
  const int per = (int)(nn_part_rows(n) / NN_ROWBLOCK);
  const int parts = (nblk + per - 1) / per;
  hipLaunchKernelGGL(k_mlp_back, dim3(parts), dim3(TR_BLOCK), 0, s, w.net, w.rec, w.gs, nblk, per, w.part);
  return {parts, losses};
}

void launch_mlp_grad(const MlpWork& w, const float* feat, const int32_t* label, int64_t n, double* grad, double* loss,
                     hipStream_t s) {
  const TrainParts t = launch_mlp_train(w, feat, label, n, s);
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((NN_NPARAM + 63) / 64), dim3(256), 0, s, w.part, t.parts, grad,
                     AdamArgs{}, w.lossp, t.losses, n, loss);
}

void launch_mlp_step(const MlpWork& w, const float* feat, const int32_t* label, int64_t n, float* P, float* m,
                     float* v, double c1, double c2, double lr, double b1, double b2, double eps, double* loss,
                     hipStream_t s) {
  const TrainParts t = launch_mlp_train(w, feat, label, n, s);
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((NN_NPARAM + 63) / 64), dim3(256), 0, s, w.part, t.parts,
                     (double*)nullptr, AdamArgs{P, m, v, c1, c2, lr, b1, b2, eps}, w.lossp, t.losses, n, loss);
}

void launch_mlp_adam(float* P, float* m, float* v, const double* g, double c1, double c2, double lr, double b1,
                     double b2, double eps, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_adam, dim3((NN_NPARAM + 255) / 256), dim3(256), 0, s,
                     AdamArgs{P, m, v, c1, c2, lr, b1, b2, eps}, g);
}

}  // namespace kgdb
