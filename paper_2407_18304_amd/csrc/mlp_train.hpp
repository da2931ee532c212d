// mlp_train.hpp -- one training pass of the warm-start network in three
// kernels (128 hidden units, BF16 operands): the rows forward and backward,
// the weight gradients, and their sum with the Adam step.
//
// The arithmetic is that of the layer-by-layer kernels in mlp.hip: operands
// rounded to BF16 where a product takes them, FP32 accumulation, FP32
// pre-activations, gradients and bias sums.  Layer by layer a step took 24
// launches that each read and wrote FP32 activations in HBM (4096 rows x 64
// groups: 240 us of column sums, 150 us of weight gradients added up with
// atomics, 140 us of forward and backward products); the floor, rows and
// weights read once and the products at the matrix cores' rate, is under 5 us,
// so what counts is the number of dependent steps.  Three kernels take 25 + 11
// + 8 us (32768 rows: 111 us a step, 1000 rows x 4 groups: 29 us).
#pragma once

namespace mgrhd {
namespace mlp {

constexpr int kRowTile = 32;     // rows of a workgroup's tile (two matrix-core tiles)
constexpr int kRowThreads = 512;  // a wave per 16 hidden units
constexpr int kMaxSplits = 32;   // most row ranges of a weight gradient
constexpr int kHT = 128;         // hidden width of this path

// Buffers of one pass.  The transposed activations and gradients are
// [unit][pitch] BF16, rows contiguous: k_train_dw reads both its operands as
// matrix-core fragments straight from them, with no LDS.
struct TrainArgs {
  const float* X;   // features, feature-major [n_in][ldx]
  const float* T;   // targets [rows][n_out]
  int64_t ldx, rows, pitch;
  const __bf16* W[4];   // [N_pad][K_pad], zero padded
  const __bf16* WT[4];  // layers 1..3: [128][kt_pad], zero padded
  const float* b[4];    // [N_pad]
  int K_pad[4], N_pad[4], kt_pad[4];
  int n_in, n_out;
  __bf16* XT;      // [K_pad[0]][pitch]
  __bf16* HT[3];   // [128][pitch]
  __bf16* dT[4];   // [N_pad][pitch]: gradient of each layer's pre-activation
  float* bias_part;  // [workgroups][3 * 128 + N_pad[3]]
  float* loss_part;  // [workgroups]
  float scale;       // 1 / (rows n_out)
};

// LDS pitch of a tile of k columns: 16-byte aligned rows, skewed banks.
__host__ __device__ constexpr int tile_pitch(int k) { return k + 8; }
__host__ __device__ inline size_t train_lds_bytes(int k_pad0, int kt_pad3) {
  const int wide = k_pad0 > kt_pad3 ? k_pad0 : kt_pad3;
  return sizeof(__bf16) * (size_t)kRowTile * (tile_pitch(wide) + 2 * tile_pitch(kHT));
}

// acc[a] = in[16a..][k] W[16 nt..][k]^T over ksteps slices of 32; in: LDS rows of
// pitch ldi, W: rows of K_pad in L2.  The weights of four slices are requested
// at once.
__device__ __forceinline__ void tile_product(const __bf16* in, int ldi,
                                             const __bf16* __restrict__ W, int K_pad, int ksteps,
                                             int nt, floatx4 (&acc)[2]) {
  const int lane = threadIdx.x % 64, r16 = lane % 16, kq = 8 * (lane / 16);
  const __bf16* w0 = W + (int64_t)(16 * nt + r16) * K_pad + kq;
#pragma unroll
  for (int a = 0; a < 2; ++a) acc[a] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int kPre = 4;
  for (int kb = 0; kb < ksteps; kb += kPre) {
    bf16x8 w[kPre];
#pragma unroll
    for (int kk = 0; kk < kPre; ++kk)
      if (kb + kk < ksteps) w[kk] = *(const bf16x8*)(w0 + 32 * (kb + kk));
#pragma unroll
    for (int kk = 0; kk < kPre; ++kk) {
      if (kb + kk >= ksteps) break;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const bf16x8 x = *(const bf16x8*)(in + (16 * a + r16) * ldi + 32 * (kb + kk) + kq);
        acc[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, w[kk], acc[a], 0, 0, 0);
      }
    }
  }
}

// Four consecutive rows of one unit, as BF16, into the LDS tile (row-major)
// and the transposed array.
__device__ __forceinline__ void put4(const floatx4& v, __bf16* tile, int ld, __bf16* trans,
                                     int64_t pitch, int row, int unit, int64_t r0) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 p;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = (__bf16)v[i];
    if (tile) tile[(row + i) * ld + unit] = p[i];
  }
  *(bf16x4*)(trans + (int64_t)unit * pitch + r0 + row) = p;
}

// The rows: forward through the four layers, the mean-squared error, and back
// to the first layer's pre-activation, a workgroup per tile.  A wave holds 16 units of
// every hidden layer in both directions, so the FP32 pre-activations stay in
// its registers until the backward pass wants their SiLU'.  Bound by the chain
// of seven dependent products, each an L2 latency and a barrier: a tile of 32
// rows leaves a workgroup for each CU at 8192 rows and costs half the chain of
// two tiles of 16.
__global__ __launch_bounds__(kRowThreads, 4) void k_train_rows(TrainArgs q) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wide = q.K_pad[0] > q.kt_pad[3] ? q.K_pad[0] : q.kt_pad[3];
  const int ldx = tile_pitch(wide), ldh = tile_pitch(kHT);
  __bf16* const Xs = (__bf16*)smem;            // input tile, then the output gradient
  __bf16* const Hs[2] = {Xs + kRowTile * ldx, Xs + kRowTile * ldx + kRowTile * ldh};
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int r16 = lane % 16, row4 = 4 * (lane / 16);
  constexpr int kWaves = kRowThreads / 64;
  static_assert(16 * kWaves == kHT, "a wave per 16 hidden units");
  const int unit = 16 * wave + r16;  // this lane's hidden unit
  const int n_tiles3 = q.N_pad[3] / 16;
  float bsum[3] = {}, bsum3[2] = {}, loss = 0.f;
  const int64_t r0 = (int64_t)blockIdx.x * kRowTile;
  {
    // a thread's features of one row, eight loads in flight
    const int r = tid % kRowTile;
    const bool live = r0 + r < q.rows;
    constexpr int kU = 8, kStep = kRowThreads / kRowTile;
    for (int f0 = tid / kRowTile; f0 < q.K_pad[0]; f0 += kU * kStep) {
      float x[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int f = f0 + u * kStep;
        x[u] = (f < q.n_in && live) ? q.X[(int64_t)f * q.ldx + r0 + r] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int f = f0 + u * kStep;
        if (f >= q.K_pad[0]) break;
        Xs[r * ldx + f] = (__bf16)x[u];
        q.XT[(int64_t)f * q.pitch + r0 + r] = (__bf16)x[u];
      }
    }
  }
  __syncthreads();
  floatx4 z[3][2];
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const __bf16* in = l == 0 ? Xs : Hs[(l - 1) % 2];
    tile_product(in, l == 0 ? ldx : ldh, q.W[l], q.K_pad[l], q.K_pad[l] / 32, wave, z[l]);
    const float bv = q.b[l][unit];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      floatx4 h;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = z[l][a][i] + bv;
        z[l][a][i] = v;
        h[i] = v / (1.f + expf(-v));
      }
      put4(h, Hs[l % 2], ldh, q.HT[l], q.pitch, 16 * a + row4, unit, r0);
    }
    __syncthreads();
  }
  // output layer, error and its gradient (the columns up to kt_pad are zero)
  for (int e = tid; e < kRowTile * (q.kt_pad[3] - q.N_pad[3]); e += kRowThreads) {
    const int w = q.kt_pad[3] - q.N_pad[3];
    Xs[(e / w) * ldx + q.N_pad[3] + e % w] = (__bf16)0.f;
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int nt = wave + kWaves * p;
    if (nt >= n_tiles3) break;
    floatx4 y[2];
    tile_product(Hs[0], ldh, q.W[3], q.K_pad[3], kHT / 32, nt, y);
    const int n = 16 * nt + r16;
    const float bv = q.b[3][n];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      floatx4 d;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = r0 + 16 * a + row4 + i;
        d[i] = 0.f;
        if (row < q.rows && n < q.n_out) {
          const float e = y[a][i] + bv - q.T[row * q.n_out + n];
          d[i] = 2.f * e * q.scale;
          loss += e * e;
        }
        bsum3[p] += d[i];
      }
      put4(d, Xs, ldx, q.dT[3], q.pitch, 16 * a + row4, n, r0);
    }
  }
  __syncthreads();
  // backward: dH_l = dZ_{l+1} W_{l+1}, dZ_l = dH_l SiLU'(z_l)
#pragma unroll
  for (int l = 2; l >= 0; --l) {
    const __bf16* in = l == 2 ? Xs : Hs[l % 2];  // dZ_3 in Xs, dZ_2 in Hs[1], dZ_1 in Hs[0]
    floatx4 d[2];
    tile_product(in, l == 2 ? ldx : ldh, q.WT[l + 1], q.kt_pad[l + 1], q.kt_pad[l + 1] / 32,
                 wave, d);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      floatx4 g;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = z[l][a][i];
        const float s = 1.f / (1.f + expf(-v));
        g[i] = d[a][i] * (s * (1.f + v * (1.f - s)));
        bsum[l] += g[i];
      }
      put4(g, l > 0 ? Hs[(l + 1) % 2] : nullptr, ldh, q.dT[l], q.pitch, 16 * a + row4, unit, r0);
    }
    __syncthreads();
  }
  // sums over this workgroup's rows: the four 4-row groups of a column are in
  // lanes 16 and 32 apart
  float* const bp = q.bias_part + (int64_t)blockIdx.x * (3 * kHT + q.N_pad[3]);
  auto over_rows = [](float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
  };
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const float v = over_rows(bsum[l]);
    if (lane < 16) bp[l * kHT + unit] = v;
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const float v = over_rows(bsum3[p]);
    const int nt = wave + kWaves * p;
    if (lane < 16 && nt < n_tiles3) bp[3 * kHT + 16 * nt + r16] = v;
  }
  float* const part = (float*)smem;  // (the tiles are done with)
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) loss += __shfl_xor(loss, m, 64);
  if (lane == 0) part[wave] = loss;
  __syncthreads();
  if (tid == 0) {
    float sum = 0.f;
    for (int w = 0; w < kWaves; ++w) sum += part[w];
    q.loss_part[blockIdx.x] = sum;
  }
}

// Weight gradients dW_l = dZ_l^T in_l over one range of rows: a workgroup per 64
// x 64 tile of one layer's matrix and range, a wave per 32 x 32, both operands
// read as fragments (rows contiguous).  Every range writes its own partial
// matrix, summed by k_train_finish: ranges of some 200 rows give 500 workgroups
// at 4096 rows, and no atomics.
struct DwArgs {
  const __bf16* A[4];  // dT[l]: [M_pad][pitch]
  const __bf16* B[4];  // the layer's input transposed: [N_pad][pitch]
  int M[4], N[4], M_pad[4], N_pad[4], tiles_n[4];
  int first[5];  // first tile of each layer
  int64_t w_off[4];
  int64_t pitch, chunk, n_params;
  float* part;   // [ranges][n_params]
};

__global__ __launch_bounds__(256) void k_train_dw(DwArgs q) {
  const int tile = blockIdx.x;
  int l = 0;
  while (tile >= q.first[l + 1]) ++l;
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  const int r16 = lane % 16, kq = 8 * (lane / 16);
  const int m0 = 64 * ((tile - q.first[l]) / q.tiles_n[l]) + 32 * (wave / 2);
  const int n0 = 64 * ((tile - q.first[l]) % q.tiles_n[l]) + 32 * (wave % 2);
  const int64_t k0 = (int64_t)blockIdx.y * q.chunk;
  const int64_t k1 = k0 + q.chunk < q.pitch ? k0 + q.chunk : q.pitch;
  const __bf16 *pa[2], *pb[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {  // (units beyond the matrix: any row, not stored)
    pa[a] = q.A[l] + (int64_t)min(m0 + 16 * a + r16, q.M_pad[l] - 1) * q.pitch + kq;
    pb[a] = q.B[l] + (int64_t)min(n0 + 16 * a + r16, q.N_pad[l] - 1) * q.pitch + kq;
  }
  floatx4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int kPre = 4;
  for (int64_t k = k0; k < k1; k += 32 * kPre) {
    bf16x8 fa[kPre][2], fb[kPre][2];
#pragma unroll
    for (int u = 0; u < kPre; ++u)
      if (k + 32 * u < k1)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          fa[u][a] = *(const bf16x8*)(pa[a] + k + 32 * u);
          fb[u][a] = *(const bf16x8*)(pb[a] + k + 32 * u);
        }
#pragma unroll
    for (int u = 0; u < kPre; ++u)
      if (k + 32 * u < k1)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[a][b] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[u][a], fb[u][b], acc[a][b], 0, 0, 0);
  }
  float* const out = q.part + (int64_t)blockIdx.y * q.n_params + q.w_off[l];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int n = n0 + 16 * b + r16;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m0 + 16 * a + 4 * (lane / 16) + i;
        if (m < q.M[l] && n < q.N[l]) out[(int64_t)m * q.N[l] + n] = acc[a][b][i];
      }
    }
}

// The parameters: gradients from the partial sums, the loss, and with ADAM the
// step on the FP32 master weights, whose BF16 copies are written with them.
// The first workgroups take 256 weights each, the others 8 biases each (32
// threads per bias over the row tiles' sums), the last one the loss too.
struct FinishArgs {
  const float* part;
  const float* bias_part;
  const float* loss_part;
  int splits, row_blocks, bias_width;
  float loss_scale;
  float *loss, *loss_out;
  float *p, *g, *m, *v;
  int64_t n_params, n_weights, n_weight_blocks;
  int64_t w_off[4], b_off[4];
  int in_dim[4], out_dim[4], K_pad[4], kt_pad[4];
  __bf16* W[4];
  __bf16* WT[4];
  float* b[4];
  float lr, b1, b2, eps, c1, c2;
};

template <bool ADAM>
__global__ __launch_bounds__(256) void k_train_finish(FinishArgs q) {
  __shared__ float red[256];
  const int tid = threadIdx.x;
  if (blockIdx.x < q.n_weight_blocks) {
    const int64_t i = (int64_t)blockIdx.x * 256 + tid;
    if (i >= q.n_weights) return;
    float s = 0.f;
    for (int k = 0; k < q.splits; ++k) s += q.part[(int64_t)k * q.n_params + i];
    q.g[i] = s;
    if (ADAM) {
      const float x = adam_update(q.p, q.m, q.v, i, s, q.lr, q.b1, q.b2, q.eps, q.c1, q.c2);
      int l = 3;
      while (i < q.w_off[l]) --l;
      const int r = (int)(i - q.w_off[l]), o = r / q.in_dim[l], c = r % q.in_dim[l];
      q.W[l][(int64_t)o * q.K_pad[l] + c] = (__bf16)x;
      if (l > 0) q.WT[l][(int64_t)c * q.kt_pad[l] + o] = (__bf16)x;
    }
    return;
  }
  // biases: i counts them over the layers, column n of the partial sums
  const int64_t i = (blockIdx.x - q.n_weight_blocks) * 8 + tid % 8;
  const bool live = i < q.n_params - q.n_weights;
  int l = 3;
  while (q.n_weights + i < q.b_off[l]) --l;
  const int o = (int)(q.n_weights + i - q.b_off[l]);
  float s = 0.f;
  if (live)
    for (int k = tid / 8; k < q.row_blocks; k += 32)
      s += q.bias_part[(int64_t)k * q.bias_width + l * kHT + o];
  red[tid] = s;
  __syncthreads();
  if (tid < 8 && live) {
    for (int k = 1; k < 32; ++k) s += red[8 * k + tid];
    const int64_t at = q.n_weights + i;
    q.g[at] = s;
    if (ADAM)
      q.b[l][o] = adam_update(q.p, q.m, q.v, at, s, q.lr, q.b1, q.b2, q.eps, q.c1, q.c2);
  }
  if (blockIdx.x == gridDim.x - 1) {
    float e = 0.f;
    for (int k = tid; k < q.row_blocks; k += 256) e += q.loss_part[k];
    __syncthreads();
    red[tid] = e;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (tid < h) red[tid] += red[tid + h];
      __syncthreads();
    }
    if (tid == 0) {
      *q.loss = red[0] * q.loss_scale;
      if (q.loss_out) *q.loss_out = red[0] * q.loss_scale;
    }
  }
}

}  // namespace mlp
}  // namespace mgrhd
