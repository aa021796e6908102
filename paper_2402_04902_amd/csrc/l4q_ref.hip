// The unfused quantizer-gradient pass (binary32 mode, unfused backward of the bfloat16 mode, and there QAT-LoRA too),
// the fixed-order sums of partial results, and the AdamW step.  No assumption on shapes beyond the
// library's divisibility rules.
#include "l4q_device.h"
#include "l4q_kernels.h"
#include "l4q_reduce.h"

namespace l4q {

namespace {

// ------------------------------------------------------------------ quantizer gradients, unfused
//   dscale[p,q] = sum_j dWq * (m ? code - w : code)   (Eq. quant_lsq_s and App. A.1 case list)
//   dzero [p,q] = sum_j dWq * (m ? 0 : 1)             (Eq. appen_lsq_b)
// and, LORA (the L4Q layer; the QAT-LoRA quantizer sees the frozen weight alone and needs neither):
//   dWq <- m * dWq                                    (Eq. appen_ste)
//   dB[p,k]     = gamma * sum_j (m * dWq)[p,j] A[k,j] (Eq. appen_l4q_b)
//
// Bound: memory (dWq and W0 read once; LORA: the masked dWq written), with the IEEE divide and the rank sums close behind.
// A workgroup takes ROWS weight rows and deals their columns out to its 4 waves in units of 256 (or a whole group where
// groups are longer), a lane owning 4 consecutive columns of all the rows: A is read once per ROWS rows, and ROWS
// independent loads per operand are in flight.  One wave per row with one row's loads in flight, the first form, took
// 137 us on 4096 x 4096 bf16 without LoRA (28 now: 100 MB at 3.5 TB/s) and 66 us on 2048 x 2048 binary32 at rank
// 16 (now 27; 4 rows per workgroup 32).
constexpr int QG_KCHUNK = 16;

// v[N] per lane -> the sum over the wave of v[lane % N]: each step halves the values held and adds the halves exchanged
template <int N, int OFF = N / 2>
__device__ __forceinline__ float wave_sum_scatter(float (&v)[N], int lane) {
  if constexpr (OFF > 0) {
    const bool upper = (lane & OFF) != 0;
#pragma unroll
    for (int c = 0; c < OFF; ++c) {
      const float keep = upper ? v[c + OFF] : v[c], give = upper ? v[c] : v[c + OFF];
      v[c] = keep + __shfl_xor(give, OFF, 64);
    }
    return wave_sum_scatter<N, OFF / 2>(v, lane);
  } else {
    float sum = v[0];
    for (int off = N; off < 64; off <<= 1) sum += __shfl_xor(sum, off, 64);
    return sum;
  }
}

template <class T, bool LORA, int ROWS>
__global__ __launch_bounds__(256, 2) void quant_grads_kernel(LayerDims d, const T* __restrict__ W0,
                                                           const T* __restrict__ A, const T* __restrict__ B,
                                                           const float* __restrict__ scale,
                                                           const float* __restrict__ zero, float* __restrict__ dW,
                                                           float* __restrict__ dscale, float* __restrict__ dzero,
                                                           float* __restrict__ dB) {
  __shared__ float dB_sums[4][64];
  __shared__ float b_lds[ROWS][LORA ? 256 : 1];  // the rows of B (rank <= 256)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t p0 = (int64_t)blockIdx.x * ROWS;
  const int64_t G = d.i / d.g;
  const int width = d.g / 4 < 64 ? d.g / 4 : 64;  // lanes that share a group within a step of 256 columns
  const int64_t unit = d.g > 256 ? d.g : 256;
  int64_t row[ROWS];  // rows past the end repeat the last one and store nothing
#pragma unroll
  for (int q = 0; q < ROWS; ++q) row[q] = p0 + q < d.o ? p0 + q : d.o - 1;

  if (LORA) {
    for (int q = 0; q < ROWS; ++q)
      for (int k = threadIdx.x; k < d.r; k += 256) b_lds[q][k] = load1(B + row[q] * d.r + k);
    __syncthreads();
  }

  // pass 0 does everything for LoRA ranks 0..15; further passes only add dB for ranks 16.., re-reading
  // the already masked dW.
  for (int k0 = 0; k0 < (LORA ? d.r : 1); k0 += QG_KCHUNK) {
    const int kn = d.r - k0 < QG_KCHUNK ? d.r - k0 : QG_KCHUNK;
    float dBacc[ROWS * QG_KCHUNK];
#pragma unroll
    for (int k = 0; k < ROWS * QG_KCHUNK; ++k) dBacc[k] = 0.f;
    for (int64_t u0 = wave * unit; u0 < d.i; u0 += 4 * unit) {
      float ds[ROWS] = {}, db[ROWS] = {};
      for (int64_t base = u0; base < u0 + unit && base < d.i; base += 256) {
        const int64_t j0 = base + lane * 4;
        const bool active = j0 < d.i;
        const int64_t jc = active ? j0 : 0;
        float g4[ROWS][4];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) load4(dW + row[q] * d.i + jc, g4[q]);
        if (k0 == 0) {
          const int64_t grp = jc / d.g;
          float w0[ROWS][4], s[ROWS], b[ROWS], acc[ROWS][4];
#pragma unroll
          for (int q = 0; q < ROWS; ++q) {
            load4(W0 + row[q] * d.i + jc, w0[q]);
            s[q] = scale[row[q] * G + grp];
            b[q] = zero[row[q] * G + grp];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[q][c] = 0.f;
          }
          if (LORA) {  // rank sums, k ascending
            const T* ap = A + jc;
#pragma unroll 8
            for (int k = 0; k < d.r; ++k, ap += d.i) {
              float a[4];
              load4(ap, a);
#pragma unroll
              for (int q = 0; q < ROWS; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[q][c] = lora_mac<T>(acc[q][c], b_lds[q][k], a[c]);
            }
          }
#pragma unroll
          for (int q = 0; q < ROWS; ++q) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float wc = LORA ? w0[q][c] + d.gamma * acc[q][c] : w0[q][c];
              const QuantOut qo = quantize_elem(wc, s[q], b[q], d.qn, d.qp);
              const float gv = active ? g4[q][c] : 0.f;
              ds[q] = fmaf(gv, qo.in_range ? qo.code - qo.w : qo.code, ds[q]);
              db[q] += qo.in_range ? 0.f : gv;
              g4[q][c] = qo.in_range ? gv : 0.f;
            }
            if (LORA && active && p0 + q < d.o) store4(dW + row[q] * d.i + jc, g4[q]);
          }
        }
        if (LORA) {
          const T* ap = A + (int64_t)k0 * d.i + jc;
#pragma unroll
          for (int k = 0; k < QG_KCHUNK; ++k) {
            float a[4];
            load4(ap, a);
            ap += k + 1 < kn ? d.i : 0;  // (ranks past the last repeat it: those sums are not stored)
#pragma unroll
            for (int q = 0; q < ROWS; ++q)
#pragma unroll
              for (int c = 0; c < 4; ++c)
                dBacc[q * QG_KCHUNK + k] = fmaf(active ? g4[q][c] : 0.f, a[c], dBacc[q * QG_KCHUNK + k]);
          }
        }
        if (k0 == 0 && (d.g <= 256 || base + 256 >= u0 + unit)) {  // the end of the lanes' groups
#pragma unroll
          for (int q = 0; q < ROWS; ++q) {
            const float ds_sum = wave_sum_width(ds[q], width), db_sum = wave_sum_width(db[q], width);
            if (active && (lane & (width - 1)) == 0 && p0 + q < d.o) {
              const int64_t at = row[q] * G + j0 / d.g;
              dscale[at] = d.accumulate ? dscale[at] + ds_sum : ds_sum;
              dzero[at] = d.accumulate ? dzero[at] + db_sum : db_sum;
            }
            ds[q] = 0.f;
            db[q] = 0.f;
          }
        }
      }
    }
    if (LORA) {
      dB_sums[wave][lane] = wave_sum_scatter<ROWS * QG_KCHUNK>(dBacc, lane);
      __syncthreads();
      if (wave == 0) {
        const int q = lane / QG_KCHUNK, k = lane % QG_KCHUNK;
        if (q < ROWS && k < kn && p0 + q < d.o) {
          const float v = d.gamma * (((dB_sums[0][lane] + dB_sums[1][lane]) + dB_sums[2][lane]) + dB_sums[3][lane]);
          float* dst = dB + (p0 + q) * d.r + k0 + k;
          *dst = d.accumulate ? *dst + v : v;
        }
      }
      __syncthreads();
    }
  }
}

}  // namespace

// second pass of launch_tn: out[e] = scale * sum_b partial[b * n + e], b ascending
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ partial, int64_t nblocks,
                                                               int64_t n, float scale, float* __restrict__ out,
                                                               bool accumulate) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  float acc = 0.f;
#pragma unroll 8
  for (int64_t b = 0; b < nblocks; ++b) acc += partial[b * n + e];
  out[e] = accumulate ? out[e] + scale * acc : scale * acc;
}

void launch_reduce_partials(const float* partial, int64_t nblocks, int64_t n, float scale, float* out,
                            bool accumulate, hipStream_t stream) {
  hipLaunchKernelGGL(reduce_partials_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, partial,
                     nblocks, n, scale, out, accumulate);
}

__global__ __launch_bounds__(256) void reduce_two_partials_kernel(TwoPartials p) {
  __shared__ float4 slice_sum[3][64];
  reduce_two_block(p, (int)blockIdx.x, slice_sum);
}

void launch_reduce_two_partials(const TwoPartials& p, hipStream_t stream) {
  hipLaunchKernelGGL(reduce_two_partials_kernel, dim3((unsigned)two_partials_blocks(p)), dim3(256), 0, stream, p);
}

// ------------------------------------------------------------------ AdamW step on {A, B, scale, zero}
// One launch over the concatenation [A | B | scale | zero]; the moments m, v are stored in that order.
__global__ __launch_bounds__(256) void adamw_kernel(AdamwArgs a) {
  const int64_t n = a.n[0] + a.n[1] + a.n[2] + a.n[3];
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
    int t = 0;
    int64_t k = e;
    while (k >= a.n[t]) { k -= a.n[t]; ++t; }
    const float g = a.grad[t][k];
    float p = a.param[t][k];
    const float m = a.beta1 * a.m[e] + (1.f - a.beta1) * g;
    const float v = a.beta2 * a.v[e] + (1.f - a.beta2) * g * g;
    a.m[e] = m;
    a.v[e] = v;
    const float mhat = m / a.bias1, vhat = v / a.bias2;
    p = p - a.lr * a.weight_decay * p - a.lr * mhat / (sqrtf(vhat) + a.eps);
    a.param[t][k] = p;
    if (t < 2 && a.copy_bf16[t]) a.copy_bf16[t][k] = f32_to_bf16(p);
  }
}

// The same for tensors whose sizes are all multiples of 4 (every bfloat16 layer): 4 consecutive elements per thread,
// 16-byte accesses.  Bound: memory and a launch (0.9 M elements, 27 MB, of a 4096 x 11008 layer at rank 16: 6.0
// against 6.8 us).
__global__ __launch_bounds__(256) void adamw_quad_kernel(AdamwArgs a) {
  const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  int t = 0;
  int64_t k = e;
  while (t < 4 && k >= a.n[t]) { k -= a.n[t]; ++t; }
  if (t == 4) return;
  float g[4], p[4], m[4], v[4];
  load4(a.grad[t] + k, g);
  load4(a.param[t] + k, p);
  load4(a.m + e, m);
  load4(a.v + e, v);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    m[c] = a.beta1 * m[c] + (1.f - a.beta1) * g[c];
    v[c] = a.beta2 * v[c] + (1.f - a.beta2) * g[c] * g[c];
    const float mhat = m[c] / a.bias1, vhat = v[c] / a.bias2;
    p[c] = p[c] - a.lr * a.weight_decay * p[c] - a.lr * mhat / (sqrtf(vhat) + a.eps);
  }
  store4(a.m + e, m);
  store4(a.v + e, v);
  store4(a.param[t] + k, p);
  if (t < 2 && a.copy_bf16[t]) store4(a.copy_bf16[t] + k, p);
}

void launch_adamw(const AdamwArgs& a, hipStream_t stream) {
  const int64_t n = a.n[0] + a.n[1] + a.n[2] + a.n[3];
  // (the moments are one array for all four tensors: a tensor of any other size would misalign the next one's)
  if (((a.n[0] | a.n[1] | a.n[2] | a.n[3]) & 3) == 0 && n < (1ll << 33)) {  // (one launch's threads)
    hipLaunchKernelGGL(adamw_quad_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, stream, a);
    return;
  }
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(adamw_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a);
}

template <class T>
void launch_quant_grads(const LayerDims& d, const T* W0, const T* A, const T* B, const float* scale,
                        const float* zero, float* dWq_inout, float* dscale, float* dzero, float* dB,
                        hipStream_t stream) {
  // Rows per workgroup: 2, and 1 where 2 leave compute units without a workgroup.  The rank sums and 16 dB sums per row take
  // registers: 2 rows leave 3 waves per SIMD where 4 leave 2.  Forward + backward of a binary32 layer at rank 16, 1 / 2 / 4
  // rows, in us: 4096 x 4096 293 / 275 / 305; 2048 x 2048 111 / 109 / 114; 2048 x 1024 78 / 76 / 88; 2048 x 256 56 / 59 / 68;
  // 256 x 256 at rank 8 33.6 / 34.7 / 38.4.  Unfused backward of a bfloat16 one: 4096 x 4096 152 / 134 / 162, at rank 64
  // 361 / 265 / 345.  Without LoRA terms (this kernel alone, 4096 x 4096): 28.7 / 28.4 / 31.1.
  const int rows = (d.o + 1) / 2 > device_compute_units() ? 2 : 1;
  dim3 grid((unsigned)((d.o + rows - 1) / rows));
#define L4Q_QG_LAUNCH(LORA, ROWS)                                                                                    \
  hipLaunchKernelGGL((quant_grads_kernel<T, LORA, ROWS>), grid, dim3(256), 0, stream, d, W0, A, B, scale, zero, dWq_inout, \
                     dscale, dzero, dB)
  if (dB && rows == 2) L4Q_QG_LAUNCH(true, 2);
  else if (dB) L4Q_QG_LAUNCH(true, 1);
  else if (rows == 2) L4Q_QG_LAUNCH(false, 2);
  else L4Q_QG_LAUNCH(false, 1);
#undef L4Q_QG_LAUNCH
}

template void launch_quant_grads<float>(const LayerDims&, const float*, const float*, const float*, const float*,
                                        const float*, float*, float*, float*, float*, hipStream_t);
template void launch_quant_grads<bf16_t>(const LayerDims&, const bf16_t*, const bf16_t*, const bf16_t*,
                                         const float*, const float*, float*, float*, float*, float*, hipStream_t);

}  // namespace l4q
