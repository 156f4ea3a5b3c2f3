// Coarse-grid MLP on MFMA: forward, backward, Adam (not in the paper; the
// learned stand-in for the exact coarse solve of Alg. fmg).
//
// Model: four dense layers n_in -> H -> H -> H -> n_out, ReLU between them.
// Weights and every layer input are stored in bfloat16 (round to nearest
// even); products run on the bf16 matrix cores with float32 accumulation
// (v_mfma_f32_16x16x32_bf16); biases, pre-activations, master weights and
// Adam moments are float32.  Loss: mean squared error over the n_out outputs.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "kernels.h"
#include "mlp.h"

namespace hhg {

// Adam on float32 masters and moments; pb, pbt: the bf16 copies (p null: none).
struct AdamArgs {
  float *p = nullptr, *m, *v;
  unsigned short *pb, *pbt;
  float lr, b1, b2, eps, c1, c2;
};
// Packing of a minibatch's input features.
struct PackArgs {
  int B = 0, n_in, Kpad;
  const float* X;
  const int* idx;
  unsigned short *A0, *A0T;
  long ldt;
  __host__ __device__ int blocks() const { return ((B + 7) / 8) * ((Kpad + 63) / 64); }
};

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f2bf(float f) {
  unsigned u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (unsigned short)((u >> 16) | 0x40);  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short b) { return __uint_as_float(((unsigned)b) << 16); }

// A training step is a chain of eight small launches, each bound by its latency
// (4 - 6 us against 0.1 us of products): a tile of 16 x 16 per wavefront
// spreads them over the most CUs, everything a tile's epilogue reads is loaded
// before its products, and what can run beside a link of the chain is in its
// launch -- the weight gradients of a layer with the input gradients of the
// layer before, the Adam update in the epilogue of the weight gradients, the
// loss in that of the last layer, the packing of the next minibatch with the
// last gradients.  Step of batch 256, 331 -> 512 -> 512 -> 512 -> 206: 15
// launches 78.7 us -> eight, 58 us.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned short v8us __attribute__((ext_vector_type(8)));

// Elements k .. k + 7 of a row of K, zero beyond it.
__device__ __forceinline__ v8bf load8(const unsigned short* __restrict__ row, int k, int K) {
  v8us v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = k + e < K ? row[k + e] : (unsigned short)0;
  return __builtin_bit_cast(v8bf, v);
}

constexpr int kKSteps = 16;  // 32-wide k steps held in registers at once (k chunk 512)

// One 16 x 16 tile of C[m][n] = sum_k A[m][k] B[n][k] (both operands row-major
// with the contraction index contiguous: lda, ldb in elements, multiples of
// 8), bf16 inputs, float32 sums, per wavefront on v_mfma_f32_16x16x32_bf16:
// lane l holds A row l % 16 and B row l % 16 at k = 8 (l / 16) + 0..7 of each
// 32-wide k step (one 16-byte load per operand; the same k slots for both
// operands, so the product is the full sum over k whatever order the unit adds
// the slots in); result lanes: row 4 (l / 16) + q, column l % 16.  A k tail (K
// not a multiple of 32) is loaded element by element and zero-filled.
// RS: also the row sums of A (row l % 16, in the lanes below 16).
struct GemmOp {
  int M, N, K;
  const unsigned short *A, *B;
  long lda, ldb;
  __host__ __device__ int tiles() const { return ((M + 15) / 16) * ((N + 15) / 16); }
};
__device__ __forceinline__ v4f gemm_tile(const GemmOp& o, int tm, int tn, bool rsum, float& asum) {
  const int lane = threadIdx.x, r = lane & 15, kg = lane >> 4;
  const int m = tm + r, n = tn + r;
  const unsigned short* arow = o.A + (long)min(m, o.M - 1) * o.lda;
  const unsigned short* brow = o.B + (long)min(n, o.N - 1) * o.ldb;
  v4f acc = {0.f, 0.f, 0.f, 0.f};
  asum = 0.f;
  auto product = [&](v8bf a, v8bf b) {
    if (rsum)
#pragma unroll
      for (int e = 0; e < 8; ++e) asum += (float)a[e];
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
  };
  // a whole k chunk of both operands is loaded before the first product, so
  // the wavefront waits for memory once per chunk, not once per step; the k
  // tail apart, so that the steps are two loads each (a checked load in every
  // step was 30 KB of code, fetched cold in every launch)
  const int full = o.K / 32;
  for (int c0 = 0; c0 < full; c0 += kKSteps) {
    v8bf a[kKSteps], b[kKSteps];
#pragma unroll
    for (int st = 0; st < kKSteps; ++st)
      if (c0 + st < full) {
        const int k = 32 * (c0 + st) + 8 * kg;
        a[st] = *reinterpret_cast<const v8bf*>(arow + k);
        b[st] = *reinterpret_cast<const v8bf*>(brow + k);
      }
#pragma unroll
    for (int st = 0; st < kKSteps; ++st)
      if (c0 + st < full) product(a[st], b[st]);
  }
  if (32 * full < o.K) {
    const int k = 32 * full + 8 * kg;
    product(load8(arow, k, o.K), load8(brow, k, o.K));
  }
  // the wait states between the last product and the first read of its result,
  // 16 where 8 are needed (4 passes + 4): the compiler's own were missing on a
  // branch taken right after a product (results of rows 2 and 3 of 4 stale), so
  // no branch but the loop's and the tail's follows one (a row sum's is before
  // it), and both lead here.  The assembly is checked by tests/test_mfma_waits.py.
  asm volatile("s_nop 15" : "+a"(acc));
  if (rsum) {  // sum over the four k lane groups of row r
    asum += __shfl_xor(asum, 16);
    asum += __shfl_xor(asum, 32);
  }
  return acc;
}

// h[q] = words of rows mm + q, q < 4, of column n: into T[n][mm + q]
// (leading dimension ldt, a multiple of 16; mm a multiple of 4), rows < M.
__device__ __forceinline__ void store_t(unsigned short* T, long ldt, int n, int mm, int M,
                                        const unsigned short (&h)[4]) {
  unsigned short* to = T + n * ldt + mm;
  if (mm + 4 <= M) {
    *reinterpret_cast<v4s*>(to) = v4s{(short)h[0], (short)h[1], (short)h[2], (short)h[3]};
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (mm + q < M) to[q] = h[q];
  }
}

// Forward layer: Z = A W^T + bias; act != null: act = bf16(relu(Z)), actT the
// same transposed (leading dimension ldt); out != null: out = Z.  y != null
// (the last layer of a training step): the mean squared error against rows
// idx[m] (null: m) of y, n_out columns: G = bf16(2 (Z - y) / (M n_out)) (0 in
// padded columns), GT transposed, the tile's sum of squares in partial.
struct FwdArgs {
  GemmOp o;
  const float* bias;
  float* out;
  unsigned short *act, *actT;
  long ldt;
  const float* y;
  const int* idx;
  int n_out;
  unsigned short *G, *GT;
  double* partial;
};
__global__ void __launch_bounds__(64) k_forward(FwdArgs f) {
  const int lane = threadIdx.x, kg = lane >> 4;
  // tiles down a column first: the four tiles that share the 128-byte lines of a
  // row of results then run on one XCD where the rows' tiles are a multiple of
  // 8 (forward of 331 -> 512 -> 512 -> 512 -> 206, batch 1024: 42.8 us along the
  // rows, 37.7 down the columns; training the same either way)
  const int tm = (int)blockIdx.x * 16, tn = (int)blockIdx.y * 16;
  const int n = tn + (lane & 15), mm = tm + 4 * kg, N = f.o.N, M = f.o.M;
  const float bias = f.bias[min(n, N - 1)];
  float yv[4] = {0.f, 0.f, 0.f, 0.f};
  if (f.y && n < f.n_out)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = min(mm + q, M - 1);
      yv[q] = f.y[(f.idx ? (long)f.idx[m] : (long)m) * f.n_out + n];
    }
  float unused;
  const v4f acc = gemm_tile(f.o, tm, tn, false, unused);
  unsigned short h[4];
  double loss = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool in = mm + q < M && n < N;
    const long at = (long)(mm + q) * N + n;
    const float z = acc[q] + bias;
    if (f.out && in) f.out[at] = z;
    float v = fmaxf(z, 0.f);
    if (f.y) {
      v = 0.f;
      if (in && n < f.n_out) {
        const float d = z - yv[q];
        loss += (double)d * d;
        v = 2.f * d / (float)(M * f.n_out);
      }
    }
    h[q] = f2bf(v);
    unsigned short* w = f.y ? f.G : f.act;
    if (w && in) w[at] = h[q];
  }
  unsigned short* t = f.y ? f.GT : f.actT;
  if (t && n < N) store_t(t, f.ldt, n, mm, M, h);
  if (f.y) {
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) loss += __shfl_xor(loss, k);
    if (lane == 0) f.partial[blockIdx.x * gridDim.y + blockIdx.y] = loss;
  }
}

// One Adam step of a parameter with gradient g; its new value.
__device__ __forceinline__ float adam(const AdamArgs& a, long t, float p, float m, float v, float g) {
  const float mm = fmaf(1.f - a.b1, g, a.b1 * m);
  const float vv = fmaf(g, (1.f - a.b2) * g, a.b2 * v);
  a.m[t] = mm;
  a.v[t] = vv;
  const float w = p - a.lr * (mm / a.c1) / (sqrtf(vv / a.c2) + a.eps);
  a.p[t] = w;
  a.pb[t] = f2bf(w);
  return w;
}

// Weight gradient of a layer, dW[n][k] = sum_b GT[n][b] aT[k][b], and its bias
// gradient, the row sums of GT (from the tiles of the first column): stored at
// grad + woff, grad + boff, or (adam.p != null) applied at once, in the
// parameters, their bf16 copies and the transposed copies (at woff, rows x
// cols transposed).
struct WgradArgs {
  GemmOp o;
  long woff, boff;
};
__device__ __forceinline__ void wgrad_tile(const WgradArgs& w, float* __restrict__ grad, const AdamArgs& ad, int tile) {
  const int lane = threadIdx.x, kg = lane >> 4, r = lane & 15;
  const int nt = (w.o.N + 15) / 16, tm = (tile / nt) * 16, tn = (tile % nt) * 16;
  const int n = tn + r, mm = tm + 4 * kg, N = w.o.N, M = w.o.M;
  float p[4] = {}, m[4] = {}, v[4] = {}, pr = 0.f, mr = 0.f, vr = 0.f;
  const bool rsum = tn == 0, rs = rsum && kg == 0 && tm + r < M;
  if (ad.p) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const long t = w.woff + (long)min(mm + q, M - 1) * N + min(n, N - 1);
      p[q] = ad.p[t], m[q] = ad.m[t], v[q] = ad.v[t];
    }
    if (rs) pr = ad.p[w.boff + tm + r], mr = ad.m[w.boff + tm + r], vr = ad.v[w.boff + tm + r];
  }
  float asum;
  const v4f acc = gemm_tile(w.o, tm, tn, rsum, asum);
  if (rs) {
    if (ad.p)
      adam(ad, w.boff + tm + r, pr, mr, vr, asum);
    else
      grad[w.boff + tm + r] = asum;
  }
  if (n >= N) return;
  unsigned short h[4] = {0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (mm + q >= M) continue;
    const long t = w.woff + (long)(mm + q) * N + n;
    if (ad.p)
      h[q] = f2bf(adam(ad, t, p[q], m[q], v[q], acc[q]));
    else
      grad[t] = acc[q];
  }
  if (ad.p) store_t(ad.pbt + w.woff, M, n, mm, M, h);
}

// Input gradient of a layer and the ReLU backward of the layer before:
// dA[b][k] = sum_n G[b][n] WT[k][n]; gout[b][k] = bf16(dA (mask[b][k] > 0)),
// goutT the same transposed.
struct XgradArgs {
  GemmOp o;
  const unsigned short* mask;
  unsigned short *gout, *goutT;
  long ldt;
};
__device__ __forceinline__ void xgrad_tile(const XgradArgs& x, int tile) {
  const int lane = threadIdx.x, kg = lane >> 4;
  const int nt = (x.o.N + 15) / 16, tm = (tile / nt) * 16, tn = (tile % nt) * 16;
  const int n = tn + (lane & 15), mm = tm + 4 * kg, N = x.o.N, M = x.o.M;
  unsigned short mk[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) mk[q] = x.mask[(long)min(mm + q, M - 1) * N + min(n, N - 1)];
  float unused;
  const v4f acc = gemm_tile(x.o, tm, tn, false, unused);
  if (n >= N) return;
  unsigned short h[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    h[q] = f2bf(bf2f(mk[q]) > 0.f ? acc[q] : 0.f);
    if (mm + q < M) x.gout[(long)(mm + q) * N + n] = h[q];
  }
  store_t(x.goutT, x.ldt, n, mm, M, h);
}

// Input features (float32, rows idx[b] of X, null: b) -> bf16, padded to Kpad
// columns, and (A0T != null) transposed into A0T[k][b] (leading dimension
// ldt).  A block takes 8 rows of 64 columns.
__device__ __forceinline__ void pack_block(const PackArgs& a, int blk) {
  const int nk = (a.Kpad + 63) / 64, b0 = (blk / nk) * 8, k = (blk % nk) * 64 + (int)threadIdx.x;
  if (k >= a.Kpad) return;
  v8us h;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int b = min(b0 + e, a.B - 1);
    const long row = a.idx ? a.idx[b] : b;  // sample row of the data set (minibatch gather)
    h[e] = k < a.n_in ? f2bf(a.X[row * a.n_in + k]) : (unsigned short)0;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (b0 + e < a.B) {
      a.A0[(long)(b0 + e) * a.Kpad + k] = h[e];
      if (a.A0T && b0 + 8 > a.B) a.A0T[k * a.ldt + b0 + e] = h[e];
    }
  if (a.A0T && b0 + 8 <= a.B) *reinterpret_cast<v8us*>(a.A0T + k * a.ldt + b0) = h;
}
__global__ void __launch_bounds__(64) k_pack_input(PackArgs a) { pack_block(a, (int)blockIdx.x); }

// One link of the backward chain: by block, the tiles of an input gradient, of
// up to two weight gradients, the loss sum (acc[0] += scale sum of the tiles'
// partials, fixed order) and the packing of the next minibatch.
struct BwdArgs {
  XgradArgs x;
  WgradArgs w[2];
  int nx, nw[2], npart, npack;  // blocks of each part (npart > 0: one block for the loss)
  float* grad;
  AdamArgs adam;
  const double* partial;
  double scale;
  double* acc;
  PackArgs pack;
};
__global__ void __launch_bounds__(64) k_backward(BwdArgs a) {
  int q = (int)blockIdx.x;
  if (q < a.nx) {
    xgrad_tile(a.x, q);
    return;
  }
  q -= a.nx;
  if (q < a.nw[0] + a.nw[1]) {
    const bool first = q < a.nw[0];
    wgrad_tile(first ? a.w[0] : a.w[1], a.grad, a.adam, first ? q : q - a.nw[0]);
    return;
  }
  q -= a.nw[0] + a.nw[1];
  if (q < a.npack) {
    pack_block(a.pack, q);
    return;
  }
  double l = 0.0;
  for (int i = threadIdx.x; i < a.npart; i += 64) l += a.partial[i];
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) l += __shfl_xor(l, k);
  if (threadIdx.x == 0) a.acc[0] += l * a.scale;
}

// out[c][r] = in[r][c] for the four weight matrices (bf16, blockIdx.y =
// layer): the transposed copies feed the input-gradient products.
__global__ void k_transpose_w(WShapes w, const unsigned short* __restrict__ in, unsigned short* __restrict__ out) {
  const int l = blockIdx.y;
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n = (long)w.rows[l] * w.cols[l];
  if (t >= n) return;
  const int r = (int)(t / w.cols[l]), c = (int)(t % w.cols[l]);
  out[w.off[l] + (long)c * w.rows[l] + r] = in[w.off[l] + t];
}

// Output (B x Npad float32) -> y (B x n_out float32).
__global__ void k_unpack_output(int B, int n_out, int Npad, const float* __restrict__ Z, float* __restrict__ y) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= B * n_out) return;
  y[t] = Z[(t / n_out) * Npad + t % n_out];
}

__global__ void k_fill_f64(double* __restrict__ x, int n) {
  if ((int)threadIdx.x < n) x[threadIdx.x] = 0.0;
}

__global__ void k_to_bf16(long n, const float* __restrict__ p, unsigned short* __restrict__ pb) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) pb[t] = f2bf(p[t]);
}

unsigned nb(long n, int b = 256) { return (unsigned)((n + b - 1) / b); }
int pad16(int n) { return (n + 15) & ~15; }

}  // namespace

// ------------------------------------------------------------------ host
Mlp::~Mlp() {
  for (void* p : allocs) (void)hipFree(p);
}

void Mlp::init(int in, int H, int out, int max_b) {
  n_in = in, hidden = H, n_out = out, max_batch = max_b;
  kin = pad16(in), kout = pad16(out), bpad = pad16(max_b);
  rows[0] = H, cols[0] = kin;
  rows[1] = H, cols[1] = H;
  rows[2] = H, cols[2] = H;
  rows[3] = kout, cols[3] = H;
  nparams_dev = 0;
  for (int l = 0; l < 4; ++l) {
    woff[l] = nparams_dev;
    nparams_dev += (long)rows[l] * cols[l];
    boff[l] = nparams_dev;
    nparams_dev += rows[l];
  }
  auto al = [&](size_t bytes) {
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, bytes ? bytes : 4);
    if (e != hipSuccess) throw Error{HHG_ERR_OOM, "hipMalloc (mlp)"};
    allocs.push_back(p);
    HHG_CHECK_HIP(hipMemset(p, 0, bytes ? bytes : 4));
    return p;
  };
  P = (float*)al(nparams_dev * 4);
  Gr = (float*)al(nparams_dev * 4);
  Mo = (float*)al(nparams_dev * 4);
  Vo = (float*)al(nparams_dev * 4);
  Pb = (unsigned short*)al(nparams_dev * 2);
  PbT = (unsigned short*)al(nparams_dev * 2);
  for (int q = 0; q < 2; ++q) {
    A0[q] = (unsigned short*)al((size_t)bpad * kin * 2);
    A0T[q] = (unsigned short*)al((size_t)bpad * kin * 2);
  }
  Zout = (float*)al((size_t)bpad * kout * 4);
  for (int l = 0; l < 4; ++l) {
    G[l] = (unsigned short*)al((size_t)bpad * rows[l] * 2);
    GT[l] = (unsigned short*)al((size_t)bpad * rows[l] * 2);
    if (l < 3) {
      Ab[l] = (unsigned short*)al((size_t)bpad * rows[l] * 2);
      AbT[l] = (unsigned short*)al((size_t)bpad * rows[l] * 2);
    }
  }
  partial = (double*)al(sizeof(double) * ((size_t)bpad * kout / 256 + 2));
  loss_acc = (double*)al(sizeof(double) * 2);
  step = 0;
}

long Mlp::host_params() const {
  long n = 0;
  const int r[4] = {hidden, hidden, hidden, n_out}, c[4] = {n_in, hidden, hidden, hidden};
  for (int l = 0; l < 4; ++l) n += (long)r[l] * c[l] + r[l];
  return n;
}

void Mlp::set_params(const float* host) {
  std::vector<float> dev(nparams_dev, 0.f);
  const int r[4] = {hidden, hidden, hidden, n_out}, c[4] = {n_in, hidden, hidden, hidden};
  long q = 0;
  for (int l = 0; l < 4; ++l) {
    for (int i = 0; i < r[l]; ++i)
      for (int j = 0; j < c[l]; ++j) dev[woff[l] + (long)i * cols[l] + j] = host[q++];
    for (int i = 0; i < r[l]; ++i) dev[boff[l] + i] = host[q++];
  }
  HHG_CHECK_HIP(hipMemcpy(P, dev.data(), nparams_dev * 4, hipMemcpyHostToDevice));
  HHG_CHECK_HIP(hipMemset(Mo, 0, nparams_dev * 4));
  HHG_CHECK_HIP(hipMemset(Vo, 0, nparams_dev * 4));
  hipLaunchKernelGGL(k_to_bf16, dim3(nb(nparams_dev)), dim3(256), 0, 0, nparams_dev, P, Pb);
  transpose_weights(0);
  HHG_CHECK_HIP(hipDeviceSynchronize());
  step = 0;
}

void Mlp::unpack(const float* dev_vec, float* host) const {
  std::vector<float> dev(nparams_dev);
  HHG_CHECK_HIP(hipMemcpy(dev.data(), dev_vec, nparams_dev * 4, hipMemcpyDeviceToHost));
  const int r[4] = {hidden, hidden, hidden, n_out}, c[4] = {n_in, hidden, hidden, hidden};
  long q = 0;
  for (int l = 0; l < 4; ++l) {
    for (int i = 0; i < r[l]; ++i)
      for (int j = 0; j < c[l]; ++j) host[q++] = dev[woff[l] + (long)i * cols[l] + j];
    for (int i = 0; i < r[l]; ++i) host[q++] = dev[boff[l] + i];
  }
}

void Mlp::transpose_weights(hipStream_t s) {
  long mx = 0;
  for (int l = 0; l < 4; ++l) mx = std::max(mx, (long)rows[l] * cols[l]);
  hipLaunchKernelGGL(k_transpose_w, dim3(nb(mx), 4), dim3(256), 0, s, shapes(), Pb, PbT);
}

WShapes Mlp::shapes() const {
  WShapes w;
  for (int l = 0; l < 4; ++l) {
    w.off[l] = woff[l];
    w.rows[l] = rows[l];
    w.cols[l] = cols[l];
  }
  return w;
}

PackArgs Mlp::pack_args(const float* x, const int* idx, int B, bool train, int buf) const {
  return PackArgs{B, n_in, kin, x, idx, A0[buf], train ? A0T[buf] : nullptr, (long)bpad};
}

// Forward layers on the packed input of buffer buf: y == null: the output in
// Zout; else (training) the transposed activations and the output gradient.
void Mlp::forward_layers(hipStream_t s, int B, int buf, const float* y, const int* idx) {
  const unsigned short* a = A0[buf];
  int ka = kin;
  for (int l = 0; l < 4; ++l) {
    // Z[b][n] = sum_k a[b][k] W[n][k] + bias[n]; hidden layers: Ab = bf16(relu(Z))
    // (padded output columns: zero weights and bias, so Z = 0 there)
    FwdArgs f{};
    f.o = GemmOp{B, rows[l], ka, a, Pb + woff[l], (long)ka, (long)cols[l]};
    f.bias = P + boff[l];
    f.ldt = bpad;
    if (l < 3) {
      f.act = Ab[l];
      f.actT = y ? AbT[l] : nullptr;
    } else if (y) {
      f.y = y, f.idx = idx, f.n_out = n_out, f.G = G[3], f.GT = GT[3], f.partial = partial;
    } else {
      f.out = Zout;
    }
    KScope ks(s, KF_MLP, 2.0 * B * rows[l] * ka);
    hipLaunchKernelGGL(k_forward, dim3((B + 15) / 16, (rows[l] + 15) / 16), dim3(64), 0, s, f);
    if (l < 3) {
      a = Ab[l];
      ka = rows[l];
    }
  }
}

void Mlp::forward(hipStream_t s, const float* x, int B, float* y) {
  const PackArgs pk = pack_args(x, nullptr, B, false, 0);
  hipLaunchKernelGGL(k_pack_input, dim3(pk.blocks()), dim3(64), 0, s, pk);
  forward_layers(s, B, 0, nullptr, nullptr);
  hipLaunchKernelGGL(k_unpack_output, dim3(nb((long)B * n_out)), dim3(256), 0, s, B, n_out, kout, Zout, y);
}

// Loss and gradients of the minibatch packed in buffer buf: into Gr, or with
// adam.p applied at once; next.B > 0: packs the next minibatch on the way.
void Mlp::loss_grad_dev(hipStream_t s, const float* y, const int* idx, int B, int buf, double* loss_acc,
                        const AdamArgs& adam, const PackArgs& next) {
  forward_layers(s, B, buf, y, idx);
  // launch l: the input gradients of layer l beside the weight gradients of the
  // layer after it (an update there must not touch weights that are still read)
  for (int l = 3; l >= 0; --l) {
    BwdArgs a{};
    double work = 0.0;
    a.grad = Gr;
    a.adam = adam;
    auto wgrad = [&](int q, int i) {
      // dW[n][k] = sum_b G[b][n] a[b][k] = sum_b GT[n][b] aT[k][b]; db[n] = sum_b GT[n][b]
      const int ka = q > 0 ? rows[q - 1] : kin;
      a.w[i].o = GemmOp{rows[q], ka, B, GT[q], q > 0 ? AbT[q - 1] : A0T[buf], (long)bpad, (long)bpad};
      a.w[i].woff = woff[q], a.w[i].boff = boff[q];
      a.nw[i] = a.w[i].o.tiles();
      work += 2.0 * rows[q] * ka * B;
    };
    if (l > 0) {
      a.x = XgradArgs{GemmOp{B, rows[l - 1], rows[l], G[l], PbT + woff[l], (long)rows[l], (long)rows[l]}, Ab[l - 1],
                      G[l - 1], GT[l - 1], (long)bpad};
      a.nx = a.x.o.tiles();
      work += 2.0 * B * rows[l - 1] * rows[l];
    }
    if (l < 3) wgrad(l + 1, 0);
    if (l == 0) wgrad(0, 1);
    if (l == 3) {
      a.npart = ((B + 15) / 16) * ((kout + 15) / 16);
      a.partial = partial, a.scale = 1.0 / ((double)B * n_out), a.acc = loss_acc;
    }
    if (l == 0 && next.B > 0) {
      a.pack = next;
      a.npack = next.blocks();
    }
    KScope ks(s, KF_MLP, work);
    hipLaunchKernelGGL(k_backward, dim3(a.nx + a.nw[0] + a.nw[1] + a.npack + (a.npart > 0)), dim3(64), 0, s, a);
  }
}

double Mlp::loss_grad(hipStream_t s, const float* x, const float* y, int B) {
  hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, loss_acc, 2);
  const PackArgs pk = pack_args(x, nullptr, B, true, 0);
  hipLaunchKernelGGL(k_pack_input, dim3(pk.blocks()), dim3(64), 0, s, pk);
  loss_grad_dev(s, y, nullptr, B, 0, loss_acc, AdamArgs{}, PackArgs{});
  double l = 0.0;
  HHG_CHECK_HIP(hipMemcpyAsync(&l, loss_acc, sizeof(double), hipMemcpyDeviceToHost, s));
  HHG_CHECK_HIP(hipStreamSynchronize(s));
  return l;
}

void Mlp::train_dev(hipStream_t s, const float* x, const float* y, int n_samples, int batch, int epochs, float lr,
                    const int* order, double* loss) {
  const int per = n_samples / batch;
  const long total = (long)epochs * per;
  auto rows_of = [&](long q) { return order + (q / per) * n_samples + (q % per) * batch; };
  const PackArgs first = pack_args(x, rows_of(0), batch, true, 0);
  hipLaunchKernelGGL(k_pack_input, dim3(first.blocks()), dim3(64), 0, s, first);
  for (long q = 0; q < total; ++q) {
    ++step;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - std::pow(b1, (float)step), c2 = 1.f - std::pow(b2, (float)step);
    const int buf = (int)(q & 1);
    loss_grad_dev(s, y, rows_of(q), batch, buf, loss + q / per, AdamArgs{P, Mo, Vo, Pb, PbT, lr, b1, b2, 1e-8f, c1, c2},
                  q + 1 < total ? pack_args(x, rows_of(q + 1), batch, true, buf ^ 1) : PackArgs{});
  }
}

}  // namespace hhg
