// Bandwidth-bound row movement around the expert GEMMs: gather into
// expert-contiguous order, gate-weighted combine (Eq. 2), and their backward
// counterparts.  All traffic is 16-byte vectors along the contiguous feature
// dimension; sums run in fp32 in a fixed slot order and are rounded once.
#include "kernels.h"
#include "lds_load.h"

namespace spes {
namespace {

// xp[inv[t*k+j], :] = x[t, :] for j < k: every input row is read once and written to its k places
template <typename T>
__global__ __launch_bounds__(256) void permute_kernel(const T* __restrict__ x, const int* __restrict__ inv, int k,
                                                      T* __restrict__ xp, long total_vec, int nvec, int d) {
  constexpr int N = Vec16<T>::N;
  const long stride = (long)gridDim.x * 256;
  for (long v = (long)blockIdx.x * 256 + threadIdx.x; v < total_vec; v += stride) {
    const long t = v / nvec;
    const int c = (int)(v - t * nvec);
    Vec16<T> q;
    q.load_once(x + t * d + c * N);
    for (int j = 0; j < k; ++j) {
      const long r = inv[t * k + j];
      q.store_once(xp + r * d + c * N);
    }
  }
}

// y[t,:] = sum_j gate[t,j] * yp[inv[t*k+j], :]; KU > 0: k == KU, all k rows are requested before the first is used
template <typename T, int KU>
__global__ __launch_bounds__(256) void combine_kernel(const T* __restrict__ yp, const int* __restrict__ inv,
                                                      const float* __restrict__ gate, T* __restrict__ y, long total_vec,
                                                      int nvec, int d, int k) {
  constexpr int N = Vec16<T>::N;
  const long stride = (long)gridDim.x * 256;
  for (long v = (long)blockIdx.x * 256 + threadIdx.x; v < total_vec; v += stride) {
    const long t = v / nvec;
    const int c = (int)(v - t * nvec);
    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.f;
    if (KU > 0) {
      Vec16<T> q[KU > 0 ? KU : 1];
      float g[KU > 0 ? KU : 1];
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        const long r = inv[t * KU + j];
        g[j] = gate[t * KU + j];
        q[j].load_once(yp + r * d + c * N);
      }
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        float f[N];
        q[j].unpack(f);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = fmaf(g[j], f[i], acc[i]);
      }
    } else {
      for (int j = 0; j < k; ++j) {
        const long r = inv[t * k + j];
        const float g = gate[t * k + j];
        Vec16<T> q;
        q.load_once(yp + r * d + c * N);
        float f[N];
        q.unpack(f);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = fmaf(g, f[i], acc[i]);
      }
    }
    Vec16<T> o;
    o.pack(acc);
    o.store_once(y + t * d + c * N);
  }
}

// out[i] (+)= sum_p partial[p*n + i], p ascending: four elements per thread, n a multiple of four.  The partials are requested eight at a
// time: one after the other, each load waited for, 32 of them took 10 to 12 us for a 32 x 2048 gradient.  (The router weight
// gradient's sum is the work of a few blocks and has nothing to do with dx: they run ahead of the dx blocks in one launch.  As a launch of its
// own it was 5 us.)
struct Partials {
  const float* partial;
  float* out;
  long n;
  int n_partial, accumulate, blocks;       // 256 threads each
};
__device__ __forceinline__ void reduce_partials(const Partials& r) {
  const long i = ((long)blockIdx.x * 256 + threadIdx.x) * 4, n = r.n;
  if (i >= n) return;
  constexpr int U = 8;
  const float4 acc = r.accumulate ? *reinterpret_cast<const float4*>(r.out + i) : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](const float4& v) { sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w; };
  int p = 0;
  for (; p + U <= r.n_partial; p += U) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4*>(r.partial + (long)(p + u) * n + i);
#pragma unroll
    for (int u = 0; u < U; ++u) add(v[u]);
  }
  for (; p < r.n_partial; ++p) add(*reinterpret_cast<const float4*>(r.partial + (long)p * n + i));
  *reinterpret_cast<float4*>(r.out + i) = make_float4(acc.x + sum.x, acc.y + sum.y, acc.z + sum.z, acc.w + sum.w);
}

// dx[t,:] = sum_j dxp[inv[t*k+j], :] + sum_e dlogits[t,e] * w_router[e,:]; one block per token
template <typename T>
__global__ __launch_bounds__(256) void dx_gather_kernel(const T* __restrict__ dxp, const int* __restrict__ inv,
                                                        const float* __restrict__ dlogits, const T* __restrict__ w_router,
                                                        T* __restrict__ dx, int d, int k, int M, const Partials red) {
  if ((int)blockIdx.x < red.blocks) { reduce_partials(red); return; }
  constexpr int N = Vec16<T>::N;
  __shared__ float dl[kMaxExperts];
  __shared__ int rows[kMaxExperts];
  const long t = (int)blockIdx.x - red.blocks;
  if (threadIdx.x < M) dl[threadIdx.x] = dlogits[t * M + threadIdx.x];
  if (threadIdx.x < k) rows[threadIdx.x] = inv[t * k + threadIdx.x];
  __syncthreads();
  const int nvec = d / N;
  for (int c = threadIdx.x; c < nvec; c += 256) {
    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.f;
    for (int j = 0; j < k; ++j) {
      Vec16<T> q;
      q.load_once(dxp + (long)rows[j] * d + c * N);
      float f[N];
      q.unpack(f);
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] += f[i];
    }
    for (int e = 0; e < M; ++e) {
      Vec16<T> q;
      q.load(w_router + (long)e * d + c * N);
      float f[N];
      q.unpack(f);
      const float s = dl[e];
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] = fmaf(s, f[i], acc[i]);
    }
    Vec16<T> o;
    o.pack(acc);
    o.store_once(dx + t * d + c * N);
  }
}

// The same in bf16 storage with the router part on the matrix cores, from the bf16 copy of dlogits (M a multiple of 8): a block takes 256
// columns of `tokens` tokens, sixteen at a time.  A wavefront's 64 columns of W_r go through LDS once, into fragments that stay in registers;
// its product of sixteen tokens goes through LDS, as a value of the storage type, to the 32 lanes that hold a token's 512 bytes of dxp.
// Up to eight rows of a token (KU) are all requested before the product is formed, further ones (MORE) eight at a time, with their
// places in dxp known by then.  Bound by the bytes of dxp and dx.  (As a GEMM of its own the product was written and read once more, and cost a
// launch, and the sum of dW_r's partials another.)  Where d is no multiple of 64, rows begin within a 128-byte line, and two wavefronts
// read the line between them: with eight lanes to a row every second one, and a streaming load drops it for the other.  So a row is 32 lanes
// wide, and such rows (LINES false) come by plain loads, which cost 4 to 15 % where d is a multiple.  The router's products, the sum and dx, in us: as
// launches of their own / one launch, eight lanes to a row, rows one by one where k is not 1, 2, 4 or 8 / now
//   64 experts, 20000 tokens x 520   k = 4: 72 / 58 / 47     k = 7: 84 / 107 / 65    k = 8: 85 / 87 / 72     k = 16: 131 / 210 / 129
//   16384 x 2056                     k = 4: 143 / 169 / 133  k = 7: 190 / 250 / 186  k = 8: 196 / 265 / 193  k = 16: 305 / 418 / 299
//   16384 x 2048                     k = 4: 128 / 102 / 102  k = 7: 172 / 199 / 147  k = 8: 180 / 161 / 162  k = 16: 279 / 364 / 271
//   1531 x 512                       k = 4: 24 / 16 / 16     k = 7: 25 / 24 / 18     k = 8: 25 / 18 / 18     k = 16: 27 / 35 / 21
template <int KU, bool MORE, bool LINES>
__global__ __launch_bounds__(256) void dx_router_kernel(const bf16_t* __restrict__ dxp, const int* __restrict__ inv,
                                                        const bf16_t* __restrict__ dlogits, const bf16_t* __restrict__ w_router,
                                                        bf16_t* __restrict__ dx, int T, int d, int k, int M, int tokens, int col_blocks, const Partials red) {
  if ((int)blockIdx.x < red.blocks) { reduce_partials(red); return; }
  constexpr int WP = 72, OP = 264;                 // pitches of a wavefront's panel of W_r and of a token's product over the block's columns
  __shared__ __attribute__((aligned(16))) bf16_t lds[4 * 64 * WP];       // the four panels, then two sets of products in turn
  static_assert(2 * 16 * OP <= 4 * 64 * WP, "the products take the panels' place");
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int block = (int)blockIdx.x - red.blocks, tile = block / col_blocks;
  const int c0 = (block - tile * col_blocks) * 256, w0 = c0 + wave * 64;
  bf16_t* const w = lds + wave * 64 * WP;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int e = i * 8 + (lane >> 3), col = w0 + (lane & 7) * 8;
    *reinterpret_cast<uint4*>(w + e * WP + (lane & 7) * 8) =
        e < M && col < d ? *reinterpret_cast<const uint4*>(w_router + (long)e * d + col) : make_uint4(0, 0, 0, 0);
  }
  wave_lds_order();
  bf16x8 fw[4][2];                                 // column l16 of the panel's sixteen columns j, experts s*32 + lq*8 .. +7
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const bf16_t* const p = w + (s * 32 + lq * 8 + (l16 >> 2)) * WP + j * 16 + (lane & 3) * 4;
      const uint2 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * WP);
      fw[j][s] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
    }
  __syncthreads();
  // lanes to a token's row, as a power of two: 32, in the last columns as few as cover them
  const int width = d - c0 < 256 ? d - c0 : 256, lanes = width > 128 ? 5 : width > 64 ? 4 : 3;
  const int cl = (tid & ((1 << lanes) - 1)) * 8, c = c0 + cl;
  const int t_first = tile * tokens, t_end = t_first + tokens < T ? t_first + tokens : T;
  for (int t0 = t_first; t0 < t_end; t0 += 16) {
    bf16_t* const out = lds + ((t0 - t_first) & 16 ? 16 * OP : 0);
    // the lane's two tokens, KU of their rows of dxp
    Vec16<bf16_t> q[2][KU];
    int row[2][KU], tok[2];
    bool live[2];
    auto find = [&](int first) {
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int j = 0; j < KU; ++j) row[v][j] = live[v] && (!MORE || first + j < k) ? inv[(long)tok[v] * (MORE ? k : KU) + first + j] : -1;
    };
    auto request = [&]() {
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int j = 0; j < KU; ++j) {
          const bf16_t* const p = dxp + (long)row[v][j] * d + c;
          if (row[v][j] < 0) q[v][j].raw = make_uint4(0, 0, 0, 0);
          else if (LINES) q[v][j].load_once(p);
          else q[v][j].load(p);
        }
    };
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int at = (v << (8 - lanes)) + (tid >> lanes);
      tok[v] = t0 + at;
      live[v] = at < 16 && tok[v] < t_end && c < d;
    }
    find(0);
    bf16x8 fl[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const bool in = t0 + l16 < t_end && s * 32 + lq * 8 < M;
      fl[s] = __builtin_bit_cast(bf16x8, in ? *reinterpret_cast<const uint4*>(dlogits + (long)(t0 + l16) * M + s * 32 + lq * 8) : make_uint4(0, 0, 0, 0));
    }
    request();
    if (MORE) find(KU);
    // prod[j][r] = the product of token l16 and column j*16 + lq*4 + r
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 prod = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 2; ++s) prod = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j][s], fl[s], prod, 0, 0, 0);
      *reinterpret_cast<uint2*>(out + l16 * OP + wave * 64 + j * 16 + lq * 4) = make_uint2(pack_bf16x2(prod[0], prod[1]), pack_bf16x2(prod[2], prod[3]));
    }
    __syncthreads();                               // (the products' other half is written when all have read it: behind the next of these)
    float acc[2][8];
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[v][i] = 0.f;
    auto add = [&](int v, const Vec16<bf16_t>& x) {
      float f[8];
      x.unpack(f);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[v][i] += f[i];
    };
    auto add_rows = [&]() {
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int j = 0; j < KU; ++j) add(v, q[v][j]);
    };
    add_rows();
    if (MORE)
      for (int first = KU; first < k; first += KU) {
        request();
        find(first + KU);
        add_rows();
      }
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      if (!live[v]) continue;
      Vec16<bf16_t> r, o;
      r.raw = *reinterpret_cast<const uint4*>(out + (tok[v] - t0) * OP + cl);
      add(v, r);
      o.pack(acc[v]);
      o.store_once(dx + (long)tok[v] * d + c);
    }
  }
}

// Backward of the weighted combine as a stand-alone step: for the k routed pairs of token t,
// dyp[inv[t*k+j], :] = gate[t,j] * dy[t, :] and dgate[t,j] = <dy[t, :], yp[inv[t*k+j], :]>.  One block per token: the
// token's dy row is read once and its k scaled copies written, the k rows of yp are read once for the dots.
// KU > 0: k == KU, the thread's k rows of yp are all requested before the first is used.
template <typename T, int KU>
__global__ __launch_bounds__(256) void grad_scatter_kernel(const T* __restrict__ dy, const T* __restrict__ yp,
                                                           const int* __restrict__ inv, const float* __restrict__ gate,
                                                           T* __restrict__ dyp, float* __restrict__ dgate, int d, int k) {
  constexpr int N = Vec16<T>::N;
  __shared__ int rows[kMaxExperts];
  __shared__ float gts[kMaxExperts];
  __shared__ float part[kMaxExperts][4];
  const long t = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid < k) { rows[tid] = inv[t * k + tid]; gts[tid] = gate[t * k + tid]; }
  __syncthreads();
  const int nvec = d / N;
  if (KU > 0) {
    float dots[KU > 0 ? KU : 1];
#pragma unroll
    for (int j = 0; j < KU; ++j) dots[j] = 0.f;
    for (int c = tid; c < nvec; c += 256) {
      Vec16<T> q, qy[KU > 0 ? KU : 1];
      q.load_once(dy + t * d + c * N);
#pragma unroll
      for (int j = 0; j < KU; ++j) qy[j].load_once(yp + (long)rows[j] * d + c * N);
      float g[N];
      q.unpack(g);
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        float f[N], o[N];
        qy[j].unpack(f);
#pragma unroll
        for (int i = 0; i < N; ++i) { dots[j] = fmaf(g[i], f[i], dots[j]); o[i] = gts[j] * g[i]; }
        Vec16<T> w;
        w.pack(o);
        w.store_once(dyp + (long)rows[j] * d + c * N);
      }
    }
#pragma unroll
    for (int j = 0; j < KU; ++j) {
      const float v = wave_sum(dots[j]);
      if (lane == 0) part[j][wv] = v;
    }
  } else {
    for (int j = 0; j < k; ++j) {
      float dot = 0.f;
      for (int c = tid; c < nvec; c += 256) {
        Vec16<T> q, qy;
        q.load(dy + t * d + c * N);                    // read again for the next pair: from the cache
        qy.load_once(yp + (long)rows[j] * d + c * N);
        float g[N], f[N], o[N];
        q.unpack(g);
        qy.unpack(f);
#pragma unroll
        for (int i = 0; i < N; ++i) { dot = fmaf(g[i], f[i], dot); o[i] = gts[j] * g[i]; }
        Vec16<T> w;
        w.pack(o);
        w.store_once(dyp + (long)rows[j] * d + c * N);
      }
      const float v = wave_sum(dot);
      if (lane == 0) part[j][wv] = v;
    }
  }
  __syncthreads();
  if (tid < k) dgate[t * k + tid] = (part[tid][0] + part[tid][1]) + (part[tid][2] + part[tid][3]);   // fixed order
}

inline int flat_grid(long total_vec) {
  long b = (total_vec + 255) / 256;       // one vector per thread where the grid allows it
  if (b < 1) b = 1;
  if (b > 1 << 20) b = 1 << 20;
  return (int)b;
}

inline int ok() { return hipGetLastError() == hipSuccess ? SPES_OK : SPES_EHIP; }

}  // namespace

int launch_permute(int dtype, const void* x, const int* inv, int k, void* xp, int T, int d, hipStream_t s) {
  if (dtype == SPES_F32) {
    const int nvec = d / 4;
    hipLaunchKernelGGL(permute_kernel<float>, dim3(flat_grid((long)T * nvec)), dim3(256), 0, s, (const float*)x, inv, k, (float*)xp,
                       (long)T * nvec, nvec, d);
  } else {
    const int nvec = d / 8;
    hipLaunchKernelGGL(permute_kernel<bf16_t>, dim3(flat_grid((long)T * nvec)), dim3(256), 0, s, (const bf16_t*)x, inv, k,
                       (bf16_t*)xp, (long)T * nvec, nvec, d);
  }
  return ok();
}

template <typename T>
void combine_dispatch(const void* yp, const int* inv, const float* gate, void* y, int Tn, int d, int k, hipStream_t s) {
  const int nvec = d / Vec16<T>::N;
  const long total = (long)Tn * nvec;
  const dim3 grid(flat_grid(total));
#define SPES_COMBINE(KU) \
  hipLaunchKernelGGL((combine_kernel<T, KU>), grid, dim3(256), 0, s, (const T*)yp, inv, gate, (T*)y, total, nvec, d, k)
  if (k == 8) SPES_COMBINE(8);
  else if (k == 4) SPES_COMBINE(4);
  else if (k == 2) SPES_COMBINE(2);
  else if (k == 1) SPES_COMBINE(1);
  else SPES_COMBINE(0);
#undef SPES_COMBINE
}

int launch_combine(int dtype, const void* yp, const int* inv, const float* gate, void* y, int T, int d, int k, hipStream_t s) {
  if (dtype == SPES_F32) combine_dispatch<float>(yp, inv, gate, y, T, d, k, s);
  else combine_dispatch<bf16_t>(yp, inv, gate, y, T, d, k, s);
  return ok();
}

template <typename T>
void grad_scatter_dispatch(const void* dy, const void* yp, const int* inv, const float* gate, void* dyp, float* dgate, int Tn,
                           int d, int k, hipStream_t s) {
#define SPES_SCATTER(KU) \
  hipLaunchKernelGGL((grad_scatter_kernel<T, KU>), dim3(Tn), dim3(256), 0, s, (const T*)dy, (const T*)yp, inv, gate, (T*)dyp, dgate, d, k)
  if (k == 8) SPES_SCATTER(8);
  else if (k == 4) SPES_SCATTER(4);
  else if (k == 2) SPES_SCATTER(2);
  else if (k == 1) SPES_SCATTER(1);
  else SPES_SCATTER(0);
#undef SPES_SCATTER
}

int launch_grad_scatter(int dtype, const void* dy, const void* yp, const int* inv, const float* gate, void* dyp, float* dgate,
                        int T, int d, int k, hipStream_t s) {
  if (dtype == SPES_F32) grad_scatter_dispatch<float>(dy, yp, inv, gate, dyp, dgate, T, d, k, s);
  else grad_scatter_dispatch<bf16_t>(dy, yp, inv, gate, dyp, dgate, T, d, k, s);
  return ok();
}

int launch_dx_gather(int dtype, const void* dxp, const int* inv, const float* dlogits, const bf16_t* dlogits_bf, const void* w_router,
                     void* dx, int T, int d, int k, int M, const float* partial, int n_partial, float* d_w_router, int accumulate,
                     hipStream_t s) {
  const long n = (long)M * d;
  const Partials red = {partial, d_w_router, n, n_partial, accumulate, cdiv(n, 1024)};
  if (dlogits_bf != nullptr) {
    // tokens per block: as many as leave four blocks per CU, so that W_r's panel is read for few of them only where tokens are few
    const int cols = cdiv(d, 256);
    int tokens = 64;
    while (tokens > 16 && (long)cdiv(T, tokens) * cols < 1024) tokens /= 2;
    const long blocks = (long)cdiv(T, tokens) * cols + red.blocks;
    if (blocks > 0x7fffffffL) return SPES_ESHAPE;
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, (const bf16_t*)dxp, inv, dlogits_bf, (const bf16_t*)w_router,
                         (bf16_t*)dx, T, d, k, M, tokens, cols, red);
    };
#define SPES_DX(KU, MORE) \
  if (d % 64 == 0) launch(dx_router_kernel<KU, MORE, true>); else launch(dx_router_kernel<KU, MORE, false>)
    switch (k) {
      case 1: SPES_DX(1, false); break;
      case 2: SPES_DX(2, false); break;
      case 3: SPES_DX(3, false); break;
      case 4: SPES_DX(4, false); break;
      case 5: SPES_DX(5, false); break;
      case 6: SPES_DX(6, false); break;
      case 7: SPES_DX(7, false); break;
      case 8: SPES_DX(8, false); break;
      default: SPES_DX(8, true);
    }
#undef SPES_DX
  } else if (dtype == SPES_F32) {
    hipLaunchKernelGGL(dx_gather_kernel<float>, dim3(T + red.blocks), dim3(256), 0, s, (const float*)dxp, inv, dlogits,
                       (const float*)w_router, (float*)dx, d, k, M, red);
  } else {
    hipLaunchKernelGGL(dx_gather_kernel<bf16_t>, dim3(T + red.blocks), dim3(256), 0, s, (const bf16_t*)dxp, inv, dlogits,
                       (const bf16_t*)w_router, (bf16_t*)dx, d, k, M, red);
  }
  return ok();
}

}  // namespace spes
