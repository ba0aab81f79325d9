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

// The same in bf16 storage with the router part on the matrix cores, from the bf16 copy of dlogits (M a multiple of 8): a wavefront takes 64
// columns of `tokens` tokens, sixteen at a time.  Its panel of W_r goes through LDS once, into fragments that stay in registers; the
// product of sixteen tokens is turned through LDS to where a token's row segment, 128 bytes of dxp, belongs to eight lanes.
// The product is rounded to bf16 before it is added: a token's router part is a value of the storage type, as when it was a GEMM's result.
// The k rows of a token are all requested before the product is formed (KU > 0: k == KU).  Bound by the bytes of dxp and dx.  (As
// a GEMM of its own the product was written and read once more, and cost a launch, and the sum of dW_r's partials another: steps
// of 3777 tokens 1536 x 1280 307 -> 296 us, 1531 tokens 512 x 352 151 -> 148, 16384 tokens 2048 x 1024 3727 -> 3667, 32768 tokens 4096 x
// 1408 16.74 -> 16.63 ms.)
template <int KU>
__global__ __launch_bounds__(256) void dx_router_kernel(const bf16_t* __restrict__ dxp, const int* __restrict__ inv,
                                                        const bf16_t* __restrict__ dlogits, const bf16_t* __restrict__ w_router,
                                                        bf16_t* __restrict__ dx, int T, int d, int k, int M, int tokens, int col_blocks, const Partials red) {
  if ((int)blockIdx.x < red.blocks) { reduce_partials(red); return; }
  constexpr int WP = 72;                           // pitch of a row of W_r's panel, and of a token's product, which take its place
  __shared__ __attribute__((aligned(16))) bf16_t panel[4][64 * WP];
  const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6), l16 = lane & 15, lq = lane >> 4;
  const int block = (int)blockIdx.x - red.blocks, tile = block / col_blocks;
  const int c0 = (block - tile * col_blocks) * 256 + wave * 64, c = c0 + (lane & 7) * 8;
  if (c0 >= d) return;                             // (the wavefronts of a block never meet)
  const bool c_in = c < d;
  bf16_t* const w = panel[wave];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int e = i * 8 + (lane >> 3);
    *reinterpret_cast<uint4*>(w + e * WP + (lane & 7) * 8) =
        e < M && c_in ? *reinterpret_cast<const uint4*>(w_router + (long)e * d + c) : make_uint4(0, 0, 0, 0);
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
  wave_lds_order();
  const int t_first = tile * tokens, t_end = t_first + tokens < T ? t_first + tokens : T;
  for (int t0 = t_first; t0 < t_end; t0 += 16) {
    // the lane's two tokens, their rows of dxp
    constexpr int KV = KU > 0 ? KU : 1;
    Vec16<bf16_t> q[2][KV];
    long row[2][KV];
    int tok[2];
    bool live[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      tok[v] = t0 + v * 8 + (lane >> 3);
      live[v] = tok[v] < t_end && c_in;
#pragma unroll
      for (int j = 0; j < KU; ++j) row[v][j] = live[v] ? inv[(long)tok[v] * KU + j] : -1;
    }
    bf16x8 fl[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const bool in = t0 + l16 < t_end && s * 32 + lq * 8 < M;
      fl[s] = __builtin_bit_cast(bf16x8, in ? *reinterpret_cast<const uint4*>(dlogits + (long)(t0 + l16) * M + s * 32 + lq * 8) : make_uint4(0, 0, 0, 0));
    }
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int j = 0; j < KU; ++j)
        if (live[v]) q[v][j].load_once(dxp + row[v][j] * d + c); else q[v][j].raw = make_uint4(0, 0, 0, 0);
    // prod[j][r] = the product of token l16 and column j*16 + lq*4 + r
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 prod = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 2; ++s) prod = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j][s], fl[s], prod, 0, 0, 0);
      *reinterpret_cast<uint2*>(w + l16 * WP + j * 16 + lq * 4) = make_uint2(pack_bf16x2(prod[0], prod[1]), pack_bf16x2(prod[2], prod[3]));
    }
    wave_lds_order();
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      float acc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = 0.f;
      auto add = [&](const Vec16<bf16_t>& x) {
        float f[8];
        x.unpack(f);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += f[i];
      };
      if (KU > 0) {
#pragma unroll
        for (int j = 0; j < KU; ++j) add(q[v][j]);
      } else if (live[v]) {
        for (int j = 0; j < k; ++j) {
          q[v][0].load_once(dxp + (long)inv[(long)tok[v] * k + j] * d + c);
          add(q[v][0]);
        }
      }
      Vec16<bf16_t> r;
      r.raw = *reinterpret_cast<const uint4*>(w + (v * 8 + (lane >> 3)) * WP + (lane & 7) * 8);
      add(r);
      Vec16<bf16_t> o;
      o.pack(acc);
      if (live[v]) o.store_once(dx + (long)tok[v] * d + c);
    }
    wave_lds_order();
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
    // tokens per wavefront: as many as leave four blocks per CU, so that W_r's panel is read for few of them only where tokens are few
    const int cols = cdiv(d, 256);
    int tokens = 64;
    while (tokens > 16 && (long)cdiv(T, tokens) * cols < 1024) tokens /= 2;
    const long blocks = (long)cdiv(T, tokens) * cols + red.blocks;
    if (blocks > 0x7fffffffL) return SPES_ESHAPE;
#define SPES_DX(KU) \
  hipLaunchKernelGGL(dx_router_kernel<KU>, dim3((unsigned)blocks), dim3(256), 0, s, (const bf16_t*)dxp, inv, dlogits_bf, \
                     (const bf16_t*)w_router, (bf16_t*)dx, T, d, k, M, tokens, cols, red)
    switch (k) {
      case 1: SPES_DX(1); break;
      case 2: SPES_DX(2); break;
      case 4: SPES_DX(4); break;
      case 8: SPES_DX(8); break;
      default: SPES_DX(0);
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
