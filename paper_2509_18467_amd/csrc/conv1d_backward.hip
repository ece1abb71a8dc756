// Adjoint of the causal depthwise conv with its pointwise feature map (paper section 4.1; the layer-wise
// distillation of section 5 trains the conv weights through it):
//   u_t = sum_{dl < W} w[dl] x_{t-dl},   y_t = phi(u_t),   du_t = dy_t phi'(u_t)   (phi' = 1, or for 1 + ELU: 1 if u > 0, else e^u)
//   dx_s = sum_{dl < W} w[dl] du_{s+dl},   dw[dl] = sum_{b,t} du_t x_{t-dl},   rows before the first token: dhalo like dx
// u is recomputed from x (one more pass of W multiply-adds beats reading a stored copy).  Streaming: a thread owns
// four adjacent channels and walks a run of tokens (plus the W - 1 tokens after it, whose du the run's last dx need)
// with x and du of the last W tokens in registers, rows of x and dy travelling four at a time, one group ahead of the
// arithmetic; 6 bytes per element moved in bf16 storage.  A strip of 64 tokens is cut into 1, 4 or 16 runs, walked by as many
// threads of the same workgroup.  dw: every (batch, strip) writes its partial sums to the workspace (those of its runs
// added through LDS, in order), a second kernel adds them, each thread a share and the shares in order (no atomics:
// repeated calls agree bit for bit).
//
// What bounds it: HBM where there is enough to do.  32768 tokens of 32 / 8 heads of 64, bf16, both kernels: 98 / 30 us, 4.4 and
// 3.6 TB/s with the partial sums; a thread per strip, one row in flight, took 109 / 80.  Groups of 2 or 8 rows instead of 4, one
// or two threads per strip, nontemporal stores: the same within 3 %, or slower.
#include "kernels.h"

namespace lawcat {
namespace {

constexpr int kStrip = 64;

struct f4 { float v[4]; };
__device__ inline f4 ld4(const float* p) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  return {{t.x, t.y, t.z, t.w}};
}
__device__ inline f4 ld4(const bf16_t* p) {
  const uint2 t = *reinterpret_cast<const uint2*>(p);
  return {{__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16),
           __uint_as_float(t.y & 0xffff0000u)}};
}
__device__ inline void st4(float* p, const f4& a) { *reinterpret_cast<float4*>(p) = make_float4(a.v[0], a.v[1], a.v[2], a.v[3]); }
__device__ inline uint32_t pack2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 h = {(__bf16)a, (__bf16)b};  // round to nearest even
  return __builtin_bit_cast(uint32_t, h);
}
__device__ inline void st4(bf16_t* p, const f4& a) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack2(a.v[0], a.v[1]), pack2(a.v[2], a.v[3]));
}

// rows travel as stored
__device__ inline f4 unpack(const float4& t) { return {{t.x, t.y, t.z, t.w}}; }
__device__ inline f4 unpack(const uint2& t) {
  return {{__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16),
           __uint_as_float(t.y & 0xffff0000u)}};
}
template <typename T> struct RawOf;
template <> struct RawOf<float> { typedef float4 type; };
template <> struct RawOf<bf16_t> { typedef uint2 type; };

constexpr int kGroup = 4;   // rows fetched together, one group ahead of the arithmetic

// grid (ceil(row / (1024 / NSUB)), strips, B), 256 threads = 256 / NSUB groups of four channels x NSUB runs of a strip's tokens;
// row = H * d channels of a token.
// WHOLE (up to four strips in all, as launch_phi() says): grid (ceil(row / 32)), 512 threads = 8 groups of four channels x all strips' runs of 4 tokens; `partial` is
// dw itself, added up in the order of the two kernels (the same bits).  A second launch for so few sums took as long as the first:
// 100 tokens of two heads, fp32, the training pass 83.3 -> 79.7 us, 256 96.0 -> 94.3; 200 of 32 / 8, bf16, 80.7 -> 79.4.  For more strips a
// workgroup's columns are too narrow for its 512 threads: 8 strips, 500 tokens of 4 / 2 125.0 / 126.8, 16, 1000 of 32 / 8 98.3 / 117.6.
template <typename T, int W, int PHI, int NSUB, bool WHOLE = false>
__global__ void __launch_bounds__(WHOLE ? 512 : 256) conv_bwd_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                      const T* __restrict__ halo, const T* __restrict__ dy,
                                                      T* __restrict__ dx, T* __restrict__ dhalo,
                                                      float* __restrict__ partial, int Tn, int row, int strips = 0, int n_partial = 0) {
  constexpr int COLS = WHOLE ? 8 : 256 / NSUB, RUN = kStrip / NSUB;
  typedef typename RawOf<T>::type Raw;
  const int col = threadIdx.x % COLS, sub = threadIdx.x / COLS;
  const int e0 = (blockIdx.x * COLS + col) * 4;
  const int all = WHOLE ? sub / NSUB : 0;      // of all sequences' strips
  const int b = WHOLE ? all / strips : blockIdx.z, strip = WHOLE ? all - b * strips : blockIdx.y;
  const int t0 = strip * kStrip + (WHOLE ? sub % NSUB : sub) * RUN, t1 = min(Tn, t0 + RUN);
  const bool active = e0 < row && t0 < Tn && (!WHOLE || all < n_partial);

  float dw[4][W];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int dl = 0; dl < W; ++dl) dw[i][dl] = 0.f;
  if (active) {
    const T* xb = x + (size_t)b * Tn * row + e0;
    const T* yb = dy + (size_t)b * Tn * row + e0;
    T* db = dx + (size_t)b * Tn * row + e0;
    const int t_end = t1 + W - 1, t_in = min(t_end, Tn);
    Raw nx[kGroup], ny[kGroup];
    auto fetch = [&](int t) {
#pragma unroll
      for (int r = 0; r < kGroup; ++r) {
        nx[r] = Raw{};
        ny[r] = Raw{};
        if (t + r < t_in) {
          nx[r] = *reinterpret_cast<const Raw*>(xb + (size_t)(t + r) * row);
          ny[r] = *reinterpret_cast<const Raw*>(yb + (size_t)(t + r) * row);
        }
      }
    };
    fetch(t0);
    float wv[4][W];
    if constexpr (W == 4) {   // the 4 x 4 taps of this thread's channels are contiguous
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f4 t = ld4(w + (size_t)(e0 + i) * 4);
#pragma unroll
        for (int dl = 0; dl < 4; ++dl) wv[i][dl] = t.v[dl];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int dl = 0; dl < W; ++dl)
          wv[i][dl] = sizeof(T) == 2 ? __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(w)[(size_t)(e0 + i) * W + dl] << 16)
                                     : reinterpret_cast<const float*>(w)[(size_t)(e0 + i) * W + dl];
    }
    // xw[j] = x_{t-j}, du[j] = du_{t-j} of the token t being worked on
    f4 xw[W], du[W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
      xw[j] = {{0.f, 0.f, 0.f, 0.f}};
      du[j] = {{0.f, 0.f, 0.f, 0.f}};
    }
#pragma unroll
    for (int j = 1; j < W; ++j) {   // history of the run's first token: x_{t0-j} goes to xw[j-1], shifted below
      const int s = t0 - j;
      if (s >= 0) xw[j - 1] = ld4(xb + (size_t)s * row);
      else if (halo != nullptr) xw[j - 1] = ld4(halo + ((size_t)b * (W - 1) + (W - 1 + s)) * row + e0);
    }
#pragma unroll 1
    for (int tg = t0; tg < t_end; tg += kGroup) {
      Raw cx[kGroup], cy[kGroup];
#pragma unroll
      for (int r = 0; r < kGroup; ++r) { cx[r] = nx[r]; cy[r] = ny[r]; }
      if (tg + kGroup < t_in) fetch(tg + kGroup);
#pragma unroll
      for (int r = 0; r < kGroup; ++r) {
        const int t = tg + r;
        if (t >= t_end) break;
#pragma unroll
        for (int j = W - 1; j >= 1; --j) {
          xw[j] = xw[j - 1];
          du[j] = du[j - 1];
        }
        f4 d0 = {{0.f, 0.f, 0.f, 0.f}};
        xw[0] = d0;
        if (t < Tn) {
          xw[0] = unpack(cx[r]);
          const f4 g = unpack(cy[r]);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float u = 0.f;
#pragma unroll
            for (int dl = 0; dl < W; ++dl) u = fmaf(wv[i][dl], xw[dl].v[i], u);
            d0.v[i] = PHI == 1 ? (u > 0.f ? g.v[i] : g.v[i] * __expf(u)) : g.v[i];
          }
        }
        du[0] = d0;
        if (t < t1) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int dl = 0; dl < W; ++dl) dw[i][dl] = fmaf(d0.v[i], xw[dl].v[i], dw[i][dl]);
        }
        // dx of token s = t - (W - 1) is complete now
        const int s = t - (W - 1);
        f4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float acc = 0.f;
#pragma unroll
          for (int dl = 0; dl < W; ++dl) acc = fmaf(wv[i][dl], du[W - 1 - dl].v[i], acc);
          o.v[i] = acc;
        }
        if (s >= t0) st4(db + (size_t)s * row, o);
        else if (s < 0 && dhalo != nullptr) st4(dhalo + ((size_t)b * (W - 1) + (W - 1 + s)) * row + e0, o);
      }
    }
  }
  if constexpr (WHOLE) {
    constexpr int N = COLS * 4 * W;      // sums
    __shared__ float sums[512 * 4 * W], strip_sums[4 * N];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int dl = 0; dl < W; ++dl) sums[threadIdx.x * 4 * W + i * W + dl] = dw[i][dl];
    __syncthreads();
    for (int k = threadIdx.x; k < n_partial * N; k += 512) {
      const int q = k / N, e = k % N;
      float acc = 0.f;
#pragma unroll
      for (int j = 0; j < NSUB; ++j) acc += sums[(q * NSUB + j) * N + e];
      strip_sums[k] = acc;
    }
    __syncthreads();
    const int first = blockIdx.x * N + threadIdx.x;
    if (threadIdx.x < N && first < row * W) {
      float acc = strip_sums[threadIdx.x];
      for (int q = 1; q < n_partial; ++q) acc += strip_sums[q * N + threadIdx.x];
      partial[first] = acc;
    }
    return;
  }
  float* out = partial + ((size_t)b * gridDim.y + strip) * row * W;
  if constexpr (NSUB == 1) {      // a thread's own 4 W sums are contiguous
    if (!active) return;
#pragma unroll
    for (int v = 0; v < W; ++v) {
      f4 t;
#pragma unroll
      for (int i = 0; i < 4; ++i) t.v[i] = dw[(4 * v + i) / W][(4 * v + i) % W];
      st4(out + (size_t)e0 * W + 4 * v, t);
    }
    return;
  }
  // the strip's runs, in order
  __shared__ float sums[256 * 4 * W];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int dl = 0; dl < W; ++dl) sums[threadIdx.x * 4 * W + i * W + dl] = dw[i][dl];
  __syncthreads();
  const int first = blockIdx.x * COLS * 4 * W, n = row * W;
  for (int e = threadIdx.x; e < COLS * 4 * W; e += 256) {
    if (first + e >= n) break;
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < NSUB; ++j) acc += sums[j * COLS * 4 * W + e];
    out[first + e] = acc;
  }
}

// dw[e] = sum of the partial sums: 32 threads per four elements take a contiguous share of them each, in (batch, strip) order,
// then the shares are added in order.  n is a multiple of 32 (64 channels at least).  One thread per element walked 512
// partial sums in 64 dependent rounds, 22 us for 8192 or 2048 elements; this takes 5.
constexpr int kShares = 32;
__global__ void __launch_bounds__(256) conv_bwd_reduce_kernel(const float* __restrict__ partial, float* __restrict__ dw,
                                                             int n_partial, int n) {
  __shared__ float sums[kShares][32];
  const int lane = threadIdx.x & 7, share = threadIdx.x >> 3;
  const int e0 = blockIdx.x * 32 + lane * 4;
  const int per = (n_partial + kShares - 1) / kShares;
  const int p0 = share * per, p1 = min(n_partial, p0 + per);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p = p0; p < p1; p += 8) {
    float4 t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      t[u] = p + u < p1 ? *reinterpret_cast<const float4*>(partial + (size_t)(p + u) * n + e0) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 8; ++u) { acc.x += t[u].x; acc.y += t[u].y; acc.z += t[u].z; acc.w += t[u].w; }
  }
  *reinterpret_cast<float4*>(&sums[share][lane * 4]) = acc;
  __syncthreads();
  if (threadIdx.x < 32) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < kShares; ++j) s += sums[j][threadIdx.x];
    dw[blockIdx.x * 32 + threadIdx.x] = s;
  }
}

// The same for up to 16 partial sums: four elements per thread, all loads at once (8 sequences of up to 4 tokens, 2 heads of 64: the
// call 6.0 us with the shares).
constexpr int kFewPartials = 16;
__global__ void __launch_bounds__(64) conv_bwd_sum_kernel(const float* __restrict__ partial, float* __restrict__ dw, int n_partial, int n) {
  const int e0 = (blockIdx.x * 64 + threadIdx.x) * 4;
  if (e0 >= n) return;
  float4 t[kFewPartials];
#pragma unroll
  for (int p = 0; p < kFewPartials; ++p)
    t[p] = p < n_partial ? *reinterpret_cast<const float4*>(partial + (size_t)p * n + e0) : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 acc = t[0];
#pragma unroll
  for (int p = 1; p < kFewPartials; ++p) { acc.x += t[p].x; acc.y += t[p].y; acc.z += t[p].z; acc.w += t[p].w; }
  *reinterpret_cast<float4*>(dw + e0) = acc;
}

template <typename T, int W, int PHI, int NSUB>
void launch_kernel(const ConvBackwardParams& p, float* partial, int row, int strips, hipStream_t stream) {
  const int cols = 256 / NSUB;
  hipLaunchKernelGGL((conv_bwd_kernel<T, W, PHI, NSUB>), dim3((row / 4 + cols - 1) / cols, strips, p.B), dim3(256), 0, stream,
                     (const T*)p.x, (const T*)p.w, (const T*)p.halo, (const T*)p.dy, (T*)p.dx, (T*)p.dhalo, partial, p.T, row, 0, 0);
}

template <typename T, int W, int PHI>
hipError_t launch_phi(const ConvBackwardParams& p, hipStream_t stream) {
  const int row = p.H * p.d;
  const int strips = (p.T + kStrip - 1) / kStrip, n_partial = p.B * strips, n = row * W;
  float* partial = n_partial == 1 ? p.dw : static_cast<float*>(p.workspace);   // a single strip: its sums are the result
  // Runs of 16 tokens (4 of the strip's threads per four channels), or of 4 where those would leave most of the chip idle: the
  // W - 1 tokens that a run reads and works out a second time cost more than the latency they hide at 128K channels x strips and
  // above (bf16, runs of 4 / 16, 2048 channels of 64 sequences of 64 tokens 21.5 / 17.5 us, of 8 of 200 12.3 / 14.1).  A thread
  // walks a strip of up to 4 tokens alone (64 sequences of one token: 7.3 us, 9.4 in runs of 4), and a longer one, shorter than a
  // whole strip, where that fills the chip: short sequences leave most runs empty (256 sequences, 2048 channels, bf16, 17 and 32
  // tokens 19.6 and 30.2 us, in runs of 16 26.1 and 33.4; from 64 on the same).
  const long long work = (long long)row * n_partial;
  // One launch as long as its workgroups find a place at once: one a compute unit with three taps or four, two with one or two.  us, two
  // launches / one: 8192 channels, 4 taps, 250 tokens 8.5 / 7.1, 9216 9.7 / 11.9, 24576, 128 tokens 10.1 / 15.8; 16384, 2 taps, 250 tokens 8.9 / 8.7,
  // 24576, 190 tokens 9.8 / 12.4.
  if (p.T > 4 && n_partial > 1 && n_partial <= 4 && work < 96 * 1024 && row <= (W <= 2 ? 16384 : 8192)) {
    hipLaunchKernelGGL((conv_bwd_kernel<T, W, PHI, 16, true>), dim3((row / 4 + 7) / 8), dim3(512), 0, stream, (const T*)p.x, (const T*)p.w,
                       (const T*)p.halo, (const T*)p.dy, (T*)p.dx, (T*)p.dhalo, p.dw, p.T, row, strips, n_partial);
    return hipGetLastError();
  }
  if (p.T <= 4 || (p.T < kStrip && work * (int)sizeof(T) >= 1 << 20)) launch_kernel<T, W, PHI, 1>(p, partial, row, strips, stream);
  else if (work >= 96 * 1024) launch_kernel<T, W, PHI, 4>(p, partial, row, strips, stream);
  else launch_kernel<T, W, PHI, 16>(p, partial, row, strips, stream);
  if (n_partial > kFewPartials)
    hipLaunchKernelGGL(conv_bwd_reduce_kernel, dim3(n / 32), dim3(256), 0, stream, partial, p.dw, n_partial, n);
  else if (n_partial > 1)
    hipLaunchKernelGGL(conv_bwd_sum_kernel, dim3((n / 4 + 63) / 64), dim3(64), 0, stream, partial, p.dw, n_partial, n);
  return hipGetLastError();
}

template <typename T, int W>
hipError_t launch_w(const ConvBackwardParams& p, hipStream_t stream) {
  return p.phi == 1 ? launch_phi<T, W, 1>(p, stream) : launch_phi<T, W, 0>(p, stream);
}

template <typename T>
hipError_t launch_t(const ConvBackwardParams& p, hipStream_t stream) {
  switch (p.W) {
    case 1: return launch_w<T, 1>(p, stream);
    case 2: return launch_w<T, 2>(p, stream);
    case 3: return launch_w<T, 3>(p, stream);
    case 4: return launch_w<T, 4>(p, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

size_t conv_backward_workspace_bytes(int B, int T, int H, int d, int W) {
  return (size_t)B * ((T + kStrip - 1) / kStrip) * H * d * W * sizeof(float);
}

hipError_t launch_conv_backward(const ConvBackwardParams& p, hipStream_t stream) {
  return p.bf16 ? launch_t<bf16_t>(p, stream) : launch_t<float>(p, stream);
}

}  // namespace lawcat
