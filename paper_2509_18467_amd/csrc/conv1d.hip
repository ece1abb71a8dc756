// Causal depthwise Conv1D across tokens (paper section 4.1, the sum over delta):
//   y[b,t,h,c] = phi( sum_{delta<W} w[h,c,delta] * x[b,t-delta,h,c] )
// Streaming kernel: each thread owns one 16-byte column group of a row and slides a
// register window down a strip of tokens, so every row is fetched from HBM once and
// the W-1 rows above a strip are the only re-reads (they hit L2).  Rows are contiguous
// H*d elements, so consecutive lanes read consecutive 16-byte pieces.
#include "kernels.h"

namespace lawcat {
namespace {

constexpr int kGroup = 4;   // rows fetched together, one group ahead of the arithmetic

template <typename T> struct Io;
template <> struct Io<float> {
  static constexpr int VEC = 4;
  typedef float4 Raw;
  __device__ static Raw load_raw(const float* p) { return *reinterpret_cast<const float4*>(p); }
  __device__ static Raw zero_raw() { return make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ static void unpack(const Raw& r, float (&f)[VEC]) { f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w; }
  __device__ static void load(const float* p, float (&f)[VEC]) {
    float4 r = *reinterpret_cast<const float4*>(p);
    f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w;
  }
  __device__ static void store(float* p, const float (&f)[VEC]) {
    *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
  }
  __device__ static float scalar(const float* p) { return *p; }
};
template <> struct Io<bf16_t> {
  static constexpr int VEC = 8;
  typedef uint4 Raw;
  __device__ static Raw load_raw(const bf16_t* p) { return *reinterpret_cast<const uint4*>(p); }
  __device__ static Raw zero_raw() { return make_uint4(0u, 0u, 0u, 0u); }
  __device__ static void unpack(const Raw& r, float (&f)[VEC]) {
    const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(u[i] << 16);
      f[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
    }
  }
  __device__ static void load(const bf16_t* p, float (&f)[VEC]) {
    uint4 r = *reinterpret_cast<const uint4*>(p);
    uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(u[i] << 16);
      f[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
    }
  }
  __device__ static uint32_t pack(float a, float b) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    bf2 v = {(__bf16)a, (__bf16)b};  // round to nearest even
    return __builtin_bit_cast(uint32_t, v);
  }
  __device__ static void store(bf16_t* p, const float (&f)[VEC]) {
    uint4 r;
    r.x = pack(f[0], f[1]); r.y = pack(f[2], f[3]); r.z = pack(f[4], f[5]); r.w = pack(f[6], f[7]);
    *reinterpret_cast<uint4*>(p) = r;
  }
  __device__ static float scalar(const bf16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }
};

__device__ inline float apply_phi(float x, int phi) {
  if (phi == 1) return x > 0.f ? 1.f + x : __expf(x);
  return x;
}

// kStrip: tokens per thread (see launch_typed).  The thread of a sequence's last strip also writes the conv cache for a
// continuation, whose rows it requests before anything else where a strip is one group (in a longer one they would take registers
// from a wave in four: 32 heads of 128, bf16, 8100 tokens 26.4 us, requested at the end 24.3): one launch instead of two (a decode step's conv, 32 heads of 64:
// 6.2 -> 4.2 us, and 3.2 with divisions of 32 bits and no arithmetic for rows past the end; 256 sequences, 32 heads of 128: 14.4 -> 6.2 -> 5.4).
template <typename T, int kStrip>
__global__ void __launch_bounds__(256) conv1d_causal_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                            const T* __restrict__ halo, T* __restrict__ y,
                                                            T* __restrict__ tail, int B, int Tn, int rowlen, int W, int phi) {
  constexpr int VEC = Io<T>::VEC;
  const int vecs = rowlen / VEC;
  const int nstrips = (Tn + kStrip - 1) / kStrip;
  int col, s, b;
  if (gridDim.x < (1u << 23)) {      // thread numbers of 32 bits, as nearly always: their divisions are a fifth of 64-bit ones
    const unsigned gid = blockIdx.x * blockDim.x + threadIdx.x, rest = gid / (unsigned)vecs;
    col = (int)(gid - rest * vecs);
    b = (int)(rest / (unsigned)nstrips);
    s = (int)(rest - (unsigned)b * nstrips);
  } else {
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    col = (int)(gid % vecs);
    const long long rest = gid / vecs;
    s = (int)(rest % nstrips);
    b = (int)(rest / nstrips);
  }
  if (b >= B) return;
  const int e0 = col * VEC;  // first element (h*d + c) of this thread's column group

  float wt[4][VEC];  // wt[delta][i]
  if (W == 4) {
    // the VEC x 4 taps of this column group are contiguous: four whole-vector loads instead of 4 VEC scalar
    // ones (the scalar form made every thread start with a long chain of small dependent loads)
    float flat[4 * VEC];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float part[VEC];
      Io<T>::load(w + (size_t)e0 * 4 + j * VEC, part);
#pragma unroll
      for (int i = 0; i < VEC; ++i) flat[j * VEC + i] = part[i];
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i)
#pragma unroll
      for (int dl = 0; dl < 4; ++dl) wt[dl][i] = flat[i * 4 + dl];
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i)
#pragma unroll
      for (int dl = 0; dl < 4; ++dl) wt[dl][i] = dl < W ? Io<T>::scalar(w + (size_t)(e0 + i) * W + dl) : 0.f;
  }

  const int t0 = s * kStrip;
  typedef typename Io<T>::Raw Raw;
  Raw last[3];         // the conv cache for a continuation: the last W - 1 rows of [halo ; x], as they are
  const bool ends = tail != nullptr && s == nstrips - 1;
  auto fetch_last = [&] {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      last[r] = Io<T>::zero_raw();
      const int src = Tn - (W - 1) + r;
      if (r >= W - 1) continue;
      if (src >= 0) last[r] = Io<T>::load_raw(x + ((size_t)b * Tn + src) * rowlen + e0);
      else if (halo != nullptr) last[r] = Io<T>::load_raw(halo + ((size_t)b * (W - 1) + (W - 1 + src)) * rowlen + e0);
    }
  };
  if (kStrip == kGroup && ends) fetch_last();
  float win[3][VEC];  // win[j] = row t-1-j
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int src = t0 - 1 - j;
    if (j >= W - 1) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) win[j][i] = 0.f;
    } else if (src >= 0) {
      Io<T>::load(x + ((size_t)b * Tn + src) * rowlen + e0, win[j]);
    } else if (halo != nullptr) {
      Io<T>::load(halo + ((size_t)b * (W - 1) + (W - 1 + src)) * rowlen + e0, win[j]);
    } else {
#pragma unroll
      for (int i = 0; i < VEC; ++i) win[j][i] = 0.f;
    }
  }
  // Rows travel in groups of kGroup, the next group's loads issued before this group's arithmetic, so that
  // every thread keeps kGroup 16-byte loads in flight.
  const T* xb = x + ((size_t)b * Tn) * rowlen + e0;
  T* yb = y + ((size_t)b * Tn) * rowlen + e0;
  Raw nxt[kGroup];
#pragma unroll
  for (int r = 0; r < kGroup; ++r) nxt[r] = (t0 + r < Tn) ? Io<T>::load_raw(xb + (size_t)(t0 + r) * rowlen) : Io<T>::zero_raw();
#pragma unroll 1
  for (int tg = t0; tg < t0 + kStrip && tg < Tn; tg += kGroup) {
    Raw cur[kGroup];
#pragma unroll
    for (int r = 0; r < kGroup; ++r) cur[r] = nxt[r];
    if (kStrip > kGroup && tg + kGroup < t0 + kStrip) {
#pragma unroll
      for (int r = 0; r < kGroup; ++r) {
        const int t = tg + kGroup + r;
        nxt[r] = (t < Tn) ? Io<T>::load_raw(xb + (size_t)t * rowlen) : Io<T>::zero_raw();
      }
    }
#pragma unroll
    for (int r = 0; r < kGroup; ++r) {
      if (kStrip == kGroup && tg + r >= Tn) break;      // (a decode step: one token of the four)
      float c[VEC], out[VEC];
      Io<T>::unpack(cur[r], c);
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        float acc = wt[0][i] * c[i];
        acc = fmaf(wt[1][i], win[0][i], acc);
        acc = fmaf(wt[2][i], win[1][i], acc);
        acc = fmaf(wt[3][i], win[2][i], acc);
        out[i] = apply_phi(acc, phi);
        win[2][i] = win[1][i];
        win[1][i] = win[0][i];
        win[0][i] = c[i];
      }
      if (tg + r < Tn) Io<T>::store(yb + (size_t)(tg + r) * rowlen, out);
    }
  }
  if (ends) {
    if (kStrip > kGroup) fetch_last();
#pragma unroll
    for (int r = 0; r < 3; ++r)
      if (r < W - 1) *reinterpret_cast<Raw*>(tail + ((size_t)b * (W - 1) + r) * rowlen + e0) = last[r];
  }
}

// tail_out[b, r] = row (T - (W-1) + r) of [halo ; x]: the conv cache for a continuation.
template <typename T>
__global__ void conv_tail_kernel(const T* __restrict__ x, const T* __restrict__ halo, T* __restrict__ tail,
                                 int B, int Tn, int rowlen, int W) {
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = (long long)B * (W - 1) * rowlen;
  if (gid >= total) return;
  const int e = (int)(gid % rowlen);
  const int r = (int)((gid / rowlen) % (W - 1));
  const int b = (int)(gid / ((long long)rowlen * (W - 1)));
  const int src = Tn - (W - 1) + r;
  T val = T(0);
  if (src >= 0) val = x[((size_t)b * Tn + src) * rowlen + e];
  else if (halo != nullptr) val = halo[((size_t)b * (W - 1) + (W - 1 + src)) * rowlen + e];
  tail[gid] = val;
}

template <typename T>
hipError_t launch_typed(const ConvParams& p, hipStream_t stream) {
  const int rowlen = p.H * p.d;
  const int vecs = rowlen / Io<T>::VEC;
  auto threads = [&](int strip) { return (long long)p.B * ((p.T + strip - 1) / strip) * vecs; };
  T* tail = p.W > 1 ? (T*)p.tail_out : nullptr;
  auto launch = [&](auto kernel, int strip, int block) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((threads(strip) + block - 1) / block)), dim3(block), 0, stream, (const T*)p.x,
                       (const T*)p.w, (const T*)p.halo, (T*)p.y, tail, p.B, p.T, rowlen, p.W, p.phi);
    return hipGetLastError();
  };
  // The longest of 64, 32 and 16 tokens per strip that leaves two workgroups for every compute unit; strips of 4, with nothing to
  // wait for but one group of rows, for less than that: the three rows that a strip reads again cost less there than a walk in
  // dependent groups, and more above.  32 heads of 64, bf16, one sequence, strips of 4 / 16: four taps, 4096 tokens 8.9 / 11.8 us,
  // 5328 in 16 sequences 13.5 / 12.9, 8100 16.9 / 15.0; two, whose taps are read one by one, 2000 tokens 8.9 / 11.3, 4096 14.4 / 12.6.
  constexpr long long kWant = 512 * 256;
  const long long few = (p.W == 2 || p.W == 3) ? 50000 : 80000;
  if (p.T <= 4 || threads(16) < few) return launch(conv1d_causal_kernel<T, 4>, 4, 64);
  // Strips of 8 between that and one round of 16: twice the waves, which read 11 rows for 8 (four taps, bf16, strips of 16 / 8: 5003
  // tokens 15.7 / 14.3 us, 6000 16.7 / 15.5, 7000 18.1 / 17.8, 8100 19.2 / 19.2, 7 x 777 16.3 / 14.8; 4096 tokens, strips of 4 / 8,
  // 12.0 / 12.5; fp32 storage, where they move twice the bytes, the same within 1 %).
  if constexpr (sizeof(T) == 2)
    if (p.W == 4 && threads(16) < kWant) return launch(conv1d_causal_kernel<T, 8>, 8, 64);
  if (threads(64) >= kWant) return launch(conv1d_causal_kernel<T, 64>, 64, 256);
  if (threads(32) >= kWant) return launch(conv1d_causal_kernel<T, 32>, 32, 256);
  return launch(conv1d_causal_kernel<T, 16>, 16, 256);
}

}  // namespace

hipError_t launch_conv1d(const ConvParams& p, hipStream_t stream) {
  return p.bf16 ? launch_typed<bf16_t>(p, stream) : launch_typed<float>(p, stream);
}

hipError_t launch_conv_tail(const ConvParams& p, hipStream_t stream) {
  if (p.W <= 1 || p.tail_out == nullptr) return hipSuccess;
  const int rowlen = p.H * p.d;
  const long long total = (long long)p.B * (p.W - 1) * rowlen;
  const unsigned grid = (unsigned)((total + 255) / 256);
  if (p.bf16)
    hipLaunchKernelGGL(conv_tail_kernel<bf16_t>, dim3(grid), dim3(256), 0, stream, (const bf16_t*)p.x,
                       (const bf16_t*)p.halo, (bf16_t*)p.tail_out, p.B, p.T, rowlen, p.W);
  else
    hipLaunchKernelGGL(conv_tail_kernel<float>, dim3(grid), dim3(256), 0, stream, (const float*)p.x,
                       (const float*)p.halo, (float*)p.tail_out, p.B, p.T, rowlen, p.W);
  return hipGetLastError();
}

}  // namespace lawcat
