// Where the gate logits of paper section 4.2 come from: two consecutive low-rank linear layers on the layer
// input (the appendix's ablation on the rank of the gate function; rank 32 in the distilled models),
//   g[b,t,n] = sum_r ( sum_c x[b,t,c] * w1[r,c] ) * w2[n,r] + bias[n],   n over the Hkv * dk key channels.
// Streaming and HBM-bound: dm * 2 bytes read and N * 2 written per token against 2 * rank * (dm + N) flops
// (26 flop/B at dm = 2048, N = 512), so the matrix cores are used for what they are, a dense contraction, and
// the kernel is laid out around the reads of x.
//   bf16 storage, rank 32: both products transposed so that no operand is ever shuffled,
//     H^T = W1 x^T   (A = 16 rows of w1, B = 16 tokens of x, both read as whole row pieces and turned into fragment layout
//                     through the wave's own LDS rows),
//     G^T = W2 H^T   (the two accumulator tiles of H^T, rounded to bf16, ARE the B operand: k slot s < 4 is
//                     rank 4g + s, slot s >= 4 rank 16 + 4g + s - 4; w2 rows are read with the same permutation),
//     a lane then holds 4 adjacent channels of one token; they pass through the wave's own LDS rows and leave
//     as whole 256-byte row pieces.  The waves of a workgroup share up to 16 or 32 tokens and split the channels
//     of both products.
//   anything else (fp32 storage, other ranks): one workgroup per token, plain fp32 FMAs.
#include <algorithm>

#include "kernels.h"

namespace lawcat {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((vector_size(16)));

constexpr int kRsrcFlags = 0x00020000;  // raw buffer, 32-bit data format of gfx9-family descriptors
constexpr int kRank = 32;               // what the matrix-core kernel is built for
constexpr int kSlab = 64;               // channels of x per step of the first product
constexpr int kGroupCh = 128;           // output channels staged per store round

__device__ inline uint32_t pack2(float a, float b) {
  bf16x2 v = {(__bf16)a, (__bf16)b};  // round to nearest even
  return __builtin_bit_cast(uint32_t, v);
}
__device__ inline float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// grid (ceil(rows / tokens)), kWaves waves; rows = B * T tokens.  A workgroup owns `tokens` of them (at most TT tiles of 16): its
// waves split the channels of x for the first product (slab w, w + kWaves, ...), add their partial H^T
// through LDS, and split the output channels for the second (group w, w + kWaves, ...): short dependent
// chains and many waves per compute unit, which is what a streaming kernel needs to keep HBM busy.
// What bounds it: w1 (256 KB at d_model 4096), which every workgroup reads from L2, twice as much as 16 tokens of x.  With w1 in
// fragment layout straight from L2 (16 rows, one cache line each, per 16 lanes) 5003 tokens at d_model 4096 took 24.2 us, in whole
// row pieces 18.6 for 16 tokens a workgroup and 16.5 for 32; without w2 on its way before the sums meet 1 more.  How many slabs are
// on their way (1 to 4) makes no difference up to 10K tokens; two are 4 % better at 32K.
template <int TT, int kWaves, int kDepth>
__global__ void __launch_bounds__(64 * kWaves) gate_project_mfma_kernel(const bf16_t* __restrict__ x,
                                                                        const bf16_t* __restrict__ w1,
                                                                        const bf16_t* __restrict__ w2,
                                                                        const bf16_t* __restrict__ bias,
                                                                        bf16_t* __restrict__ g, long long rows, int dm, int N, int tokens) {
  constexpr int NR = 16 * TT;             // most tokens of a workgroup, which takes `tokens` of them
  constexpr int SS = kSlab * 2 + 16;      // LDS row stride of a slab's rows of x and of w1, bytes
  constexpr int RS = kGroupCh * 2 + 16;   // of staged logits (a 256-byte row piece plus padding)
  constexpr int kMine = (NR + kRank) * SS > NR * RS ? (NR + kRank) * SS : NR * RS;
  __shared__ __attribute__((aligned(16))) unsigned char stage[kWaves * kMine];
  __shared__ __attribute__((aligned(16))) float part[kWaves][TT][2][64][4];
  const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = l & 15, gq = l >> 4;
  const long long row0 = (long long)blockIdx.x * tokens;   // first token of this workgroup
  const int nrows = (int)((rows - row0) < tokens ? (rows - row0) : tokens);
  // the rows of x and of g, each through a descriptor of its own: rows past the last token read as zero and are
  // not written
  const __amdgpu_buffer_rsrc_t xsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<const char*>(x) + (size_t)row0 * dm * 2), 0, nrows * dm * 2, kRsrcFlags);
  const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc((void*)w1, 0, kRank * dm * 2, kRsrcFlags);
  const __amdgpu_buffer_rsrc_t gdst = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<char*>(g) + (size_t)row0 * N * 2), 0, nrows * N * 2, kRsrcFlags);

  // ---- H^T[rank][token] = sum_c w1[rank][c] x[token][c], this wave's slabs of 64 channels
  // The slab's rows of x and of w1 are read as whole row pieces (8 lanes per row, 8 rows per instruction: read in fragment layout,
  // 16 lanes of a load touch 16 rows, and the cache serves a line at a time), kDepth slabs ahead, pass through this wave's own LDS
  // rows and come back in fragment layout (lane (row n, group gq): 16 bytes at 64 j + 16 gq).
  floatx4 acc[TT][2];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) { acc[tt][0] = floatx4{0.f, 0.f, 0.f, 0.f}; acc[tt][1] = floatx4{0.f, 0.f, 0.f, 0.f}; }
  unsigned char* mine = stage + (size_t)wv * kMine;
  const int lr = l >> 3, lp = l & 7;                                    // row within a group of 8, 16-byte piece
  const unsigned off = (unsigned)lr * dm * 2 + lp * 16;
  struct Slab { u32x4 x[2 * TT], w[kRank / 8]; };
  auto fetch = [&](int k0, Slab& o) {
    // (a slab past the last channel: offsets that no descriptor covers read as zero)
    const unsigned at = k0 < dm ? off + (unsigned)k0 * 2 : 0xF0000000u, step = k0 < dm ? (unsigned)dm * 16 : 0u;
#pragma unroll
    for (int it = 0; it < 2 * TT; ++it) o.x[it] = __builtin_amdgcn_raw_buffer_load_b128(xsrc, (int)(at + it * step), 0, 0);
#pragma unroll
    for (int it = 0; it < kRank / 8; ++it) o.w[it] = __builtin_amdgcn_raw_buffer_load_b128(wsrc, (int)(at + it * step), 0, 0);
  };
  constexpr int kStep = kSlab * kWaves;
  Slab buf[kDepth];
#pragma unroll
  for (int d = 0; d < kDepth; ++d) fetch(wv * kSlab + d * kStep, buf[d]);
#pragma unroll 1
  for (int k0 = wv * kSlab; k0 < dm; k0 += kStep * kDepth) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
      // this slab's rows into LDS (the previous slab's fragment reads were issued before these writes, and LDS
      // serves one wave's requests in order)
#pragma unroll
      for (int it = 0; it < 2 * TT; ++it) *reinterpret_cast<u32x4*>(mine + (8 * it + lr) * SS + lp * 16) = buf[d].x[it];
#pragma unroll
      for (int it = 0; it < kRank / 8; ++it) *reinterpret_cast<u32x4*>(mine + (NR + 8 * it + lr) * SS + lp * 16) = buf[d].w[it];
      __builtin_amdgcn_wave_barrier();
      fetch(k0 + (d + kDepth) * kStep, buf[d]);
#pragma unroll
      for (int j = 0; j < kSlab / 32; ++j) {
        const unsigned char* p = mine + n * SS + 64 * j + 16 * gq;
        const bf16x8 a0 = *reinterpret_cast<const bf16x8*>(p + NR * SS), a1 = *reinterpret_cast<const bf16x8*>(p + (NR + 16) * SS);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const bf16x8 b = *reinterpret_cast<const bf16x8*>(p + 16 * tt * SS);
          acc[tt][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b, acc[tt][0], 0, 0, 0);
          acc[tt][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b, acc[tt][1], 0, 0, 0);
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  // this wave's first group of w2's rows, on the way while the sums meet
  uint2 w2lo[kGroupCh / 16], w2hi[kGroupCh / 16];
  auto fetch2 = [&](int c0) {
#pragma unroll
    for (int ct = 0; ct < kGroupCh / 16; ++ct) {
      const bf16_t* wr = w2 + (size_t)(c0 + 16 * ct + n) * kRank;      // row of w2 = 32 ranks = 64 bytes
      w2lo[ct] = *reinterpret_cast<const uint2*>(wr + 4 * gq);
      w2hi[ct] = *reinterpret_cast<const uint2*>(wr + 16 + 4 * gq);
    }
  };
  if (wv * kGroupCh < N) fetch2(wv * kGroupCh);
  // the waves' partial sums meet in LDS; every wave adds them up in the same order
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    *reinterpret_cast<floatx4*>(&part[wv][tt][0][l][0]) = acc[tt][0];
    *reinterpret_cast<floatx4*>(&part[wv][tt][1][l][0]) = acc[tt][1];
  }
  __syncthreads();
  bf16x8 hb[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      floatx4 sum = *reinterpret_cast<const floatx4*>(&part[0][tt][mt][l][0]);
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        const floatx4 p = *reinterpret_cast<const floatx4*>(&part[w][tt][mt][l][0]);
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] += p[i];
      }
      acc[tt][mt] = sum;
    }
    // lane (token n, group gq): acc[tt][mt][i] = H^T[16 mt + 4 gq + i][16 tt + n]; as the next product's B operand
    const u32x4 hbits = {pack2(acc[tt][0][0], acc[tt][0][1]), pack2(acc[tt][0][2], acc[tt][0][3]),
                         pack2(acc[tt][1][0], acc[tt][1][1]), pack2(acc[tt][1][2], acc[tt][1][3])};
    hb[tt] = __builtin_bit_cast(bf16x8, hbits);
  }

  // ---- G^T[channel][token] = sum_r w2[channel][r] H^T[r][token] + bias[channel], this wave's groups of 128 channels
  // (staged for the store in the same LDS rows: every wave is past its slabs, the barrier above says so)
  for (int c0 = wv * kGroupCh; c0 < N; c0 += kGroupCh * kWaves) {
#pragma unroll
    for (int ct = 0; ct < kGroupCh / 16; ++ct) {
      const u32x4 abits = {w2lo[ct].x, w2lo[ct].y, w2hi[ct].x, w2hi[ct].y};
      float bv[4] = {0.f, 0.f, 0.f, 0.f};
      if (bias != nullptr) {
        const uint2 bb = *reinterpret_cast<const uint2*>(bias + c0 + 16 * ct + 4 * gq);
        bv[0] = bf_lo(bb.x); bv[1] = bf_hi(bb.x); bv[2] = bf_lo(bb.y); bv[3] = bf_hi(bb.y);
      }
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        floatx4 out = {bv[0], bv[1], bv[2], bv[3]};
        out = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, abits), hb[tt], out, 0, 0, 0);
        // lane (token 16 tt + n, gq): channels c0 + 16 ct + 4 gq + i
        *reinterpret_cast<uint2*>(mine + (16 * tt + n) * RS + (16 * ct + 4 * gq) * 2) =
            make_uint2(pack2(out[0], out[1]), pack2(out[2], out[3]));
      }
    }
    if (c0 + kGroupCh * kWaves < N) fetch2(c0 + kGroupCh * kWaves);
    __builtin_amdgcn_wave_barrier();   // LDS serves one wave's requests in order: the rows are complete below
#pragma unroll
    for (int it = 0; it < NR * (kGroupCh / 8) / 64; ++it) {
      const int idx = it * 64 + l;
      const int r = idx / (kGroupCh / 8), vec = idx % (kGroupCh / 8);
      const u32x4 u = *reinterpret_cast<const u32x4*>(mine + r * RS + vec * 16);
      __builtin_amdgcn_raw_buffer_store_b128(u, gdst, (int)((unsigned)r * N * 2 + (c0 + vec * 8) * 2), 0, 0);
    }
    __builtin_amdgcn_wave_barrier();   // the rows are read before the next round overwrites them
  }
}

// Any storage type, any rank: one workgroup per token.
template <typename T>
__device__ inline float to_f(T v);
template <>
__device__ inline float to_f<float>(float v) { return v; }
template <>
__device__ inline float to_f<bf16_t>(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ inline void from_f(float v, float* p) { *p = v; }
__device__ inline void from_f(float v, bf16_t* p) { *p = (bf16_t)(pack2(v, 0.f) & 0xffffu); }

template <typename T>
__global__ void __launch_bounds__(256) gate_project_generic_kernel(const T* __restrict__ x, const T* __restrict__ w1,
                                                                   const T* __restrict__ w2, const T* __restrict__ bias,
                                                                   T* __restrict__ g, int dm, int rank, int N) {
  extern __shared__ float sm[];   // x row (dm floats), then h (rank floats)
  float* xs = sm;
  float* h = sm + dm;
  const size_t row = blockIdx.x;
  for (int c = threadIdx.x; c < dm; c += 256) xs[c] = to_f<T>(x[row * dm + c]);
  __syncthreads();
  for (int r = threadIdx.x; r < rank; r += 256) {
    float acc = 0.f;
    for (int c = 0; c < dm; ++c) acc = fmaf(xs[c], to_f<T>(w1[(size_t)r * dm + c]), acc);
    h[r] = acc;
  }
  __syncthreads();
  for (int nn = threadIdx.x; nn < N; nn += 256) {
    float acc = bias != nullptr ? to_f<T>(bias[nn]) : 0.f;
    for (int r = 0; r < rank; ++r) acc = fmaf(h[r], to_f<T>(w2[(size_t)nn * rank + r]), acc);
    from_f(acc, g + row * N + nn);
  }
}

}  // namespace

hipError_t launch_gate_project(const GateProjectParams& p, hipStream_t stream) {
  const long long rows = (long long)p.B * p.T;
  if (rows > 0x7fffffffLL) return hipErrorInvalidValue;
  if (p.bf16 && p.rank == kRank && p.dm % 128 == 0 && p.N % kGroupCh == 0 && (long long)32 * p.dm * 2 < (1ll << 31) &&
      (long long)32 * p.N * 2 < (1ll << 31)) {
    // The tokens are spread evenly over the compute units: as many workgroups for each as 32 tokens a workgroup call for, and of those the
    // same number of tokens.  Eight waves share a workgroup's tokens while a unit has one, four after that (two slabs on their way): 16384
    // tokens at d_model 4096 with 1024 outputs, 32 to four / to eight 39.0 / 41.9 us; 4096, to eight 12.7.  us, spread evenly / 16 tokens a
    // workgroup up to 4096 and from 8193 to 16352, else 32, whatever the count: d_model 4096 with 1024 outputs, 4200 tokens 12.3 / 16.2, 9500
    // 26.5 / 31.5, 12500 34.0 / 45.4, 17500 46.9 / 56.7; 2048 with 512, 5003 8.9 / 9.5, 12500 14.6 / 21.3, 17500 21.1 / 23.9.
    // Not where the workgroups added cost more, which is w1 and w2 once each:
    //   up to 4096 tokens 12 a workgroup at least, or 16 where x is narrow.  4 at least / 12 / 16: d_model 4096 with 1024, 300 tokens 8.19 /
    //     8.06 / 8.05, 1024 9.03 / 8.77 / 8.84, 2048 (8 each) 10.21 / 9.25 / 9.51; 3200, 13 each / 16, 10.2 / 11.0; 1024 with 512, 5.66 / 5.42;
    //   a narrow x past that: d_model 512 with 512, 6000 tokens 6.48 / 6.45, 8200 8.31 / 7.72 (12500 9.57 / 9.70, 17500 12.1 / 12.6);
    //   from the fourth to a unit on, which waits for one of three to end, with narrow x and few outputs: 2048 with 512, 24600 37.9 / 36.7, 26000
    //     39.1 / 37.6 (30000 42.6 / 44.1); 1024 with 512, 28000 23.7 / 22.3; 2048 with 1024, 24600 43.6 / 48.9; 4096 with 512, 54.5 / 64.8.
    auto launch = [&](auto kernel, int tokens, int waves) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)((rows + tokens - 1) / tokens)), dim3(64 * waves), 0, stream, (const bf16_t*)p.x,
                         (const bf16_t*)p.w1, (const bf16_t*)p.w2, (const bf16_t*)p.bias, (bf16_t*)p.g, rows, p.dm, p.N, tokens);
    };
    const long long each = (rows + 32 * 256 - 1) / (32 * 256);   // workgroups per compute unit
    const int share = (int)((rows + 256 * each - 1) / (256 * each));
    if (rows <= 16 * 256) {
      launch(gate_project_mfma_kernel<1, 8, 1>, p.dm < 2048 ? 16 : std::max(12, share), 8);
    } else {
      const bool even = p.dm >= 1024 && (each <= 3 || (long long)p.dm * p.N >= 2048 * 1024);
      if (each == 1) launch(gate_project_mfma_kernel<2, 8, 1>, even ? share : 32, 8);
      else launch(gate_project_mfma_kernel<2, 4, 2>, even ? share : 32, 4);
    }
    return hipGetLastError();
  }
  const size_t lds = (size_t)(p.dm + p.rank) * sizeof(float);
  if (lds > 64 * 1024) return hipErrorInvalidValue;
  if (p.bf16)
    hipLaunchKernelGGL(gate_project_generic_kernel<bf16_t>, dim3((unsigned)rows), dim3(256), lds, stream, (const bf16_t*)p.x,
                       (const bf16_t*)p.w1, (const bf16_t*)p.w2, (const bf16_t*)p.bias, (bf16_t*)p.g, p.dm, p.rank, p.N);
  else
    hipLaunchKernelGGL(gate_project_generic_kernel<float>, dim3((unsigned)rows), dim3(256), lds, stream, (const float*)p.x,
                       (const float*)p.w1, (const float*)p.w2, (const float*)p.bias, (float*)p.g, p.dm, p.rank, p.N);
  return hipGetLastError();
}

}  // namespace lawcat
