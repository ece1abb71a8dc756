// The layer that follows the conv in paper section 4.1: a linear layer with nonlinearity, the same for the
// query and the key,
//   y[b,t,h,f] = phi( sum_c x~[b,t,h,c] * Wf[h / group, c, f] ),   x~ = causal depthwise conv of x (no phi)
// fused with that conv: one kernel reads the raw rows, slides the conv window in registers, keeps the conv
// output of a tile in LDS and multiplies it by the head's d x d matrix.
//   bf16 storage: the product runs on the matrix cores (v_mfma_f32_16x16x32_bf16, fp32 accumulate), computed
//     transposed (y^T = Wf^T x~^T) so that a lane ends up with four adjacent features of one token; the results
//     go back through LDS and leave as whole rows; the conv output is rounded to bf16 once, as an MFMA operand.
//   fp32 storage: plain fp32 FMAs (the 1e-4 bar leaves no room for bf16 operands).
// Streaming and HBM-bound: 2 bytes read and 2 written per element; the matrix (8 or 32 KB) is read from L2 once
// per workgroup, which walks a run of tiles.  5003 tokens, 32 / 8 heads of 128: 24.7 / 9.6 us with the rows kept for a
// continuation (3.3 and 2.1 TB/s); 32.9 / 18.0 when the matrix was transposed into LDS two bytes at a time, the taps were
// read one by one and a second launch copied those rows.  Both in the layer's one launch 28.3, now 26.0 (the matrix in registers).
#include "segment_scan.h"

namespace lawcat {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;        // fp32 kernel: tokens per tile
constexpr int kTilesPerBlock = 4;
constexpr int kShare = 3;        // bf16 kernel: workgroups that share a compute unit

typedef unsigned int u32x4 __attribute__((vector_size(16)));

__device__ inline float apply_phi(float x, int phi) { return phi == 1 ? (x > 0.f ? 1.f + x : __expf(x)) : x; }
template <bool ELU>
__device__ inline float apply_phi(float x) { return ELU ? (x > 0.f ? 1.f + x : __expf(x)) : x; }
__device__ inline float bf_to_f(bf16_t u) { return __uint_as_float((uint32_t)u << 16); }
__device__ inline uint32_t pack2(float a, float b) {
  bf16x2 v = {(__bf16)a, (__bf16)b};  // round to nearest even
  return __builtin_bit_cast(uint32_t, v);
}

__device__ inline bf16x8 make8(uint2 a, uint2 b) { return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y)); }
// 4 x 16 elements of 16 bits in LDS, read transposed: lane (g, n) gets column n of the four rows at its group's address
__device__ inline uint2 read_tr(const unsigned char* p) {
  typedef short short4v __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)p));
}

// ---- fp32 kernel: conv of one 64-token tile into LDS (no phi).  Thread = one channel pair x a run of tokens.
// xs: [kTile][D] elements of XS (bf16_t packed pairs or float), row stride `rs` bytes.
template <typename T, int D>
__device__ inline void conv_tile(const T* __restrict__ x, const T* __restrict__ w, const T* __restrict__ halo, int b,
                                 int h, int H, int Tn, int W, int t0, unsigned char* xs, int rs) {
  constexpr int PAIRS = D / 2;
  constexpr int NTOK = kTile * PAIRS / 256;   // tokens per thread: 8 (d = 64) or 16 (d = 128)
  const int cp = threadIdx.x % PAIRS, tg = threadIdx.x / PAIRS;
  const int c0 = 2 * cp;
  float wt[2][4];
#pragma unroll
  for (int ch = 0; ch < 2; ++ch)
#pragma unroll
    for (int dl = 0; dl < 4; ++dl) {
      float v = 0.f;
      if (dl < W) {
        const T* p = w + ((size_t)h * D + c0 + ch) * W + dl;
        if constexpr (sizeof(T) == 2) v = bf_to_f(*p); else v = *p;
      }
      wt[ch][dl] = v;
    }
  auto row = [&](int t, float (&v)[2]) {   // raw row t of this thread's two channels; rows < 0 from the halo or zero
    v[0] = 0.f; v[1] = 0.f;
    const T* p = nullptr;
    if (t >= 0 && t < Tn) p = x + (((size_t)b * Tn + t) * H + h) * D + c0;
    else if (t < 0 && halo != nullptr && t >= -(W - 1)) p = halo + (((size_t)b * (W - 1) + (W - 1 + t)) * H + h) * D + c0;
    if (p != nullptr) {
      if constexpr (sizeof(T) == 2) {
        const uint32_t u = *reinterpret_cast<const uint32_t*>(p);
        v[0] = __uint_as_float(u << 16); v[1] = __uint_as_float(u & 0xffff0000u);
      } else {
        const float2 f = *reinterpret_cast<const float2*>(p);
        v[0] = f.x; v[1] = f.y;
      }
    }
  };
  const int ts = t0 + tg * NTOK;
  float win[3][2];
#pragma unroll
  for (int j = 0; j < 3; ++j) row(ts - 1 - j, win[j]);
#pragma unroll
  for (int i = 0; i < NTOK; ++i) {
    float cur[2];
    row(ts + i, cur);
    float out[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      float acc = wt[ch][0] * cur[ch];
      acc = fmaf(wt[ch][1], win[0][ch], acc);
      acc = fmaf(wt[ch][2], win[1][ch], acc);
      acc = fmaf(wt[ch][3], win[2][ch], acc);
      out[ch] = acc;
      win[2][ch] = win[1][ch]; win[1][ch] = win[0][ch]; win[0][ch] = cur[ch];
    }
    unsigned char* dst = xs + (size_t)(tg * NTOK + i) * rs;
    if constexpr (sizeof(T) == 2) *reinterpret_cast<uint32_t*>(dst + c0 * 2) = pack2(out[0], out[1]);
    else *reinterpret_cast<float2*>(dst + c0 * 4) = make_float2(out[0], out[1]);
  }
}

// bf16 storage, matrix cores.  One workgroup (4 waves) walks `tiles_per_block` consecutive tiles of one
// (batch, head group): a tile is TT tokens x GH adjacent heads that share one matrix, ROWS = TT * GH rows of D
// channels (at D = 64 256 rows of four heads or 128 of one, at D = 128 64).
//   load  : thread = 8 adjacent channels (16 bytes) x a run of 8 tokens (256 rows) or 4; the run's raw rows and the
//           three before it in registers, read through a buffer descriptor over the workgroup's own token range, so
//           that rows before the first token and past the last read as zero without a branch; the next tile's
//           rows are requested before the current tile's products start
//   conv  : in registers, fp32; rounded to bf16 into LDS, row = token * GH + head (the order in memory)
//   matrix: wave w takes the 16-row groups w, w + 4, ...: B operand = the 16 rows, A operand = Wf^T (Wf read transposed from LDS),
//           so a lane ends up with 4 adjacent features of one row; phi; back into the same LDS rows.  Head dim 128: wave w takes features
//           32 w .. of all rows, its share of the matrix in registers (from LDS, 64 reads of it per 16 rows, each a latency of its own:
//           the layer at 5003 tokens 103.1 -> 102.1 us, at 16000 235.5 -> 232.5), results in LDS rows of their own
//   store : the wave reads its 16 finished rows (head dim 128: the workgroup the tile) back 16 bytes per lane and stores whole
//           128/256-byte rows (buffer stores: rows past the last token are dropped)
// WT: the conv width when it is the paper's 4 (no per-tap branches), 0 = any width up to 4, read from W.
template <int D> constexpr bool held = D == 128;
struct FeatureArgs {
  const bf16_t *x, *w, *halo, *wf;
  bf16_t *y, *tail;
  int Tn, H, group, W, tiles_per_block;
  int runs;                                  // workgroups per (batch, head group)
};
template <int D, int GH, int TT, bool ELU, int WT>
__device__ __forceinline__ void feature_tiles(const FeatureArgs& a, int block, unsigned char* smem) {
  const bf16_t *__restrict__ x = a.x, *__restrict__ w = a.w, *__restrict__ halo = a.halo, *__restrict__ wf = a.wf;
  bf16_t *__restrict__ y = a.y, *__restrict__ tail = a.tail;
  const int Tn = a.Tn, H = a.H, group = a.group, tiles_per_block = a.tiles_per_block;
  const int bx = block % a.runs, by = block / a.runs;
  const int W = WT != 0 ? WT : a.W;
  constexpr int RS = D * 2 + 16;              // LDS row stride in bytes (16-byte reads of 16 rows hit distinct banks)
  constexpr int KS = D / 32, FT = D / 16;
  constexpr int ROWS = TT * GH;
  constexpr int VPH = D / 8;                  // 16-byte vectors per head row
  constexpr int VECS = GH * VPH;              // per token
  constexpr int NTOK = ROWS * VPH / 256;      // tokens per thread
  constexpr int kRsrcFlags = 0x00020000;      // raw buffer, 32-bit data format of gfx9-family descriptors
  static_assert(ROWS * VPH == 256 * NTOK && 256 % VECS == 0, "tile must give every thread NTOK tokens of one vector");
  // HELD (head dim 128): a wave keeps 32 features' columns of the matrix in registers and takes all rows of a tile, results in LDS rows of
  // their own; the matrix passes through both.  Otherwise it stays in LDS and a wave takes 16 rows at a time.
  constexpr bool HELD = held<D>;
  static_assert(!HELD || 2 * ROWS == D);
  unsigned char* wts = smem;                  // Wf: [c][f] bf16
  unsigned char* xs = smem + (HELD ? 0 : D * RS);     // the tile: [row][c] bf16
  unsigned char* ys = smem + ROWS * RS;       // HELD: its results
  const int hgroups = H / GH;
  const int b = by / hgroups, h0 = (by % hgroups) * GH;
  const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
  const int n = l & 15, g = l >> 4;
  const int v = tid % VECS, run = tid / VECS;
  const int hh = v / VPH, c0 = (v % VPH) * 8;
  const unsigned stride = (unsigned)H * D * 2;                 // bytes per token row
  const unsigned coff = (unsigned)((h0 + hh) * D + c0) * 2;    // this thread's columns, in bytes

  const int ntiles = (Tn + TT - 1) / TT;
  const int tile0 = bx * tiles_per_block;
  const int tile_end = min(ntiles, tile0 + tiles_per_block);
  // this workgroup's tokens [first, last) and the three rows before them; the host has checked that the range
  // stays far below 2^32 bytes, so that the wrapped offsets of rows -3 .. -1 fall outside the descriptor
  const int first = tile0 * TT, last = min(tile_end * TT, Tn), lo = max(first - 3, 0);
  const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<const char*>(x) + ((size_t)b * Tn + lo) * stride), 0, (int)((unsigned)(last - lo) * stride),
      kRsrcFlags);
  const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<char*>(y) + ((size_t)b * Tn + first) * stride), 0, (int)((unsigned)(last - first) * stride),
      kRsrcFlags);

  u32x4 raw[NTOK + 3];
  auto load_tile = [&](int t0) {
    const unsigned base = (unsigned)(t0 + run * NTOK - 3 - lo) * stride + coff;
#pragma unroll
    for (int j = 0; j < NTOK + 3; ++j) raw[j] = __builtin_amdgcn_raw_buffer_load_b128(src, (int)(base + j * stride), 0, 0);
  };
  load_tile(first);
  if (first == 0 && halo != nullptr && run == 0) {
    // the rows before the first token come from the caller's halo (oldest row first, W - 1 rows)
    const __amdgpu_buffer_rsrc_t hsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(reinterpret_cast<const char*>(halo) + (size_t)b * (W - 1) * stride), 0, (int)((unsigned)(W - 1) * stride),
        kRsrcFlags);
#pragma unroll
    for (int j = 0; j < 3; ++j)
      if (j - 3 >= -(W - 1)) raw[j] = __builtin_amdgcn_raw_buffer_load_b128(hsrc, (int)((unsigned)(W - 4 + j) * stride + coff), 0, 0);
  }
  // conv weights of this thread's 8 channels
  float wt[8][4];
  if constexpr (WT == 4) {       // contiguous: four 16-byte loads
    const u32x4* wsrc = reinterpret_cast<const u32x4*>(w + ((size_t)(h0 + hh) * D + c0) * 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u32x4 u = wsrc[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        wt[2 * j + (i >> 1)][2 * (i & 1)] = __uint_as_float(u[i] << 16);
        wt[2 * j + (i >> 1)][2 * (i & 1) + 1] = __uint_as_float(u[i] & 0xffff0000u);
      }
    }
  } else {
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
      for (int dl = 0; dl < 4; ++dl) wt[c][dl] = dl < W ? bf_to_f(w[((size_t)(h0 + hh) * D + c0 + c) * W + dl]) : 0.f;
  }
  // the matrix into LDS
  {
    const bf16_t* wsrc = wf + (size_t)(h0 / group) * D * D;
    for (int e = tid; e < D * D / 8; e += 256) {
      const int c = e / VPH, f0 = (e % VPH) * 8;
      *reinterpret_cast<uint4*>(wts + c * RS + f0 * 2) = *reinterpret_cast<const uint4*>(wsrc + (size_t)c * D + f0);
    }
  }

  bf16x8 held_a[HELD ? 2 : 1][KS];     // features 32 wv + 16 f + n of channels 32 ks + {4 g + i, 16 + 4 g + i}
  if constexpr (HELD) {
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const unsigned char* p = wts + (32 * ks + 4 * g + (n >> 2)) * RS + (32 * wv + 16 * f + 4 * (n & 3)) * 2;
        held_a[f][ks] = make8(read_tr(p), read_tr(p + 16 * RS));
      }
    __syncthreads();
  }

  for (int tile = tile0; tile < tile_end; ++tile) {
    const int t0 = tile * TT;
    // conv of this thread's 8 tokens x 8 channels; taps beyond W are skipped, not multiplied by zero
#pragma unroll
    for (int i = 0; i < NTOK; ++i) {
      float acc[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] = 0.f;
#pragma unroll
      for (int dl = 0; dl < 4; ++dl) {
        if (dl < W) {
          const u32x4 r = raw[i + 3 - dl];
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const float xv = (c & 1) ? __uint_as_float(r[c >> 1] & 0xffff0000u) : __uint_as_float(r[c >> 1] << 16);
            acc[c] = fmaf(wt[c][dl], xv, acc[c]);
          }
        }
      }
      const uint4 pk = make_uint4(pack2(acc[0], acc[1]), pack2(acc[2], acc[3]), pack2(acc[4], acc[5]), pack2(acc[6], acc[7]));
      *reinterpret_cast<uint4*>(xs + (size_t)((run * NTOK + i) * GH + hh) * RS + c0 * 2) = pk;
    }
    __syncthreads();                          // the tile (and, the first time, the matrix) is in LDS
    if (tile + 1 < tile_end) load_tile(t0 + TT);
    if constexpr (HELD) {
      bf16x8 b[2][KS];          // the next row group's operands travel while this one's products run
      auto load_rows = [&](int rg, bf16x8 (&o)[KS]) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const unsigned char* p = xs + (16 * rg + n) * RS + (32 * ks + 4 * g) * 2;
          o[ks] = make8(*reinterpret_cast<const uint2*>(p), *reinterpret_cast<const uint2*>(p + 32));
        }
      };
      load_rows(0, b[0]);
#pragma unroll
      for (int rg = 0; rg < ROWS / 16; ++rg) {
        if (rg + 1 < ROWS / 16) load_rows(rg + 1, b[(rg + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int f = 0; f < 2; ++f) acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(held_a[f][ks], b[rg & 1][ks], acc[f], 0, 0, 0);
        // lane (n, g): features 32 wv + 16 f + 4 g + i of row n
#pragma unroll
        for (int f = 0; f < 2; ++f)
          *reinterpret_cast<uint2*>(ys + (16 * rg + n) * RS + (32 * wv + 16 * f + 4 * g) * 2) =
              make_uint2(pack2(apply_phi<ELU>(acc[f][0]), apply_phi<ELU>(acc[f][1])), pack2(apply_phi<ELU>(acc[f][2]), apply_phi<ELU>(acc[f][3])));
      }
      __syncthreads();       // (the next tile's rows go to xs, its results to ys, behind another barrier)
#pragma unroll
      for (int it = 0; it < ROWS * VPH / 256; ++it) {
        const int idx = it * 256 + tid, grow = idx / VPH, vec = idx % VPH;
        const u32x4 u = *reinterpret_cast<const u32x4*>(ys + grow * RS + vec * 16);
        const unsigned off = (unsigned)(t0 - first + grow / GH) * stride + (unsigned)((h0 + grow % GH) * D + vec * 8) * 2;
        __builtin_amdgcn_raw_buffer_store_b128(u, dst, (int)off, 0, 0);
      }
      continue;
    }
#pragma unroll 1
    for (int rg = wv; rg < ROWS / 16; rg += 4) {
      unsigned char* rows = xs + (size_t)(16 * rg) * RS;
      bf16x8 bfrag[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const unsigned char* p = rows + n * RS + (32 * ks + 4 * g) * 2;
        bfrag[ks] = make8(*reinterpret_cast<const uint2*>(p), *reinterpret_cast<const uint2*>(p + 32));
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          // feature 16 ft + n of channels 32 ks + {4 g + i, 16 + 4 g + i}: two transposing reads
          const unsigned char* p = wts + (32 * ks + 4 * g + (n >> 2)) * RS + (16 * ft + 4 * (n & 3)) * 2;
          const bf16x8 afrag = make8(read_tr(p), read_tr(p + 16 * RS));
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afrag, bfrag[ks], acc, 0, 0, 0);
        }
        // lane (n, g): features 16 ft + 4 g + i of row n; every lane of the wave has read the rows already
        *reinterpret_cast<uint2*>(rows + n * RS + (16 * ft + 4 * g) * 2) =
            make_uint2(pack2(apply_phi<ELU>(acc[0]), apply_phi<ELU>(acc[1])),
                       pack2(apply_phi<ELU>(acc[2]), apply_phi<ELU>(acc[3])));
      }
      __builtin_amdgcn_wave_barrier();        // LDS serves one wave's requests in order: the rows are complete below
#pragma unroll
      for (int it = 0; it < 16 * VPH / 64; ++it) {
        const int idx = it * 64 + l;
        const int r = idx / VPH, vec = idx % VPH;
        const int grow = 16 * rg + r;          // row of the tile: token * GH + head
        const u32x4 u = *reinterpret_cast<const u32x4*>(rows + r * RS + vec * 16);
        const unsigned off = (unsigned)(t0 - first + grow / GH) * stride + (unsigned)((h0 + grow % GH) * D + vec * 8) * 2;
        __builtin_amdgcn_raw_buffer_store_b128(u, dst, (int)off, 0, 0);
      }
    }
    __syncthreads();                          // every wave is done with the tile before the next conv overwrites it
  }
  // the workgroup of the last tile keeps the last W - 1 raw rows of [halo ; x] for a continuation
  if (tail != nullptr && tile_end == ntiles) {
    for (int i = tid; i < (W - 1) * VECS; i += 256) {
      const int r = i / VECS, from = Tn - (W - 1) + r;
      const size_t col = (size_t)h0 * D + (i % VECS) * 8, row = (size_t)H * D;
      u32x4 u = {0u, 0u, 0u, 0u};
      if (from >= 0) u = *reinterpret_cast<const u32x4*>(x + ((size_t)b * Tn + from) * row + col);
      else if (halo != nullptr) u = *reinterpret_cast<const u32x4*>(halo + ((size_t)b * (W - 1) + (W - 1 + from)) * row + col);
      *reinterpret_cast<u32x4*>(tail + ((size_t)b * (W - 1) + r) * row + col) = u;
    }
  }
}

// grid: the workgroups of one tensor, or of the queries and then of the keys (two shapes of tile, one launch: the keys' few bytes
// travel beside the queries').  The whole layer, 5003 tokens, 32 / 8 heads of 128, gates included: 112.6 -> 106.2 us, 500 tokens 55.2 -> 47.5.
template <int D, int GH, int TT, int GH2, int TT2, bool ELU, int WT>
__global__ void __launch_bounds__(256, kShare) conv_feature_mfma_kernel(const FeatureArgs a, const FeatureArgs a2, int first) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if ((int)blockIdx.x < first) feature_tiles<D, GH, TT, ELU, WT>(a, blockIdx.x, smem);
  else if constexpr (GH2 > 0) feature_tiles<D, GH2, TT2, ELU, WT>(a2, blockIdx.x - first, smem);
}

// fp32 storage, plain FMAs.  Same grid.
template <int D>
__global__ void __launch_bounds__(256) conv_feature_f32_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                               const float* __restrict__ halo,
                                                               const float* __restrict__ wf, float* __restrict__ y,
                                                               int B, int Tn, int H, int group, int W, int phi) {
  constexpr int RS = (D + 2) * 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* xs = smem;
  const int bh = blockIdx.y, b = bh / H, h = bh % H;
  const int tid = threadIdx.x;
  const float* wsrc = wf + (size_t)(h / group) * D * D;
  for (int tile = 0; tile < kTilesPerBlock; ++tile) {
    const int t0 = (blockIdx.x * kTilesPerBlock + tile) * kTile;
    if (t0 >= Tn) break;
    __syncthreads();
    conv_tile<float, D>(x, w, halo, b, h, H, Tn, W, t0, xs, RS);
    __syncthreads();
    for (int e = tid; e < kTile * D; e += 256) {
      const int tl = e / D, f = e % D;
      const float* xr = reinterpret_cast<const float*>(xs + (size_t)tl * RS);
      float acc = 0.f;
      for (int c = 0; c < D; ++c) acc = fmaf(xr[c], wsrc[(size_t)c * D + f], acc);
      if (t0 + tl < Tn) y[(((size_t)b * Tn + t0 + tl) * H + h) * D + f] = apply_phi(acc, phi);
    }
  }
}

}  // namespace

namespace {

constexpr int kComputeUnits = 256;   // MI355X

constexpr int feature_lds(int d, int rows) { return (d == 128 ? 2 * rows : d + rows) * (d * 2 + 16); }
// workgroups per compute unit (LDS, registers)
constexpr int resident(int lds) { return (160 * 1024 / lds) < kShare ? (160 * 1024 / lds) : kShare; }

// Tiles of one tensor: `places` workgroups for all of its (batch, head group) pairs, each walking a contiguous run of tiles (the
// matrix goes into LDS once per workgroup).
template <int D, int GH, int TT>
bool feature_args(const ConvParams& p, const void* wf, int group, int places, FeatureArgs& a, int& blocks) {
  const int ntiles = (p.T + TT - 1) / TT;
  const long long nbh = (long long)p.B * (p.H / GH);
  const long long per_bh = places / nbh > 0 ? places / nbh : 1;
  const int tpb = (int)((ntiles + per_bh - 1) / per_bh);
  // a workgroup addresses its own token range with 32-bit byte offsets
  if (((unsigned long long)tpb * TT + 16) * p.H * D * 2 >= (1ull << 31) || nbh > 65535) return false;
  a.x = (const bf16_t*)p.x; a.w = (const bf16_t*)p.w; a.halo = (const bf16_t*)p.halo; a.wf = (const bf16_t*)wf;
  a.y = (bf16_t*)p.y; a.tail = p.W > 1 ? (bf16_t*)p.tail_out : nullptr;
  a.Tn = p.T; a.H = p.H; a.group = group; a.W = p.W; a.tiles_per_block = tpb;
  a.runs = (ntiles + tpb - 1) / tpb;
  if ((unsigned long long)a.runs * nbh >= (1ull << 30)) return false;
  blocks = (int)(a.runs * nbh);
  return true;
}

// One tensor (k null), or queries and keys in one launch (GH2 > 0).
template <int D, int GH, int TT, int GH2, int TT2>
hipError_t launch_mfma(const ConvParams& p, const ConvParams* k, const void* wf, int group, hipStream_t stream) {
  constexpr int rows = TT * GH > TT2 * GH2 ? TT * GH : TT2 * GH2, lds = feature_lds(D, rows);
  constexpr int kPlaces = kComputeUnits * resident(lds);      // one round of workgroups
  FeatureArgs a, a2{};
  int first, second = 0;
  // the two tensors' workgroups in proportion to their elements
  const int mine = k ? (int)((long long)kPlaces * p.H / (p.H + k->H)) : kPlaces;
  if (!feature_args<D, GH, TT>(p, wf, group, mine, a, first)) return hipErrorInvalidValue;
  if constexpr (GH2 > 0)
    if (!feature_args<D, GH2, TT2>(*k, wf, 1, kPlaces - mine, a2, second)) return hipErrorInvalidValue;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(first + second), dim3(256), lds, stream, a, a2, first);
    return hipGetLastError();
  };
#define LAWCAT_KERNEL(ELU, WT) conv_feature_mfma_kernel<D, GH, TT, GH2, TT2, ELU, WT>
#define LAWCAT_LAUNCH(ELU, WT)                                       \
  {                                                                  \
    const hipError_t e = set_lds<LAWCAT_KERNEL(ELU, WT)>(lds);       \
    return e != hipSuccess ? e : launch(LAWCAT_KERNEL(ELU, WT));     \
  }
  if (p.W == 4) {
    if (p.phi == 1) LAWCAT_LAUNCH(true, 4)
    LAWCAT_LAUNCH(false, 4)
  }
  if (p.phi == 1) LAWCAT_LAUNCH(true, 0)
  LAWCAT_LAUNCH(false, 0)
#undef LAWCAT_LAUNCH
#undef LAWCAT_KERNEL
}

}  // namespace

hipError_t launch_conv_feature(const ConvParams& p, const void* wf, int group, hipStream_t stream) {
  if (p.bf16) {
    // four adjacent heads per workgroup where they share a matrix (wider contiguous rows), else one
    const bool four = group % 4 == 0;
    // rows per tile: 256 (four heads) or 128 at d = 64, 64 at d = 128: three workgroups to a compute unit in LDS and registers, where
    // tiles twice as long leave two.  Single heads at d = 64, 5003 tokens: 6.3 us as taken, 7.4 twice as long; the layer at d = 128,
    // 5003 tokens: 102.6 and 105.7
    if (p.d == 64) return four ? launch_mfma<64, 4, 64, 0, 0>(p, nullptr, wf, group, stream) : launch_mfma<64, 1, 128, 0, 0>(p, nullptr, wf, group, stream);
    return four ? launch_mfma<128, 4, 16, 0, 0>(p, nullptr, wf, group, stream) : launch_mfma<128, 1, 64, 0, 0>(p, nullptr, wf, group, stream);
  }
  const dim3 grid((p.T + kTile * kTilesPerBlock - 1) / (kTile * kTilesPerBlock), p.B * p.H);
  if (p.d == 64) {
    constexpr int lds = kTile * (64 + 2) * 4;
    hipLaunchKernelGGL(conv_feature_f32_kernel<64>, grid, dim3(256), lds, stream, (const float*)p.x, (const float*)p.w,
                       (const float*)p.halo, (const float*)wf, (float*)p.y, p.B, p.T, p.H, group, p.W, p.phi);
  } else {
    constexpr int lds = kTile * (128 + 2) * 4;
    hipLaunchKernelGGL(conv_feature_f32_kernel<128>, grid, dim3(256), lds, stream, (const float*)p.x, (const float*)p.w,
                       (const float*)p.halo, (const float*)wf, (float*)p.y, p.B, p.T, p.H, group, p.W, p.phi);
  }
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_conv_tail(p, stream);
}

hipError_t launch_conv_feature_pair(const ConvParams& q, const ConvParams& k, const void* wf, hipStream_t stream) {
  const int group = q.H / k.H;
  if (q.bf16) {
    const bool four = group % 4 == 0;
    if (q.d == 64) return four ? launch_mfma<64, 4, 64, 1, 128>(q, &k, wf, group, stream) : launch_mfma<64, 1, 128, 1, 128>(q, &k, wf, group, stream);
    return four ? launch_mfma<128, 4, 16, 1, 64>(q, &k, wf, group, stream) : launch_mfma<128, 1, 64, 1, 64>(q, &k, wf, group, stream);
  }
  const hipError_t e = launch_conv_feature(q, wf, group, stream);
  return e != hipSuccess ? e : launch_conv_feature(k, wf, 1, stream);
}

}  // namespace lawcat
