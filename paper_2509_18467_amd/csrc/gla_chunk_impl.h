// bf16 matrix-core prefill of the normalized gated linear attention (paper section 4.2)
// with the causal depthwise Conv1D of section 4.1 and the pointwise feature map fused into
// the load stage.  Included by one translation unit per head dimension.
//
// Algebra.  Split the sum over i in the state/output equations of section 4.2 at the start
// of a 16-token chunk.  With E_t = prod of alpha over the chunk's tokens up to t (per key
// channel) and a per-channel reference rho the output of token t in the chunk is
//   num_t = (q_t (.) E_t/rho) (rho (.) S_start) + sum_{i<=t} [(q_t (.) E_t/rho) . (k_i rho/E_i)] v_i
//   den_t = (q_t (.) E_t/rho) (rho (.) z_start) + sum_{i<=t} [(q_t (.) E_t/rho) . (k_i rho/E_i)]
// and the state after the chunk is S_end = diag(E_last) S_start + sum_i (k_i E_last/E_i)^T v_i.
// rho is 1 for a channel whose decay over the whole chunk stays above 2^-100 (then 1/E_i cannot overflow), and
// otherwise the decay up to the middle of the chunk (E of its eighth token), so that neither E_t/rho nor
// rho/E_i spans more than eight steps of decay.  A chunk in which every channel has rho = 1 (the usual case)
// skips the scaling of the state operand.
// All the products are bf16 MFMAs with fp32 accumulation.  The normalizer z is carried as one more
// (replicated) column tile of the state, updated by the same MFMAs against an all-ones value operand.
//
// Parallel decomposition.  One team of d/16 waves owns one (batch, kv head) and one segment of the sequence and walks it in granules
// of 64 tokens; a wave holds 16 value columns of the state in MFMA accumulators (and its share of z); the query heads of the group share
// k, v, the decay and the state.  With more than one segment a first pass computes each segment's state contribution and total
// decay, a small scan turns them into segment start states (or, with few segments, each workgroup of the output pass folds
// its predecessors' contributions itself), and the output pass starts from those.
//
// Output pass, head dim 64: a wave forms Q' and K' of one of the granule's four chunks and takes the outputs of that chunk, all value
// columns of them, so that they never leave it; only k (.) E_last/E and V go to the other waves, and the state at each chunk's start, as
// bf16 operands, comes back from them: two barriers a granule, and a wave's stores cover 64 bytes of a row.  With every wave forming 16
// columns of all outputs (scores and denominators shared per chunk, six barriers a granule, 32 bytes of a row per store) 32768 tokens
// of 32 heads on 8 took 107.4 us, now 96.7; 8192 46.5 and 43.3, 64 9.5 and 7.7.  What bounds it: the output pass moves 386 MB in 80 us at its
// quickest, 93 % of the rate of a large copy, in 85 to 92 on average; the state pass and the launches in between are the rest.
// Head dim 128: the state at four chunks' starts would fill the LDS, so each wave forms its 16 columns of all outputs.  z, scores and
// denominators of a granule come first, two (chunk, head) a wave, then outputs and state without a barrier: 16384 tokens of 32 heads
// on 8 127.5 -> 123 us, 5000 of 16 on 8 50.2 -> 46.6, 700 27.9 -> 26.3, 128K tokens 830 -> 800 (scores per chunk, by half of the waves
// while the others waited, z in all waves' registers).  Its stages do not overlap: the compute stage (5.9 of 14.3 us a granule) is
// bound by the vector ALUs, outputs and state (5.7) by LDS, 26 KB a wave and chunk.  Granules of 32 tokens in two sets of operands, the
// two waves of a SIMD in opposite stages, took 151 us.
// Long sequences with conv take a form of its own there (gla_wide.h: two workgroups of four waves a compute unit).
//
// Per-step decay is floored at 2^-13 so that eight steps of 1/alpha stay below 2^104; the floor changes
// a state by at most 2^-13 of what the step before it held.
#pragma once
#include <hip/hip_ext.h>

#include <algorithm>

#include "segment_scan.h"

namespace lawcat {
namespace chunk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kAlphaMin = 1.220703125e-4f;   // 2^-13
constexpr float kInvAlphaMax = 8192.f;         // 2^13
constexpr float kLog2AlphaMin = -13.f;
constexpr float kSafeDecay = 7.888609052210118e-31f;  // 2^-100: a chunk that decays less keeps the chunk-start reference
constexpr int kChunk = 16;

// MODE of the load stage
constexpr int kPlain = 0;     // q, k are already q-dot, k-dot (lawcat_gla_prefill)
constexpr int kConvId = 1;    // conv, identity feature map
constexpr int kConvElu = 2;   // conv, 1 + ELU

// Optional start/stop events of the output-pass kernel (measurement entry point only).
struct TraceEvents {
  hipEvent_t start, stop;
};

struct ChunkArgs {
  const bf16_t *q, *k, *v, *g, *wq, *wk, *q_halo, *k_halo;
  const float *S0, *z0;
  bf16_t* o;
  float* den_out;
  float* S_out;
  float* z_out;
  bf16_t *q_tail, *k_tail;
  float* ws;
  int* seg_live;   // one per workspace slot: written by the state pass, 0 = the segment's total decay is exactly zero in every channel
  // Sequences of different lengths packed along the token axis: device array of B + 1 row offsets, or null for B
  // sequences of T tokens each (nseg segments of seg_len, grid (nseg, B * Hkv)).  With it, T is the longest length and nseg the segment
  // count of that length: every sequence has nseg workspace slots, is cut by cut_sequence(), and `places` says which workgroup
  // takes which segment.
  const int* seq_start;
  int B, T, Hq, Hkv, W;
  int group;   // query heads per kv head (Hq / Hkv)
  int qh0;     // first query head, within its group, that this launch of the output pass covers (its z index: GR heads each)
  int most;    // most query heads that a workgroup of the output pass takes: 4, 2 or 1
  int seg_len, nseg;
  int per_head;     // packed batches: workgroups per kv head
  double inv_len;   // 1 / seg_len
  int places;       // which workgroup takes which segment
  int wide;    // head dim 128: the output pass in its form for many workgroups (gla_wide.h)
  int fold;    // few segments: the output pass folds its predecessors' contributions itself, there is no scan
  float gate_scale, eps;
};

// S_out, z_out are S0, z0
inline bool in_place(const ChunkArgs& a) { return a.S0 == a.S_out || a.z0 == a.z_out; }

// most segments before one whose contributions the output pass folds
template <int D> constexpr int kFoldMost = D == 64 ? 11 : 8;

// which workgroup takes which segment (see find_place)
constexpr int kDirect = 0, kInOrder = 1, kByLength = 2;

template <int D, int GR, int MODE>
struct Geo {
  static constexpr int NW = D / 16;          // waves per team: one per 16 value columns
  static constexpr int TEAM = 64 * NW;       // threads per team
  static constexpr int CH = D / 64;          // 64-channel slabs per row = waves per 16-token chunk in the load stage
  static constexpr int NTG = 64;             // tokens per granule (one load stage of the team)
  static constexpr int MCG = NTG / kChunk;   // chunks per granule
  static constexpr int RT = D / 16;          // 16-row tiles of the state (key channels)
  static constexpr int KS = D / 32;          // k-steps of a 16x16x32 MFMA over the key channels
  static constexpr int QRS = D * 2 + 8;      // LDS row stride (bytes) of token-major bf16 rows
  static constexpr int TRS = NTG * 2 + 8;    // LDS row stride (bytes) of channel-major bf16 rows
  // OWN: a wave keeps its chunk's Q', K' (see the top); S at each chunk's start, in MFMA operands, [chunk][16 value columns][k-step]
  // [64 lanes] x 16 B.
  static constexpr bool OWN = D == 64 && GR > 0, WIDE = false;
  static constexpr int kSn = 0;
  static constexpr int kSnChunk = D * D * 2;
  static constexpr int kQp = 0;
  static constexpr int kKp = kQp + GR * NTG * QRS;
  static constexpr int kKd = OWN ? MCG * kSnChunk : kKp + (GR > 0 ? NTG * QRS : 0);  // GR == 0: the state pass keeps no Q', K'
  static constexpr int kVt = kKd + D * TRS;
  static constexpr int kEb = kVt + D * TRS;
  static constexpr int kEf = kEb + MCG * D * 4;   // the reference rho of each chunk and channel, fp32
  static constexpr int kWl = kEf + MCG * D * 4;
  // conv weights (none without conv: 54.8 KB at head dim 64 would leave two workgroups a compute unit, 52.8 leave three), then
  static constexpr int kPs = kWl + (MODE == kPlain ? 0 : (GR + 1) * D * 16);   // shared scores: [chunk][head][64 lanes] x 16 B (4 high parts, 4 residuals)
  static constexpr int kDn = kPs + (OWN ? 0 : MCG * GR * 1024);    // shared denominators: [chunk][head][16 queries] fp32
  static constexpr int kZs = kDn + (OWN ? 0 : MCG * GR * 64);      // z at each chunk's start, bf16
  static constexpr int kFl = kZs + (GR > 0 ? MCG * D * 2 : 0);     // per load-stage wave: 1 if one of its channels uses the mid-chunk reference
  static constexpr int kBytes = kFl + 32;
  static constexpr int kSlot = D * D + 2 * D;  // floats per workspace slot: S | z | decay
};

__device__ inline float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ inline uint32_t pack2(float a, float b) {
  bf16x2 v = {(__bf16)a, (__bf16)b};  // v_cvt_pk_bf16_f32, round to nearest even
  return __builtin_bit_cast(uint32_t, v);
}
// value of the lane whose byte index (lane * 4) is given; callers form the index once, not per exchange (the
// generic shuffle recomputes it with half a dozen instructions every time)
__device__ inline float lane_get(int byte_index, float v) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(byte_index, __float_as_int(v)));
}
__device__ inline bf16x8 make8(uint2 a, uint2 b) { return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y)); }
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Raw input rows of one granule held in registers between the load and the compute stage:
// one dword = two adjacent channels of one token.  Index j is row tok0 - 3 + j: three rows of conv
// history (keys and queries only), then the patch's eight tokens.
template <int NQ>
struct Raw {
  uint32_t g[11];
  uint32_t k[11];
  uint32_t v[11];
  uint32_t q[NQ][11];
};

// Uniform (per workgroup) row addressing of one input tensor: a raw buffer descriptor over the rows of this
// batch element, starting at this head's columns.  A load whose byte offset falls outside [0, bytes) returns
// zero, which supplies the zero rows before the first token (their offsets wrap around to huge values) and
// past the last one without a branch.
struct RowSrc {
  __amdgpu_buffer_rsrc_t rsrc;
  const char* halo;   // nullable: first halo row of this batch, at this head's columns
  unsigned stride;    // bytes per token row
  unsigned width;     // bytes of a row that belong to this workgroup's heads
};

__device__ inline RowSrc make_row_src(const char* base, const char* halo, unsigned stride, int T, unsigned width) {
  // stride field 0 (raw buffer); 0x00020000 = 32-bit data format of gfx9-family descriptors.  The host has
  // checked that (T + 4) * stride fits 32 bits.
  const unsigned bytes = (unsigned)(T - 1) * stride + width;
  return RowSrc{__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000), halo, stride, width};
}

// Rows t0-3 .. t0+7 (+ this thread's patch offset, folded into voff) of one tensor.  t0 is uniform.  HALO: it may be 0 (elsewhere the
// halo's branch would only lead the compiler to wait for rows in flight: 98.4 -> 96.8 us at 32768 tokens of 64).
template <bool CONV, bool HALO>
__device__ inline void load_rows(const RowSrc& s, int t0, int tl0, int W, unsigned voff, unsigned coff,
                                 uint32_t (&raw)[11]) {
#pragma unroll
  for (int j = CONV ? 0 : 3; j < 11; ++j)
    raw[j] = __builtin_amdgcn_raw_buffer_load_b32(s.rsrc, (int)(voff + (unsigned)(t0 - 3 + j) * s.stride), 0, 0);
  if (HALO && t0 == 0 && s.halo != nullptr && tl0 == 0) {
    // the rows before the first token come from the caller's halo (oldest row first, W-1 rows), read through a
    // descriptor of its own with 32-bit offsets (64-bit row addresses would be kept in registers across the
    // whole granule loop for this one use)
    const __amdgpu_buffer_rsrc_t hr =
        __builtin_amdgcn_make_buffer_rsrc((void*)s.halo, 0, (int)((unsigned)(W - 2) * s.stride + s.width), 0x00020000);
#pragma unroll
    for (int j = 0; j < 3; ++j)
      if (j - 3 >= -(W - 1))
        raw[j] = __builtin_amdgcn_raw_buffer_load_b32(hr, (int)((unsigned)(W - 4 + j) * s.stride + coff), 0, 0);
  }
}

// conv (section 4.1 sum over delta) + feature map on the 8 tokens x 2 channels of a patch.
// For MODE kConvElu the weights arrive pre-multiplied by log2(e): with y' = y log2(e),
// 1 + ELU(y) = ln2 * max(y', 0) + min(2^y', 1).
template <int MODE>
__device__ inline void conv_phi(const uint32_t (&raw)[11], const float* wts /*[2][4] in LDS*/, float (&y)[8][2]) {
  if (MODE == kPlain) {
#pragma unroll
    for (int i = 0; i < 8; ++i) { y[i][0] = bf_lo(raw[i + 3]); y[i][1] = bf_hi(raw[i + 3]); }
    return;
  }
  const floatx4 w0 = *reinterpret_cast<const floatx4*>(wts);
  const floatx4 w1 = *reinterpret_cast<const floatx4*>(wts + 4);
  float x0[11], x1[11];
#pragma unroll
  for (int j = 0; j < 11; ++j) { x0[j] = bf_lo(raw[j]); x1[j] = bf_hi(raw[j]); }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float a0 = w0[0] * x0[i + 3];
    a0 = fmaf(w0[1], x0[i + 2], a0); a0 = fmaf(w0[2], x0[i + 1], a0); a0 = fmaf(w0[3], x0[i], a0);
    float a1 = w1[0] * x1[i + 3];
    a1 = fmaf(w1[1], x1[i + 2], a1); a1 = fmaf(w1[2], x1[i + 1], a1); a1 = fmaf(w1[3], x1[i], a1);
    if (MODE == kConvElu) {
      // med3(x, 0, 1) of a non-negative x is min(x, 1); written this way it folds into the clamp bit of v_exp_f32
      a0 = fmaf(fmaxf(a0, 0.f), kLn2, __builtin_amdgcn_fmed3f(fast_exp2(a0), 0.f, 1.f));
      a1 = fmaf(fmaxf(a1, 0.f), kLn2, __builtin_amdgcn_fmed3f(fast_exp2(a1), 0.f, 1.f));
    }
    y[i][0] = a0;
    y[i][1] = a1;
  }
}

// What a wave keeps of its chunk between the stages (head dim 64): Q' as MFMA operands, masked scores as high parts and residuals
template <int D, int NQ>
struct Chunk {
  bf16x8 q[NQ][D / 32];
  uint4 p[NQ];
};

// Head dim 128, output pass, four waves: granules of 32 tokens, 32 value columns of the state a wave.  Two workgroups share a compute
// unit, so that one's loads and vector instructions run beside the other's MFMA stage; see gla_wide.h.
template <int GR, int MODE>
struct WideGeo {
  static constexpr int D = 128, NW = 4, TEAM = 64 * NW, CH = 2, NTG = 32, MCG = NTG / kChunk;
  static constexpr int RT = D / 16, KS = D / 32, CT = 2;      // CT: tiles of value columns a wave
  static constexpr int QRS = D * 2 + 8, TRS = NTG * 2 + 8;
  static constexpr bool OWN = false, WIDE = true;
  static constexpr int HW = (GR + 1) / 2;                     // heads whose scores a wave sums up
  static constexpr int kQp = 0;
  static constexpr int kKd = kQp + GR * NTG * QRS;            // (K' passes through the last head's Q' rows)
  static constexpr int kVt = kKd + D * TRS;
  static constexpr int kEb = kVt + D * TRS;
  static constexpr int kEf = kEb + MCG * D * 4;
  static constexpr int kWl = kEf + MCG * D * 4;
  static constexpr int kPs = kWl + (MODE == kPlain ? 0 : (GR + 1) * D * 16);   // parts of scores, then scores: [chunk][head][64 lanes] x 16 B
  static constexpr int kZs = kPs + MCG * GR * 1024;
  static constexpr int kDn = kZs + MCG * D * 2;               // denominators: [chunk][head][16 queries] fp32
  static constexpr int kFl = kDn + MCG * GR * 64;
  static constexpr int kBytes = kFl + 32;
  static constexpr int kSlot = D * D + 2 * D;
  static_assert(2 * ((kBytes + 1279) / 1280 * 1280) <= 160 * 1024);
};
// Scores of a chunk over the wave's 64 channels, of the heads that it sums up
template <int GR>
struct Part { floatx4 p[(GR + 1) / 2]; };

// Causal scores of a chunk, P^T[key 4 g4 + i][query n] for key <= query, as a k = 32 operand: slots 0..3 the high parts, 4..7 the
// residuals of this lane's 4 keys.  The weights of the few nearest keys dominate the output, so their bf16 rounding would not
// average out.
__device__ inline uint4 pack_scores(floatx4 pt, int g4, int n) {
#pragma unroll
  for (int i = 0; i < 4; ++i) pt[i] = (4 * g4 + i <= n) ? pt[i] : 0.f;
  const uint32_t ph0 = pack2(pt[0], pt[1]), ph1 = pack2(pt[2], pt[3]);
  const uint32_t pl0 = pack2(pt[0] - bf_lo(ph0), pt[1] - bf_hi(ph0));
  const uint32_t pl1 = pack2(pt[2] - bf_lo(ph1), pt[3] - bf_hi(ph1));
  return make_uint4(ph0, ph1, pl0, pl1);
}

template <int D, int GR, int MODE, bool OUTPUT, typename GEO = Geo<D, GR, MODE>>
struct Kernel {
  using G = GEO;
  static constexpr bool OWN = OUTPUT && G::OWN;
  static constexpr bool CONV = MODE != kPlain;
  static constexpr int NQ = OUTPUT ? GR : 1;

  // ---- HBM -> registers: the raw rows of the granule starting at token t0
  // Gate logits, keys and values are issued one stage ahead (under the MFMA stage); the query heads are fetched
  // inside the compute stage, two heads ahead of their use (fetch_head).  Prefetching query heads a stage ahead
  // as well measured slower at every count tried (larger bursts into the memory pipeline, more registers live
  // across the MFMA stage).
  template <bool FIRST>     // the granule may be the sequence's first
  __device__ static inline void fetch(Raw<NQ>& raw, const RowSrc& srcK, const RowSrc& srcG, const RowSrc& srcV,
                                      int t0, int tl0, unsigned coff, int W) {
    const unsigned voffkv = (unsigned)tl0 * srcK.stride + coff;
    load_rows<false, false>(srcG, t0, tl0, 1, voffkv, coff, raw.g);
    load_rows<CONV, CONV && FIRST>(srcK, t0, tl0, W, voffkv, coff, raw.k);
    load_rows<false, false>(srcV, t0, tl0, 1, voffkv, coff, raw.v);
  }

  // One query head of the granule at t0.
  template <bool FIRST>
  __device__ static inline void fetch_head(Raw<NQ>& raw, const RowSrc& srcQ, int hh, int t0, int tl0,
                                           unsigned coff, int W) {
    load_rows<CONV, CONV && FIRST>(srcQ, t0, tl0, W, (unsigned)tl0 * srcQ.stride + coff + hh * D * 2, coff + hh * D * 2, raw.q[hh]);
  }

  // ---- registers -> LDS operands: gate products, conv + phi, scaling by the decay, bf16 packing
  template <bool EDGE, bool GS1, typename OWN_T>
  __device__ static inline void compute(Raw<NQ>& raw, const RowSrc& srcQ, unsigned coff, int W, unsigned char* smem,
                                        const float* wl, int t0, int s1, int tl0, int c0, int mcw, int th,
                                        float gate_scale, OWN_T& own) {
    const int tok0 = t0 + tl0;
    const int idx32 = (int)(((threadIdx.x & 63) ^ 32) << 2);  // the lane that holds the other half of the chunk
    // OWN: rows of the wave's chunk in LDS on their way from patches to operands, where S of the same chunk will be: nothing else
    // reads either
    // WIDE: this wave's part, 64 channels of its chunk, of the last head's Q' rows
    unsigned char* rows;
    if constexpr (G::WIDE) rows = smem + G::kQp + ((GR - 1) * G::NTG + kChunk * mcw) * G::QRS;
    else rows = smem + G::kSn + mcw * G::kSnChunk;
    // query heads are fetched two heads ahead of their use
    if (OUTPUT) fetch_head<EDGE>(raw, srcQ, 0, t0, tl0, coff, W);
    if (OUTPUT && NQ > 1) fetch_head<EDGE>(raw, srcQ, 1, t0, tl0, coff, W);
    // keys first: conv + phi into kf, which the gate loop below scales in place by 1/E as it goes
    float kf[8][2];
    conv_phi<MODE>(raw.k, wl + ((size_t)GR * D + c0) * 4, kf);
    float E[8][2];
    float run[2] = {1.f, 1.f}, irun[2] = {1.f, 1.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        const float gl = ch ? bf_hi(raw.g[i + 3]) : bf_lo(raw.g[i + 3]);
        float u = fast_exp2(-kLog2e * gl);  // exp(-g)
        float al, ia;
        if (!GS1) u = fminf(u, 1e30f);      // (else an infinity ends at the floor too)
        if (GS1) {
          ia = fminf(1.f + u, kInvAlphaMax);  // 1/sigmoid(g) = 1 + exp(-g)
          al = fmaxf(fast_rcp(1.f + u), kAlphaMin);
        } else {
          const float a2 = fmaxf(-gate_scale * fast_log2(1.f + u), kLog2AlphaMin);
          al = fast_exp2(a2);
          ia = fast_exp2(-a2);
        }
        if (EDGE && tok0 + i >= s1) { al = 1.f; ia = 1.f; }
        run[ch] *= al;
        irun[ch] *= ia;
        E[i][ch] = run[ch];
        kf[i][ch] = (EDGE && tok0 + i >= s1) ? 0.f : kf[i][ch] * irun[ch];
      }
    }
    // Reference rho of the in-chunk factors Q' = q E_t / rho, K' = k rho / E_i.  A lane's running products start
    // at its own half of the chunk; the other half lives 32 lanes away, and one exchange gives both halves'
    // totals.  Usual case (the whole chunk decays by less than 2^100): rho = 1, the second half multiplies in the
    // first half's total.  Otherwise rho = the decay over the first half: the second half is already relative
    // to it, and the first half needs run_t / run_7 and run_7 / run_i, with this lane's own totals.
    float pre[2], ipre[2], kdf[2];
    {
      float elast[2], rho[2];
      bool mid = false;
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        const float ot = lane_get(idx32, run[ch]);
        const float t0 = th ? ot : run[ch];   // decay over the first half
        const float t1 = th ? run[ch] : ot;   // decay over the second half
        elast[ch] = t0 * t1;
        const bool safe = elast[ch] >= kSafeDecay;
        pre[ch] = safe ? (th ? t0 : 1.f) : (th ? 1.f : irun[ch]);
        ipre[ch] = safe ? (th ? fast_rcp(t0) : 1.f) : (th ? 1.f : run[ch]);
        kdf[ch] = safe ? elast[ch] : t1;      // from the reference point on to the end of the chunk
        rho[ch] = safe ? 1.f : t0;
        mid |= !safe;
      }
      if (th == 0) {
        float* eb = reinterpret_cast<float*>(smem + G::kEb) + mcw * D + c0;
        *reinterpret_cast<float2*>(eb) = make_float2(kdf[0], kdf[1]);   // E_last / rho
        float* ef = reinterpret_cast<float*>(smem + G::kEf) + mcw * D + c0;
        *reinterpret_cast<float2*>(ef) = make_float2(rho[0], rho[1]);
      }
      if (OUTPUT) {
        const bool any_mid = __builtin_amdgcn_ballot_w64(mid) != 0;
        if ((threadIdx.x & 63) == 0) *reinterpret_cast<int*>(smem + G::kFl + (threadIdx.x >> 6) * 4) = any_mid ? 1 : 0;
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // keep the sections apart: bounds live registers
    // keys: K' = k/E (in-chunk scores) and Kdec = k E_last/E (state update)
    unsigned char* kp;
    if constexpr (OWN || G::WIDE) kp = rows + 8 * th * G::QRS + c0 * 2;
    else kp = smem + G::kKp + tl0 * G::QRS + c0 * 2;
    float kdv[8][2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        E[i][ch] *= pre[ch];
        const float kprime = kf[i][ch] * ipre[ch];
        kf[i][ch] = kprime;
        kdv[i][ch] = kprime * kdf[ch];
      }
      if (OUTPUT) *reinterpret_cast<uint32_t*>(kp + i * G::QRS) = pack2(kf[i][0], kf[i][1]);
    }
    // rows of the channel-major arrays are 8-byte aligned: 8-byte writes
    unsigned char* kdp = smem + G::kKd + c0 * G::TRS + tl0 * 2;
    *reinterpret_cast<uint2*>(kdp) = make_uint2(pack2(kdv[0][0], kdv[1][0]), pack2(kdv[2][0], kdv[3][0]));
    *reinterpret_cast<uint2*>(kdp + 8) = make_uint2(pack2(kdv[4][0], kdv[5][0]), pack2(kdv[6][0], kdv[7][0]));
    *reinterpret_cast<uint2*>(kdp + G::TRS) = make_uint2(pack2(kdv[0][1], kdv[1][1]), pack2(kdv[2][1], kdv[3][1]));
    *reinterpret_cast<uint2*>(kdp + G::TRS + 8) = make_uint2(pack2(kdv[4][1], kdv[5][1]), pack2(kdv[6][1], kdv[7][1]));
    __builtin_amdgcn_sched_barrier(0);
    // values, transposed to channel-major (rows past the end were fetched as zero)
    uint32_t v0[4], v1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t ra = raw.v[3 + 2 * i], rb = raw.v[4 + 2 * i];
      v0[i] = __builtin_amdgcn_perm(rb, ra, 0x05040100u);  // low halves:  ra.lo | rb.lo << 16
      v1[i] = __builtin_amdgcn_perm(rb, ra, 0x07060302u);  // high halves: ra.hi | rb.hi << 16
    }
    unsigned char* vp = smem + G::kVt + c0 * G::TRS + tl0 * 2;
    *reinterpret_cast<uint2*>(vp) = make_uint2(v0[0], v0[1]);
    *reinterpret_cast<uint2*>(vp + 8) = make_uint2(v0[2], v0[3]);
    *reinterpret_cast<uint2*>(vp + G::TRS) = make_uint2(v1[0], v1[1]);
    *reinterpret_cast<uint2*>(vp + G::TRS + 8) = make_uint2(v1[2], v1[3]);
    if (OUTPUT) {
      const int g4 = (threadIdx.x >> 4) & 3, n = threadIdx.x & 15;
      constexpr int KO = G::WIDE ? 2 : G::KS;      // k-steps over what the wave holds
      bf16x8 kop[KO], qop[G::WIDE ? 2 : 1][KO];
      const int slab = G::WIDE ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) % G::CH : 0;
      auto operands = [&](bf16x8 (&o)[KO], const unsigned char* rows) {
        __builtin_amdgcn_wave_barrier();   // LDS serves one wave's requests in order: the rows are complete here, and read before they change
#pragma unroll
        for (int ks = 0; ks < KO; ++ks) {
          const unsigned char* p = rows + n * G::QRS + g4 * 8 + 64 * ks + (G::WIDE ? 128 * slab : 0);
          o[ks] = make8(*reinterpret_cast<const uint2*>(p), *reinterpret_cast<const uint2*>(p + 32));
        }
        __builtin_amdgcn_wave_barrier();
      };
      auto scores = [&](int hh) {
        floatx4 pt = {0.f, 0.f, 0.f, 0.f};
        if constexpr (G::WIDE) {
          // over the wave's 64 channels: one of the two waves of a chunk sums a head's up, the other hands it its part
#pragma unroll
          for (int ks = 0; ks < KO; ++ks) pt = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[ks], qop[hh & 1][ks], pt, 0, 0, 0);
          if (hh / G::HW == slab) own.p[hh % G::HW] = pt;
          else *reinterpret_cast<floatx4*>(smem + G::kPs + (mcw * GR + hh) * 1024 + (threadIdx.x & 63) * 16) = pt;
        } else {
#pragma unroll
          for (int ks = 0; ks < G::KS; ++ks) pt = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[ks], own.q[hh][ks], pt, 0, 0, 0);
          own.p[hh] = pack_scores(pt, g4, n);
        }
      };
      if constexpr (OWN || G::WIDE) operands(kop, rows);
      // queries: conv + phi, times E
#pragma unroll
      for (int hh = 0; hh < NQ; ++hh) {
        __builtin_amdgcn_sched_barrier(0);
        if (hh + 2 < NQ) fetch_head<EDGE>(raw, srcQ, hh + 2, t0, tl0, coff, W);
        float qf[8][2];
        conv_phi<MODE>(raw.q[hh], wl + ((size_t)hh * D + c0) * 4, qf);
        unsigned char* qp = (OWN ? rows + 8 * th * G::QRS : smem + G::kQp + (hh * G::NTG + tl0) * G::QRS) + c0 * 2;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          *reinterpret_cast<uint32_t*>(qp + i * G::QRS) = pack2(qf[i][0] * E[i][0], qf[i][1] * E[i][1]);
        if constexpr (OWN) {
          operands(own.q[hh], rows);
          if (hh > 0) scores(hh - 1);
        } else if constexpr (G::WIDE) {
          operands(qop[hh & 1], smem + G::kQp + (hh * G::NTG + kChunk * mcw) * G::QRS);
          if (hh > 0) scores(hh - 1);
        }
      }
      if constexpr (OWN || G::WIDE) scores(NQ - 1);
    }
    // vmcnt(0): every row has been used, nothing is in flight; said so that the compiler, which merges what is in flight in the four
    // forms of this function, does not wait after it, or before the last of them, for the next granule's rows and for all stores.  (The
    // count of exports, of which there are none, keeps it from moving the four waits to one behind where they merge.)
    __builtin_amdgcn_s_waitcnt(0x0F70 - (EDGE ? 0x20 : 0) - (GS1 ? 0x10 : 0));
  }
  // ---- state pass only: registers -> LDS operands for S_segment = sum_i (k_i (.) D_i)^T v_i, where D_i is the
  // decay from token i to the END of the segment.  The segment is walked backwards, so D_i is a product of
  // (suffix inside the 8-token patch) x (second half of the chunk) x (later chunks of the granule) x (later
  // granules, `rgran`), all <= 1, and the accumulators never need rescaling.  Contains one team barrier.
  template <bool EDGE, bool GS1>
  __device__ static inline void compute_state(const Raw<NQ>& raw, unsigned char* smem, const float* wl, int t0,
                                              int s1, int tl0, int c0, int mcw, int th, float gate_scale,
                                              float (&rgran)[2]) {
    const int tok0 = t0 + tl0;
    const int idx32 = (int)(((threadIdx.x & 63) ^ 32) << 2);  // the lane that holds the other half of the chunk
    float al[8][2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        const float gl = ch ? bf_hi(raw.g[i + 3]) : bf_lo(raw.g[i + 3]);
        float u = fast_exp2(-kLog2e * gl);  // exp(-g)
        if (!GS1) u = fminf(u, 1e30f);
        float a1;
        if (GS1) a1 = fmaxf(fast_rcp(1.f + u), kAlphaMin);
        else a1 = fast_exp2(fmaxf(-gate_scale * fast_log2(1.f + u), kLog2AlphaMin));
        if (EDGE && tok0 + i >= s1) a1 = 1.f;
        al[i][ch] = a1;
      }
    }
    // exclusive suffix products inside the patch, then to the end of the chunk
    float suf[8][2], ptot[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      float r = 1.f;
#pragma unroll
      for (int i = 7; i >= 0; --i) { suf[i][ch] = r; r *= al[i][ch]; }
      ptot[ch] = r;
    }
    float btot[2], tail[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      const float ot = lane_get(idx32, ptot[ch]);
      tail[ch] = th ? 1.f : ot;               // first half of the chunk is also decayed by the second half
      btot[ch] = th ? ot * ptot[ch] : ptot[ch] * ot;
    }
    float* ebp = reinterpret_cast<float*>(smem + G::kEb);
    if (th == 0) *reinterpret_cast<float2*>(ebp + mcw * D + c0) = make_float2(btot[0], btot[1]);
    __syncthreads();
    // decay of the later chunks of this granule and of everything after the granule
    float carry[2] = {rgran[0] * tail[0], rgran[1] * tail[1]};
#pragma unroll
    for (int m = G::MCG - 1; m >= 0; --m) {
      const float2 e = *reinterpret_cast<const float2*>(ebp + m * D + c0);
      if (m > mcw) { carry[0] *= e.x; carry[1] *= e.y; }
      rgran[0] *= e.x;
      rgran[1] *= e.y;
    }
    __builtin_amdgcn_sched_barrier(0);
    float kf[8][2];
    conv_phi<MODE>(raw.k, wl + ((size_t)GR * D + c0) * 4, kf);
    float kdv[8][2];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        const float kk = (EDGE && tok0 + i >= s1) ? 0.f : kf[i][ch];
        kdv[i][ch] = kk * (suf[i][ch] * carry[ch]);
      }
    unsigned char* kdp = smem + G::kKd + c0 * G::TRS + tl0 * 2;
    *reinterpret_cast<uint2*>(kdp) = make_uint2(pack2(kdv[0][0], kdv[1][0]), pack2(kdv[2][0], kdv[3][0]));
    *reinterpret_cast<uint2*>(kdp + 8) = make_uint2(pack2(kdv[4][0], kdv[5][0]), pack2(kdv[6][0], kdv[7][0]));
    *reinterpret_cast<uint2*>(kdp + G::TRS) = make_uint2(pack2(kdv[0][1], kdv[1][1]), pack2(kdv[2][1], kdv[3][1]));
    *reinterpret_cast<uint2*>(kdp + G::TRS + 8) = make_uint2(pack2(kdv[4][1], kdv[5][1]), pack2(kdv[6][1], kdv[7][1]));
    uint32_t v0[4], v1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t ra = raw.v[3 + 2 * i], rb = raw.v[4 + 2 * i];
      v0[i] = __builtin_amdgcn_perm(rb, ra, 0x05040100u);
      v1[i] = __builtin_amdgcn_perm(rb, ra, 0x07060302u);
    }
    unsigned char* vp = smem + G::kVt + c0 * G::TRS + tl0 * 2;
    *reinterpret_cast<uint2*>(vp) = make_uint2(v0[0], v0[1]);
    *reinterpret_cast<uint2*>(vp + 8) = make_uint2(v0[2], v0[3]);
    *reinterpret_cast<uint2*>(vp + G::TRS) = make_uint2(v1[0], v1[1]);
    *reinterpret_cast<uint2*>(vp + G::TRS + 8) = make_uint2(v1[2], v1[3]);
  }
};

// x / most for 0 <= x < 2^31, most >= 64: the quotient is off by less than 2^-20, and x + 1/2 lies 1 / (2 most) from the next whole multiple
__device__ inline int over(int x, double inv_most) { return (int)(((double)x + 0.5) * inv_most); }

// What workgroup (x, y) of a packed batch works on (uniform): sequence and segment; seg < 0: nothing.
//   kDirect: segment x of sequence y / Hkv, as where all sequences are equally long; shorter ones leave workgroups without work.
//   kInOrder: 64 lanes look at 64 sequences at a time: sequence b has those from first row / seg_len + b on (no more tokens lie before it
//     than first row / seg_len segments hold, and each of the b sequences rounds up once, so these ranges do not overlap, whatever the
//     lengths; a few at their ends have nothing to do).
//   kByLength (up to 64 sequences, one per lane): the longest segments first (workgroups are placed in order, and those
//     past what the chip holds at once should be the shortest ones), a kv head's after the other's, an odd number each, so that the
//     segments of all heads spread alike over the eight dies, and no workgroup without work among them: one that leaves at
//     once still takes a place in turn, and those behind it wait for that place (24 sequences, 26K tokens: the last began 57 us late).
struct Place { int hk, b, seg, T, nseg, len, row0; };
__device__ inline void cut_place(const ChunkArgs& a, Place& p) {
  // cut_sequence(), with a division only where it matters
  p.nseg = over(p.T + a.seg_len - 1, a.inv_len);
  if (p.nseg > 1 && a.seg_len > 64) p.len = cut_sequence(p.T, a.seg_len).len;
}
__device__ inline Place find_place(const ChunkArgs& a, int l) {
  const int* seq_start = a.seq_start;
  int row = 0, end = 0, at, lane;
  Place p{(int)blockIdx.y, 0, (int)blockIdx.x, 0, 0, a.seg_len, 0};
  if (a.places == kByLength) {
    int n = 0;
    float len = 0.f;       // about how long its segments are
    if (l < a.B) {
      row = seq_start[l];
      end = seq_start[l + 1];
      n = over(end - row + a.seg_len - 1, a.inv_len);
      len = (float)(end - row) * __builtin_amdgcn_rcpf((float)n);
    }
    int first = 0, all = 0;
#pragma unroll 4
    for (int j = 0; j < ((a.B + 3) & ~3); ++j) {      // (lanes past the last sequence hold none)
      const float lj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(len), j));
      const int nj = __builtin_amdgcn_readlane(n, j);
      first += ((lj > len) | ((lj == len) & (j < l))) ? nj : 0;
      all += nj;
    }
    const unsigned odd = all | 1;
    p.hk = blockIdx.x / odd;
    const int e = blockIdx.x - p.hk * odd;
    if (p.hk >= a.Hkv || e >= all) {
      p.seg = -1;
      return p;
    }
    lane = __builtin_ctzll(__builtin_amdgcn_ballot_w64(first <= e && e < first + n));
    p.seg = e - __builtin_amdgcn_readlane(first, lane);
    p.b = lane;
  } else {
    const int e = blockIdx.x;
    int lo = 0, n = a.B, cnt;
    do {
      const int stride = (n + 63) / 64, i = lo + l * stride;
      const bool in = l * stride < n;
      if (in) { row = seq_start[i]; end = seq_start[i + 1]; }
      at = over(row, a.inv_len) + i;
      cnt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(in && at <= e));
      lo += (cnt - 1) * stride;
      n = min(stride, a.B - lo);
    } while (n > 1);
    lane = cnt - 1;
    p.b = lo;
    p.seg = e - __builtin_amdgcn_readlane(at, lane);
  }
  p.row0 = __builtin_amdgcn_readlane(row, lane);
  p.T = __builtin_amdgcn_readlane(end, lane) - p.row0;
  cut_place(a, p);
  return p;
}

// The conv cache of a workgroup's heads: the last W - 1 raw rows of [halo ; x].
template <int D>
__device__ inline void store_tails(const ChunkArgs& a, int b, int hk, int qh0, int heads, bool keeps, int T, size_t row0, int tid, int threads) {
  const int Wm = a.W - 1;
  for (int e = tid; e < (heads + (keeps ? 1 : 0)) * Wm * D; e += threads) {
    const int c = e % D, r = (e / D) % Wm, hh = e / (D * Wm);
    const bool isq = hh < heads;
    bf16_t* dst = isq ? a.q_tail : a.k_tail;
    if (dst == nullptr) continue;
    const int H = isq ? a.Hq : a.Hkv, head = isq ? hk * a.group + qh0 + hh : hk;
    const bf16_t* x = isq ? a.q : a.k;
    const bf16_t* halo = isq ? a.q_halo : a.k_halo;
    const int src = T - Wm + r;
    bf16_t val = 0;
    if (src >= 0) val = x[((row0 + src) * H + head) * D + c];
    else if (halo != nullptr) val = halo[(((size_t)b * Wm + (Wm + src)) * H + head) * D + c];
    dst[(((size_t)b * Wm + r) * H + head) * D + c] = val;
  }
}

// One or two query heads, no conv: registers and LDS for three workgroups a compute unit.  Calls of more than 512 workgroups, three / two
// to a unit, us: 8 heads of 64, 200 sequences of 64 tokens 21.4 / 24.3, 800 81.2 / 92.4, 96 of 300 44.8 / 47.0 (256 of 300, where two make
// whole rounds, 106.3 / 102.6); 16 on 8, 29.6 / 30.8, 97.3 / 101.3, 52.3 / 56.0 (129.4 / 126.3).  Up to 512 both take the same.
template <int D, int GR, int MODE, bool OUTPUT> constexpr bool three_share = OUTPUT && D == 64 && GR <= 2 && MODE == kPlain;

// One workgroup = one team of d/16 waves.  At head dim 64 two workgroups share a compute unit (256 VGPRs each).
template <int D, int GR, int MODE, bool OUTPUT>
__global__ void __launch_bounds__(D * 4, D == 64 ? (three_share<D, GR, MODE, OUTPUT> ? 3 : 2) : 1)
    gla_chunk_kernel(const ChunkArgs a) {
  using KK = Kernel<D, GR, MODE, OUTPUT>;
  using G = Geo<D, GR, MODE>;
  constexpr bool CONV = MODE != kPlain, OWN = KK::OWN, kThree = three_share<D, GR, MODE, OUTPUT>;
  static_assert(!kThree || 3 * ((G::kBytes + 1279) / 1280 * 1280) <= 160 * 1024);      // (LDS is given out in pieces of 1280 bytes)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_all[];
  unsigned char* smem = smem_all;
  const int tid = threadIdx.x;
  // the wave index is wave-uniform: keep it in a scalar register so that everything that depends on it
  // (LDS bases, branches) is uniform control flow and scalar address math
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;   // lane
  const int g4 = l >> 4;    // MFMA lane group
  const int n = l & 15;     // MFMA row/column within a tile
  // this workgroup's sequence (first row in the packed tensors, length, segments; token indices below are relative to row0), kv head
  // and segment
  Place p{0, 0, (int)blockIdx.x, a.T, a.nseg, a.seg_len, 0};
  size_t row0;
  if (__builtin_expect(a.places == kDirect, 1)) {
    p.b = blockIdx.y / a.Hkv;
    p.hk = blockIdx.y - p.b * a.Hkv;
    row0 = (size_t)p.b * a.T;
    if (a.seq_start != nullptr) {
      p.row0 = a.seq_start[p.b];
      p.T = a.seq_start[p.b + 1] - p.row0;
      cut_place(a, p);
      row0 = (size_t)p.row0;
    }
  } else {
    p = find_place(a, l);
    if (p.seg < 0) return;      // (the whole team, before the first barrier)
    row0 = (size_t)__builtin_amdgcn_readfirstlane(p.row0);
  }
  // (left in vector registers, as divisions leave them, they make every load of the state pass without conv a loop over lanes that
  // looks for equal descriptors: 16384 tokens, 8 heads, 13.5 us instead of 10.7)
  auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  const int hk = uniform(p.hk), b = uniform(p.b), seg = uniform(p.seg), T = uniform(p.T), nseg = uniform(p.nseg), seg_len = uniform(p.len);
  const int bh = b * a.Hkv + hk;
  const size_t slot0 = (size_t)bh * a.nseg;      // workspace slot of this head's first segment
  const int qh0 = OUTPUT ? a.qh0 + (int)blockIdx.z * GR : 0;   // first query head, within its group, of this workgroup
  const bool keeps = qh0 == 0;   // of the workgroups of a group: the one that stores the final state and the keys' cache
  const int nseg_pass = OUTPUT ? nseg : nseg - 1;  // the first pass skips the last segment
  // workgroups past a sequence's last segment (packed batches) have nothing to do either
  if (seg >= nseg_pass) return;
  const int s0 = seg * seg_len;
  const int s1 = min(T, s0 + seg_len);

  // load-stage patch of this thread: 8 tokens x 2 channels
  const int cp = l & 31, th = l >> 5;
  const int mcw = w / G::CH;                       // chunk of the granule this wave loads
  const int c0 = 64 * (w % G::CH) + 2 * cp;        // first of the two channels
  const int tl0 = kChunk * mcw + 8 * th;           // first token of the patch within the granule

  // Output pass: did the scan run for this head?  It leaves the workspace untouched when no segment of the head
  // passes anything on (every total decay exactly zero): then a segment starts from its predecessor's
  // contribution as the state pass wrote it, the first from S0, z0.  With few segments (fold): lane j, whether segment j, before
  // this one, passes anything on.  The prologue's loads are issued in the order in which they are waited for: these, the conv
  // weights, the start state, the first granule's rows.
  int live_any = 0;
  if (OUTPUT) {
    if (a.fold) live_any = l >= seg || a.seg_live[slot0 + l] != 0;
    else
      for (int j = tid; j < nseg - 1; j += G::TEAM) live_any |= a.seg_live[slot0 + j];
  }
  // ... and z and decay of every segment before this one
  constexpr int kZd = OUTPUT ? (kFoldMost<D> * 2 * D + G::TEAM - 1) / G::TEAM : 1;
  static_assert(!OUTPUT || kFoldMost<D> * 2 * D * 4 <= G::kWl);
  float zraw[kZd];
  if (OUTPUT && a.fold) {
#pragma unroll
    for (int j = 0; j < kZd; ++j) {
      const int e = tid + j * G::TEAM;
      zraw[j] = e < seg * 2 * D ? a.ws[(slot0 + e / (2 * D)) * G::kSlot + D * D + e % (2 * D)] : 0.f;
    }
  }

  float* wl = reinterpret_cast<float*>(smem + G::kWl);
  // conv weights as fp32 [head][channel][4 taps], taps beyond W zero; row GR is the key head.  All of a thread's loads are issued
  // here (a channel's four taps in one) and used below, after the granule's and the state's.
  constexpr int kRows = OUTPUT ? GR + 1 : 1, kWeights = (kRows * D + G::TEAM - 1) / G::TEAM;   // channels per thread
  uint2 wraw[kWeights];
  if (CONV) {
#pragma unroll
    for (int j = 0; j < kWeights; ++j) {
      // (threads past the last channel load it again: behind a branch, the two-head kernel without phi spilled 80 registers at
      // head dim 128, where it spills none now: 16384 tokens, 16 heads on 8, 110.5 -> 101.1 us when the branch went)
      const int e = min(tid + j * G::TEAM, kRows * D - 1), c = e % D, hh = OUTPUT ? e / D : GR;
      const bf16_t* src = hh < GR ? a.wq + ((size_t)(hk * a.group + qh0 + hh) * D + c) * a.W
                                  : a.wk + ((size_t)hk * D + c) * a.W;
      if (a.W == 4) {
        wraw[j] = *reinterpret_cast<const uint2*>(src);
      } else {
        wraw[j] = make_uint2(src[0], 0);
        if (a.W > 1) wraw[j].x |= (uint32_t)src[1] << 16;
        if (a.W > 2) wraw[j].y = src[2];
      }
    }
  }

  // uniform row sources
  const unsigned kvstride = (unsigned)a.Hkv * D * 2, qstride = (unsigned)a.Hq * D * 2;
  const RowSrc srcK = make_row_src(
      (const char*)a.k + (row0 * a.Hkv + hk) * D * 2,
      (CONV && a.k_halo) ? (const char*)a.k_halo + ((size_t)b * (a.W - 1) * a.Hkv + hk) * D * 2 : nullptr, kvstride, T, D * 2);
  const RowSrc srcG = make_row_src((const char*)a.g + (row0 * a.Hkv + hk) * D * 2, nullptr, kvstride, T, D * 2);
  const RowSrc srcV = make_row_src((const char*)a.v + (row0 * a.Hkv + hk) * D * 2, nullptr, kvstride, T, D * 2);
  const RowSrc srcQ = make_row_src(
      (const char*)a.q + (row0 * a.Hq + hk * a.group + qh0) * D * 2,
      (CONV && a.q_halo) ? (const char*)a.q_halo + ((size_t)b * (a.W - 1) * a.Hq + hk * a.group + qh0) * D * 2 : nullptr, qstride, T,
      (GR > 0 ? GR : 1) * D * 2);
  const unsigned coff = (unsigned)c0 * 2;
  // This lane's part of the LDS address of a token-major row, formed once so that the chunk loop only adds a
  // uniform offset.  (Left to the compiler, row index times stride became a 64-bit multiply-add whose unused
  // high half aliased a register with a prefetch in flight, and the chunk loop then began by waiting for the
  // whole prefetch.)
  const unsigned lrow = (unsigned)n * G::QRS + (unsigned)g4 * 8;
  // This lane's value column.  OWN: of each two waves the columns alternate by fours, so that a lane of an output tile pair holds
  // eight adjacent ones.
  const int col = OWN ? 32 * (w >> 1) + 8 * (n >> 2) + 4 * (w & 1) + (n & 3) : 16 * w + n;

  // the output pass walks its segment forwards, the state pass backwards (see compute_state)
  const int nseg_gran = (s1 - s0 + G::NTG - 1) / G::NTG;
  const int tfirst = OUTPUT ? s0 : s0 + (nseg_gran - 1) * G::NTG;
  const int tstep = OUTPUT ? G::NTG : -G::NTG;
  Raw<KK::NQ> raw;
  // The output pass requests its first rows after its start state, so that it does not wait for that behind them: 1984 tokens, 8 heads of
  // 128, 35.4 -> 33.7 us, 64 tokens of 64 9.4 -> 9.2; 8192, 32 heads on 8 of 64, 44.0 -> 43.4.  Before it where that measured better (of
  // 128, 32 on 8, 16384 tokens, 128.3, after it 129.8; without conv, 200 sequences of 64 tokens, 16 heads on 8, 27.3 and 28.8), and behind the
  // fold with one head and no conv (16 of 300 20.9, before the state 21.2).
  constexpr bool kRowsFirst = !OUTPUT || (CONV ? D == 128 && GR == 4 : GR > 1), kRowsLast = OUTPUT && !CONV && GR == 1;
  if (kRowsFirst) KK::template fetch<true>(raw, srcK, srcG, srcV, tfirst, tl0, coff, a.W);
  // ---- state in accumulators: Sacc[rt][i] = S[16 rt + 4 g4 + i][col], zacc[i] = z[16 w + 4 g4 + i], the same in all n
  floatx4 Sacc[G::RT], zacc;
  const int zrow = 16 * w + 4 * g4;
  {
    const float* Sin = nullptr;
    const float* zin = nullptr;
    int first = seg;   // fold: first segment whose contribution is still to be added
    if (OUTPUT) {
      bool scanned = false;
      if (a.fold) {
        // after the last of the predecessors whose total decay is exactly zero nothing earlier counts
        const unsigned long long m = __builtin_amdgcn_ballot_w64(live_any == 0);
        first = m ? 64 - __builtin_clzll(m) : 0;
      } else if (nseg > 1) {
        // team-wide OR through the per-wave flag words (free until the granule loop; the barrier that ends the
        // prologue separates these reads from the loop's first writes)
        const bool wave_any = __builtin_amdgcn_ballot_w64(live_any != 0) != 0;
        if (l == 0) *reinterpret_cast<int*>(smem + G::kFl + w * 4) = wave_any ? 1 : 0;
        __syncthreads();
        int any = 0;
#pragma unroll
        for (int j = 0; j < G::NW; ++j) any |= *reinterpret_cast<const int*>(smem + G::kFl + j * 4);
        scanned = __builtin_amdgcn_readfirstlane(any) != 0;
      }
      if (a.fold ? first > 0 : scanned || (nseg > 1 && seg > 0)) {
        Sin = a.ws + (slot0 + (a.fold ? first - 1 : scanned ? seg : seg - 1)) * G::kSlot;
        zin = Sin + D * D;
      } else {
        if (a.S0 != nullptr) Sin = a.S0 + (size_t)bh * D * D;
        if (a.z0 != nullptr) zin = a.z0 + (size_t)bh * D;
      }
    }
#pragma unroll
    for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) Sacc[rt][i] = Sin ? Sin[(size_t)(16 * rt + 4 * g4 + i) * D + col] : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) zacc[i] = zin ? zin[zrow + i] : 0.f;
    if (!kRowsFirst && !kRowsLast) KK::template fetch<true>(raw, srcK, srcG, srcV, tfirst, tl0, coff, a.W);
    if (CONV) {
      const float wscale = MODE == kConvElu ? kLog2e : 1.f;
#pragma unroll
      for (int j = 0; j < kWeights; ++j) {
        const int e = tid + j * G::TEAM;
        if (e < kRows * D)
          *reinterpret_cast<floatx4*>(wl + ((size_t)(OUTPUT ? e : e + GR * D)) * 4) =
              floatx4{bf_lo(wraw[j].x) * wscale, bf_hi(wraw[j].x) * wscale, bf_lo(wraw[j].y) * wscale, bf_hi(wraw[j].y) * wscale};
      }
    }
    if (OUTPUT && first < seg) {
      // state <- decay (.) state + contribution, segment by segment (in the scan's order).  z and the decays, alike in 16 lanes, come
      // through LDS, all predecessors' at once; S goes straight to its lanes, the next segment's on its way meanwhile.  (With z and
      // decays in registers too, 64 of the 96 a slot took at head dim 128: spills there, and at 64 226 registers instead of 158 in the
      // one-head kernels, two workgroups a compute unit instead of three: 200 sequences of 64 tokens, 8 heads, 27.5 us and 23.6;
      // one of 130 tokens of 8 heads of 128, 22.8 and 21.8.)
      float* zd = reinterpret_cast<float*>(smem);      // [predecessor][z | decay]: free until the first granule
#pragma unroll
      for (int j = 0; j < kZd; ++j) {
        const int e = tid + j * G::TEAM;
        if (e < seg * 2 * D) zd[e] = zraw[j];
      }
      struct Rows { float s[4][4]; };      // 4 row tiles of S: a slot at head dim 64, half of one at 128
      auto load = [&](int j, int r0, Rows& o) {
        // (a descriptor: one offset register for all rows)
        const __amdgpu_buffer_rsrc_t slot =
            __builtin_amdgcn_make_buffer_rsrc((void*)(a.ws + (slot0 + j) * G::kSlot), 0, D * D * 4, 0x00020000);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            o.s[rt][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(slot, (4 * g4 * D + col) * 4, (16 * (r0 + rt) + i) * D * 4, 0));
      };
      auto add = [&](int j, int r0, const Rows& o) {
        // (all of a piece's decays at once: one latency, not one per row tile: 517 tokens 16.6 -> 15.95 us, 700 17.2 -> 16.5)
        const float* at = zd + j * 2 * D;
        floatx4 dec[4], dz, zdec;
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) dec[rt] = *reinterpret_cast<const floatx4*>(at + D + 16 * (r0 + rt) + 4 * g4);
        if (r0 == 0) {
          dz = *reinterpret_cast<const floatx4*>(at + zrow);
          zdec = *reinterpret_cast<const floatx4*>(at + D + zrow);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i) Sacc[r0 + rt][i] = fmaf(dec[rt][i], Sacc[r0 + rt][i], o.s[rt][i]);
        if (r0 == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) zacc[i] = fmaf(zdec[i], zacc[i], dz[i]);
        }
      };
      Rows x, y;
      load(first, 0, x);
      __syncthreads();
      if constexpr (D == 64) {
#pragma unroll 1
        for (int j = first; j < seg; j += 2) {
          load(min(j + 1, seg - 1), 0, y);
          add(j, 0, x);
          if (j + 1 >= seg) break;
          load(min(j + 2, seg - 1), 0, x);
          add(j + 1, 0, y);
        }
      } else {
#pragma unroll 1
        for (int j = first; j < seg; ++j) {
          load(j, 4, y);
          add(j, 0, x);
          load(min(j + 1, seg - 1), 0, x);
          add(j, 4, y);
        }
      }
    }
  }
  float rgran[2] = {1.f, 1.f};  // state pass: decay of everything after the current granule, this lane's 2 channels

  const bool gs1 = a.gate_scale == 1.0f;
  Chunk<D, KK::NQ> own;
  if (kRowsLast) KK::template fetch<true>(raw, srcK, srcG, srcV, tfirst, tl0, coff, a.W);
  __syncthreads();  // conv weights are in LDS

  // Per granule: compute stage, barrier, MFMA stage, barrier (OWN: none at its end, as only this wave reads its chunk's S and V there).
  bool dead = false;   // state pass: after the last granule walked, the segment's total decay is exactly zero
#pragma unroll 1
  for (int gi = 0; gi < nseg_gran; ++gi) {
    const int t0 = tfirst + gi * tstep;
      {
        // =========================== compute stage: registers -> LDS operands ===========================
        const bool edge = (t0 < 3) || (t0 + G::NTG > s1);
        if (!OUTPUT) {
          if (!edge && gs1)
            KK::template compute_state<false, true>(raw, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, rgran);
          else if (!edge)
            KK::template compute_state<false, false>(raw, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, rgran);
          else if (gs1)
            KK::template compute_state<true, true>(raw, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, rgran);
          else
            KK::template compute_state<true, false>(raw, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, rgran);
        } else if (!edge && gs1)
          KK::template compute<false, true>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
        else if (!edge)
          KK::template compute<false, false>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
        else if (gs1)
          KK::template compute<true, true>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
        else
          KK::template compute<true, false>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
      }
      if (!OUTPUT) {
        // State pass: everything before this granule is multiplied by rgran.  Once that is exactly zero in every
        // channel, the operands of all remaining (earlier) granules are exactly zero and add nothing to the
        // accumulators, so the walk can stop: same bits, fewer rows read.  (With gate logits ~ N(0,1) the decay
        // underflows after about 150 tokens; a slowly decaying state walks its whole segment.)
        const bool alive = __builtin_amdgcn_ballot_w64(rgran[0] != 0.f || rgran[1] != 0.f) != 0;
        if (l == 0) *reinterpret_cast<int*>(smem + G::kFl + w * 4) = alive ? 1 : 0;
      }
      // (and nothing of the prologue's is: with waits for it in the MFMA stage and at the loop's end 32768 tokens of 64 took 102.5 us,
      // without 98.4; 700 of 128 28.2 and 27.9)
      if (OUTPUT) __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      dead = false;
      if (!OUTPUT) {
        int any = 0;
#pragma unroll
        for (int j = 0; j < G::NW; ++j) any |= *reinterpret_cast<const int*>(smem + G::kFl + j * 4);
        dead = __builtin_amdgcn_readfirstlane(any) == 0;
      }
      // the waves of the chunk's latency-bound MFMA chains go ahead of a co-resident workgroup's load stage
      if (OUTPUT && D == 64) __builtin_amdgcn_s_setprio(3);
      {
        // next granule's rows travel while the matrix cores work
        if (gi + 1 < nseg_gran && !dead) KK::template fetch<!OUTPUT>(raw, srcK, srcG, srcV, t0 + tstep, tl0, coff, a.W);

        // chunks of this granule in which some channel uses the mid-chunk reference (bit mc)
        int midmask = 0;
        if (OUTPUT) {
#pragma unroll
          for (int j = 0; j < G::NW; ++j)
            midmask |= *reinterpret_cast<const int*>(smem + G::kFl + j * 4) << (j / G::CH);
          midmask = __builtin_amdgcn_readfirstlane(midmask);
        }
        const short4v ones4 = {0x3F80, 0x3F80, 0x3F80, 0x3F80};   // the state update of the normalizer z
        if constexpr (OWN) {
          // =========================== MFMA stage, head dim 64 ===========================
          // The state through the granule's chunks, 16 value columns a wave; what it is at each chunk's start goes to LDS as bf16
          // operands (rows = value columns, k = key channels {4 g4 + i, 16 + 4 g4 + i} of each 32).
          struct Update { uint2 kd; floatx4 eb; };     // (j == RT: this wave's share of z)
          auto load_value = [&](int mc) { return *reinterpret_cast<const uint2*>(smem + G::kVt + col * G::TRS + (kChunk * mc + 4 * g4) * 2); };
          auto load_update = [&](int mc, int j) {
            const int rt = j < G::RT ? j : w;
            return Update{*reinterpret_cast<const uint2*>(smem + G::kKd + (16 * rt + n) * G::TRS + (kChunk * mc + 4 * g4) * 2),
                          *reinterpret_cast<const floatx4*>(smem + G::kEb + (mc * D + 16 * rt + 4 * g4) * 4)};
          };
          // With one or two query heads, whose calls are latency, the next chunk's operands are requested before this one's results are
          // awaited (8192 tokens of 8 heads 30.2 -> 29.6 us); with four they spill
          constexpr bool kAhead = CONV && GR < 4;
          Update up[kAhead ? G::RT + 1 : 1];
          uint2 vb = load_value(0);
          if constexpr (kAhead) {
#pragma unroll
            for (int j = 0; j <= G::RT; ++j) up[j] = load_update(0, j);
          }
          auto through = [&](auto mid) {
#pragma unroll
            for (int mc = 0; mc < G::MCG; ++mc) {
              if (!kAhead && mc > 0) vb = load_value(mc);
              if constexpr (decltype(mid)::value) {
                // Some channel of the granule uses the mid-chunk reference.  The accumulators take rho in place (rho (.) S is what
                // the chunk's MFMAs need), and the update below continues from there: its decay factor is E_last / rho.
                const float* ef = reinterpret_cast<const float*>(smem + G::kEf) + mc * D + 4 * g4;
#pragma unroll
                for (int rt = 0; rt < G::RT; ++rt) Sacc[rt] *= *reinterpret_cast<const floatx4*>(ef + 16 * rt);
                zacc *= *reinterpret_cast<const floatx4*>(ef + 16 * w);
              }
#pragma unroll
              for (int ks = 0; ks < G::KS; ++ks) {
                const floatx4 lo = Sacc[2 * ks], hi = Sacc[2 * ks + 1];
                *reinterpret_cast<uint4*>(smem + G::kSn + mc * G::kSnChunk + (w * G::KS + ks) * 1024 + l * 16) =
                    make_uint4(pack2(lo[0], lo[1]), pack2(lo[2], lo[3]), pack2(hi[0], hi[1]), pack2(hi[2], hi[3]));
              }
              if (n == 0)
                *reinterpret_cast<uint2*>(smem + G::kZs + (mc * D + 16 * w + 4 * g4) * 2) = make_uint2(pack2(zacc[0], zacc[1]), pack2(zacc[2], zacc[3]));
              if (kAhead) __builtin_amdgcn_sched_barrier(0);
              // S <- diag(E_last / rho) (rho S) + Kdec^T V, z likewise with ones
#pragma unroll
              for (int j = 0; j <= G::RT; ++j) {
                const Update u = kAhead ? up[j % (kAhead ? G::RT + 1 : 1)] : load_update(mc, j);
                floatx4& acc = j < G::RT ? Sacc[j % G::RT] : zacc;
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, u.kd), j < G::RT ? __builtin_bit_cast(short4v, vb) : ones4,
                                                                acc * u.eb, 0, 0, 0);
              }
              if (kAhead && mc + 1 < G::MCG) {
                __builtin_amdgcn_sched_barrier(0);
                vb = load_value(mc + 1);
#pragma unroll
                for (int j = 0; j <= G::RT; ++j) up[j % (kAhead ? G::RT + 1 : 1)] = load_update(mc + 1, j);
                __builtin_amdgcn_sched_barrier(0);
              }
            }
          };
          if (midmask != 0) through(std::true_type{});
          else through(std::false_type{});
          __syncthreads();  // S and z at every chunk's start are in LDS
          // Outputs of the wave's own chunk: o^T[dv][query] = S^T (q (.) E)^T + [V,V]^T [P_hi;P_lo]^T, den = q' . z + (column sums of
          // P), by a ones operand against the packed scores: it sums exactly the high parts and residuals that the values meet.
          if (t0 + kChunk * w < s1) {
            const bf16x8 ones8 = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
            const int tok = t0 + kChunk * w + n;
            const size_t orow = (row0 + tok) * a.Hq + hk * a.group + qh0;
            float rden[GR];
            bf16x8 zf[G::KS];
#pragma unroll
            for (int ks = 0; ks < G::KS; ++ks) {
              const unsigned char* pz = smem + G::kZs + (w * D + 32 * ks + 4 * g4) * 2;
              zf[ks] = make8(*reinterpret_cast<const uint2*>(pz), *reinterpret_cast<const uint2*>(pz + 32));
            }
            // All four tiles of a head at a time (two at a time: 96.2 -> 98.0 us at 32768 tokens), or two where that keeps three
            // workgroups on a compute unit.  Each two hold a lane's eight adjacent columns of its token.
            constexpr int CT = kThree ? 2 : G::NW;
#pragma unroll
            for (int ct0 = 0; ct0 < G::NW; ct0 += CT) {
              if (kThree) __builtin_amdgcn_sched_barrier(0);
              bf16x8 sf[CT][G::KS], vf[CT];
#pragma unroll
              for (int e = 0; e < CT; ++e) {
                const int ct = ct0 + e;
#pragma unroll
                for (int ks = 0; ks < G::KS; ++ks)
                  sf[e][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(smem + G::kSn + w * G::kSnChunk + (ct * G::KS + ks) * 1024 + l * 16));
                // (the same four tokens fill both halves of the operand)
                const uint2 v = *reinterpret_cast<const uint2*>(smem + G::kVt + (32 * (ct >> 1) + 8 * (n >> 2) + 4 * (ct & 1) + (n & 3)) * G::TRS + (kChunk * w + 4 * g4) * 2);
                vf[e] = make8(v, v);
              }
#pragma unroll
              for (int hh = 0; hh < GR; ++hh) {
                const bf16x8 pp = __builtin_bit_cast(bf16x8, own.p[hh]);
                floatx4 dz = {0.f, 0.f, 0.f, 0.f};
                if (ct0 == 0) {
#pragma unroll
                  for (int ks = 0; ks < G::KS; ++ks) dz = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[ks], own.q[hh][ks], dz, 0, 0, 0);
                  dz = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones8, pp, dz, 0, 0, 0);
                }
                floatx4 acc[CT];
#pragma unroll
                for (int e = 0; e < CT; ++e) {
                  acc[e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                  for (int ks = 0; ks < G::KS; ++ks) acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sf[e][ks], own.q[hh][ks], acc[e], 0, 0, 0);
                  acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[e], pp, acc[e], 0, 0, 0);
                }
                const float den = dz[0] + a.eps;
                if (ct0 == 0) rden[hh] = fast_rcp(den);
                if (tok < s1) {
#pragma unroll
                  for (int e = 0; e < CT; e += 2) {
                    const floatx4 x = acc[e] * rden[hh], y = acc[e + 1] * rden[hh];
                    *reinterpret_cast<uint4*>(a.o + (orow + hh) * D + 16 * (ct0 + e) + 8 * g4) = make_uint4(pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(y[0], y[1]), pack2(y[2], y[3]));
                  }
                  if (ct0 == 0 && a.den_out != nullptr && g4 == 0) a.den_out[orow + hh] = den;
                }
              }
            }
          }
        } else if constexpr (OUTPUT) {
          // =========================== MFMA stage, head dim 128 ===========================
          // z through the granule's chunks, a wave's 16 channels; what it is at each chunk's start goes to LDS as bf16
#pragma unroll
          for (int mc = 0; mc < G::MCG; ++mc) {
            const unsigned at = (mc * D + 16 * w + 4 * g4) * 4;
            const uint2 kd = *reinterpret_cast<const uint2*>(smem + G::kKd + (16 * w + n) * G::TRS + (kChunk * mc + 4 * g4) * 2);
            if (midmask != 0) zacc *= *reinterpret_cast<const floatx4*>(smem + G::kEf + at);      // (see the state below)
            if (n == 0)
              *reinterpret_cast<uint2*>(smem + G::kZs + (mc * D + 16 * w + 4 * g4) * 2) = make_uint2(pack2(zacc[0], zacc[1]), pack2(zacc[2], zacc[3]));
            zacc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, kd), ones4, zacc * *reinterpret_cast<const floatx4*>(smem + G::kEb + at), 0, 0, 0);
          }
          __syncthreads();
          // Scores and denominators, P^T = K' Q'^T and den = q' . z + (column sums of the masked P), of chunk w % 4, half of the heads a
          // wave, shared through LDS.
          {
            constexpr int HW = (GR + 1) / 2;
            const int bc = w % G::MCG, bh0 = w / G::MCG * HW;
            if (bh0 < GR && t0 + kChunk * bc < s1) {
              bf16x8 kf[G::KS], zf[G::KS];
#pragma unroll
              for (int ks = 0; ks < G::KS; ++ks) {
                const unsigned char* pk = smem + G::kKp + (kChunk * bc) * G::QRS + lrow + 64 * ks;
                const unsigned char* pz = smem + G::kZs + (bc * D + 32 * ks + 4 * g4) * 2;
                kf[ks] = make8(*reinterpret_cast<const uint2*>(pk), *reinterpret_cast<const uint2*>(pk + 32));
                zf[ks] = make8(*reinterpret_cast<const uint2*>(pz), *reinterpret_cast<const uint2*>(pz + 32));
              }
#pragma unroll
              for (int j = 0; j < HW; ++j) {
                const int hh = bh0 + j;
                floatx4 pt = {0.f, 0.f, 0.f, 0.f}, dz = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < G::KS; ++ks) {
                  const unsigned char* pq = smem + G::kQp + (hh * G::NTG + kChunk * bc) * G::QRS + lrow + 64 * ks;
                  const bf16x8 qf = make8(*reinterpret_cast<const uint2*>(pq), *reinterpret_cast<const uint2*>(pq + 32));
                  pt = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf, pt, 0, 0, 0);
                  dz = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[ks], qf, dz, 0, 0, 0);
                }
                const uint4 pp = pack_scores(pt, g4, n);
                *reinterpret_cast<uint4*>(smem + G::kPs + (bc * GR + hh) * 1024 + l * 16) = pp;
                // column sums over the 16 keys: a ones operand against the packed scores adds them to q'.z in every row of the tile (it
                // sums exactly the high parts and residuals that the value product below uses)
                const bf16x8 ones8 = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
                dz = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones8, __builtin_bit_cast(bf16x8, pp), dz, 0, 0, 0);
                if (g4 == 0) *reinterpret_cast<float*>(smem + G::kDn + ((bc * GR + hh) * 16 + n) * 4) = dz[0] + a.eps;
              }
            }
          }
          __syncthreads();
          // Outputs and state, 16 value columns a wave, from here on without a barrier: o^T[dv][query] = S^T (q (.) E)^T + [V,V]^T
          // [P_hi;P_lo]^T, then S <- diag(E_last / rho) (rho S) + Kdec^T V.  Operands of the next head travel while this head's chain
          // runs, those of the state's update while the heads' do; the scheduling barriers keep the compiler from requesting them behind
          // the chain.  (Only that: an LDS load may come right behind an MFMA that reads the registers it fills, as operands or as
          // accumulator input.  The update loops of these kernels are full of such loads, and 72000 repeated calls agreed bit for bit.)
#pragma unroll 1
          for (int mc = 0; mc < G::MCG; ++mc) {
            const int tq = t0 + kChunk * mc;  // first token of the chunk
            if (tq >= s1) break;
            struct HeadOps { bf16x8 qb[G::KS]; bf16x8 pp; float den; };
            auto load_ops = [&](int hh, HeadOps& o) {
#pragma unroll
              for (int ks = 0; ks < G::KS; ++ks) {
                const unsigned char* p = smem + G::kQp + (hh * G::NTG + kChunk * mc) * G::QRS + lrow + 64 * ks;
                o.qb[ks] = make8(*reinterpret_cast<const uint2*>(p), *reinterpret_cast<const uint2*>(p + 32));
              }
              o.pp = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(smem + G::kPs + (mc * GR + hh) * 1024 + l * 16));
              o.den = *reinterpret_cast<const float*>(smem + G::kDn + ((mc * GR + hh) * 16 + n) * 4);
            };
            // V[tok 4 g4 .. +3][dv 16 w + n]; serves as A (V^T, the same four tokens in both halves) and as B (V)
            const uint2 vraw = *reinterpret_cast<const uint2*>(smem + G::kVt + col * G::TRS + (kChunk * mc + 4 * g4) * 2);
            // Heads per step, and row tiles of the update requested ahead: two and none with two heads (5000 tokens of 16 heads on 8 46.5 us, one
            // and all 46.8), one and all with four (16384 tokens 122.0 us, two and all 125.1, two and none 126.0).
            constexpr int NS = GR == 2 ? 2 : 1, kAheadRows = GR == 4 ? G::RT : 0;
            HeadOps ops[2][NS];
#pragma unroll
            for (int e = 0; e < NS; ++e) load_ops(e, ops[0][e]);
            if ((midmask >> mc) & 1) {
              // Rare: some channel of this chunk uses the mid-chunk reference.  The accumulators take rho in place (rho (.) S is
              // what the chunk's MFMAs need), and the state update below continues from there: its decay factor is E_last / rho.
#pragma unroll
              for (int rt = 0; rt < G::RT; ++rt) Sacc[rt] *= *reinterpret_cast<const floatx4*>(smem + G::kEf + (mc * D + 16 * rt + 4 * g4) * 4);
            }
            bf16x8 sa[G::KS];   // rows = value columns, k = key channels {4 g4 + i, 16 + 4 g4 + i} of each 32
#pragma unroll
            for (int ks = 0; ks < G::KS; ++ks) {
              const floatx4 lo = Sacc[2 * ks], hi = Sacc[2 * ks + 1];
              sa[ks] = __builtin_bit_cast(bf16x8, make_uint4(pack2(lo[0], lo[1]), pack2(lo[2], lo[3]), pack2(hi[0], hi[1]), pack2(hi[2], hi[3])));
            }
            const bf16x8 vv = make8(vraw, vraw);
            uint2 kd[G::RT];
            floatx4 eb[G::RT];
            auto load_update = [&](int rt) {
              kd[rt] = *reinterpret_cast<const uint2*>(smem + G::kKd + (16 * rt + n) * G::TRS + (kChunk * mc + 4 * g4) * 2);
              eb[rt] = *reinterpret_cast<const floatx4*>(smem + G::kEb + (mc * D + 16 * rt + 4 * g4) * 4);
            };
#pragma unroll
            for (int h0 = 0; h0 < GR; h0 += NS) {
              const HeadOps(&o)[NS] = ops[(h0 / NS) & 1];
#pragma unroll
              for (int e = 0; e < NS; ++e)
                if (h0 + NS + e < GR) load_ops(h0 + NS + e, ops[(h0 / NS + 1) & 1][e]);
              if (h0 + NS == GR) {
#pragma unroll
                for (int rt = 0; rt < kAheadRows; ++rt) load_update(rt);
              }
              __builtin_amdgcn_sched_barrier(0);
              floatx4 acc[NS];
#pragma unroll
              for (int e = 0; e < NS; ++e) acc[e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
                for (int e = 0; e < NS; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sa[ks], o[e].qb[ks], acc[e], 0, 0, 0);
#pragma unroll
              for (int e = 0; e < NS; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, o[e].pp, acc[e], 0, 0, 0);
              const int tok = tq + n;
#pragma unroll
              for (int e = 0; e < NS; ++e) acc[e] *= fast_rcp(o[e].den);
              if (tok < s1) {
                const size_t orow = (row0 + tok) * a.Hq + hk * a.group + qh0 + h0;
#pragma unroll
                for (int e = 0; e < NS; ++e) {
                  *reinterpret_cast<uint2*>(a.o + (orow + e) * D + 16 * w + 4 * g4) = make_uint2(pack2(acc[e][0], acc[e][1]), pack2(acc[e][2], acc[e][3]));
                  if (a.den_out != nullptr && w == 0 && g4 == 0) a.den_out[orow + e] = o[e].den;
                }
              }
              __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int rt = kAheadRows; rt < G::RT; ++rt) load_update(rt);
#pragma unroll
            for (int rt = 0; rt < G::RT; ++rt)
              Sacc[rt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, kd[rt]), __builtin_bit_cast(short4v, vraw), Sacc[rt] * eb[rt], 0, 0, 0);
          }
        } else {
          // =========================== MFMA stage, state pass: operands decayed to the segment's end ===========================
          struct Update { uint2 v, kd[G::RT + 1]; } up[2];
          auto load_update = [&](int mc, Update& u) {
            u.v = *reinterpret_cast<const uint2*>(smem + G::kVt + col * G::TRS + (kChunk * mc + 4 * g4) * 2);
#pragma unroll
            for (int j = 0; j <= G::RT; ++j)      // (the last: this wave's share of z)
              u.kd[j] = *reinterpret_cast<const uint2*>(smem + G::kKd + (16 * (j < G::RT ? j : w) + n) * G::TRS + (kChunk * mc + 4 * g4) * 2);
          };
          load_update(0, up[0]);
#pragma unroll
          for (int mc = 0; mc < G::MCG; ++mc) {
            if (mc + 1 < G::MCG) load_update(mc + 1, up[(mc + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            const Update& u = up[mc & 1];
#pragma unroll
            for (int rt = 0; rt < G::RT; ++rt)
              Sacc[rt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, u.kd[rt]), __builtin_bit_cast(short4v, u.v), Sacc[rt], 0, 0, 0);
            zacc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, u.kd[G::RT]), ones4, zacc, 0, 0, 0);
          }
        }
      }  // MFMA stage
    if (OUTPUT && D == 64) __builtin_amdgcn_s_setprio(0);
    if (!OWN) __syncthreads();
    if (dead) break;
  }

  // ---- state out: first pass -> workspace slot (S | z | decay); last segment of the output pass -> S_out, z_out
  float* Sdst = nullptr;
  float* zdst = nullptr;
  float* ddst = nullptr;
  if (!OUTPUT) {
    Sdst = a.ws + (slot0 + seg) * G::kSlot;
    zdst = Sdst + D * D;
    ddst = zdst + D;
  } else if (seg == nseg - 1 && keeps) {
    Sdst = a.S_out + (size_t)bh * D * D;
    zdst = a.z_out + (size_t)bh * D;
  }
  if (Sdst != nullptr) {
#pragma unroll
    for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = 16 * rt + 4 * g4 + i;
        Sdst[(size_t)c * D + col] = Sacc[rt][i];
      }
    if (n == 0) *reinterpret_cast<floatx4*>(zdst + zrow) = zacc;
    // total decay of the segment: the waves that loaded chunk 0 hold it for their two channels
    if (ddst != nullptr && mcw == 0 && th == 0) *reinterpret_cast<float2*>(ddst + c0) = make_float2(rgran[0], rgran[1]);
    if (!OUTPUT && tid == 0) a.seg_live[slot0 + seg] = dead ? 0 : 1;
  }
  if (OUTPUT && CONV && seg == nseg - 1 && a.W > 1) store_tails<D>(a, b, hk, qh0, GR, keeps, T, row0, tid, G::TEAM);
}

template <int GR, int MODE>
__global__ void gla_wide_kernel(const ChunkArgs a);     // gla_wide.h

template <int D, int GR, int MODE>
hipError_t launch_all(const ChunkArgs& a, int parts, hipStream_t stream, bool with_state_pass, const TraceEvents& ev) {
  using G = Geo<D, GR, MODE>;
  const int heads = a.B * a.Hkv;
  const bool direct = !a.seq_start || a.places == kDirect;
  const int x = direct ? a.nseg : a.places == kByLength ? (a.per_head | 1) * a.Hkv : a.per_head | 1, y = direct ? heads : a.places == kByLength ? 1 : a.Hkv;
  hipError_t e;
  if (a.nseg > 1 && with_state_pass) {
    // GR = 0: key side only
    auto k1 = gla_chunk_kernel<D, 0, MODE, false>;
    constexpr int lds1 = Geo<D, 0, MODE>::kBytes;
    e = set_lds<gla_chunk_kernel<D, 0, MODE, false>>(lds1);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k1, dim3(direct ? x - 1 : x, y), dim3(G::TEAM), lds1, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!a.fold) {
      hipLaunchKernelGGL(segment_scan_kernel<D>, dim3(scan_blocks<D>(heads), heads), dim3(256), 0, stream, a.ws, a.seg_live,
                         a.S0, a.z0, a.nseg, a.seq_start, a.Hkv, a.seg_len, in_place(a));
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  // measurement entry point: the two events take the kernel's own start and stop timestamps (no dispatch gaps)
  auto output = [&](auto kernel, int team, int bytes) {
    if (ev.start != nullptr && ev.stop != nullptr)
      hipExtLaunchKernelGGL(kernel, dim3(x, y, parts), dim3(team), bytes, stream, ev.start, ev.stop, 0, a);
    else
      hipLaunchKernelGGL(kernel, dim3(x, y, parts), dim3(team), bytes, stream, a);
    return hipGetLastError();
  };
  if constexpr (D == 128) {
    if constexpr (MODE != kPlain) if (a.wide) {
      using W = WideGeo<GR, MODE>;
      e = set_lds<gla_wide_kernel<GR, MODE>>(W::kBytes);
      return e != hipSuccess ? e : output(gla_wide_kernel<GR, MODE>, W::TEAM, W::kBytes);
    }
  }
  e = set_lds<gla_chunk_kernel<D, GR, MODE, true>>(G::kBytes);
  return e != hipSuccess ? e : output(gla_chunk_kernel<D, GR, MODE, true>, G::TEAM, G::kBytes);
}

// A group of any size is covered by output-pass launches whose workgroups take 4, 2 or 1 of its query heads each; they
// share one state pass and one scan (the key side does not depend on the query heads).  The workgroup of the first heads stores the
// state; in place its launch is the last, after all that read the start state, and takes four heads at most (see launch_gla_chunk).
template <int D>
hipError_t launch_d(const ChunkArgs& a0, int group, int mode, hipStream_t stream, const TraceEvents& ev0) {
  ChunkArgs a = a0;
  a.group = group;
  bool first = true;
  for (int done = 0; done < group;) {
    const int left = group - done, rest = left % 4;
    const int gr = in_place(a) ? (rest == 0 ? 4 : rest == 2 ? 2 : 1) : left >= a.most ? a.most : (left >= 2 ? 2 : 1);
    const int parts = in_place(a) ? 1 : left / gr;
    a.qh0 = in_place(a) ? left - gr : done;
    const TraceEvents ev = first ? ev0 : TraceEvents{nullptr, nullptr};
    hipError_t e;
#define LAWCAT_CASE(GRV)                                                                      \
  case GRV:                                                                                   \
    e = mode == kPlain    ? launch_all<D, GRV, kPlain>(a, parts, stream, first, ev)           \
        : mode == kConvId ? launch_all<D, GRV, kConvId>(a, parts, stream, first, ev)          \
                          : launch_all<D, GRV, kConvElu>(a, parts, stream, first, ev);        \
    break;
    switch (gr) {
      LAWCAT_CASE(1)
      LAWCAT_CASE(2)
      LAWCAT_CASE(4)
      default: e = hipErrorInvalidValue;
    }
#undef LAWCAT_CASE
    if (e != hipSuccess) return e;
    first = false;
    done += gr * parts;
  }
  return hipSuccess;
}

}  // namespace chunk
}  // namespace lawcat
