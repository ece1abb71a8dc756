// Normalized gated linear attention (paper section 4.2) in fp32 accuracy:
//   S_t = diag(alpha_t) S_{t-1} + k_t^T v_t,  z_t = alpha_t (.) z_{t-1} + k_t,
//   o_t = q_t S_t / (q_t . z_t + eps)
// Three kernels: gla_walk_kernel walks a whole sequence or a segment of it (prefill with fp32 storage, where bf16 matrix-core operands
// would not meet the fp32 error bound, and blocks of decode steps; gla_span_kernel forms what segments add to the state),
// gla_few_kernel takes a few tokens one after the other (the same calls), gla_step_kernel is the decode step (lawcat_gla_step, one
// token, state updated in place).
//
// gla_walk_kernel: 16 tokens at a time on the matrix cores.  Within a block of up to 16 tokens, with E_t the decay after the
// block's first token up to t, Q' = q (.) E, K' = k / E and S~, z~ the state decayed by the first token's alpha:
//   num_t = Q'_t S~ + sum_{i<=t} (Q'_t . K'_i) v_i,   den_t = Q'_t . z~ + sum_{i<=t} Q'_t . K'_i + eps
// and, with F the block's whole decay and D_i the decay after token i up to the block's end,
//   S <- F (.) S + (k (.) D)^T V
// One workgroup of d / 16 waves owns a (batch, kv head).  A wave plays two parts: up to the first barrier it owns 16 key
// channels (gates, Q', K', its channels' part of the scores and of Q' . z~, all from its own rows in LDS: no barrier in
// between), after it 16 value columns (their slice of the state in accumulators, the outputs, the update; V never passes
// through LDS).
//
// Accuracy: the errors against 64-bit arithmetic are to be no larger than those of the recurrence token by token in fp32.
// So the state takes products of decays and never their quotients; decays are multiplied up, and the state is updated, in 64
// bits (fp64 MFMAs), rounded once a chunk.  The outputs' sums are fp64 MFMAs where the outputs are stored in fp32, and fp32
// ones in bf16 storage.  2-norm errors against the fp64 oracle, 256 tokens, fp32 storage: o 5.8e-8, S 3.5e-8, z 3.9e-8; token
// by token 6.5e-8, 4.5e-8, 3.9e-8 (gates of unit scale; with slowly decaying ones the gap is wider).
//
// What bounds it: the serial chain of one workgroup (gates, lane exchanges, LDS round trips, dependent MFMAs: of a chunk's 16K
// cycles 112 fp32 MFMAs take 3.6K and 16 fp64 ones 1K), about 4 us per chunk in fp32 storage and 6 for four query heads in bf16, at head
// dim 64.  8 sequences of 32 tokens, 32 query heads on 8 kv
// heads, bf16: 18 us, fp32, 256 tokens, 2 heads: 67 us; token by token on the vector ALUs the same took 115 and 235.
#include <algorithm>

#include "chunk_f32.h"

namespace lawcat {
namespace {
using namespace f32c;

__device__ inline float ldf(const float* p) { return *p; }
__device__ inline float ldf(const bf16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }
__device__ inline void stf(float* p, float v) { *p = v; }
__device__ inline void stf(bf16_t* p, float v) {
  __bf16 h = (__bf16)v;  // round to nearest even
  *p = __builtin_bit_cast(bf16_t, h);
}

struct WalkArgs {
  const void *q, *k, *v, *g;
  const float *S0, *z0;
  void* o;
  float *den_out, *S_out, *z_out;
  int T, Hq, Hkv, group;
  int heads;             // query heads that one workgroup takes
  float gate_scale, eps;
  double* slots;         // [B * Hkv][nseg - 1]: what each segment adds to the state
  int seg_len, nseg;     // segments of seg_len tokens, a multiple of kSpan; one: all of the sequence
};

// A segment's contribution in the workspace, in 64 bits (rounded there, S after 100 slowly decaying tokens was 2 % further from 64-bit
// arithmetic than the walk in one piece): S [key channel][value column], z, the decay over the segment.
template <int D> constexpr int slot_doubles() { return D * D + 2 * D; }
constexpr int kSpan = 32;     // tokens at a time of the pass that forms them

// One tensor's rows of a sequence at this workgroup's head; a descriptor covers one chunk (any length of sequence).
struct Source {
  const char* base;
  unsigned stride, width;
};
__device__ inline Rows chunk_rows(const Source& s, int row0, int T) {
  return make_rows(s.base, (size_t)row0 * s.stride, s.stride, min(kC, T - row0), s.width);
}

template <int D, int HB>
struct WalkLds {
  static constexpr int NW = D / 16;
  static constexpr int kSet = kC * f32_row_bytes<D>();   // fp32 rows of one head's (or K') chunk
  static constexpr int kRow64 = 8 * D + 16;              // k (.) D, fp64
  static constexpr int oKd = kSet;
  static constexpr int oQ = oKd + kC * kRow64;
  static constexpr int oPart = oQ + HB * kSet;           // scores, one tile per wave and head
  static constexpr int oQz = oPart + NW * HB * 1024;     // Q' . z~, 16 tokens per wave and head
  static constexpr int oA = oQz + NW * HB * 64;          // per channel: alpha of the block's first token (fp32) ...
  static constexpr int oF = oA + D * 4;                  // ... decay of the whole block (fp64)
  static constexpr int oFlag = oF + D * 8;
  static constexpr int kBytes = oFlag + 32;
};

// one element of a row as stored
template <typename T>
__device__ inline float load_one(const Rows& r, unsigned off) {
  if constexpr (sizeof(T) == 2) return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r.rsrc, (int)off, 0, 0) << 16);
  else return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r.rsrc, (int)off, 0, 0));
}

// grid (B * Hkv, parts, segments), 4 D threads; a part takes `heads` of the group's query heads, a multiple of HB, and part 0 of the last
// segment stores the state.  With one part and one segment S_out, z_out may be S0, z0: a wave reads and writes the same elements of both.
// Layouts of a 16 x 16 tile in a lane (g, n): "patch" = rows 4 g + i, column n (an fp32 accumulator; rows are tokens, columns
// the wave's channels); "strided" = rows 4 i + g (an fp64 accumulator, and the tokens of step i of a contraction over them).
template <typename T, int D, int HB>
__global__ void __launch_bounds__(4 * D, 2) gla_walk_kernel(const WalkArgs a) {
  typedef Store<T> St;
  typedef WalkLds<D, HB> L;
  constexpr int NW = L::NW, RT = D / 16;
  constexpr bool kWide = sizeof(T) == 4;      // outputs stored in fp32: fp64 sums
  // fp32 storage: operands from LDS as they are used.  At head dim 128 there are no registers for more, and at 64 the fp64 chains hide
  // those reads: in batches, with the wait in the loop below, 8 sequences of 300 tokens of 8 heads on 2 took 34.0 us, now 32.9, 2000
  // tokens of 32 on 8 98.4 and 95.7, 16 of 100 45.8 and 43.5, 8192 361 and 351, blocks of 200 tokens 120.5 and 117.8.
  constexpr bool kLean = kWide;
  constexpr bool kWaitOnce = kWide && D == 64;
  constexpr int kBatch = HB > 1 && D == 64 ? 2 : 1;      // heads whose operands are in registers at once
  extern __shared__ __attribute__((aligned(16))) unsigned char sm[];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, g = l >> 4, n = l & 15;
  const Lanes ln = make_lanes(l);
  const Quad qd = make_quad(l);
  const int bh = blockIdx.x, b = bh / a.Hkv, hk = bh % a.Hkv;
  const int s0 = kWide ? blockIdx.z * a.seg_len : 0, rows = kWide ? min(a.T - s0, a.seg_len) : a.T;      // this segment's tokens
  const int nb = a.heads / HB, nchunk = (rows + kC - 1) / kC;
  const int hq0 = hk * a.group + blockIdx.y * a.heads;      // first query head
  const unsigned kvs = (unsigned)a.Hkv * D * St::kBytes, qs = (unsigned)a.Hq * D * St::kBytes;
  const size_t kv1 = (((size_t)b * a.T + s0) * a.Hkv + hk) * D * St::kBytes;
  const size_t q1 = (((size_t)b * a.T + s0) * a.Hq + hq0) * D * St::kBytes;
  const Source K{(const char*)a.k + kv1, kvs, D * St::kBytes}, V{(const char*)a.v + kv1, kvs, D * St::kBytes},
      Gt{(const char*)a.g + kv1, kvs, D * St::kBytes}, Q{(const char*)a.q + q1, qs, (unsigned)a.heads * D * St::kBytes},
      O{(const char*)a.o + q1, qs, (unsigned)a.heads * D * St::kBytes};
  const unsigned offk = St::offset(chunk_rows(K, 0, rows), g, n, 16 * w), offq = St::offset(chunk_rows(Q, 0, rows), g, n, 16 * w);
  const unsigned own = (unsigned)(16 * w + n) * St::kBytes;

  typename St::Raw rq[HB], rk, rg;
  float rv[4];
  auto fetch = [&](int ci, int hb) {
    if (hb == 0) {
      rg = St::load(chunk_rows(Gt, ci * kC, rows), offk, 0);
      rk = St::load(chunk_rows(K, ci * kC, rows), offk, 0);
      const Rows v = chunk_rows(V, ci * kC, rows);
#pragma unroll
      for (int i = 0; i < 4; ++i) rv[i] = load_one<T>(v, (unsigned)(4 * i + g) * kvs + own);
    }
    const Rows q = chunk_rows(Q, ci * kC, rows);
#pragma unroll
    for (int h = 0; h < HB; ++h) rq[h] = St::load(q, offq + (unsigned)(hb * HB + h) * D * St::kBytes, 0);
  };
  fetch(0, 0);

  // S[16 rt + 4 g + i][16 w + n] and z[16 w + n] before the block
  floatx4 X[RT];
  // (through a descriptor, with 32-bit offsets; a missing start state reads as zero)
  const unsigned soff = (unsigned)(4 * g * D + 16 * w + n) * 4;
  const Rows Sin = make_rows(a.S0, (size_t)bh * D * D * 4, D * 4, a.S0 ? D : 0, D * 4);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      X[rt][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(Sin.rsrc, (int)soff, (16 * rt + i) * D * 4, 0));
  double z = a.z0 ? a.z0[(size_t)bh * D + 16 * w + n] : 0.f;
  if (kWide && blockIdx.z > 0) {
    // ... then the segments before this one, in 64 bits, rounded once
    double Y[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) Y[rt][i] = (double)X[rt][i];
    struct Part { double s[RT][4], dec[RT][4], z, zdec; };
    auto load_part = [&](int j, Part& o) {
      const double *slot = a.slots + ((size_t)bh * (a.nseg - 1) + j) * slot_doubles<D>(), *zd = slot + D * D;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = 16 * rt + 4 * g + i;
          o.s[rt][i] = slot[c * D + 16 * w + n];
          o.dec[rt][i] = zd[D + c];
        }
      o.z = zd[16 * w + n];
      o.zdec = zd[D + 16 * w + n];
    };
    auto add_part = [&](const Part& o) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) Y[rt][i] = fma(o.dec[rt][i], Y[rt][i], o.s[rt][i]);
      z = fma(o.zdec, z, o.z);
    };
    const int before = blockIdx.z;
    Part x, y;
    // At head dim 64 the next one travels meanwhile; at 128 there are no registers for it, and 28 of the first one's spill, here alone:
    // four row tiles at a time, where next to none do, measure within 2 % on either side (2 heads, 512 tokens 74.2 / 73.6 us, 1500 157.5 / 157.8).
    if constexpr (D == 64) {
      load_part(0, x);
#pragma unroll 1
      for (int j = 0; j < before; j += 2) {
        load_part(min(j + 1, before - 1), y);
        add_part(x);
        if (j + 1 >= before) break;
        load_part(min(j + 2, before - 1), x);
        add_part(y);
      }
    } else {
#pragma unroll 1
      for (int j = 0; j < before; ++j) {
        load_part(j, x);
        add_part(x);
      }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) X[rt][i] = (float)Y[rt][i];
  }

  int* flags = reinterpret_cast<int*>(sm + L::oFlag);
  Decay d;
  float kk[4], vv[4], E[4], zt = 0.f;    // patch, strided, patch; z~
  floatx4 kf = {0.f, 0.f, 0.f, 0.f};
  const bool gs1 = a.gate_scale == 1.0f;
  // a chunk's gates, keys and values from what was fetched, and into how many blocks this wave needs it to be cut
  auto gates = [&](int row0) {
    float gl[4];
    St::patch(qd, rg, gl);
    St::patch(qd, rk, kk);
    bool tame = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // alpha = sigmoid(g)^gate_scale; at gate_scale 1 directly 1 / (1 + e^-g)
      const float al = gs1 ? 1.f / (1.f + expf(-gl[i])) : expf(a.gate_scale * log_sigmoid(gl[i]));
      d.al[i] = row0 + 4 * g + i < rows ? al : 1.f;
      vv[i] = rv[i];
      tame = tame && fabsf(kk[i]) < kTame && fabsf(vv[i]) < kTame;
    }
    int cut = whole_chunk(d, ln, g);
    if (__builtin_amdgcn_ballot_w64(!tame) != 0) cut = kC;
    if (l == 0) flags[w] = cut;
  };
  gates(0);
  __syncthreads();

  if (kWaitOnce) __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): the start state and the first rows (see the loop's)
  int ci = 0, blk = 0, hb = 0, nblk = 1, lo = 0, hi = kC;
  while (ci < nchunk) {
    const int row0 = ci * kC;
    // ---- own 16 key channels: once per block the decays, K' and k (.) D; Q' of HB heads
    if (hb == 0) {
      if (blk == 0) {
        int m = 1;
#pragma unroll
        for (int j = 0; j < NW; ++j) m = max(m, flags[j]);
        nblk = __builtin_amdgcn_readfirstlane(m);
      }
      lo = blk * (kC / nblk);
      hi = lo + kC / nblk;
      double e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) e[i] = (4 * g + i > lo && 4 * g + i < hi) ? (double)d.al[i] : 1.0;
      const double p1 = e[0] * e[1], s1 = e[2] * e[3], tot = p1 * s1;
      const double x1 = lane_get(ln.x1, tot), x2 = lane_get(ln.x2, tot), x3 = lane_get(ln.x3, tot), x23 = x2 * x3;
      const double before = ((g & 1) ? x1 : 1.0) * ((g & 2) ? x23 : 1.0), after = ((g & 1) ? 1.0 : x1) * ((g & 2) ? 1.0 : x23);
      const int r = lo & 3;
      const float first = lane_get(ln.n4 + ((lo >> 2) << 6), r == 0 ? d.al[0] : r == 1 ? d.al[1] : r == 2 ? d.al[2] : d.al[3]);
      const double last = (tot * x1) * x23, F = last * (double)first;
      // of E and of the first token's alpha: in channels that nearly close, queries keep their bits down to 2^-94 (not 2^-62) and
      // up to 2^95
      const Center c = center_of((float)last);
      const float firstc = first * c.down;
      E[0] = (float)(before * e[0]) * c.up; E[1] = (float)(before * p1) * c.up;
      E[2] = (float)(before * p1 * e[2]) * c.up; E[3] = (float)(before * tot) * c.up;
      const double Dc[4] = {after * s1 * e[1], after * s1, after * e[3], after};
      float kp[4];
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = 4 * g + i >= lo && 4 * g + i < hi;
        const double x = in ? (double)kk[i] * Dc[i] : 0.0;
        s += x;
        *reinterpret_cast<double*>(sm + L::oKd + (4 * g + i) * L::kRow64 + (16 * w + n) * 8) = x;
        kp[i] = in ? kk[i] / E[i] : 0.f;
      }
      f32_to_lds<D>(sm, g, n, 16 * w, kp);
      s += lane_get(ln.x1, s);
      s += lane_get(ln.x2, s);
      zt = (float)z * firstc;
      z = fma(z, F, s);
      if (g == 0) {
        *reinterpret_cast<float*>(sm + L::oA + (16 * w + n) * 4) = firstc;
        *reinterpret_cast<double*>(sm + L::oF + (16 * w + n) * 8) = F;
      }
      __builtin_amdgcn_wave_barrier();   // LDS serves one wave's requests in order: its rows are complete below
      // the scores' rows come out in strided order: row m of the operand is token 4 (m % 4) + m / 4
      kf = *reinterpret_cast<const floatx4*>(sm + (4 * (n & 3) + (n >> 2)) * f32_row_bytes<D>() + (16 * w + 4 * g) * 4);
    }
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      float qp[4];
      floatx4 s;
      St::patch(qd, rq[h], qp);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        qp[i] = (4 * g + i >= lo && 4 * g + i < hi) ? qp[i] * E[i] : 0.f;
        s[i] = row16_sum(qp[i] * zt);
      }
      f32_to_lds<D>(sm + L::oQ + h * L::kSet, g, n, 16 * w, qp);
      if (n == 0) *reinterpret_cast<floatx4*>(sm + L::oQz + ((w * HB + h) * kC + 4 * g) * 4) = s;
    }
    const int hb1 = hb + 1 < nb ? hb + 1 : 0;
    const int blk1 = hb1 ? blk : (blk + 1 < nblk ? blk + 1 : 0);
    const int ci1 = (hb1 || blk1) ? ci : ci + 1;
    // vmcnt(0): nothing is in flight but the outputs of the chunk before and, the first time, the start state.  (Taken to be possibly in
    // flight, it let every chunk wait for the next one's rows below.)
    if (!kWaitOnce) __builtin_amdgcn_s_waitcnt(0x0F70);
    if (ci1 < nchunk) fetch(ci1, hb1);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      const floatx4 qf = f32_row_frag<D>(sm + L::oQ + h * L::kSet, g, n, w);
      floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) s = mfma_f32(kf[i], qf[i], s);       // [token 4 i + g of K'][token n of Q']
      *reinterpret_cast<floatx4*>(sm + L::oPart + (w * HB + h) * 1024 + l * 16) = s;
    }
    __syncthreads();
    // ---- own 16 value columns
    const Rows orow = chunk_rows(O, row0, rows);
    float vm[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) vm[i] = (4 * i + g >= lo && 4 * i + g < hi) ? vv[i] : 0.f;
    // Operands come from LDS in batches, the next head's while this one's products run.  One by one, as the compiler places them, each
    // was a latency of its own, and S~ was formed per head: 4 sequences of 200 tokens, 32 heads on 8, with the wait above 101.0 -> 98.8
    // us, 8 of 32 of 128 45.1 -> 42.6 (for two and five spilled registers with two and four heads at a time), of 64 25.8 -> 25.4.
    auto first_alpha = [&](int rt) { return *reinterpret_cast<const floatx4*>(sm + L::oA + (16 * rt + 4 * g) * 4); };
    floatx4 Xs[kLean ? 1 : RT];      // S~
    if constexpr (!kLean) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) Xs[rt] = first_alpha(rt);
    }
    struct HeadOps { floatx4 p[NW], q[kLean ? 1 : RT], z[kWide ? 1 : NW]; } ops[kBatch];      // scores, Q', and Q' . z~ in parts
    auto load_z = [&](int h, HeadOps& o) {
      const float* qz = reinterpret_cast<const float*>(sm + L::oQz) + h * kC;
#pragma unroll
      for (int j = 0; j < NW; ++j) o.z[j] = *reinterpret_cast<const floatx4*>(qz + j * HB * kC + 4 * g);
    };
    auto load_ops = [&](int h, HeadOps& o) {
#pragma unroll
      for (int j = 0; j < NW; ++j) o.p[j] = *reinterpret_cast<const floatx4*>(sm + L::oPart + (j * HB + h) * 1024 + l * 16);
      if constexpr (!kLean) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) o.q[rt] = f32_row_frag<D>(sm + L::oQ + h * L::kSet, g, n, rt);
      }
      if constexpr (D == 64 && !kWide) load_z(h, o);
    };
    load_ops(0, ops[0]);
    if (!kLean) __builtin_amdgcn_sched_barrier(0);
    if constexpr (!kLean) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) Xs[rt] *= X[rt];
    }
    auto store_den = [&](int h, int t, float den) {
      if (a.den_out != nullptr && w == 0 && n == 0 && t >= lo && t < hi && row0 + t < rows)
        a.den_out[((size_t)b * a.T + s0 + row0 + t) * a.Hq + hq0 + hb * HB + h] = den;
    };
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      HeadOps& o = ops[h % kBatch];
      if (kBatch == 1 && h > 0) load_ops(h, o);
      if (kBatch > 1 && h + 1 < HB) load_ops(h + 1, ops[(h + 1) % kBatch]);
      if (!kLean) __builtin_amdgcn_sched_barrier(0);
      floatx4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < NW; ++j) p += o.p[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = (4 * i + g >= lo && 4 * i + g <= n) ? p[i] : 0.f;
      if constexpr (kWide) {
        const float* qz = reinterpret_cast<const float*>(sm + L::oQz) + h * kC;
        doublex4 num = {0.0, 0.0, 0.0, 0.0}, ps = num;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ps = mfma_f64((double)p[i], 1.0, ps);
          num = mfma_f64((double)p[i], (double)vm[i], num);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const floatx4 qf = kLean ? f32_row_frag<D>(sm + L::oQ + h * L::kSet, g, n, rt) : o.q[kLean ? 0 : rt], xs = kLean ? X[rt] * first_alpha(rt) : Xs[kLean ? 0 : rt];
#pragma unroll
          for (int i = 0; i < 4; ++i) num = mfma_f64((double)qf[i], (double)xs[i], num);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = 4 * i + g;
          double den = ps[i] + (double)a.eps;
#pragma unroll
          for (int j = 0; j < NW; ++j) den += (double)qz[j * HB * kC + t];
          const unsigned off = (unsigned)t * qs + own + (unsigned)(hb * HB + h) * D * 4;
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)num[i] / (float)den), orow.rsrc, (int)(t >= lo && t < hi ? off : kNowhere), 0, 0);
          store_den(h, t, (float)den);
        }
      } else {
        floatx4 num = {0.f, 0.f, 0.f, 0.f}, pv = num, ps = num;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pv = mfma_f32(p[i], vm[i], pv);
          ps = mfma_f32(p[i], 1.f, ps);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
          for (int i = 0; i < 4; ++i) num = mfma_f32(o.q[rt][i], Xs[rt][i], num);
        }
        if constexpr (D == 128) load_z(h, o);
        floatx4 den = {a.eps, a.eps, a.eps, a.eps};
#pragma unroll
        for (int j = 0; j < NW; ++j) den += o.z[j];
        float ov[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          den[i] += ps[i];
          ov[i] = (num[i] + pv[i]) / den[i];
          store_den(h, 4 * g + i, den[i]);
        }
        St::store(orow, qd, offq + (unsigned)(hb * HB + h) * D * St::kBytes, 0, g, n, lo, hi, ov);
      }
    }
    if (hb1 == 0) {
      // rows of the operand in strided order: the tile comes out as a patch
      struct Update { double kd[4]; double F[4]; };
      auto load_update = [&](int rt) {
        const double* kd = reinterpret_cast<const double*>(sm + L::oKd + (16 * rt + strided(n)) * 8);
        const double* F = reinterpret_cast<const double*>(sm + L::oF) + 16 * rt + 4 * g;
        Update u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          u.kd[i] = kd[(4 * i + g) * (L::kRow64 / 8)];
          u.F[i] = F[i];
        }
        return u;
      };
      constexpr int kRows = kLean ? 1 : D == 64 ? 4 : 2;      // row tiles at a time
#pragma unroll
      for (int r0 = 0; r0 < RT; r0 += kRows) {
        Update u[kRows];
        if (kLean) __builtin_amdgcn_sched_barrier(0);      // bounds the operands in flight: fewer spills
#pragma unroll
        for (int e = 0; e < kRows; ++e) u[e] = load_update(r0 + e);
        if (!kLean) __builtin_amdgcn_sched_barrier(0);
        doublex4 t[kRows];
#pragma unroll
        for (int e = 0; e < kRows; ++e) t[e] = kZero64;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int e = 0; e < kRows; ++e) t[e] = mfma_f64(u[e].kd[i], (double)vm[i], t[e]);
#pragma unroll
        for (int e = 0; e < kRows; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i) X[r0 + e][i] = (float)fma((double)X[r0 + e][i], u[e].F[i], t[e][i]);
      }
      if (ci1 > ci && ci1 < nchunk) gates(ci1 * kC);
    }
    __syncthreads();
    ci = ci1; blk = blk1; hb = hb1;
  }
  // the state after the last token
  if (blockIdx.y != 0 || (kWide && (int)blockIdx.z != a.nseg - 1)) return;
  if (g == 0) a.z_out[(size_t)bh * D + 16 * w + n] = (float)z;
  const Rows Sout = make_rows(a.S_out, (size_t)bh * D * D * 4, D * 4, D, D * 4);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)X[rt][i]), Sout.rsrc, (int)soff, (16 * rt + i) * D * 4, 0);
}

// What a segment adds to the state at its end, sum_i (k_i (.) decay from i to the end)^T v_i, its z and its decay, from fp32 storage: products
// and sums in 64 bits as in the walk.  grid (nseg - 1, B * Hkv), 4 D threads; 32 tokens at a time, the last first.
// Latency: two lane exchanges, one barrier and D / 2 fp64 MFMAs per wave and 32 tokens: 6 us for 32 tokens at head dim 64, launch included.
template <int D>
__global__ void __launch_bounds__(4 * D) gla_span_kernel(const WalkArgs a) {
  typedef Store<float> St;
  constexpr int RT = D / 16, NM = kSpan / kC, kRow = 8 * D + 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char sm[];      // k (.) decay, fp64 rows
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, g = l >> 4, n = l & 15;
  const Lanes ln = make_lanes(l);
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / a.Hkv, hk = bh % a.Hkv, s0 = seg * a.seg_len;
  const unsigned kvs = (unsigned)a.Hkv * D * 4;
  const size_t kv1 = (((size_t)b * a.T + s0) * a.Hkv + hk) * D * 4;
  const Source K{(const char*)a.k + kv1, kvs, D * 4}, V{(const char*)a.v + kv1, kvs, D * 4}, Gt{(const char*)a.g + kv1, kvs, D * 4};
  const unsigned off = (unsigned)(4 * g) * kvs + (16 * w + n) * 4;
  const bool gs1 = a.gate_scale == 1.0f;
  doublex4 S[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) S[rt] = kZero64;
  double z = 0.0, run = 1.0;
  St::Raw rk[NM], rg[NM];
  float rv[NM][4];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      rg[m] = St::load(chunk_rows(Gt, t0 + kC * m, a.seg_len), off, 0);
      rk[m] = St::load(chunk_rows(K, t0 + kC * m, a.seg_len), off, 0);
      const Rows v = chunk_rows(V, t0 + kC * m, a.seg_len);
#pragma unroll
      for (int i = 0; i < 4; ++i) rv[m][i] = load_one<float>(v, (unsigned)(4 * i + g) * kvs + (16 * w + n) * 4);
    }
  };
  fetch(a.seg_len - kSpan);
#pragma unroll 1
  for (int t0 = a.seg_len - kSpan; t0 >= 0; t0 -= kSpan) {      // (only whole segments have a successor)
#pragma unroll
    for (int m = NM - 1; m >= 0; --m) {
      double e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float gl = rg[m].v[i];
        e[i] = (double)(gs1 ? 1.f / (1.f + expf(-gl)) : expf(a.gate_scale * log_sigmoid(gl)));
      }
      const double s1 = e[2] * e[3], s0x = e[1] * s1, tot = e[0] * s0x;
      const double x1 = lane_get(ln.x1, tot), x2 = lane_get(ln.x2, tot), x3 = lane_get(ln.x3, tot), x23 = x2 * x3;
      const double after = ((g & 1) ? 1.0 : x1) * ((g & 2) ? 1.0 : x23) * run;
      const double Dc[4] = {s0x * after, s1 * after, e[3] * after, after};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double x = (double)rk[m].v[i] * Dc[i];
        z += x;
        *reinterpret_cast<double*>(sm + (kC * m + 4 * g + i) * kRow + (16 * w + n) * 8) = x;
      }
      run *= (tot * x1) * x23;
    }
    __syncthreads();
    float vv[NM][4];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) vv[m][i] = rv[m][i];
    if (t0 > 0) fetch(t0 - kSpan);
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)     // rows of the operand in strided order: the tile comes out as a patch
          S[rt] = mfma_f64(*reinterpret_cast<const double*>(sm + (kC * m + 4 * i + g) * kRow + (16 * rt + strided(n)) * 8), (double)vv[m][i], S[rt]);
    __syncthreads();
  }
  double *slot = a.slots + ((size_t)bh * (a.nseg - 1) + seg) * slot_doubles<D>(), *zd = slot + D * D;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) slot[(16 * rt + 4 * g + i) * D + 16 * w + n] = S[rt][i];
  z += lane_get(ln.x1, z);
  z += lane_get(ln.x2, z);
  if (g == 0) {
    zd[16 * w + n] = z;
    zd[D + 16 * w + n] = run;
  }
}

// Decode step (T = 1), state in place.  One block per (batch, kv head).  Thread t owns value column
// t % D and a contiguous band of D*D/256 key channels of it, so a wave reads and writes whole 256-byte
// rows of S; alpha, k, z and the query heads are staged in LDS and read as broadcasts; the partial
// q.S sums of the 256/D bands are combined through LDS.  Query heads go four at a time, a wave holds one of them and
// forms its q.z.
// Few sequences: bound by latency, so everything is requested at once, before the first barrier (state and queries behind one each,
// and q.z summed by every thread, were three latencies in a row).  Many: by the state's traffic, about 5 TB/s for 256.  With both convs, in
// a graph, 32 query heads on 8 kv heads, us (before, the convs included, in brackets): head dim 64, one sequence 9.6 (11.4), 200 16.6 (19.5);
// 128, one 11.2 (14.2), 64 18.3 (23.1), 200 42.7 (47.0).
template <typename T, int D>
__global__ void __launch_bounds__(256) gla_step_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                       const T* __restrict__ v, const T* __restrict__ g,
                                                       float* S, float* z, T* __restrict__ o, int Hq, int Hkv,
                                                       float gate_scale, float eps) {
  constexpr int NPART = 256 / D;      // bands of key channels
  constexpr int RPT = D / NPART;      // key channels per thread
  constexpr int HT = 4;               // query heads per pass
  constexpr int NQ = D / 64;          // channels of its head in a lane: l, l + 64
  __shared__ float sh_a[D], sh_k[D], sh_z[D], sh_q[HT][D], sh_part[HT][NPART][D], sh_den[HT];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const Lanes ln = make_lanes(l);
  const int bh = blockIdx.x;  // b * Hkv + hk
  const int b = bh / Hkv, hk = bh % Hkv;
  const int group = Hq / Hkv;
  const size_t head0 = (size_t)b * Hq + (size_t)hk * group;
  float* Sh = S + (size_t)bh * D * D;
  const int col = tid % D, part = tid / D;
  float gl = 0.f, kk = 0.f, z0 = 0.f;
  if (tid < D) {
    gl = ldf(g + (size_t)bh * D + tid);
    kk = ldf(k + (size_t)bh * D + tid);
    z0 = z[(size_t)bh * D + tid];
  }
  float qv[NQ];
  auto fetch_q = [&](int h0) {
#pragma unroll
    for (int i = 0; i < NQ; ++i) qv[i] = h0 + w < group ? ldf(q + (head0 + h0 + w) * D + 64 * i + l) : 0.f;
  };
  fetch_q(0);
  const float vv = ldf(v + (size_t)bh * D + col);
  float sreg[RPT];
#pragma unroll
  for (int r = 0; r < RPT; ++r) sreg[r] = Sh[(size_t)(part * RPT + r) * D + col];
  if (tid < D) {
    const float alpha = expf(gate_scale * log_sigmoid(gl));
    const float zn = fmaf(alpha, z0, kk);
    sh_a[tid] = alpha;
    sh_k[tid] = kk;
    sh_z[tid] = zn;
    z[(size_t)bh * D + tid] = zn;
  }
  auto stage_q = [&] {
#pragma unroll
    for (int i = 0; i < NQ; ++i) sh_q[w][64 * i + l] = qv[i];
    __syncthreads();
  };
  stage_q();
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int c = part * RPT + r;
    sreg[r] = fmaf(sh_a[c], sreg[r], sh_k[c] * vv);
    Sh[(size_t)c * D + col] = sreg[r];
  }
  for (int h0 = 0;;) {
    float d = qv[0] * sh_z[l];
#pragma unroll
    for (int i = 1; i < NQ; ++i) d = fmaf(qv[i], sh_z[64 * i + l], d);
    d = row16_sum(d);
    d += lane_get(ln.x1, d);
    d += lane_get(ln.x2, d);
    if (l == 0) sh_den[w] = d + eps;
    float pn[HT] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      if (D == 128 && r % 16 == 0) __builtin_amdgcn_sched_barrier(0);     // bounds the operands in flight
      const int c = part * RPT + r;
#pragma unroll
      for (int hh = 0; hh < HT; ++hh) pn[hh] = fmaf(sh_q[hh][c], sreg[r], pn[hh]);
    }
#pragma unroll
    for (int hh = 0; hh < HT; ++hh) sh_part[hh][part][col] = pn[hh];
    __syncthreads();
    // thread (hh = part', col): one output element each for up to 256 / D heads at a time
    for (int hh = part; hh < min(HT, group - h0); hh += NPART) {
      float num = 0.f;
#pragma unroll
      for (int pp = 0; pp < NPART; ++pp) num += sh_part[hh][pp][col];
      stf(o + (head0 + h0 + hh) * D + col, num / sh_den[hh]);
    }
    h0 += HT;
    if (h0 >= group) break;
    fetch_q(h0);
    __syncthreads();  // this pass is done with sh_q / sh_part
    stage_q();
  }
}

// grid (B * Hkv, parts), 4 D threads.  A few tokens, one after the other, the state in registers in 64 bits and rounded once at the end, as the walk rounds it once
// a chunk.  A thread owns value column t % D and a quarter of its key channels; the next token's rows are requested a token ahead;
// a part takes `heads` of the group's query heads, and part 0 stores the state.  The sums of the outputs are 64-bit ones where the outputs are stored in fp32.  With one part S_out, z_out may be S0, z0:
// a thread reads and writes the same elements of both.
template <typename T, int D>
__global__ void __launch_bounds__(4 * D) gla_few_kernel(const WalkArgs a) {
  typedef std::conditional_t<sizeof(T) == 4, double, float> Acc;
  constexpr int NPART = 4, RPT = D / NPART, HT = 4, NWD = D / 64;
  __shared__ float sh_a[D], sh_k[D], sh_q[HT][D];
  __shared__ double sh_z[2][D];
  __shared__ Acc sh_part[HT][NPART][D], sh_den[HT][NWD];
  const int tid = threadIdx.x, col = tid % D, part = tid / D;
  const int bh = blockIdx.x, b = bh / a.Hkv, hk = bh % a.Hkv;
  const int hq0 = hk * a.group + blockIdx.y * a.heads;      // first query head
  const T* q = static_cast<const T*>(a.q) + ((size_t)b * a.T * a.Hq + hq0) * D;
  const size_t kv1 = ((size_t)b * a.T * a.Hkv + hk) * D, kvs = (size_t)a.Hkv * D, qs = (size_t)a.Hq * D;
  const T *k = static_cast<const T*>(a.k) + kv1, *v = static_cast<const T*>(a.v) + kv1, *g = static_cast<const T*>(a.g) + kv1;
  T* o = static_cast<T*>(a.o) + ((size_t)b * a.T * a.Hq + hq0) * D;
  const bool gs1 = a.gate_scale == 1.0f;
  const Lanes ln = make_lanes(tid & 63);

  float nk = 0.f, ng = 0.f, nv, nq;
  auto fetch = [&](int t) {
    if (tid < D) {
      nk = ldf(k + t * kvs + tid);
      ng = ldf(g + t * kvs + tid);
    }
    nv = ldf(v + t * kvs + col);
    nq = part < a.heads ? ldf(q + t * qs + tid) : 0.f;
  };
  fetch(0);
  const float* S0 = a.S0 ? a.S0 + (size_t)bh * D * D : nullptr;
  double S[RPT], z = 0.0;
#pragma unroll
  for (int r = 0; r < RPT; ++r) S[r] = S0 ? S0[(size_t)(part * RPT + r) * D + col] : 0.f;
  if (tid < D && a.z0) z = a.z0[(size_t)bh * D + tid];
  for (int t = 0; t < a.T; ++t) {
    if (tid < D) {
      const float al = gs1 ? 1.f / (1.f + expf(-ng)) : expf(a.gate_scale * log_sigmoid(ng));
      z = fma((double)al, z, (double)nk);
      sh_a[tid] = al;
      sh_k[tid] = nk;
      sh_z[t & 1][tid] = z;      // (the token before may still be read)
    }
    const float vv = nv, qq = nq;
    __syncthreads();
    if (t + 1 < a.T) fetch(t + 1);
#pragma unroll
    for (int r = 0; r < RPT; ++r) S[r] = fma((double)sh_a[part * RPT + r], S[r], (double)sh_k[part * RPT + r] * (double)vv);
    for (int h0 = 0; h0 < a.heads; h0 += HT) {
      const int nh = min(HT, a.heads - h0);
      if (h0 > 0) __syncthreads();      // the pass before is done with sh_q / sh_part
      if (part < nh) sh_q[part][col] = h0 == 0 ? qq : ldf(q + t * qs + (size_t)h0 * D + tid);
      __syncthreads();
#pragma unroll
      for (int hh = 0; hh < HT; ++hh) {
        if (hh >= nh) break;
        Acc pn[2] = {0, 0};
#pragma unroll
        for (int r = 0; r < RPT; ++r) pn[r & 1] = fma((Acc)sh_q[hh][part * RPT + r], (Acc)S[r], pn[r & 1]);
        sh_part[hh][part][col] = pn[0] + pn[1];
      }
      if (part < nh) {                  // a wave: 64 channels of q . z of its head
        Acc d = row16_sum((Acc)sh_q[part][col] * (Acc)sh_z[t & 1][col]);
        d += lane_get(ln.x1, d);
        d += lane_get(ln.x2, d);
        if ((tid & 63) == 0) sh_den[part][col / 64] = d;
      }
      __syncthreads();
      if (part < nh) {
        Acc num = 0, den = a.eps;
#pragma unroll
        for (int pp = 0; pp < NPART; ++pp) num += sh_part[part][pp][col];
#pragma unroll
        for (int i = 0; i < NWD; ++i) den += sh_den[part][i];
        stf(o + t * qs + (size_t)(h0 + part) * D + col, (float)num / (float)den);
        if (a.den_out != nullptr && col == 0) a.den_out[((size_t)b * a.T + t) * a.Hq + hq0 + h0 + part] = (float)den;
      }
    }
  }
  if (blockIdx.y != 0) return;
  if (tid < D) a.z_out[(size_t)bh * D + tid] = (float)z;
#pragma unroll
  for (int r = 0; r < RPT; ++r) a.S_out[((size_t)bh * D + part * RPT + r) * D + col] = (float)S[r];
}

template <typename T, int D>
hipError_t launch_step_d(const RecurrentParams& p, hipStream_t stream) {
  hipLaunchKernelGGL((gla_step_kernel<T, D>), dim3(p.B * p.Hkv), dim3(256), 0, stream, (const T*)p.q, (const T*)p.k,
                     (const T*)p.v, (const T*)p.g, p.S_out, p.z_out, (T*)p.o, p.Hq, p.Hkv, p.gate_scale, p.eps);
  return hipGetLastError();
}

template <typename T, int D, int HB>
hipError_t launch_sized(const WalkArgs& a, int heads, hipStream_t stream) {
  const hipError_t e = set_lds<gla_walk_kernel<T, D, HB>>(WalkLds<D, HB>::kBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gla_walk_kernel<T, D, HB>), dim3(heads, a.group / a.heads, a.nseg), dim3(4 * D), (WalkLds<D, HB>::kBytes), stream, a);
  return hipGetLastError();
}

// Segments of a fp32 prefill: the walk is one serial chain per query head, so while those are few each is cut into up to kMostSegments
// that are walked side by side, from states that two more steps provide (gla_span_kernel, and the fold at the head of the walk).
// A training pass of 2 heads, us, whole / up to 4 / 8 / 16 segments: 256 tokens of 64 143.7 / 105.5 / 98.7 / 99.1, 512 of 128 427 / 276 / 232 /
// 295 (the fold grows with the segments; 2048 tokens, 32 heads of 64, 684 / 341 / 257 / 240).  Two segments of 32 tokens at head dim 128 gain
// nothing (151 / 152).
constexpr int kMostSegments = 8;
struct Split { int seg_len, nseg; };
Split split_of(int B, int T, int Hq, int Hkv, int d) {
  const long long places = (d == 64 ? 512 : 256) / ((long long)B * Hq > 0 ? (long long)B * Hq : 1);
  const int most = (int)std::min<long long>(places, kMostSegments);
  if (most < 2 || T < (d == 64 ? 2 : 3) * kSpan) return {T, 1};
  const int len = ((T + most - 1) / most + kSpan - 1) / kSpan * kSpan;
  return {len, (T + len - 1) / len};
}
size_t slots_bytes(int heads, int d, int nseg) { return (size_t)heads * (nseg - 1) * (d * d + 2 * d) * sizeof(double); }

template <typename T, int D>
hipError_t launch_walk(const RecurrentParams& p, bool in_place, hipStream_t stream) {
  WalkArgs a{};
  a.q = p.q; a.k = p.k; a.v = p.v; a.g = p.g; a.S0 = p.S0; a.z0 = p.z0; a.o = p.o; a.den_out = p.den_out;
  a.S_out = p.S_out; a.z_out = p.z_out; a.T = p.T; a.Hq = p.Hq; a.Hkv = p.Hkv; a.group = p.Hq / p.Hkv;
  a.gate_scale = p.gate_scale; a.eps = p.eps; a.seg_len = p.T; a.nseg = 1;
  const int heads = p.B * p.Hkv;
  a.heads = a.group;
  // A workgroup per query head where they are all resident at once (two of four waves per compute unit at head dim 64, one of
  // eight at 128): the walk is serial, and the state's update, which every one of them repeats, is the smaller part of it.
  // fp32, 256 tokens, 32 query heads on 8 kv heads, head dim 64 / 128: 68 / 137 us, where one workgroup for the four heads of a
  // group takes 147 / 344.  (Not in place: they would read a state that part 0 replaces.)
  const bool spread = !in_place && (long long)p.B * p.Hq <= (D == 64 ? 512 : 256);
  // A few tokens go one after the other, where the walk pays for a chunk of 16 and, in one workgroup, for one batch of query heads
  // after the other.  us at 1, 3 (in place) or 4 tokens, few / walk: in place, 8 kv heads, one query head each, 8 sequences, head dim
  // 64, bf16 5.0 / 6.4, -, 8.5 / 6.4; four each, one sequence 5.0 / 9.0, 7.7 / 9.1, 9.1 / 9.1, 64 sequences, fp32 7.1 / 18.5, 10.8 / 18.1,
  // 12.8 / 18.1.  Prefill, fp32, 64 sequences: one query head on each of 8 of dim 64 6.4 / 11.3, -, 11.7 / 11.4; eight on each of 4
  // of dim 128 12.3 / 45.9, 6 tokens 39.1 / 46.7, 8 48.8 / 46.6; sixteen on one of dim 128 7.4 / 79.4, 12 tokens 36.8 / 80.6.  Out of
  // place up to 512 workgroups take four query heads each (16 on one of dim 128, one token: 6.3 us, in one workgroup 14.9).
  const int most = in_place ? std::min(4, a.group) : std::max(3, spread ? 0 : 3 * a.group / 4);
  if (p.T <= most) {
    if (!in_place && a.group % 4 == 0 && (long long)heads * (a.group / 4) <= 512) a.heads = 4;
    hipLaunchKernelGGL((gla_few_kernel<T, D>), dim3(heads, a.group / a.heads), dim3(4 * D), 0, stream, a);
    return hipGetLastError();
  }
  if (spread) a.heads = 1;
  if constexpr (sizeof(T) == 4) {
    const Split s = in_place ? Split{p.T, 1} : split_of(p.B, p.T, p.Hq, p.Hkv, D);
    if (s.nseg > 1 && p.workspace != nullptr && p.workspace_bytes >= slots_bytes(heads, D, s.nseg)) {
      a.seg_len = s.seg_len; a.nseg = s.nseg; a.slots = static_cast<double*>(p.workspace);
      constexpr int lds = kSpan * (8 * D + 16);
      const hipError_t e = set_lds<gla_span_kernel<D>>(lds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(gla_span_kernel<D>, dim3(a.nseg - 1, heads), dim3(4 * D), lds, stream, a);
    }
  }
  // four query heads at a time; two where fp64 sums at head dim 128 would not leave registers for four (256, and 44 spilled)
  if constexpr (sizeof(T) == 2 || D == 64)
    if (a.heads % 4 == 0) return launch_sized<T, D, 4>(a, heads, stream);
  if (a.heads % 2 == 0) return launch_sized<T, D, 2>(a, heads, stream);
  return launch_sized<T, D, 1>(a, heads, stream);
}

hipError_t launch_walk(const RecurrentParams& p, bool in_place, hipStream_t stream) {
  if (p.bf16) return p.d == 64 ? launch_walk<bf16_t, 64>(p, in_place, stream) : launch_walk<bf16_t, 128>(p, in_place, stream);
  return p.d == 64 ? launch_walk<float, 64>(p, in_place, stream) : launch_walk<float, 128>(p, in_place, stream);
}

}  // namespace

hipError_t launch_gla_step(const RecurrentParams& p, hipStream_t stream) {
  if (p.bf16) return p.d == 64 ? launch_step_d<bf16_t, 64>(p, stream) : launch_step_d<bf16_t, 128>(p, stream);
  return p.d == 64 ? launch_step_d<float, 64>(p, stream) : launch_step_d<float, 128>(p, stream);
}

size_t gla_recurrent_workspace_bytes(int B, int T, int Hq, int Hkv, int d) {
  const Split s = split_of(B, T, Hq, Hkv, d);
  return s.nseg > 1 ? slots_bytes(B * Hkv, d, s.nseg) : 0;
}

// S0, z0 may be the same memory as S_out, z_out here too
hipError_t launch_gla_recurrent(const RecurrentParams& p, hipStream_t stream) {
  const bool in_place = p.S0 == p.S_out || p.z0 == p.z_out;
  return launch_walk(p, in_place, stream);
}

// n consecutive decode steps: the same walk, from and into the caller's state
hipError_t launch_gla_steps(const RecurrentParams& p, hipStream_t stream) { return launch_walk(p, true, stream); }

}  // namespace lawcat
