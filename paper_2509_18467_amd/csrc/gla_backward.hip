// Adjoint of the normalized gated linear attention of paper section 4.2 (what the layer-wise distillation of
// section 5 differentiates through): given dO = dL/do and the forward's den, the gradients with respect to
// q-dot, k-dot, v, the gate logits and the start state.  With v^ = [v, 1], S^ = [S | z]:
//   dnum = dO / den,  dden = -(dO . o) / den = -(q_t S_t dnum^T) / den,   d^ = [dnum | dden]
//   (o is never read: rounded to the storage type it would spoil dq, where S dnum^T and z dden nearly cancel)
//   dq_t = S^_t d^_t^T
//   Gr_t = alpha_{t+1} (.) Gr_{t+1} + sum_h q_{h,t}^T d^_{h,t}
//   dk_t = Gr_t v^_t^T,   dv_t = k_t Gr_t[:, :dv]
//   dlog alpha_t = sum_{s >= t} ( sum_h q_{h,s} (.) dq_{h,s} - k_s (.) dk_s )     (every pair i < t <= s carries
//                  alpha_t once, in the query's gradient and not in the key's)
//   dg_t = dlog alpha_t * gate_scale * (1 - sigmoid(g_t))
//
// Chunked form, in fp32 accuracy (chunk_f32.h).  Within a chunk of up to 16 tokens, with E_t the decay from the
// chunk's first token on, Q' = q (.) E, K' = k / E, S~ the state decayed up to and including the first token and
// R~ = E_last (.) (the gradient that flows into the chunk's end):
//   dq_t = [ E_t (.) ( S~ dO_t + sum_{i<=t} (dO_t . v_i) K'_i ) ] / den_t + z_t dden_t,   z_t = E_t (.) ( z~ + sum_{i<=t} K'_i )
//   S~ <- S~ + K'^T V   (times E_last and the next alpha when the next chunk begins)
//   dk_i = [ R~ v_i + R~z + sum_{h, s>=i} Q'_s ( (dO_s . v_i) / den_s + dden_s ) ] / E_i
//   dv_i = K'_i R~ + sum_{h, s>=i} (Q'_s . K'_i / den_s) dO_s
//   R~ <- R~ + sum_h Q'^T d^   (times alpha of the chunk's first token when the chunk before it begins)
// Where a channel decays too fast for the quotients k / E, the forward sweep takes the chunk token by token on the vector ALUs,
// S_t and z_t in registers.  So does the reverse sweep, for all chunks of the segment: one loop with both forms in it took registers
// from the ordinary one (fp32 storage, 32768 tokens, 1520 us where two loops take 1063).  And a token whose operands or denominator
// are not finite may spoil only what the equations say: the sums above run over masked matrices, where a zero weight times an
// infinity is a NaN.  The forward sweep flags a segment with such a token, and the reverse sweep goes token by token there.
// bf16 / fp32 storage, 32768 tokens, 32 / 8 heads of 64, us a call: ordinary gates 412 / 1063, one channel's logits at -30 1290 /
// 1830, in blocks of one token with the matrices 3000 / 9450; 2 tokens of 100 closed in all channels 995 / 1615 (in blocks 666 / 1925).
// Launches: with one segment, the forward sweep (dq, dden, and the segments' contributions to the gradient that flows backwards) and
// the reverse sweep (dk, dv, dg).  With more, the segments' contributions to the state come first (walked backwards, so that the walk
// stops once nothing earlier can reach the segment's end); beyond a few, a scan follows them, and another one the forward sweep.
// The gate's sum over all later tokens is split at segment ends, where it equals sum_j S^[c, j] Gr[c, j], the states on the two
// sides of the boundary: no pass over the sequence is needed for it.
//
// What it measures (32768 tokens, 32 query heads on 8 kv heads, d = 64, bf16), kernel by kernel in a training pass under a profiler, at their
// quickest / on average: state 14 / 15, scans 4, forward sweep 155 / 172, reverse sweep 152 / 171 (on a slower card 164 / 181, 163 / 182).  The two sweeps move 0.57 and 0.54 GB (q, dO,
// k, v, g once each, the gate term in fp32, the gradients), 105 us each at the rate of a large copy; what bounds them is a workgroup's dependent
// chain through a chunk's sections between two barriers, at two waves per SIMD, whose registers leave room for no third (a limit of
// 168 spilled: forward 636 us, reverse 423).  The training pass, us, step by step: 645; the reverse sweep's products of two fp32 operands as bf16 terms
// (chunk_f32.h) 638; dO and v, which only go to LDS, loaded as whole rows (a load of a patch touched 16 rows for 32 bytes, and the
// issue of a chunk's twelve took a sixth of it) 613; no branch around the reverse sweep's loads, whose join waited for all of them,
// 599; 32-bit offsets and the operands of the state's update read together 597; patches with a row's four lanes side by side, whose loads
// then are 16 accesses and not 64, 586.  Nothing or worse: patches transposed through LDS (667), rows a chunk ahead through LDS (624), loads spread over the
// stage (627), a denominator load per wave (623).
//
// fp32 storage: the sums of every contraction are fp64 MFMAs and decays are multiplied up in 64 bits, rounded per chunk, because
// chains of fp32 MFMAs alone were up to 2.4 times further from 64-bit arithmetic than sums token by token.  2-norm errors of
// gradients, 20 tokens of 2 heads, 256 sequences, all sums token by token in fp32 / as it is: dq 3.7e-7 / 2.9e-7, dk 1.6e-7 / 9.5e-8,
// dv 6.1e-8 / 4.6e-8, dS0 8.2e-8 / 8.0e-8, dz0 1.1e-7 / 9.5e-8; logits ~ N(0, 5^2), where chunks go token by token, 40 tokens, 8 heads
// on 2: dq 2.2e-7 / 1.9e-7, dk 1.7e-7 / 1.4e-7, dv 6.1e-8 / 5.0e-8, dg 2.7e-6 / 2.1e-6.  256 tokens of 2 heads: 124 / 55 us.
#include "chunk_f32.h"

namespace lawcat {
namespace {
using namespace f32c;

// A chunk in which a channel decays by more than this from its first token on goes token by token: centred (chunk_f32.h), the
// operands of its products stand within 2^40 of unscaled values.
constexpr float kWhole = 8.271806125530277e-25f;   // 2^-80

template <typename T> using Wide = std::conditional_t<sizeof(T) == 4, double, float>;
template <typename T> __device__ inline float inverse(float x) { return sizeof(T) == 4 ? 1.f / x : __builtin_amdgcn_rcpf(x); }

struct BwdArgs {
  const void *q, *k, *v, *g, *dO;
  const float* den;
  const float *S0, *z0;
  void *dq, *dk, *dv, *dg;
  float *dS0, *dz0;
  float* dden;       // [heads][tokens][group], a chunk's as [group][its tokens]
  float* qdq;        // sum_h q (.) dq: [heads][tokens][D], a chunk's in the patch layout ([D / 16][64 lanes][4 tokens]), or, of
                     // fewer than 16 tokens, as [D][its tokens]
  uint8_t* serial;   // [heads][segments]: whether the reverse sweep goes token by token
  float* slots_f;    // [heads][nseg - 1][D*D + 2D]: forward contributions, then the states after the segments
  float* slots_r;    // the same for Gr, segments in reverse order
  int *live_f, *live_r;   // [heads][nseg]: 0 = the segment's total decay is exactly zero in every channel
  int B, T, Hq, Hkv, group, seg_len, nseg;
  int fold;          // few segments: the sweeps fold their predecessors' contributions, there are no scans
  float gate_scale;
};

template <int D> constexpr int slot_floats() { return D * D + 2 * D; }

// This lane's part (channel c, value columns 16 jt + 4 g ..) of the state before segment `seg`: what the scan left (it leaves the
// contributions as they are where no segment passes its start state on: they are the states after them then), or, with few
// segments, the contributions before it folded here, from after the last segment whose total decay is exactly zero.
// slots, live: of this head; S0, z0: its start state or null.  Uniform.
template <int D>
__device__ inline void start_state(const float* slots, const int* live, bool fold, int seg, const float* S0, const float* z0,
                                   int c, int g, floatx4 (&X)[D / 16], float& z) {
  int first = seg;                           // first segment whose contribution is still to be added
  const float *src = nullptr, *zsrc = nullptr;
  if (fold) {
    const int l = threadIdx.x & 63;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(l < seg && live[l] == 0);
    first = m ? 64 - __builtin_clzll(m) : 0;
  }
  if (first > 0) {
    src = slots + (size_t)(first - 1) * slot_floats<D>();
    zsrc = src + D * D;
  } else {
    src = S0;
    zsrc = z0;
  }
#pragma unroll
  for (int jt = 0; jt < D / 16; ++jt)
    X[jt] = src ? *reinterpret_cast<const floatx4*>(src + (size_t)c * D + 16 * jt + 4 * g) : floatx4{0.f, 0.f, 0.f, 0.f};
  z = zsrc ? zsrc[c] : 0.f;
#pragma unroll 1
  for (int j = first; j < seg; ++j) {
    const float* slot = slots + (size_t)j * slot_floats<D>();
    const float dec = slot[D * D + D + c];
    z = fmaf(dec, z, slot[D * D + c]);
#pragma unroll
    for (int jt = 0; jt < D / 16; ++jt) {
      const floatx4 x = *reinterpret_cast<const floatx4*>(slot + (size_t)c * D + 16 * jt + 4 * g);
#pragma unroll
      for (int i = 0; i < 4; ++i) X[jt][i] = fmaf(dec, X[jt][i], x[i]);
    }
  }
}

// ---- contribution of a segment to the state at its end: sum_i (k_i (.) decay from i to the end)^T v^_i.
// grid (nseg - 1, heads).  Granules of 64 tokens, last one first; stops when the decay is exactly zero in all channels.
template <typename T, int D>
__global__ void __launch_bounds__(4 * D) bwd_state_kernel(const BwdArgs a) {
  typedef Store<T> St;
  constexpr int NW = D / 16, NM = 4;
  __shared__ __attribute__((aligned(16))) unsigned char vrows[NM * kC * St::template row_bytes<D>()];
  __shared__ int flags[NW];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, g = l >> 4, n = l & 15;
  const Lanes ln = make_lanes(l);
  const Turn qd = make_turn(l);
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / a.Hkv, hk = bh % a.Hkv;
  const int s0 = seg * a.seg_len, rows = min(a.T, s0 + a.seg_len) - s0;
  const unsigned stride = (unsigned)a.Hkv * D * St::kBytes;
  const size_t first = (((size_t)b * a.T + s0) * a.Hkv + hk) * D * St::kBytes;
  const Rows K = make_rows(a.k, first, stride, rows, D * St::kBytes), V = make_rows(a.v, first, stride, rows, D * St::kBytes),
             Gt = make_rows(a.g, first, stride, rows, D * St::kBytes);
  const unsigned off = St::row_offset(K, g, n, 16 * w);
  floatx4 X[D / 16];
#pragma unroll
  for (int jt = 0; jt < D / 16; ++jt) X[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
  float z = 0.f, run = 1.f;
  constexpr bool kRows = sizeof(T) == 2;        // v as whole rows
  typename St::Raw rk[NM], rv[kRows ? 1 : NM], rg[NM];
  WholeRows<D, 1> wv[kRows ? NM : 1];
  const unsigned offv = WholeRows<D, 1>::offset(V, threadIdx.x);
  auto fetch = [&](int t0) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      rg[m] = St::load(Gt, off, t0 + kC * m);
      rk[m] = St::load(K, off, t0 + kC * m);
      if constexpr (kRows) wv[m].load(V, offv, t0 + kC * m);
      else rv[m] = St::load(V, off, t0 + kC * m);
    }
  };
  int t0 = (rows - 1) / (NM * kC) * (NM * kC);
  fetch(t0);
  bool live = true;
  for (;;) {
    float kd[NM][4];
#pragma unroll
    for (int m = NM - 1; m >= 0; --m) {
      if constexpr (kRows) wv[m].to_lds(vrows + m * kC * St::template row_bytes<D>(), St::template row_bytes<D>(), threadIdx.x);
      else St::template to_lds<D>(vrows + m * kC * St::template row_bytes<D>(), g, n, 16 * w, rv[m]);
      float gl[4], kk[4], al[4];
      St::row_patch(qd, rg[m], gl);
      St::row_patch(qd, rk[m], kk);
      alphas_of(gl, a.gate_scale, rows - (t0 + kC * m + 4 * g), al);
      const float s2 = al[3], s1 = al[2] * s2, s0x = al[1] * s1, tot = al[0] * s0x;
      const float x1 = lane_get(ln.x1, tot), x2 = lane_get(ln.x2, tot), x3 = lane_get(ln.x3, tot);
      const float after = ((g & 1) ? 1.f : x1) * ((g & 2) ? 1.f : x2 * x3) * run;
      kd[m][0] = kk[0] * (s0x * after); kd[m][1] = kk[1] * (s1 * after); kd[m][2] = kk[2] * (s2 * after); kd[m][3] = kk[3] * after;
      run *= (tot * x1) * (x2 * x3);
      z += (kd[m][0] + kd[m][1]) + (kd[m][2] + kd[m][3]);
    }
    live = __builtin_amdgcn_ballot_w64(run != 0.f) != 0;
    if (l == 0) flags[w] = live;
    __syncthreads();
    int any = 0;
#pragma unroll
    for (int j = 0; j < NW; ++j) any |= flags[j];
    live = __builtin_amdgcn_readfirstlane(any) != 0;
    t0 -= NM * kC;
    const bool more = t0 >= 0 && live;
    if (more) fetch(t0);
    accumulate<T, D, NM>(X, vrows, g, n, kd);
    if (!more) break;
    __syncthreads();
  }
  float* slot = a.slots_f + ((size_t)bh * (a.nseg - 1) + seg) * slot_floats<D>();
  const int c = 16 * w + St::channel(n);
#pragma unroll
  for (int jt = 0; jt < D / 16; ++jt) *reinterpret_cast<floatx4*>(slot + (size_t)c * D + 16 * jt + 4 * g) = X[jt];
  z += lane_get(ln.x1, z);
  z += lane_get(ln.x2, z);
  if (g == 0) {
    slot[D * D + c] = z;
    slot[D * D + D + c] = run;
  }
  if (threadIdx.x == 0) a.live_f[(size_t)bh * a.nseg + seg] = live;
}

// A word of an array, by a 32-bit offset from a uniform pointer.  (One wave reads the chunk's denominators, and the others wait for it at
// the next barrier: with 64-bit indices 300 of a chunk's 8500 cycles more.  Training pass, 9001 tokens of 16 / 8 heads of 64 206.1 -> 202.9
// us, 700 of 32 / 8 95.1 -> 94.2; with a head's denominators per wave 32768 tokens 612.7 -> 622.9.)
__device__ inline float at32(const float* base, unsigned word) { return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + (size_t)(word * 4u)); }

template <typename T, int D, int HB>
struct Sweep {
  typedef Store<T> St;
  static constexpr int NW = D / 16;                               // waves: 16 key channels each
  static constexpr int kRow = St::template row_bytes<D>();
  static constexpr int kSet = kC * kRow;                          // one head's (or v's) rows of a chunk
  static constexpr int kO = HB * kSet;                            // dO rows of HB heads
  static constexpr int kPairs = 2 * HB * kC * 4;                  // two floats per head and token
  // fp32 storage: dO . v (at head dim 64 also the scores, whose tiles would not fit at 128) formed by each wave over its own channels
  // and added up, where otherwise every wave forms all of it in fp64 MFMAs, which bound these sweeps (32768 tokens of 32 / 8 heads of
  // 64: 1077 us and 1256; of 128, dO . v alone, 4000 tokens 500 and 586, 500 tokens of 8 / 2 heads 243 and 287)
  static constexpr bool kDaParts = sizeof(T) == 4, kParts = kDaParts && D == 64;
  // bf16 storage, reverse: a head's dO . v formed by one wave and read by all from behind the barrier that the scores need.  32768 tokens
  // of 32 / 8 heads of 64, the training pass 678.3 -> 669.5 us, 8000 of 128 494.6 -> 485.0, 4000 of 8 / 8 heads of 128 209.1 -> 207.1; 8000
  // of 8 / 8 heads of 64, where it is two MFMAs, 174.7 / 175.7.
  static constexpr bool kDaOnce = !kDaParts && (HB > 1 || D == 128);
  // bf16 storage, head dim 64, two workgroups to a compute unit: the one in its chain of products goes first (forward: between the two
  // barriers; reverse: from the scores on to the next chunk's rows).  32768 tokens of 32 / 8 heads, the training pass 659.0 -> 648.6 us,
  // 16000 slowly decaying 415.6 -> 403.8; the other way round in either sweep 663-674 of 670 to 659.  500 tokens, where units have one
  // workgroup, 91.8 / 92.5; fp32 storage 256 tokens of 2 heads 96.3 / 96.9 with it.  Which sweeps take it for how many workgroups: see
  // launch_sized().
  static constexpr bool kPair = sizeof(T) == 2 && D == 64;
  // bf16 storage, reverse: products of two fp32 operands, too, go through the matrix cores as bf16 terms (mfma_terms(), 192 cycles
  // where fp32 MFMAs take 512): q E / den is split once, for the update of R~, dk and the scores, R~ for dk and dv, a head's dO . v by the
  // wave that forms it.  The matrix cores are busy for 1184 cycles a wave and chunk instead of 2144, 32768 tokens of 32 / 8 heads of 64, the
  // training pass, 649 -> 638 us, 9001 of 16 / 8 heads 217.3 -> 210.4; bf16 results that differ from rounded exact ones, 3001 to
  // 65536 tokens of 32 / 8, 16 / 8 and 32 / 4 heads, N(0, 1) and slow gates: dk 0.75 to 0.97, dv 0.58 to 0.77, dg 0.80 to 0.97 times as many.  Head dim 128, whose terms do not fit the LDS (dk alone: 389 -> 395 us for 6000 tokens, registers), and one query
  // head a pass (three workgroups a compute unit) keep fp32 MFMAs.
  static constexpr bool kScoreTerms = kDaOnce && D == 64;
  static constexpr int kDaWave = NW >= 2 * HB ? HB : 0;           // the first of these waves, after those with the scores where there are
  static constexpr int kTile = 2048;
  // forward, twice, in turn, so that no wave waits for the others to be done with a chunk before it begins the next: dO rows | v rows |
  // 1 / den, den per head and token | one word per wave
  static constexpr int oV = kO;
  static constexpr int oDen = oV + kSet;
  static constexpr int oFlag = oDen + kPairs;
  static constexpr int kTurn = oFlag + 32;
  // once: partial q . u of every wave | parts of dO . v | the state before a chunk that goes token by token
  static constexpr int oPart = 2 * kTurn;
  static constexpr int oDa = oPart + NW * HB * kC * 4;
  static constexpr int oX = oDa + (kDaParts ? NW * HB * kTile : 0);
  static constexpr int kForward = oX + D * D * 4;
  // reverse: dO rows (in bf16 storage twice, in turn: they are read last in a chunk, unless their operands are read ahead) | v rows |
  // 1 / den, dden | K' rows | R~ [channel][value column] | Q' rows of HB heads | scores
  static constexpr int rV = kDaParts || kScoreTerms ? kO : 2 * kO;
  static constexpr int rDen = rV + kSet;
  static constexpr int kTriples = 3 * HB * kC * 4;                // (dden as it is, too)
  static constexpr int rK = rDen + (kScoreTerms ? 2 * kTriples : kPairs);
  static constexpr int kTerms = 3 * D * kC * 2;                   // a row per channel and term: 16 tokens
  static constexpr int rR = rK + (kScoreTerms ? kTerms : kC * f32_row_bytes<D>());
  static constexpr int kStateTerms = 3 * D * D * 2;
  static constexpr int rQ = rR + (kScoreTerms ? kStateTerms : D * f32_row_bytes<D>());
  static constexpr int rSc = rQ + HB * (kScoreTerms ? kTerms : kC * f32_row_bytes<D>());
  static constexpr int kScore = sizeof(T) == 2 ? 3 * 512 : 2048;  // per head: three terms of 8 bytes per lane, or one fp64 tile
  // (or parts of the scores), then dO . v per head or its parts
  static constexpr int rDa = rSc + HB * (kParts ? NW * kTile : kScore);
  static constexpr int kDa = kScoreTerms ? 3 * 512 : 1024;        // kDaOnce: per head three terms of 8 bytes per lane, or fp32
  static constexpr int kReverse = rDa + (kDaParts ? NW * HB * kTile : kDaOnce ? HB * kDa : 0);
  static_assert(kForward <= 160 * 1024 / (D == 64 ? 2 : 1) && kReverse <= 160 * 1024 / (D == 64 ? 2 : 1));
};

// ---- forward sweep: dq, dden, sum_h q (.) dq, and the segment's contribution to the gradient flowing backwards.
// grid (nseg, heads), 4 D threads.
template <typename T, int D, int HB, bool PAIR>
__global__ void __launch_bounds__(4 * D, 2) bwd_forward_kernel(const BwdArgs a) {
  typedef Store<T> St;
  typedef Sweep<T, D, HB> L;
  constexpr int NW = L::NW;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  unsigned char* sm = lds;      // this chunk's turn of the rows
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, g = l >> 4, n = l & 15;
  const Lanes ln = make_lanes(l);
  const Turn qd = make_turn(l);
  constexpr bool kWide = sizeof(T) == 4;      // fp32 storage: contractions summed in 64 bits
  const int row = kWide ? strided(n) : n;     // the A operand's row in this lane
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / a.Hkv, hk = bh % a.Hkv;
  const int s0 = seg * a.seg_len, rows = min(a.T, s0 + a.seg_len) - s0;
  const int nb = a.group / HB;
  const unsigned kvs = (unsigned)a.Hkv * D * St::kBytes, qs = (unsigned)a.Hq * D * St::kBytes;
  const size_t kv1 = (((size_t)b * a.T + s0) * a.Hkv + hk) * D * St::kBytes;
  const size_t q1 = (((size_t)b * a.T + s0) * a.Hq + (size_t)hk * a.group) * D * St::kBytes;
  const Rows K = make_rows(a.k, kv1, kvs, rows, D * St::kBytes), V = make_rows(a.v, kv1, kvs, rows, D * St::kBytes),
             Gt = make_rows(a.g, kv1, kvs, rows, D * St::kBytes), Q = make_rows(a.q, q1, qs, rows, a.group * D * St::kBytes),
             O = make_rows(a.dO, q1, qs, rows, a.group * D * St::kBytes), dQ = make_rows(a.dq, q1, qs, rows, a.group * D * St::kBytes);
  const unsigned offk = St::row_offset(K, g, n, 16 * w), offq = St::row_offset(Q, g, n, 16 * w);
  const int c = 16 * w + St::channel(n);

  // state before the next chunk's first token (to be decayed by f), normalizer; gradient contribution
  floatx4 X[D / 16], R[D / 16];
  float z = 0.f;
  double Rz = 0.0;       // a long sum of signed terms: 64 bits
  start_state<D>(a.slots_f + (size_t)bh * (a.nseg - 1) * slot_floats<D>(), a.live_f + (size_t)bh * a.nseg, a.fold, seg,
                 a.S0 ? a.S0 + (size_t)bh * D * D : nullptr, a.z0 ? a.z0 + (size_t)bh * D : nullptr, c, g, X, z);
#pragma unroll
  for (int jt = 0; jt < D / 16; ++jt) R[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
  float pend = 1.f;      // E_last of the chunk before
  float P = 1.f;         // decay from the segment's start up to the chunk before
  float qdq[4] = {0.f, 0.f, 0.f, 0.f};

  // inputs of the next item, in registers.  Item = (chunk, HB query heads).
  constexpr bool kRows = sizeof(T) == 2;        // dO and v as whole rows
  typename St::Raw rq[HB], rk, rg, ro[kRows ? 1 : HB], rv;
  WholeRows<D, HB> wo;
  WholeRows<D, 1> wv;
  const unsigned offwo = WholeRows<D, HB>::offset(O, tid), offwv = WholeRows<D, 1>::offset(V, tid);
  const float* dens = a.den + ((size_t)b * a.T + s0) * a.Hq + (size_t)hk * a.group;     // (its rows lie within 32-bit offsets, as those of q do)
  float rden = 1.f;
  auto fetch = [&](int ci, int hb) {
    const int row0 = ci * kC;
    if (hb == 0) {
      rg = St::load(Gt, offk, row0);
      rk = St::load(K, offk, row0);
      if constexpr (kRows) wv.load(V, offwv, row0);
      else rv = St::load(V, offk, row0);
    }
    if constexpr (kRows) wo.load(O, offwo + (unsigned)(hb * HB) * D * St::kBytes, row0);
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      const unsigned ho = (unsigned)(hb * HB + h) * D * St::kBytes;
      if constexpr (!kRows) ro[h] = St::load(O, offq + ho, row0);
      rq[h] = St::load(Q, offq + ho, row0);
    }
    if (tid < HB * kC) {
      const int t = row0 + (tid & 15);
      rden = t < rows ? at32(dens, (unsigned)(t * a.Hq + hb * HB + (tid >> 4))) : 1.f;
    }
  };

  const int nchunk = (rows + kC - 1) / kC;
  int ci = 0, hb = 0;
  // What follows takes some instructions out of the four heads' pass, with row16_sums() below: 32768 tokens of 32 / 8 heads of 64, the
  // training pass 680.0 -> 673.5 us, 16000 that decay slowly 426.0 -> 421.1 (with one or two heads it gives nothing).
  constexpr bool kAlways = HB == 4;           // rows past the last chunk are requested too (they read as zero): no registers change places
  constexpr bool kSkip = HB == 4 && D == 64;  // no sums for the segment's start that nothing reaches; at head dim 128 the branch's
                                              // registers spill (8000 tokens 498.6 / 519)
  constexpr int kSharp = 1, kBad = 2;
  bool sharp = false, serial = false;   // a wave's channels decay too fast for products over the chunk; any wave's: token by token
  bool any_serial = false;
  bool bad = false;      // a token of the chunk has a query too large, or operands or a denominator that are not finite
  Decay d;
  float kk[4], kp[4], zt[4], wf = 0.f;
  if (nchunk > 0) fetch(0, 0);
  while (ci < nchunk) {
    const int row0 = ci * kC;
    const size_t token = (size_t)bh * a.T + s0 + row0;
    const int len = min(kC, rows - row0);        // the chunk's tokens
    // ---- rows to LDS, gates
    if (hb == 0) {
      float gl[4];
      St::row_patch(qd, rg, gl);
      St::row_patch(qd, rk, kk);
      alphas_of(gl, a.gate_scale, rows - (row0 + 4 * g), d.al);
      bool tame = true;
#pragma unroll
      for (int i = 0; i < 4; ++i) tame = tame && fabsf(kk[i]) < kTame;
      whole_chunk<Wide<T>>(d, ln, g);
      sharp = __builtin_amdgcn_ballot_w64(!tame || !(d.last >= kWhole)) != 0;
      bad = false;
    }
    // (v in every turn: the registers hold it for all of the chunk's heads)
    if constexpr (kRows) {
      wv.to_lds(sm + L::oV, L::kRow, tid);
      wo.to_lds(sm, L::kRow, tid);
    } else {
      St::template to_lds<D>(sm + L::oV, g, n, 16 * w, rv);
#pragma unroll
      for (int h = 0; h < HB; ++h) St::template to_lds<D>(sm + h * L::kSet, g, n, 16 * w, ro[h]);
    }
    if constexpr (L::kDaParts) {
      __builtin_amdgcn_wave_barrier();   // LDS serves one wave's requests in order: its rows are complete below
#pragma unroll
      for (int h = 0; h < HB; ++h) dot_part64<D>(sm + L::oV, sm + h * L::kSet, w, g, n, lds + L::oDa + (w * HB + h) * L::kTile);
    }
    if (tid < HB * kC) {
      float* den = reinterpret_cast<float*>(sm + L::oDen);
      den[tid] = 1.f / rden;
      den[HB * kC + tid] = rden;
    }
    float qq[HB][4];
#pragma unroll
    for (int h = 0; h < HB; ++h) St::row_patch(qd, rq[h], qq[h]);
    float top = 0.f;       // largest |q|
#pragma unroll
    for (int h = 0; h < HB; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) top = fmaxf(top, fabsf(qq[h][i]));
    bad = bad || __builtin_amdgcn_ballot_w64(!(top < kTame)) != 0;
    int* flags = reinterpret_cast<int*>(sm + L::oFlag);
    if (l == 0) flags[w] = (sharp ? kSharp : 0) | (bad ? kBad : 0);
    __syncthreads();
    if (PAIR) __builtin_amdgcn_s_setprio(1);
    if (hb == 0) {
      int any = 0;
#pragma unroll
      for (int j = 0; j < NW; ++j) any |= flags[j];
      serial = __builtin_amdgcn_readfirstlane(any & kSharp) != 0;
    }
    const int hb1 = hb + 1 < nb ? hb + 1 : 0;
    const int ci1 = hb1 ? ci : ci + 1;
    if (!serial && (kAlways || ci1 < nchunk)) fetch(ci1, hb1);
    // ---- once per chunk: decays, K', the state decayed up to the first token, z_t
    if (hb == 0 && serial) {
#pragma unroll
      for (int jt = 0; jt < D / 16; ++jt)
#pragma unroll
        for (int i = 0; i < 4; ++i) X[jt][i] *= pend;
      z *= pend;
      wf = P * d.first;
      P *= d.first * d.last;
      pend = 1.f;
    } else if (hb == 0) {
      center(d);
      const float f = d.first * pend;
#pragma unroll
      for (int jt = 0; jt < D / 16; ++jt)
#pragma unroll
        for (int i = 0; i < 4; ++i) X[jt][i] *= f;
      z *= f;
      float ones[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        kp[i] = kk[i] * inverse<T>(d.E[i]);
        // running sums over the tokens: a lower triangle of ones against K'
        ones[i] = 4 * g + i <= row ? 1.f : 0.f;
      }
      const floatx4 pz = token_steps<kWide>(ones, kp, floatx4{z, z, z, z});
#pragma unroll
      for (int i = 0; i < 4; ++i) zt[i] = d.E[i] * pz[i];
      z = lane_get(ln.n4 + 192, pz[3]);      // all of the chunk's tokens
      wf = P * d.first;
      P *= d.first * d.last;
      pend = d.last;
    }
    const bool last_head = hb + 1 == nb;
    floatx4 u[HB];
    if (serial) {
      // ---- token by token: S_t, z_t, u_t = S_t dO_t
      int lane = l;                                   // not known to be l: nothing of this loop is formed before it
      asm volatile("" : "+v"(lane));
      const int gs = lane >> 4, ns = lane & 15;
      const Lanes lns = make_lanes(lane);
      floatx4* before = reinterpret_cast<floatx4*>(lds + L::oX) + tid;
      const float z0 = z;
      if (!last_head) {
#pragma unroll
        for (int jt = 0; jt < D / 16; ++jt) before[4 * D * jt] = X[jt];
      }
#pragma unroll 1
      for (int tg = 0; tg < 4; ++tg) {
        const int from = ((tg << 4) + ns) << 2;       // the lane that holds tokens 4 tg .. of this channel
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned char* col = sm + (4 * tg + i) * L::kRow + 4 * gs * St::kBytes;
          const float al = lane_get(from, d.al[i]), kt = lane_get(from, kk[i]);
          z = fmaf(al, z, kt);
          if (gs == tg) zt[i] = z;
          constexpr int NP = kWide ? 4 : 1;            // partial sums
          float part[HB][NP] = {};
#pragma unroll
          for (int jt = 0; jt < D / 16; ++jt) {
            const floatx4 v4 = St::four(col + L::oV + 16 * jt * St::kBytes);
#pragma unroll
            for (int e = 0; e < 4; ++e) X[jt][e] = fmaf(al, X[jt][e], kt * v4[e]);
#pragma unroll
            for (int h = 0; h < HB; ++h) {
              const floatx4 o4 = St::four(col + h * L::kSet + 16 * jt * St::kBytes);
#pragma unroll
              for (int e = 0; e < 4; ++e) part[h][e % NP] = fmaf(X[jt][e], o4[e], part[h][e % NP]);
            }
          }
#pragma unroll
          for (int h = 0; h < HB; ++h) {
            float sum = kWide ? (part[h][0] + part[h][1 % NP]) + (part[h][2 % NP] + part[h][3 % NP]) : part[h][0];
            sum += lane_get(lns.x1, sum);
            sum += lane_get(lns.x2, sum);
            u[h][i] = gs == tg ? sum : (tg == 0 ? 0.f : u[h][i]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (kAlways || ci1 < nchunk) fetch(ci1, hb1);     // not before: its registers are the loop's
      if (!last_head) {
        z = z0;
#pragma unroll
        for (int jt = 0; jt < D / 16; ++jt) X[jt] = before[4 * D * jt];
      }
    } else {
      // ---- u_t = E_t ( S~ dO_t + sum_{i <= t} (dO_t . v_i) K'_i )
#pragma unroll
      for (int h = 0; h < HB; ++h) u[h] = floatx4{0.f, 0.f, 0.f, 0.f};
      contract<T, D, HB>(X, sm, g, n, u);
#pragma unroll
      for (int h = 0; h < HB; ++h) {
        floatx4 da;    // [token i of v][token `row` of dO]
        if constexpr (L::kDaParts) da = add64(floatx4{0.f, 0.f, 0.f, 0.f}, sum_parts64<NW>(lds + L::oDa + h * L::kTile, HB * L::kTile, g, n));
        else da = dot_rows<T, D, kWide>(sm + L::oV, sm + h * L::kSet, g, n);
        float am[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) am[i] = 4 * g + i <= row ? da[i] : 0.f;
        const floatx4 s = token_steps<kWide>(am, kp, floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int i = 0; i < 4; ++i) u[h][i] = (u[h][i] + s[i]) * d.E[i];
      }
    }
    float* part = reinterpret_cast<float*>(lds + L::oPart);
    if constexpr (HB == 4) {
      float qu[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) qu[j] = qq[j >> 2][j & 3] * u[j >> 2][j & 3];
      part[(w * HB + (n >> 2)) * kC + 4 * g + (n & 3)] = row16_sums(qu, n);
    } else {
#pragma unroll
      for (int h = 0; h < HB; ++h) {
        floatx4 s;
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = row16_sum(qq[h][i] * u[h][i]);
        if (n == 0) *reinterpret_cast<floatx4*>(part + (w * HB + h) * kC + 4 * g) = s;
      }
    }
    __syncthreads();
    if (PAIR) __builtin_amdgcn_s_setprio(0);
    // ---- dden = -(q . u) / den^2, dq = u / den + z dden
    const bool carries = __builtin_amdgcn_ballot_w64(wf != 0.f) != 0;   // this wave's channels still reach the segment's start
    float qw[HB][4];
    Wide<T> rz = 0;
    // dden of head (n / 4) % HB and token 4 g + n % 4 in this lane: the waves' parts summed in 64 bits, rounded once (every
    // lane forming all of its row's sixteen, in fp32: 489 us for the call at 32768 tokens, this 471)
    float mine;
    {
      const int h = (n >> 2) & (HB - 1), t = 4 * g + (n & 3), at = h * kC + t;
      double s = 0.0;
#pragma unroll
      for (int j = 0; j < NW; ++j) s += (double)part[j * HB * kC + at];
      const float* den = reinterpret_cast<const float*>(sm + L::oDen);
      const double r = den[at], rr = r + r * (1.0 - (double)den[HB * kC + at] * r);
      mine = (float)(-(s * rr) * rr);
      if (w == 0 && n < 4 * HB && t < len) (a.dden + token * a.group)[(unsigned)((hb * HB + h) * len + t)] = mine;
    }
    const float dds[16] = {row16_get<0>(mine), row16_get<1>(mine), row16_get<2>(mine), row16_get<3>(mine),
                           row16_get<4>(mine), row16_get<5>(mine), row16_get<6>(mine), row16_get<7>(mine),
                           row16_get<8>(mine), row16_get<9>(mine), row16_get<10>(mine), row16_get<11>(mine),
                           row16_get<12>(mine), row16_get<13>(mine), row16_get<14>(mine), row16_get<15>(mine)};
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      const floatx4 rd = *reinterpret_cast<const floatx4*>(sm + L::oDen + (h * kC + 4 * g) * 4);
      float dq[4];
      floatx4 dd;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dd[i] = dds[4 * h + i];
        dq[i] = fmaf(zt[i], dd[i], u[h][i] * rd[i]);
        qdq[i] = fmaf(qq[h][i], dq[i], qdq[i]);
      }
      if (carries || !kSkip) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float qe = wf * d.E[i] * qq[h][i];
          rz = fma((Wide<T>)qe, (Wide<T>)dd[i], rz);
          qw[h][i] = qe * rd[i];
        }
      }
      St::row_store(dQ, qd, offq + (unsigned)(hb * HB + h) * D * St::kBytes, row0, g, n, dq);
    }
    Rz += rz;
    // q and dO reach rz through dden, and a denominator of zero does: what is not finite in any of them shows here
    bad = bad || __builtin_amdgcn_ballot_w64(!(rz - rz == 0) || (kSkip && !(mine - mine == 0))) != 0;
    if (seg > 0 && carries) accumulate<T, D, HB>(R, sm, g, n, qw);
    if (last_head) {
      float kp1[1][4] = {{kp[0], kp[1], kp[2], kp[3]}};
      if (!serial) accumulate<T, D, 1>(X, sm + L::oV, g, n, kp1);
      float* out = a.qdq + token * D;
      if (len == kC) {
        *reinterpret_cast<floatx4*>(out + (w * 64 + l) * 4) = floatx4{qdq[0], qdq[1], qdq[2], qdq[3]};
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * g + i < len) out[c * len + 4 * g + i] = qdq[i];
      }
      if (tid == 0) {
        int any = bad;
#pragma unroll
        for (int j = 0; j < NW; ++j) any |= flags[j];
        any_serial = any_serial || any != 0;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) qdq[i] = 0.f;
    }
    ci = ci1; hb = hb1;
    sm = sm == lds ? lds + L::kTurn : lds;
  }
  if (tid == 0) a.serial[(size_t)bh * a.nseg + seg] = any_serial;
  if (seg > 0) {
    float* slot = a.slots_r + ((size_t)bh * (a.nseg - 1) + (a.nseg - 1 - seg)) * slot_floats<D>();
#pragma unroll
    for (int jt = 0; jt < D / 16; ++jt) *reinterpret_cast<floatx4*>(slot + (size_t)c * D + 16 * jt + 4 * g) = R[jt];
    Rz += lane_get(ln.x1, Rz);
    Rz += lane_get(ln.x2, Rz);
    if (g == 0) {
      slot[D * D + c] = (float)Rz;
      slot[D * D + D + c] = P;
    }
    const int any = __syncthreads_or(P != 0.f);
    if (tid == 0) a.live_r[(size_t)bh * a.nseg + (a.nseg - 1 - seg)] = any != 0;
  }
}

// ---- reverse sweep: dk, dv, dg, and the start state's gradient.  grid (nseg, heads), 4 D threads.
// kTokens: every chunk of the segment token by token.
template <typename T, int D, int HB, bool PAIR, bool kTokens>
__device__ __forceinline__ void reverse_sweep(const BwdArgs& a) {
  typedef Store<T> St;
  typedef Sweep<T, D, HB> L;
  constexpr int NW = L::NW;
  extern __shared__ __attribute__((aligned(16))) unsigned char sm[];
  unsigned char* orows = sm;    // this chunk's turn of the dO rows
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, g = l >> 4, n = l & 15;
  const Lanes ln = make_lanes(l);
  const Turn qd = make_turn(l);
  const Quad qv = make_quad(l);      // (dv: lanes are value columns as they come)
  constexpr bool kWide = sizeof(T) == 4;      // fp32 storage: contractions summed in 64 bits
  const int row = kWide ? strided(n) : n;     // the A operand's row in this lane
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / a.Hkv, hk = bh % a.Hkv;
  const int s0 = seg * a.seg_len, rows = min(a.T, s0 + a.seg_len) - s0;
  const int nb = a.group / HB;
  const unsigned kvs = (unsigned)a.Hkv * D * St::kBytes, qs = (unsigned)a.Hq * D * St::kBytes;
  const size_t kv1 = (((size_t)b * a.T + s0) * a.Hkv + hk) * D * St::kBytes;
  const size_t q1 = (((size_t)b * a.T + s0) * a.Hq + (size_t)hk * a.group) * D * St::kBytes;
  const Rows K = make_rows(a.k, kv1, kvs, rows, D * St::kBytes), V = make_rows(a.v, kv1, kvs, rows, D * St::kBytes),
             Gt = make_rows(a.g, kv1, kvs, rows, D * St::kBytes), Q = make_rows(a.q, q1, qs, rows, a.group * D * St::kBytes),
             O = make_rows(a.dO, q1, qs, rows, a.group * D * St::kBytes), dK = make_rows(a.dk, kv1, kvs, rows, D * St::kBytes),
             dV = make_rows(a.dv, kv1, kvs, rows, D * St::kBytes), dG = make_rows(a.dg, kv1, kvs, rows, D * St::kBytes);
  const unsigned offk = St::row_offset(K, g, n, 16 * w), offq = St::row_offset(Q, g, n, 16 * w);
  const int c = 16 * w + St::channel(n), vc = 16 * w + n;      // this lane's key channel, and value column

  // the gradient flowing into the segment's end, and the gate's sum over everything after it
  floatx4 R[D / 16];
  float Rz0 = 0.f, later = 0.f;
#pragma unroll
  for (int jt = 0; jt < D / 16; ++jt) R[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (seg + 1 < a.nseg) {
    floatx4 end[D / 16];     // the state at the segment's end
    float zend;
    start_state<D>(a.slots_f + (size_t)bh * (a.nseg - 1) * slot_floats<D>(), a.live_f + (size_t)bh * a.nseg, a.fold, seg + 1,
                   a.S0 ? a.S0 + (size_t)bh * D * D : nullptr, a.z0 ? a.z0 + (size_t)bh * D : nullptr, c, g, end, zend);
    start_state<D>(a.slots_r + (size_t)bh * (a.nseg - 1) * slot_floats<D>(), a.live_r + (size_t)bh * a.nseg, a.fold, a.nseg - 1 - seg,
                   nullptr, nullptr, c, g, R, Rz0);
#pragma unroll
    for (int jt = 0; jt < D / 16; ++jt)
#pragma unroll
      for (int i = 0; i < 4; ++i) later = fmaf(R[jt][i], end[jt][i], later);
    later += lane_get(ln.x1, later);
    later += lane_get(ln.x2, later);
    later = fmaf(Rz0, zend, later);
  }
  double Rz = Rz0;
  float pend = 1.f;      // alpha of the first token of the chunk after

  // 1 / den, and dden (times den where it meets q E / den), of a chunk's heads and tokens: in LDS ahead of its rows where q E / den goes
  // there
  constexpr bool kAhead = L::kScoreTerms && !kTokens;
  unsigned char* dn = sm + L::rDen;      // this chunk's turn
  constexpr bool kRows = sizeof(T) == 2;        // dO and v as whole rows
  typename St::Raw rq[HB], rk, rg, ro[kRows ? 1 : HB], rv;
  WholeRows<D, HB> wo;
  WholeRows<D, 1> wv;
  const unsigned offwo = WholeRows<D, HB>::offset(O, tid), offwv = WholeRows<D, 1>::offset(V, tid);
  floatx4 rqdq = {0.f, 0.f, 0.f, 0.f};
  const float* den_rows = a.den + ((size_t)b * a.T + s0) * a.Hq + (size_t)hk * a.group;
  float rden = 1.f, rdd = 0.f;
  // whole: a chunk that is not the first to be taken and so has 16 tokens, where it matters (of the first one, more query heads at most).
  // With a load in the loop that depends on it, every chunk waited for all loads under way there, 1500 of its 10100 cycles: 32768 tokens
  // of 32 / 8 heads of 64, the training pass, 613.9 -> 599.1 us (of 128 nothing, with one query head a pass 205.0 -> 206.5: left as it was).
  constexpr std::bool_constant<(D == 64 || HB > 1)> kWhole16{};
  auto fetch = [&](int ci, int hb, auto whole) {
    const int row0 = ci * kC;
    const size_t token = (size_t)bh * a.T + s0 + row0;
    const int len = min(kC, rows - row0);
    auto dens = [&] {
      if (tid < HB * kC) {
        const int t = row0 + (tid & 15), h = hb * HB + (tid >> 4);
        rden = t < rows ? at32(den_rows, (unsigned)(t * a.Hq + h)) : 1.f;
        rdd = t < rows ? at32(a.dden + token * a.group, (unsigned)(h * len + (tid & 15))) : 0.f;
      }
    };
    if (kAhead) dens();
    if (hb == 0) {
      rg = St::load(Gt, offk, row0);
      rk = St::load(K, offk, row0);
      if constexpr (kRows) wv.load(V, offwv, row0);
      else rv = St::load(V, offk, row0);
      const float* in = a.qdq + token * D;
      if (whole || len == kC) {
        rqdq = *reinterpret_cast<const floatx4*>(in + (w * 64 + l) * 4);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) rqdq[i] = 4 * g + i < len ? in[c * len + 4 * g + i] : 0.f;
      }
    }
    if constexpr (kRows) wo.load(O, offwo + (unsigned)(hb * HB) * D * St::kBytes, row0);
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      const unsigned ho = (unsigned)(hb * HB + h) * D * St::kBytes;
      if constexpr (!kRows) ro[h] = St::load(O, offq + ho, row0);
      rq[h] = St::load(Q, offq + ho, row0);
    }
    if (!kAhead) dens();
  };

  const int nchunk = (rows + kC - 1) / kC;
  int ci = nchunk - 1, hb = 0;
  Decay d;
  float kk[4], kp[4], rE[4], sig[4], qdq[4];
  Split4 rs[L::kScoreTerms ? D / 16 : 1];      // R~
  floatx4 dk0, dk, dv0, dv;     // from after the chunk (state products), within it
  doublex4 dvw;                 // fp32 storage: dv0 + dv
  if (ci >= 0) fetch(ci, 0, std::false_type{});
  auto put_dens = [&](unsigned char* to) {
    if (tid < HB * kC) {
      float* den = reinterpret_cast<float*>(to);
      den[tid] = 1.f / rden;
      den[HB * kC + tid] = kAhead ? rdd * rden : rdd;
      if (kAhead) den[2 * HB * kC + tid] = rdd;
    }
  };
  if (kAhead) {
    put_dens(dn);
    __syncthreads();
  }
  while (ci >= 0) {
    const int row0 = ci * kC;
    // ---- once per chunk: decays, K', R~; rows to LDS
    if (hb == 0) {
      float gl[4];
      St::row_patch(qd, rg, gl);
      St::row_patch(qd, rk, kk);
      alphas_of(gl, a.gate_scale, rows - (row0 + 4 * g), d.al);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sig[i] = __builtin_amdgcn_rcpf(1.f + __expf(gl[i]));       // 1 - sigmoid(g)
        qdq[i] = rqdq[i];
      }
      whole_chunk<Wide<T>>(d, ln, g);
      if constexpr (kTokens) {
        Rz *= pend;
#pragma unroll
        for (int i = 0; i < 4; ++i) d.E[i] = rE[i] = 1.f;
#pragma unroll
        for (int jt = 0; jt < D / 16; ++jt)
#pragma unroll
          for (int i = 0; i < 4; ++i) R[jt][i] *= pend;
        dk0 = dk = dv0 = dv = floatx4{0.f, 0.f, 0.f, 0.f};
        dvw = kZero64;
      } else {
        center(d);
        const float f = d.last * pend;
        Rz *= f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          rE[i] = inverse<T>(d.E[i]);
          kp[i] = kk[i] * rE[i];
        }
        if constexpr (L::kScoreTerms) terms_to_lds(sm + L::rK, D * 32, g, n, 16 * w, split4(kp[0], kp[1], kp[2], kp[3]));
        else f32_to_lds<D>(sm + L::rK, g, n, 16 * w, kp);
#pragma unroll
        for (int jt = 0; jt < D / 16; ++jt) {
#pragma unroll
          for (int i = 0; i < 4; ++i) R[jt][i] *= f;
          if constexpr (L::kScoreTerms) {
            rs[jt] = split4(R[jt][0], R[jt][1], R[jt][2], R[jt][3]);
            state_terms_to_lds(sm + L::rR, D * D * 2, g, n, 16 * w, jt, rs[jt]);
          } else {
            *reinterpret_cast<floatx4*>(sm + L::rR + vc * f32_row_bytes<D>() + (16 * jt + 4 * g) * 4) = R[jt];      // (a row per lane, as K')
          }
        }
      }
      pend = d.first;
      if constexpr (kRows) wv.to_lds(sm + L::rV, L::kRow, tid);
      else St::template to_lds<D>(sm + L::rV, g, n, 16 * w, rv);
    }
    if constexpr (kRows) {
      wo.to_lds(orows, L::kRow, tid);
    } else {
#pragma unroll
      for (int h = 0; h < HB; ++h) St::template to_lds<D>(orows + h * L::kSet, g, n, 16 * w, ro[h]);
    }
    unsigned char* das = sm + L::rDa;     // parts of dO . v
    if constexpr (L::kDaParts) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int h = 0; h < HB; ++h) dot_part64<D>(orows + h * L::kSet, sm + L::rV, w, g, n, das + (w * HB + h) * L::kTile);
    }
    const float* den = reinterpret_cast<const float*>(dn);
    if (!kAhead) put_dens(dn);
    float qp[HB][4];
    Split4 qs[HB];         // q E / den
    Wide<T> rzt[4] = {0, 0, 0, 0};
#pragma unroll
    for (int h = 0; h < HB; ++h) {
      St::row_patch(qd, rq[h], qp[h]);
#pragma unroll
      for (int i = 0; i < 4; ++i) qp[h][i] *= d.E[i];
      if constexpr (kAhead) {
        const floatx4 rd = *reinterpret_cast<const floatx4*>(dn + (h * kC + 4 * g) * 4), dd = *reinterpret_cast<const floatx4*>(dn + ((2 * HB + h) * kC + 4 * g) * 4);
        float qw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          qw[i] = qp[h][i] * rd[i];
          rzt[i] = fma((Wide<T>)qp[h][i], (Wide<T>)dd[i], rzt[i]);
        }
        qs[h] = split4(qw[0], qw[1], qw[2], qw[3]);
        terms_to_lds(sm + L::rQ + h * L::kTerms, D * 32, g, n, 16 * w, qs[h]);
      } else if constexpr (!kTokens) {
        f32_to_lds<D>(sm + L::rQ + h * kC * f32_row_bytes<D>(), g, n, 16 * w, qp[h]);
      }
    }
    if constexpr (L::kParts && !kTokens) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int h = 0; h < HB; ++h) dot_part64<D>(sm + L::rQ + h * kC * f32_row_bytes<D>(), sm + L::rK, w, g, n, sm + L::rSc + (w * HB + h) * L::kTile);
    }
    __syncthreads();
    if (PAIR) __builtin_amdgcn_s_setprio(0);
    const int hb1 = hb + 1 < nb ? hb + 1 : 0;
    const int ci1 = hb1 ? ci : ci - 1;
    if (!kTokens && ci1 >= 0) fetch(ci1, hb1, kWhole16);
    if constexpr (kTokens) {
      // ---- token by token, these query heads' part: Gr_t, dk_t = Gr_t v^_t, dv_t = k_t Gr_t (over the channels through LDS)
      int lane = l;                                   // not known to be l: nothing of this loop is formed before it
      asm volatile("" : "+v"(lane));
      const int gs = lane >> 4, ns = lane & 15;
      const Lanes lns = make_lanes(lane);
      floatx4 Y[D / 16];
      double y = hb == 0 ? Rz : 0.0;
#pragma unroll
      for (int jt = 0; jt < D / 16; ++jt) Y[jt] = hb == 0 ? R[jt] : floatx4{0.f, 0.f, 0.f, 0.f};
      float* dvp = reinterpret_cast<float*>(sm + L::rR);
      float aln = 1.f;       // alpha of the token after
#pragma unroll 1
      for (int tg = 3; tg >= 0; --tg) {
        const int from = ((tg << 4) + ns) << 2;
#pragma unroll
        for (int i = 3; i >= 0; --i) {
          const unsigned char *col = sm + L::rV + (4 * tg + i) * L::kRow + 4 * gs * St::kBytes, *ocol = orows + (4 * tg + i) * L::kRow + 4 * gs * St::kBytes;
          const float kt = lane_get(from, kk[i]);
          float wt[HB];
          y *= aln;
#pragma unroll
          for (int h = 0; h < HB; ++h) {
            const float qv = lane_get(from, qp[h][i]);
            wt[h] = qv * den[h * kC + 4 * tg + i];
            y = fma((double)qv, (double)den[(HB + h) * kC + 4 * tg + i], y);
          }
          float part[4] = {};
#pragma unroll
          for (int jt = 0; jt < D / 16; ++jt) {
            floatx4 x = Y[jt] * aln;
#pragma unroll
            for (int h = 0; h < HB; ++h) {
              const floatx4 o4 = St::four(ocol + h * L::kSet + 16 * jt * St::kBytes);
#pragma unroll
              for (int e = 0; e < 4; ++e) x[e] = fmaf(wt[h], o4[e], x[e]);
            }
            Y[jt] = x;
            const floatx4 v4 = St::four(col + 16 * jt * St::kBytes);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              part[e] = fmaf(x[e], v4[e], part[e]);
              x[e] = row16_sum(kt * x[e]);
            }
            if (ns == 0) *reinterpret_cast<floatx4*>(dvp + (w * kC + 4 * tg + i) * D + 16 * jt + 4 * gs) = x;
          }
          float acc = (part[0] + part[1]) + (part[2] + part[3]);
          acc += lane_get(lns.x1, acc);
          acc += lane_get(lns.x2, acc);
          if (gs == tg) dk[i] += acc + (float)y;
          aln = lane_get(from, d.al[i]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      Rz = hb == 0 ? y : Rz + y;
#pragma unroll
      for (int jt = 0; jt < D / 16; ++jt) R[jt] = hb == 0 ? Y[jt] : R[jt] + Y[jt];
      if (ci1 >= 0) fetch(ci1, hb1, kWhole16);          // not before: its registers are the loop's
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        Wide<T> s = 0;
#pragma unroll
        for (int j = 0; j < NW; ++j) s += dvp[(j * kC + 4 * g + i) * D + vc];
        if (kWide) dvw[i] += s;
        else dv[i] += s;
      }
    } else {
    if (hb == 0) {
      // ---- what flows in from after the chunk: dk gets R~ v^, dv gets K' R~
      floatx4 acc[1] = {floatx4{(float)Rz, (float)Rz, (float)Rz, (float)Rz}};
      if constexpr (L::kScoreTerms) acc[0] = contract_terms<D>(rs, sm + L::rV, g, n, acc[0]);
      else contract<T, D, 1>(R, sm + L::rV, g, n, acc);
      dk0 = acc[0];
      dk = dv0 = dv = floatx4{0.f, 0.f, 0.f, 0.f};
      dvw = kZero64;
      if constexpr (L::kScoreTerms) {
        dv0 = mfma_terms(terms_frag(sm + L::rK, D * 32, g, n, 0), state_terms_frag(sm + L::rR, D * D * 2, g, n, w, 0),
                         terms_frag(sm + L::rK, D * 32, g, n, 1), state_terms_frag(sm + L::rR, D * D * 2, g, n, w, 1));
      } else
#pragma unroll
      for (int ct = 0; ct < D / 16; ++ct) {
        const floatx4 f = f32_row_frag<D>(sm + L::rK, g, row, ct);
        float fa[4], r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          fa[i] = f[i];
          r[i] = *reinterpret_cast<const float*>(sm + L::rR + (16 * ct + 4 * g + i) * f32_row_bytes<D>() + vc * 4);
        }
        if constexpr (kWide) {
#pragma unroll
          for (int i = 0; i < 4; ++i) dvw = mfma_f64(fa[i], r[i], dvw);
        } else {
          dv0 = token_steps<false>(fa, r, dv0);
        }
      }
    }
    // ---- scores of head w: Q'_s . K'_i / den_s for i <= s, shared through LDS (in the terms the product below uses)
    if (!L::kParts && w < HB) {
      const unsigned char* qrows = sm + L::rQ + w * kC * f32_row_bytes<D>();
      const floatx4 rd = *reinterpret_cast<const floatx4*>(dn + (w * kC + 4 * g) * 4);
      unsigned char* p = sm + L::rSc + w * L::kScore;
      if constexpr (sizeof(T) == 2) {
        floatx4 sc = {0.f, 0.f, 0.f, 0.f};       // [s][`row`]
        if constexpr (L::kScoreTerms) {
          sc = mfma_terms(terms_frag(sm + L::rQ + w * L::kTerms, D * 32, g, n, 0), terms_frag(sm + L::rK, D * 32, g, n, 0),
                          terms_frag(sm + L::rQ + w * L::kTerms, D * 32, g, n, 1), terms_frag(sm + L::rK, D * 32, g, n, 1));
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[i] = row <= 4 * g + i ? sc[i] : 0.f;
        } else {
          sc = dot_rows<float, D>(qrows, sm + L::rK, g, n);
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[i] = row <= 4 * g + i ? sc[i] * rd[i] : 0.f;
        }
        const Split4 s = split4(sc[0], sc[1], sc[2], sc[3]);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2*>(p + k * 512 + l * 8) = s.t[k];
      } else {
        doublex4 sc = dot_rows64<D>(qrows, sm + L::rK, g, n);
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[i] = row <= 4 * g + i ? sc[i] * (double)rd[i] : 0.0;
        *reinterpret_cast<doublex4*>(p + l * 32) = sc;
      }
    }
    // ---- dO_s . v_i + dden_s den_s for i <= s, of a head, the same way
    if constexpr (L::kDaOnce) {
      if (w >= L::kDaWave && w < L::kDaWave + HB) {
        const int h = w - L::kDaWave;
        const floatx4 rd = *reinterpret_cast<const floatx4*>(dn + (h * kC + 4 * g) * 4);
        const floatx4 dd = *reinterpret_cast<const floatx4*>(dn + ((HB + h) * kC + 4 * g) * 4);      // (kAhead: dden den)
        const floatx4 da = dot_rows<T, D, kWide>(orows + h * L::kSet, sm + L::rV, g, n);
        floatx4 am;
#pragma unroll
        for (int i = 0; i < 4; ++i) am[i] = row <= 4 * g + i ? (kAhead ? da[i] + dd[i] : fmaf(da[i], rd[i], dd[i])) : 0.f;
        if constexpr (kAhead) {
          const Split4 s = split4(am[0], am[1], am[2], am[3]);
#pragma unroll
          for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2*>(das + h * L::kDa + k * 512 + l * 8) = s.t[k];
        } else {
          *reinterpret_cast<floatx4*>(das + h * L::kDa + l * 16) = am;
        }
      }
    }
    // ---- dk within the chunk, and what the chunk adds to the gradient flowing on
    const bool wide = seg == 0 && ci == 0 && a.dS0 != nullptr;     // dS0 is fp32 whatever the storage
    if constexpr (kAhead) {
      if (wide) {
        float qw[HB][4];
#pragma unroll
        for (int h = 0; h < HB; ++h) join4(qs[h], qw[h]);
        accumulate_wide<T, D, HB>(R, orows, g, n, qw);
      } else {
#pragma unroll
        for (int h = 0; h < HB; h += 2) accumulate_pair<D, false>(R, orows + h * L::kSet, orows + (h + 1) * L::kSet, g, n, pair_terms(qs[h], qs[h + 1]));
      }
    } else {
      float qw[HB][4];
#pragma unroll
      for (int h = 0; h < HB; ++h) {
        const floatx4 rd = *reinterpret_cast<const floatx4*>(dn + (h * kC + 4 * g) * 4);
        const floatx4 dd = *reinterpret_cast<const floatx4*>(dn + ((HB + h) * kC + 4 * g) * 4);
        if constexpr (!L::kDaOnce) {
          floatx4 da;    // [token s of dO][token `row` of v]
          if constexpr (L::kDaParts) da = add64(floatx4{0.f, 0.f, 0.f, 0.f}, sum_parts64<NW>(das + h * L::kTile, HB * L::kTile, g, n));
          else da = dot_rows<T, D, kWide>(orows + h * L::kSet, sm + L::rV, g, n);
          float am[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) am[i] = row <= 4 * g + i ? fmaf(da[i], rd[i], dd[i]) : 0.f;
          dk = token_steps<kWide>(am, qp[h], dk);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          rzt[i] = fma((Wide<T>)qp[h][i], (Wide<T>)dd[i], rzt[i]);
          qw[h][i] = qp[h][i] * rd[i];
        }
      }
      if (wide) accumulate_wide<T, D, HB>(R, orows, g, n, qw);
      else accumulate<T, D, HB>(R, orows, g, n, qw);
    }
    double rz = (((double)rzt[3] + (double)rzt[2]) + (double)rzt[1]) + (double)rzt[0];
    rz += lane_get(ln.x1, rz);
    rz += lane_get(ln.x2, rz);
    Rz += rz;
    uint2 of[HB];          // dO as the operands of dv, read ahead where its rows are one set
    if constexpr (L::kScoreTerms) {
#pragma unroll
      for (int h = 0; h < HB; ++h) of[h] = St::template col_frag<D>(orows + h * L::kSet, g, n, w);
    }
    if (kAhead) put_dens(dn == sm + L::rDen ? dn + L::kTriples : sm + L::rDen);
    if constexpr (!L::kParts) __syncthreads();
    if (PAIR) __builtin_amdgcn_s_setprio(1);
    if constexpr (kAhead) {
      auto term = [&](int h, int k) { return *reinterpret_cast<const uint2*>(das + h * L::kDa + k * 512 + l * 8); };
      auto da = [&](int h) { return Terms{make8(term(h, 0), term(h + 1, 0)), make8(term(h, 1), term(h + 1, 1)), make8(term(h, 2), term(h + 1, 2))}; };
      if constexpr (HB == 4) {
        dk += mfma_terms(da(0), pair_terms(qs[0], qs[1]), da(2), pair_terms(qs[2], qs[3]));
      } else {
        dk += mfma_terms(da(0), pair_terms(qs[0], qs[1]));
      }
    } else if constexpr (L::kDaOnce) {
#pragma unroll
      for (int h = 0; h < HB; ++h) {
        const floatx4 f = *reinterpret_cast<const floatx4*>(das + h * L::kDa + l * 16);
        const float am[4] = {f[0], f[1], f[2], f[3]};
        dk = token_steps<kWide>(am, qp[h], dk);
      }
    }
    // ---- dv within the chunk: this wave's 16 value columns
    if constexpr (sizeof(T) == 2) {
      if constexpr (HB == 1) {
        const unsigned char* p = sm + L::rSc + l * 8;
        const uint2 f = St::template col_frag<D>(orows, g, n, w);
#pragma unroll
        for (int k = 2; k >= 0; --k) dv = mfma_bf16_k16(*reinterpret_cast<const uint2*>(p + k * 512), f, dv);
      } else {
#pragma unroll
        for (int h = 0; h < HB; h += 2) {
          const unsigned char* p = sm + L::rSc + h * L::kScore + l * 8;
          bf16x8 f;
          if constexpr (L::kScoreTerms) f = make8(of[h], of[h + 1]);
          else f = make8(St::template col_frag<D>(orows + h * L::kSet, g, n, w), St::template col_frag<D>(orows + (h + 1) * L::kSet, g, n, w));
#pragma unroll
          for (int k = 2; k >= 0; --k)
            dv = mfma_bf16(make8(*reinterpret_cast<const uint2*>(p + k * 512), *reinterpret_cast<const uint2*>(p + L::kScore + k * 512)), f, dv);
        }
      }
    } else {
#pragma unroll
      for (int h = 0; h < HB; ++h) {
        doublex4 sc;
        if constexpr (L::kParts) {
          const floatx4 rd = *reinterpret_cast<const floatx4*>(dn + (h * kC + 4 * g) * 4);
          sc = sum_parts64<NW>(sm + L::rSc + h * L::kTile, HB * L::kTile, g, n);
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[i] = row <= 4 * g + i ? sc[i] * (double)rd[i] : 0.0;
        } else {
          sc = *reinterpret_cast<const doublex4*>(sm + L::rSc + h * L::kScore + l * 32);
        }
        const floatx4 f = f32_col_frag<D>(orows + h * L::kSet, g, n, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) dvw = mfma_f64(sc[i], f[i], dvw);
      }
    }
    }
    if (hb + 1 == nb) {
      // ---- outputs; the gate's sum over this token and all later ones (by additions: no later token's sum
      // holds an earlier token's term, finite or not)
      float dkv[4], dvv[4], dgv[4];
      Wide<T> x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dkv[i] = (dk0[i] + dk[i]) * rE[i];
        dvv[i] = kWide ? (float)dvw[i] : dv0[i] + dv[i];
        x[i] = fmaf(-kk[i], dkv[i], qdq[i]);
      }
#pragma unroll
      for (int i = 2; i >= 0; --i) x[i] += x[i + 1];
      const Wide<T> x1 = lane_get(ln.x1, x[0]), x2 = lane_get(ln.x2, x[0]), x3 = lane_get(ln.x3, x[0]);
      const Wide<T> after = (g & 2) ? ((g & 1) ? Wide<T>(0) : x1) : ((g & 1) ? x2 + x3 : x1 + (x2 + x3));
      const Wide<T> rest = after + (Wide<T>)later;
#pragma unroll
      for (int i = 0; i < 4; ++i) dgv[i] = (float)(x[i] + rest) * a.gate_scale * sig[i];
      later = lane_get(ln.n4, (float)(x[0] + rest));
      St::row_store(dK, qd, offk, row0, g, n, dkv);
      St::store(dV, qv, St::offset(dV, g, n, 16 * w), row0, g, n, 0, kC, dvv);
      St::row_store(dG, qd, offk, row0, g, n, dgv);
    }
    // What is read after the barrier before dv (the scores, dO . v, dO) is written next after the first barrier of the next chunk, or in the other
    // turn's rows; everything else was read before it.  (One turn of rows, parts, and tokens one by one, are read up to here.)
    if constexpr (L::kDaParts || kTokens) __syncthreads();
    else if constexpr (!L::kScoreTerms) orows = orows == sm ? sm + L::kO : sm;
    if (kAhead) dn = dn == sm + L::rDen ? dn + L::kTriples : sm + L::rDen;
    ci = ci1; hb = hb1;
  }
  if (seg == 0) {
    if (a.dS0 != nullptr) {
#pragma unroll
      for (int jt = 0; jt < D / 16; ++jt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) R[jt][i] *= pend;
        *reinterpret_cast<floatx4*>(a.dS0 + ((size_t)bh * D + c) * D + 16 * jt + 4 * g) = R[jt];
      }
    }
    if (a.dz0 != nullptr && g == 0) a.dz0[(size_t)bh * D + c] = (float)(pend * Rz);
  }
}

template <typename T, int D, int HB, bool PAIR>
__global__ void __launch_bounds__(4 * D, 2) bwd_reverse_kernel(const BwdArgs a) {
  if (a.serial[(size_t)blockIdx.y * a.nseg + blockIdx.x] != 0) reverse_sweep<T, D, HB, PAIR, true>(a);
  else reverse_sweep<T, D, HB, PAIR, false>(a);
}

template <int D>
void launch_scan(float* slots, int* live, const float* S0, const float* z0, const BwdArgs& a, hipStream_t stream) {
  const int heads = a.B * a.Hkv, x = scan_blocks<D>(heads);
  hipLaunchKernelGGL((segment_scan_kernel<D, true>), dim3(x, heads), dim3(256), 0, stream, slots, live, S0, z0, a.nseg,
                     (const int*)nullptr, a.Hkv, a.seg_len, false);
}

template <typename T, int D, int HB, bool FORWARD_PAIR, bool REVERSE_PAIR>
hipError_t launch_sweeps(const BwdArgs& a, hipStream_t stream) {
  typedef Sweep<T, D, HB> L;
  const auto forward = bwd_forward_kernel<T, D, HB, FORWARD_PAIR>;
  const auto reverse = bwd_reverse_kernel<T, D, HB, REVERSE_PAIR>;
  const int heads = a.B * a.Hkv;
  hipError_t e = set_lds<bwd_forward_kernel<T, D, HB, FORWARD_PAIR>>(L::kForward);
  if (e != hipSuccess) return e;
  e = set_lds<bwd_reverse_kernel<T, D, HB, REVERSE_PAIR>>(L::kReverse);
  if (e != hipSuccess) return e;
  if (a.nseg > 1) {
    hipLaunchKernelGGL((bwd_state_kernel<T, D>), dim3(a.nseg - 1, heads), dim3(4 * D), 0, stream, a);
    if (!a.fold) launch_scan<D>(a.slots_f, a.live_f, a.S0, a.z0, a, stream);
  }
  hipLaunchKernelGGL(forward, dim3(a.nseg, heads), dim3(4 * D), L::kForward, stream, a);
  if (a.nseg > 1 && !a.fold) launch_scan<D>(a.slots_r, a.live_r, nullptr, nullptr, a, stream);
  hipLaunchKernelGGL(reverse, dim3(a.nseg, heads), dim3(4 * D), L::kReverse, stream, a);
  return hipGetLastError();
}

template <typename T, int D, int HB>
hipError_t launch_sized(const BwdArgs& a, hipStream_t stream) {
  constexpr bool kPair = Sweep<T, D, HB>::kPair;
  if constexpr (kPair) {
    // The order of two workgroups (kPair): in the forward sweep where there are up to two to a compute unit, in the reverse one also past
    // that; with one query head per pass in neither where units have one.  us, neither / both / reverse only: 500 tokens of 24 heads on 8 (64
    // workgroups) 65.2 / 66.2 / 66.0, 2000 of 8 (256) 47.4 / 47.8 / 47.7; 8000 of 8 (504) 92.0 / 89.2 / 90.3, of 24 on 8 145.8 / 143.6 / 145.0,
    // of 32 on 8 130.8 / 126.3; 16000 of 8 (672) 168.4 / 168.9 / 165.1, of 24 on 8 283.8 / 291.0 / 281.0; 40 x 100 of 16 on 8 (640) 71.3 / 73.4 /
    // 72.4, 66 x 64 of 32 on 8 (528) 76.1 / 77.4 / 76.7, 35 x 300 (840) 197.4 / 194.6 / 196.0.
    const long long blocks = (long long)a.nseg * a.B * a.Hkv;
    if (HB == 1 && blocks <= 256) return launch_sweeps<T, D, HB, false, false>(a, stream);
    if (blocks > 512) return launch_sweeps<T, D, HB, false, true>(a, stream);
  }
  return launch_sweeps<T, D, HB, kPair, kPair>(a, stream);
}

template <typename T, int D>
hipError_t launch_typed(const BwdArgs& a, hipStream_t stream) {
  // query heads per pass: four, in fp32 storage two, whose 64-bit sums would spill with four.  us with one, two and four: head dim
  // 64, 500 tokens, 2 x 8 heads on 2, 122.5, 109.8, 136.5; 128, 512 tokens, 8 heads on 2, 323, 291, 305
  if constexpr (sizeof(T) == 2)
    if (a.group % 4 == 0) return launch_sized<T, D, 4>(a, stream);
  if (a.group % 2 == 0) return launch_sized<T, D, 2>(a, stream);
  return launch_sized<T, D, 1>(a, stream);
}

struct Sizes {
  size_t qdq, slots, serial, live, dden, total;   // floats / words, and bytes in all
};
Sizes workspace_sizes(int B, int T, int Hq, int Hkv, int d, int nseg) {
  const size_t heads = (size_t)B * Hkv;
  Sizes s;
  s.qdq = heads * T * d;
  s.slots = heads * (nseg - 1) * (d * d + 2 * d);
  s.serial = (heads * nseg + 15) / 16 * 4;
  s.live = heads * nseg;
  s.dden = (size_t)B * T * Hq;
  // the size is two states and a row per segment beside both tensors, as callers may have kept it; what is used is less (but
  // for sequences of millions of tokens)
  const size_t used = s.qdq + 2 * s.slots + s.serial + 2 * s.live + s.dden, rule = s.qdq + s.dden + heads * nseg * (2 * (d * d + 2 * d) + d);
  s.total = (used > rule ? used : rule) * 4 + 256;
  return s;
}

}  // namespace

bool gla_backward_supports(int d, int group) { return group * d <= 2048; }

// Segments of the sequence, a multiple of 64 tokens: as many as make one round of the workgroups that the chip holds over all
// (batch, kv head) pairs, which is what the sweeps' registers allow: at head dim 64 two per compute unit (of four waves), with one query
// head per pass in bf16 storage three in the reverse sweep (a limit of registers for three in the forward one too spilled: 96.7 us
// and 101.1 for 8192 tokens of 8 heads), at 128 one (of eight).  bf16, 32 / 8 heads, 32768 tokens of 64 or 16384 of 128: two rounds,
// with twice the contributions and start states, take 447 and 627 us, one 409 and 582.  Two rounds where one would leave many
// places empty (300 pairs: two rounds of a third of the sequence, not one of all of it).  A segment's rows are addressed with
// 32-bit offsets from its first row.
void gla_backward_plan(int B, int T, int Hq, int Hkv, int d, int bf16, int* seg_len, int* nseg) {
  const long long heads = (long long)B * Hkv, places = d == 128 ? 256 : (bf16 && (Hq / Hkv) % 2 ? 768 : 512);
  const long long one = places / heads, two = (places < 512 ? 512 : 1024) / heads;   // segments per head
  long long want = 10 * two > 22 * one ? two : one;
  if (want < 1) want = 1;
  long long len = (T + want - 1) / want;
  const long long most = (1ll << 31) / ((long long)Hq * d * 4) / 64 * 64;
  len = (len + 63) / 64 * 64;
  if (len > most && most >= 64) len = most;
  *seg_len = (int)len;
  *nseg = (int)((T + len - 1) / len);
}

size_t gla_backward_workspace_bytes(int B, int T, int Hq, int Hkv, int d, int bf16) {
  int seg_len, nseg;
  gla_backward_plan(B, T, Hq, Hkv, d, bf16, &seg_len, &nseg);
  return workspace_sizes(B, T, Hq, Hkv, d, nseg).total;
}

hipError_t launch_gla_backward(const GlaBackwardParams& p, hipStream_t stream) {
  BwdArgs a{};
  a.q = p.q; a.k = p.k; a.v = p.v; a.g = p.g; a.dO = p.dO; a.den = p.den; a.S0 = p.S0; a.z0 = p.z0;
  a.dq = p.dq; a.dk = p.dk; a.dv = p.dv; a.dg = p.dg; a.dS0 = p.dS0; a.dz0 = p.dz0;
  a.B = p.B; a.T = p.T; a.Hq = p.Hq; a.Hkv = p.Hkv; a.group = p.Hq / p.Hkv;
  a.gate_scale = p.gate_scale;
  gla_backward_plan(p.B, p.T, p.Hq, p.Hkv, p.d, p.bf16, &a.seg_len, &a.nseg);
  if (!gla_backward_supports(p.d, a.group)) return hipErrorInvalidValue;
  // Fold / scan, us a call: head dim 64, fp32, 2 heads, 4 segments 54.8 / 58.3, 8 segments 59.0 / 59.2, bf16, 8 kv heads, 16
  // segments 69.1 / 61.1; head dim 128, fp32, 8 heads on 2, 5 segments 294 / 290, 8 segments 306 / 291 (with fewer heads, whose
  // calls are shorter, 5 are about equal)
  a.fold = a.nseg > 1 && a.nseg <= (p.d == 64 ? 8 : 5);
  const Sizes s = workspace_sizes(p.B, p.T, p.Hq, p.Hkv, p.d, a.nseg);
  float* w = static_cast<float*>(p.workspace);
  a.qdq = w; w += s.qdq;
  a.slots_f = w; w += s.slots;
  a.slots_r = w; w += s.slots;
  a.serial = reinterpret_cast<uint8_t*>(w); w += s.serial;
  a.live_f = reinterpret_cast<int*>(w); w += s.live;
  a.live_r = reinterpret_cast<int*>(w); w += s.live;
  a.dden = w;
  if (p.bf16) return p.d == 64 ? launch_typed<bf16_t, 64>(a, stream) : launch_typed<bf16_t, 128>(a, stream);
  return p.d == 64 ? launch_typed<float, 64>(a, stream) : launch_typed<float, 128>(a, stream);
}

}  // namespace lawcat
