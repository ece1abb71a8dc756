// Output pass at head dim 128, with conv, for calls of many long segments: four waves instead of eight, granules of 32 tokens instead of
// 64, 32 value columns of the state a wave instead of 16 (gla_chunk_impl.h has the algebra, the load stage and the other form).
//
// With eight waves one workgroup fills a compute unit: its load stage (vector instructions) and its MFMA stage (LDS) take turns, 5.9 and
// 5.7 of 14.3 us a granule.  Here two workgroups share the unit, 73 KB of LDS and 239 registers each, and one's load stage runs beside
// the other's MFMA stage; and the queries' operands, most of what the MFMA stage reads from LDS, serve twice as many value columns of a
// wave: 33 KB a wave and chunk for 32 columns instead of 26 for 16.  To fit, K' keeps no rows of its own: the two waves that load a chunk
// form the scores over their 64 channels each, through the last head's Q' rows before that head's go there, and add them up.
// 131072 tokens of 32 heads on 8 777 -> 686 us a call, 65536 402.6 -> 363.1; its rule is in gla_chunk.hip: twice as many segments make the
// state pass read more.  What bounds it: HBM, 4.5 TB/s.  LDS addresses are formed from a lane index that is not known to be the
// loop's: kept over the loop for all four forms of the load stage they took 18 registers too many, spilled (131072 tokens 694 us).
#pragma once
#include "gla_chunk_impl.h"

namespace lawcat {
namespace chunk {

template <int GR, int MODE>
__global__ void __launch_bounds__(256, 2) gla_wide_kernel(const ChunkArgs a) {
  constexpr int D = 128;
  using G = WideGeo<GR, MODE>;
  using KK = Kernel<D, GR, MODE, true, G>;
  constexpr bool CONV = MODE != kPlain;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63, g4 = l >> 4, n = l & 15;
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
    if (p.seg < 0) return;
    row0 = (size_t)__builtin_amdgcn_readfirstlane(p.row0);
  }
  auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  const int hk = uniform(p.hk), b = uniform(p.b), seg = uniform(p.seg), T = uniform(p.T), nseg = uniform(p.nseg), seg_len = uniform(p.len);
  const int bh = b * a.Hkv + hk;
  const size_t slot0 = (size_t)bh * a.nseg;
  const int qh0 = a.qh0 + (int)blockIdx.z * GR;
  const bool keeps = qh0 == 0;
  if (seg >= nseg) return;
  const int s0 = seg * seg_len, s1 = min(T, s0 + seg_len);

  // load-stage patch: 8 tokens x 2 channels; a chunk is loaded by two waves, 64 channels each
  const int cp = l & 31, th = l >> 5, mcw = w / G::CH;
  const int c0 = 64 * (w % G::CH) + 2 * cp, tl0 = kChunk * mcw + 8 * th;

  // Did the scan run for this head, or (fold) which segments before this one pass anything on
  int live_any = 0;
  if (a.fold) live_any = l >= seg || a.seg_live[slot0 + l] != 0;
  else
    for (int j = tid; j < nseg - 1; j += G::TEAM) live_any |= a.seg_live[slot0 + j];
  constexpr int kZd = (kFoldMost<D> * 2 * D + G::TEAM - 1) / G::TEAM;
  static_assert(kFoldMost<D> * 2 * D * 4 <= G::kWl);      // (the conv weights there are written before)
  float zraw[kZd];
  if (a.fold) {
#pragma unroll
    for (int j = 0; j < kZd; ++j) {
      const int e = tid + j * G::TEAM;
      zraw[j] = e < seg * 2 * D ? a.ws[(slot0 + e / (2 * D)) * G::kSlot + D * D + e % (2 * D)] : 0.f;
    }
  }
  float* wl = reinterpret_cast<float*>(smem + G::kWl);
  constexpr int kRows = GR + 1, kWeights = (kRows * D + G::TEAM - 1) / G::TEAM;
  uint2 wraw[kWeights];
  if (CONV) {
#pragma unroll
    for (int j = 0; j < kWeights; ++j) {
      const int e = min(tid + j * G::TEAM, kRows * D - 1), c = e % D, hh = e / D;
      const bf16_t* src = hh < GR ? a.wq + ((size_t)(hk * a.group + qh0 + hh) * D + c) * a.W : a.wk + ((size_t)hk * D + c) * a.W;
      if (a.W == 4) {
        wraw[j] = *reinterpret_cast<const uint2*>(src);
      } else {
        wraw[j] = make_uint2(src[0], 0);
        if (a.W > 1) wraw[j].x |= (uint32_t)src[1] << 16;
        if (a.W > 2) wraw[j].y = src[2];
      }
    }
  }
  const unsigned kvstride = (unsigned)a.Hkv * D * 2, qstride = (unsigned)a.Hq * D * 2;
  const RowSrc srcK = make_row_src((const char*)a.k + (row0 * a.Hkv + hk) * D * 2,
                                   (CONV && a.k_halo) ? (const char*)a.k_halo + ((size_t)b * (a.W - 1) * a.Hkv + hk) * D * 2 : nullptr, kvstride, T, D * 2);
  const RowSrc srcG = make_row_src((const char*)a.g + (row0 * a.Hkv + hk) * D * 2, nullptr, kvstride, T, D * 2);
  const RowSrc srcV = make_row_src((const char*)a.v + (row0 * a.Hkv + hk) * D * 2, nullptr, kvstride, T, D * 2);
  const RowSrc srcQ = make_row_src((const char*)a.q + (row0 * a.Hq + hk * a.group + qh0) * D * 2,
                                   (CONV && a.q_halo) ? (const char*)a.q_halo + ((size_t)b * (a.W - 1) * a.Hq + hk * a.group + qh0) * D * 2 : nullptr,
                                   qstride, T, GR * D * 2);
  const unsigned coff = (unsigned)c0 * 2;

  // ---- state in accumulators: Sacc[ct][rt][i] = S[16 rt + 4 g4 + i][col + 4 ct] (columns alternate by fours, so that a lane of a pair of
  // output tiles holds eight adjacent ones), zacc[e][i] = z[zrow + 16 e + i], the same in all n
  const int col = 32 * w + 8 * (n >> 2) + (n & 3), zrow = 32 * w + 4 * g4;
  floatx4 Sacc[G::CT][G::RT], zacc[2];
  Raw<GR> raw;
  {
    const float* Sin = nullptr;
    const float* zin = nullptr;
    int first = seg;
    bool scanned = false;
    if (a.fold) {
      const unsigned long long m = __builtin_amdgcn_ballot_w64(live_any == 0);
      first = m ? 64 - __builtin_clzll(m) : 0;
    } else if (nseg > 1) {
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
#pragma unroll
    for (int ct = 0; ct < G::CT; ++ct)
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) Sacc[ct][rt][i] = Sin ? Sin[(size_t)(16 * rt + 4 * g4 + i) * D + col + 4 * ct] : 0.f;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) zacc[e][i] = zin ? zin[zrow + 16 * e + i] : 0.f;
    KK::template fetch<true>(raw, srcK, srcG, srcV, s0, tl0, coff, a.W);
    if (CONV) {
      const float wscale = MODE == kConvElu ? kLog2e : 1.f;
#pragma unroll
      for (int j = 0; j < kWeights; ++j) {
        const int e = tid + j * G::TEAM;
        if (e < kRows * D)
          *reinterpret_cast<floatx4*>(wl + (size_t)e * 4) =
              floatx4{bf_lo(wraw[j].x) * wscale, bf_hi(wraw[j].x) * wscale, bf_lo(wraw[j].y) * wscale, bf_hi(wraw[j].y) * wscale};
      }
    }
    if (first < seg) {
      // state <- decay (.) state + contribution, segment by segment, in quarters of a slot
      float* zd = reinterpret_cast<float*>(smem);      // [predecessor][z | decay]: free until the first granule
#pragma unroll
      for (int j = 0; j < kZd; ++j) {
        const int e = tid + j * G::TEAM;
        if (e < seg * 2 * D) zd[e] = zraw[j];
      }
      struct Rows { float s[4][4]; };
      auto load = [&](int j, int q, Rows& o) {
        const __amdgpu_buffer_rsrc_t slot =
            __builtin_amdgcn_make_buffer_rsrc((void*)(a.ws + (slot0 + j) * G::kSlot), 0, D * D * 4, 0x00020000);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            o.s[rt][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(slot, (4 * g4 * D + col) * 4, ((16 * (4 * (q & 1) + rt) + i) * D + 4 * (q >> 1)) * 4, 0));
      };
      auto add = [&](int j, int q, const Rows& o) {
        const float* at = zd + j * 2 * D;
        floatx4 dec[4];
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) dec[rt] = *reinterpret_cast<const floatx4*>(at + D + 16 * (4 * (q & 1) + rt) + 4 * g4);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i) Sacc[q >> 1][4 * (q & 1) + rt][i] = fmaf(dec[rt][i], Sacc[q >> 1][4 * (q & 1) + rt][i], o.s[rt][i]);
        if (q == 0) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const floatx4 dz = *reinterpret_cast<const floatx4*>(at + zrow + 16 * e), zdec = *reinterpret_cast<const floatx4*>(at + D + zrow + 16 * e);
#pragma unroll
            for (int i = 0; i < 4; ++i) zacc[e][i] = fmaf(zdec[i], zacc[e][i], dz[i]);
          }
        }
      };
      Rows x, y;
      load(first, 0, x);
      __syncthreads();
#pragma unroll 1
      for (int j = first; j < seg; ++j) {
        load(j, 1, y);
        add(j, 0, x);
        load(j, 2, x);
        add(j, 1, y);
        load(j, 3, y);
        add(j, 2, x);
        load(min(j + 1, seg - 1), 0, x);
        add(j, 3, y);
      }
    }
  }
  const bool gs1 = a.gate_scale == 1.0f;
  Part<GR> own;
  __syncthreads();  // conv weights are in LDS, the folded segments' z and decays read

  const int granules = (s1 - s0 + G::NTG - 1) / G::NTG;
#pragma unroll 1
  for (int gi = 0; gi < granules; ++gi) {
    const int t0 = s0 + gi * G::NTG;
    const bool edge = (t0 < 3) || (t0 + G::NTG > s1);
    // (not known to be the lane's, so that no LDS address of the four forms is kept over the loop: they spilled)
    int lane = l;
    asm volatile("" : "+v"(lane));
    const int th = lane >> 5, c0 = 64 * (w % G::CH) + 2 * (lane & 31), tl0 = kChunk * mcw + 8 * th;
    const unsigned coff = (unsigned)c0 * 2;
    if (!edge && gs1)
      KK::template compute<false, true>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
    else if (!edge)
      KK::template compute<false, false>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
    else if (gs1)
      KK::template compute<true, true>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
    else
      KK::template compute<true, false>(raw, srcQ, coff, a.W, smem, wl, t0, s1, tl0, c0, mcw, th, a.gate_scale, own);
    __builtin_amdgcn_s_waitcnt(0x0F70);      // (nothing is in flight: see the other kernel)
    __syncthreads();
    __builtin_amdgcn_s_setprio(3);
    // next granule's rows travel while the matrix cores work
    if (gi + 1 < granules) KK::template fetch<false>(raw, srcK, srcG, srcV, t0 + G::NTG, tl0, coff, a.W);
    asm volatile("" : "+v"(lane));
    const int l = lane, g4 = l >> 4, n = l & 15, col = 32 * w + 8 * (n >> 2) + (n & 3), zrow = 32 * w + 4 * g4;
    const unsigned lrow = (unsigned)n * G::QRS + (unsigned)g4 * 8;      // this lane's part of a token-major row's LDS address
    int midmask = 0;
#pragma unroll
    for (int j = 0; j < G::NW; ++j) midmask |= *reinterpret_cast<const int*>(smem + G::kFl + j * 4) << (j / G::CH);
    midmask = __builtin_amdgcn_readfirstlane(midmask);
    const short4v ones4 = {0x3F80, 0x3F80, 0x3F80, 0x3F80};
    // z through the granule's chunks, a wave's 32 channels; what it is at each chunk's start goes to LDS as bf16
#pragma unroll
    for (int mc = 0; mc < G::MCG; ++mc)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const unsigned at = (mc * D + zrow + 16 * e) * 4;
        const uint2 kd = *reinterpret_cast<const uint2*>(smem + G::kKd + (32 * w + 16 * e + n) * G::TRS + (kChunk * mc + 4 * g4) * 2);
        if (midmask != 0) zacc[e] *= *reinterpret_cast<const floatx4*>(smem + G::kEf + at);
        if (n == 0) *reinterpret_cast<uint2*>(smem + G::kZs + (mc * D + zrow + 16 * e) * 2) = make_uint2(pack2(zacc[e][0], zacc[e][1]), pack2(zacc[e][2], zacc[e][3]));
        zacc[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, kd), ones4, zacc[e] * *reinterpret_cast<const floatx4*>(smem + G::kEb + at), 0, 0, 0);
      }
    __syncthreads();
    // the chunk's scores of this wave's heads, its part and the other wave's, and denominators: q' . z + (column sums of the masked scores)
    {
      const bf16x8 ones8 = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
      bf16x8 zf[G::KS];
#pragma unroll
      for (int ks = 0; ks < G::KS; ++ks) {
        const unsigned char* pz = smem + G::kZs + (mcw * D + 32 * ks + 4 * g4) * 2;
        zf[ks] = make8(*reinterpret_cast<const uint2*>(pz), *reinterpret_cast<const uint2*>(pz + 32));
      }
#pragma unroll
      for (int j = 0; j < G::HW; ++j) {
        const int hh = G::HW * (w % G::CH) + j;
        if (hh < GR) {
          unsigned char* at = smem + G::kPs + (mcw * GR + hh) * 1024 + l * 16;
          const uint4 pp = pack_scores(own.p[j] + *reinterpret_cast<const floatx4*>(at), g4, n);
          floatx4 dz = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < G::KS; ++ks) {
            const unsigned char* pq = smem + G::kQp + (hh * G::NTG + kChunk * mcw) * G::QRS + lrow + 64 * ks;
            dz = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[ks], make8(*reinterpret_cast<const uint2*>(pq), *reinterpret_cast<const uint2*>(pq + 32)), dz, 0, 0, 0);
          }
          *reinterpret_cast<uint4*>(at) = pp;
          dz = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones8, __builtin_bit_cast(bf16x8, pp), dz, 0, 0, 0);
          if (g4 == 0) *reinterpret_cast<float*>(smem + G::kDn + ((mcw * GR + hh) * 16 + n) * 4) = dz[0] + a.eps;
        }
      }
    }
    __syncthreads();
    // Outputs and state, 32 value columns a wave: o^T[dv][query] = S^T (q (.) E)^T + [V,V]^T [P_hi;P_lo]^T, then S <- diag(E_last / rho)
    // (rho S) + Kdec^T V.
#pragma unroll 1
    for (int mc = 0; mc < G::MCG; ++mc) {
      const int tq = t0 + kChunk * mc;
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
      HeadOps ops[2];
      load_ops(0, ops[0]);
      uint2 vraw[G::CT];
#pragma unroll
      for (int ct = 0; ct < G::CT; ++ct) vraw[ct] = *reinterpret_cast<const uint2*>(smem + G::kVt + (col + 4 * ct) * G::TRS + (kChunk * mc + 4 * g4) * 2);
      if ((midmask >> mc) & 1) {
        // some channel of this chunk uses the mid-chunk reference: the accumulators take rho in place, the update continues from there
#pragma unroll
        for (int rt = 0; rt < G::RT; ++rt) {
          const floatx4 ef = *reinterpret_cast<const floatx4*>(smem + G::kEf + (mc * D + 16 * rt + 4 * g4) * 4);
#pragma unroll
          for (int ct = 0; ct < G::CT; ++ct) Sacc[ct][rt] *= ef;
        }
      }
      bf16x8 sa[G::CT][G::KS];   // rows = value columns, k = key channels {4 g4 + i, 16 + 4 g4 + i} of each 32
#pragma unroll
      for (int ct = 0; ct < G::CT; ++ct)
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) {
          const floatx4 lo = Sacc[ct][2 * ks], hi = Sacc[ct][2 * ks + 1];
          sa[ct][ks] = __builtin_bit_cast(bf16x8, make_uint4(pack2(lo[0], lo[1]), pack2(lo[2], lo[3]), pack2(hi[0], hi[1]), pack2(hi[2], hi[3])));
        }
      const int tok = tq + n;
      const size_t orow = (row0 + tok) * a.Hq + hk * a.group + qh0;
#pragma unroll
      for (int hh = 0; hh < GR; ++hh) {
        const HeadOps& o = ops[hh & 1];
        if (hh + 1 < GR) load_ops(hh + 1, ops[(hh + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        floatx4 acc[G::CT];
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct) acc[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
          for (int ct = 0; ct < G::CT; ++ct) acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sa[ct][ks], o.qb[ks], acc[ct], 0, 0, 0);
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct) acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(make8(vraw[ct], vraw[ct]), o.pp, acc[ct], 0, 0, 0);
        const float r = fast_rcp(o.den);
        if (tok < s1) {
          const floatx4 x = acc[0] * r, y = acc[1] * r;
          *reinterpret_cast<uint4*>(a.o + (orow + hh) * D + 32 * w + 8 * g4) = make_uint4(pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(y[0], y[1]), pack2(y[2], y[3]));
          if (a.den_out != nullptr && w == 0 && g4 == 0) a.den_out[orow + hh] = o.den;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt) {
        const uint2 kd = *reinterpret_cast<const uint2*>(smem + G::kKd + (16 * rt + n) * G::TRS + (kChunk * mc + 4 * g4) * 2);
        const floatx4 eb = *reinterpret_cast<const floatx4*>(smem + G::kEb + (mc * D + 16 * rt + 4 * g4) * 4);
#pragma unroll
        for (int ct = 0; ct < G::CT; ++ct)
          Sacc[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, kd), __builtin_bit_cast(short4v, vraw[ct]), Sacc[ct][rt] * eb, 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
  }

  // ---- state and conv cache out
  if (seg == nseg - 1 && keeps) {
    float* S = a.S_out + (size_t)bh * D * D;
#pragma unroll
    for (int ct = 0; ct < G::CT; ++ct)
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) S[(size_t)(16 * rt + 4 * g4 + i) * D + col + 4 * ct] = Sacc[ct][rt][i];
    if (n == 0)
#pragma unroll
      for (int e = 0; e < 2; ++e) *reinterpret_cast<floatx4*>(a.z_out + (size_t)bh * D + zrow + 16 * e) = zacc[e];
  }
  if (CONV && seg == nseg - 1 && a.W > 1) store_tails<D>(a, b, hk, qh0, GR, keeps, T, row0, tid, G::TEAM);
}

}  // namespace chunk
}  // namespace lawcat
