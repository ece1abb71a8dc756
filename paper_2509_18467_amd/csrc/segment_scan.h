// What the two-level state carry of the prefill (gla_chunk_impl.h) and of its adjoint (gla_backward.hip) share: the
// scan over the segments of a head, and the dynamic-LDS limit of a kernel.
#pragma once
#include <mutex>
#include <type_traits>

#include "kernels.h"

namespace lawcat {
namespace {   // one copy per translation unit: the kernels are registered by address

// Segments of one sequence of a packed batch: as few as segments of up to `most` tokens give, equally long up to a granule of 64
// (n = ceil(T / most) segments of ceil(T / n), rounded up to 64, are n: `most` is a multiple of 64 and not below that).
struct Cut { int nseg, len; };
__host__ __device__ inline Cut cut_sequence(int T, int most) {
  const unsigned n = ((unsigned)T + most - 1) / (unsigned)most;
  return {(int)n, (int)(((unsigned)(T + 63) / 64 + n - 1) / n * 64)};
}

// Turns per-segment contributions into segment start states, in place:
//   slot[seg] <- state before segment seg;  state <- decay[seg] (.) state + contribution[seg].
// `always`: for a call whose final state replaces its start state, also where no segment passes anything on.
// AFTER: slot[seg] <- state after segment seg, for all but the last, which has no slot (nseg_max - 1 of them per head).
// The recurrence is linear, so the segments are cut into 8 groups: 8 threads per 1 or 4 state elements each
// reduce their group to (product of decays, contribution from a zero start), the eight pairs are
// combined through LDS, and each thread replays its group from its true start.  All loads of a group are independent of the running state and issued together.
//
// What bounds it: latency, two rounds of dependent loads in a launch of microseconds.  8 heads, every segment passed on: 64
// segments at head dim 64 6.3 us, 9 segments 4.6, 27 segments at head dim 128 7.4 (one element per thread and a second
// read of the slots: 6.5, 5.6, 13.2).  U and the elements per thread go together: eight segments of four elements at 128 take
// registers that cost more than the second read (9.7).  Loads past a short group's end repeat its last segment: a branch
// between them cost 2 us.
// A thread keeps its group in registers up to 8 U contributions per head, 64 at head dim 64 and 32 at 128; beyond that it reads the
// slots a second time.
// adjacent state elements of a thread: one at head dim 64, four at 128
template <int D> constexpr int kScanVec = D == 64 ? 1 : 4;
template <int D, bool AFTER = false>
__global__ void __launch_bounds__(256) segment_scan_kernel(float* __restrict__ ws, int* __restrict__ seg_live,
                                                          const float* __restrict__ S0, const float* __restrict__ z0,
                                                          int nseg_max, const int* __restrict__ seq_start, int Hkv,
                                                          int seg_len, bool always) {
  constexpr int kSlot = D * D + 2 * D;
  constexpr int NG = 8, V = kScanVec<D>, U = D == 64 ? 8 : 4;
  typedef float Vec __attribute__((ext_vector_type(V)));
  __shared__ Vec agg_x[NG][32], agg_a[NG][32];
  const int el = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int bh = blockIdx.y;
  // slots are laid out for the longest sequence; this head's sequence may use fewer
  int nseg = nseg_max;
  if (seq_start != nullptr) {
    const int b = bh / Hkv;
    nseg = cut_sequence(seq_start[b + 1] - seq_start[b], seg_len).nseg;
  }
  if (nseg < 2) return;
  if (always) {
    if (blockIdx.x == 0 && threadIdx.x == 0) seg_live[(size_t)bh * nseg_max] = 1;      // the output pass finds every start state in its slot
  } else {
    // No segment of this head passes anything on (every total decay is exactly zero: the usual case with gate
    // logits ~ N(0,1) and segments of hundreds of tokens): each start state is the predecessor's contribution,
    // which the output pass reads where it lies.  Nothing to do, and nothing is written.
    int any = 0;
    for (int j = threadIdx.x; j < nseg - 1; j += 256) any |= seg_live[(size_t)bh * nseg_max + j];
    if (__syncthreads_or(any) == 0) return;
  }
  float* slot = ws + (size_t)bh * (AFTER ? nseg_max - 1 : nseg_max) * kSlot;
  const int last = nseg - 1;                 // segments 0 .. last-1 carry contributions
  const int spg = (last + NG - 1) / NG;      // segments per group
  const int sb = min(last, grp * spg), se = min(last, sb + spg);
  // 32 V state elements per round; the grid's x extent covers them in one round when there are few heads and in several when
  // there are many (the launch stays a few thousand workgroups)
  constexpr int kTiles = (D * D + D + 32 * V - 1) / (32 * V);
  for (int tile = blockIdx.x; tile < kTiles; tile += gridDim.x) {
    const int e = (tile * 32 + el) * V;
    const bool live = e < D * D + D, isz = e >= D * D;
    const int ec = live ? e : 0, c = !live ? 0 : (isz ? e - D * D : e / D);
    Vec delta[U], dec[U];
    // segments sg .. sg + U - 1 of the group: an element of S takes its row's decay, one of z its own
    auto load = [&](int sg) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float* p = slot + (size_t)max(0, min(sg + u, se - 1)) * kSlot;
        delta[u] = *reinterpret_cast<const Vec*>(p + ec);
        if (isz) {
          dec[u] = *reinterpret_cast<const Vec*>(p + D * D + D + c);
        } else {
          const float d = p[D * D + D + c];
          dec[u] = Vec(d);
        }
      }
    };
    auto step = [](Vec& x, const Vec& a, const Vec& d) {
#pragma unroll
      for (int i = 0; i < V; ++i) x[i] = fmaf(a[i], x[i], d[i]);
    };
    // phase 1: (A, X) of the group from a zero start
    Vec A = Vec(1.f), X = Vec(0.f);
    for (int seg = sb; seg < se; seg += U) {
      load(seg);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (seg + u < se) {
          step(X, dec[u], delta[u]);
          A *= dec[u];
        }
    }
    agg_a[grp][el] = A;
    agg_x[grp][el] = X;
    __syncthreads();
    // phase 2: true start of the group
    Vec st = Vec(0.f);
    if (live) {
      if (!isz) { if (S0) st = *reinterpret_cast<const Vec*>(S0 + (size_t)bh * D * D + e); }
      else if (z0) st = *reinterpret_cast<const Vec*>(z0 + (size_t)bh * D + c);
    }
    for (int j = 0; j < grp; ++j) step(st, agg_a[j][el], agg_x[j][el]);
    // phase 3: replay, writing start states over the contributions
    for (int seg = sb; seg < se; seg += U) {
      if (spg > U) load(seg);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (seg + u < se) {
          if (live && !AFTER) *reinterpret_cast<Vec*>(slot + (size_t)(seg + u) * kSlot + e) = st;
          step(st, dec[u], delta[u]);
          if (live && AFTER) *reinterpret_cast<Vec*>(slot + (size_t)(seg + u) * kSlot + e) = st;
        }
    }
    // the group that ends at the last contribution also owns the start state of the last segment
    if (!AFTER && live && se == last && sb < se) *reinterpret_cast<Vec*>(slot + (size_t)last * kSlot + e) = st;
    __syncthreads();   // the partial products in LDS are free for the next round
  }
}

// grid's x extent: one workgroup per round and head, unless that is more than a few thousand workgroups
template <int D>
int scan_blocks(long long heads) {
  constexpr int tiles = (D * D + D + 32 * kScanVec<D> - 1) / (32 * kScanVec<D>);
  return tiles * heads <= 8192 ? tiles : (int)(4096 / heads > 1 ? 4096 / heads : 1);
}

// Raises the kernel's dynamic LDS limit once per device (the attribute is per device and per process); safe to
// call from several host threads.  The kernel is a template argument so that every kernel has its own flags.
template <auto kernel>
hipError_t set_lds(int bytes) {
  constexpr int kMaxDev = 64;
  static std::once_flag once[kMaxDev];
  static hipError_t result[kMaxDev];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  auto set = [&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
  if (dev < 0 || dev >= kMaxDev) return set();
  std::call_once(once[dev], [&] { result[dev] = set(); });
  return result[dev];
}

}  // namespace
}  // namespace lawcat
