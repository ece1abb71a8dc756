// Host side of the bf16 matrix-core prefill: segment plan, workspace size, dispatch to the
// per-head-dimension translation units.
#include "gla_chunk_impl.h"

namespace lawcat {
namespace chunk {
hipError_t launch_d64(const ChunkArgs& a, int group, int mode, hipStream_t stream, const TraceEvents& ev);
hipError_t launch_d128(const ChunkArgs& a, int group, int mode, hipStream_t stream, const TraceEvents& ev);
}  // namespace chunk

bool chunk_path_supports(int group) { return group >= 1 && group <= 64; }

// Most segments of a head whose contributions the output pass folds in one launch (see launch_gla_chunk).
static int fold_most(int heads, int group, int d) {
  return d == 64 ? std::min(chunk::kFoldMost<64> + 1, 9 + heads / 4) : std::min(group < 8 ? chunk::kFoldMost<128> + 1 : 7, 4 + heads / 8);
}

GroupCover cover_group(int group, long long walks) {
  const int most = walks * group <= 256 ? 1 : walks * ((group + 1) / 2) <= 256 ? 2 : 4;     // (see launch_gla_chunk)
  int launches = 0;
  for (int left = group; left > 0; ++launches) {
    const int heads = left >= most ? most : (left >= 2 ? 2 : 1);
    left -= left / heads * heads;
  }
  return {most, launches};
}

ChunkPlan make_chunk_plan(int B, int T, int Hq, int Hkv, int d, int carry_mode, int segment, bool conv, size_t room) {
  ChunkPlan p{};
  const int heads = B * Hkv;
  int seg_len;
  auto cut = [&](int len) {
    p.seg_len = len;
    p.nseg = (T + len - 1) / len;
    // per (head, segment): contribution or start state S | z | total decay, then one flag word each
    p.workspace_bytes = p.nseg > 1 ? (size_t)heads * p.nseg * ((d * d + 2 * d) * sizeof(float) + sizeof(int)) : 0;
  };
  if (carry_mode == 1) {
    seg_len = (T + 63) / 64 * 64;
  } else if (segment > 0) {
    seg_len = segment;
  } else {
    // enough workgroups (of up to four query heads each) to fill 256 compute units once (two 4-wave teams per unit at head dim
    // 64, one 8-wave team at 128), in segments of two granules (128 tokens) at least ...
    const int slots = d == 64 ? 512 : 256;
    const long long groups = (long long)heads * std::max(1, Hq / Hkv / 4);   // workgroups per segment
    // Head dim 128 with conv: two 4-wave teams per unit (gla_wide.h), in twice as many segments, where those are long enough that the
    // state pass, which reads up to 192 tokens of each, costs less than the output pass gains, and if the workspace has the slots.  us a
    // call, eight waves / four (segments of .. tokens): 32 on 8 heads, 8192 tokens (128) 76.6 / 90.9, 16384 (256) 128.0 / 129.3, 18000 (320) 133.7 /
    // 131.4, 24000 165.1 / 159.9, 65536 402.6 / 363.1, 131072 777 / 686, x 16, 2000 (512) 205.0 / 193.0, x 32, 700 145.7 / 144.5; two heads a
    // workgroup, 20000 (320) 116.6 / 116.2, 30000 150.9 / 146.3; one, 30000 (512) 124.1 / 125.3, 36000 (576) 144.9 / 140.2; groups of more than one
    // workgroup, whose state pass is half as many, 32 on 4, 8192 (128) 71.2 / 71.7, 12000 (192) 92.5 / 85.2.  Without conv, where there is less
    // beside the MFMA stage to run, 16384 tokens of the feature-map layer 224.8 / 240.0.
    if (d == 128 && conv) {
      const int group = std::max(1, Hq / Hkv), most = (int)((512 + groups - 1) / groups);
      const int len = ((T + most - 1) / most + 63) / 64 * 64;
      cut(len);
      p.wide = len >= (group >= 8 ? 192 : group == 1 ? 576 : 320) && p.workspace_bytes <= room;
      if (p.wide) return p;
    }
    const int want = (int)((slots + groups - 1) / groups);
    seg_len = (T + want - 1) / want;
    seg_len = (seg_len + 63) / 64 * 64;
    if (seg_len < 128) {
      // ... or of one granule, which halves the serial work of a workgroup, where they still fit the chip at once, unless
      //   two granules hold the whole sequence: no state pass then (one granule / two, 128 tokens, 8 heads of 64 x 2 15.3 / 14.7 us, x 24
      //     20.2 / 16.2, of 128 23.1 / 20.2, 30.9 / 21.9 x 16);
      //   at head dim 64 twice the contributions to fold cost more than the granule saves, which grows with both their number and the
      //     workgroups that read them: 8 heads x 3, 512 tokens 22.1 / 23.8, 800 27.4 / 23.9; x 5, 448 22.1 / 22.7, 512 27.2 / 24.4; x 8, 300
      //     21.1 / 22.1, 500 30.0 / 25.7; 32 on 8 x 12, 190 25.4 / 27.3, 390 39.1 / 37.4;
      //   at head dim 128 they are too many to fold, and half as many are not: 8 heads x 3, 390 tokens 32.0 / 33.5, 512 40.5 / 37.1, 600 38.8 /
      //     36.9.
      // (Few heads leave most of the chip idle: there the shorter walk is the better one at any length, 8 x 2, 1000 tokens 24.3 / 26.5,
      // of 128 39.0 / 42.7.)
      const int one = (T + 63) / 64, two = (T + 127) / 128, fold = std::min(7, fold_most(heads, Hq / Hkv, d));
      const bool pays = heads <= 16 || (d == 64 ? (long long)one * (heads + 18) <= 460 : one <= fold || two > fold);
      seg_len = two > 1 && one * groups <= slots && pays ? 64 : 128;
    }
  }
  cut(seg_len);
  return p;
}

hipError_t launch_gla_chunk(const ChunkParams& p, hipStream_t stream) {
  chunk::ChunkArgs a;
  a.q = (const bf16_t*)p.q; a.k = (const bf16_t*)p.k; a.v = (const bf16_t*)p.v; a.g = (const bf16_t*)p.g;
  a.wq = (const bf16_t*)p.wq; a.wk = (const bf16_t*)p.wk;
  a.q_halo = (const bf16_t*)p.q_halo; a.k_halo = (const bf16_t*)p.k_halo;
  a.S0 = p.S0; a.z0 = p.z0; a.o = (bf16_t*)p.o; a.den_out = p.den_out; a.S_out = p.S_out; a.z_out = p.z_out;
  a.q_tail = (bf16_t*)p.q_tail; a.k_tail = (bf16_t*)p.k_tail;
  a.ws = (float*)p.workspace;
  a.seq_start = p.seq_start;
  a.per_head = p.plan.per_head; a.inv_len = 1.0 / p.plan.seg_len;
  a.seg_live = reinterpret_cast<int*>(a.ws + (size_t)p.B * p.Hkv * p.plan.nseg * (p.d * p.d + 2 * p.d));
  a.B = p.B; a.T = p.T; a.Hq = p.Hq; a.Hkv = p.Hkv; a.W = p.W;
  a.seg_len = p.plan.seg_len; a.nseg = p.plan.nseg; a.wide = p.plan.wide;
  // A workgroup of the output pass takes four query heads of a group, or two or one where that still gives no more workgroups than
  // compute units: each is a serial walk, and those for two heads or one are shorter, at the price of forming the keys' side again.
  // us a call with four / two / one, 8 kv heads: of 64, 32 query heads, 64 tokens 13.7 / 11.9 / 10.7, 517 20.4 / 19.1 / -; 1500, where
  // two would be 384 workgroups, 21.8 / 22.6 / 27 (on 4 kv heads); of 128, 64 tokens 19.2 / 16.6 / 14.2, 1000 36.6 / 33.9 / 41.9 (512).
  // In place one workgroup per launch takes a segment, so that none reads a start state that another one replaces: the last launch
  // stores the state, and with several segments they all start from their slots (no fold).
  const int nseg = p.plan.nseg, heads = p.B * p.Hkv, group = p.Hq / p.Hkv;
  const long long walks = p.seq_start ? (long long)p.Hkv * p.plan.segments : (long long)nseg * heads;
  const bool in_place = chunk::in_place(a);
  a.most = in_place ? 4 : cover_group(group, walks).most;
  // With few segments the output pass folds its predecessors' contributions itself instead of waiting for a scan: a launch less,
  // and, with many heads, less traffic, against a walk over the predecessors' slots in each of the output pass's launches (more than
  // one for groups that are no multiple of 4).  Scan / fold, us a call in segments of 128 tokens: of 64, 2 heads, 8 segments 23.3 / 22.6,
  // 9 23.4 / 23.1, 11 23.2 / 23.9; 8 heads, 11 25.2 / 24.9, 12 25.7 / 25.8; 32 on 8 x 2 12 35.2 / 33.3, x 8 10 69.4 / 59.4.  Of 128, 2 heads,
  // 4 segments 32.2 / 32.3, 5 32.4 / 33.3; 8 heads, 5 34.9 / 34.6, 6 35.9 / 36.9; 32 on 8 x 2 6 44.2 / 42.6, x 4 9 83.8 / 82.7, x 8 8
  // 115.3 / 113.3; 32 on 4, whose groups are two workgroups, x 8 7 87.6 / 85.8, 8 92.9 / 102.0.
  // Packed batches (see find_place): a grid of all sequences by the longest one's segments where it has no workgroup without work, or
  // they all find a place on the chip at once: to find its segment costs a workgroup of the other grids 0.3 to 1 us a pass (by length up to 6 with 64
  // sequences, 10 before its loop lost its branches).  Else in
  // order of the rows, where that grid fits, else by length.  us a call by sequence / in order / by length, 32 query heads on 8 kv heads:
  // of 64, 128 x 200 tokens 96 / 122 / 120, 30 x 333 47 / 65 / 52, 12 of 60 to 280 24.2 / 26.4 / 29.3; 4 short ones beside one of 2000 47.5 /
  // 29.8 / 30.9, 12 of 88 to 1439 54.9 / 39.2 / 41.8; 24 of 101 to 3364 190 / 115 / 95, 48 of 204 to 691 135 / 120 / 97.  Of 128, 16 of 480 to
  // 520 84 / 128 / 88; 3 of 337 to 855 63 / 47 / 48; 24 of 300 to 498 161 / 146 / 106.  (At head dim 64 a few workgroups too many, which leave
  // at once, cost less than to order them, while a walk is short: 24 of 300 to 498, 9/8 of the chip, 48.8 / 50.1 / 51.1, but 8 of 4111 to
  // 7197, segments of 832, 172 / 140 / 140; of 128, 12 of 208 to 352, 63 / 71 / 50.)
  a.places = chunk::kDirect;
  if (p.seq_start) {
    const long long places = p.d == 64 || p.plan.wide ? 512 : 256, parts = in_place ? 1 : std::max(1, group / a.most);     // at once on the chip; workgroups per segment
    const long long direct = (long long)p.B * nseg, in_order = p.plan.per_head;
    if (direct <= p.plan.segments || direct * p.Hkv * parts <= places) a.places = chunk::kDirect;
    else if (p.B > 64) a.places = direct <= in_order ? chunk::kDirect : chunk::kInOrder;
    else if (in_order * p.Hkv * parts <= places) a.places = chunk::kInOrder;
    else a.places = p.d == 64 && p.plan.seg_len <= 256 && direct * p.Hkv * parts <= places * 9 / 8 ? chunk::kDirect : chunk::kByLength;
  }
  const int passes = group % 4 == 0 || a.most == 1 ? 1 : group / 4 + (group % 4 + 1) / 2;
  a.fold = !in_place && nseg > 1 && nseg * passes <= fold_most(heads, group, p.d);
  a.gate_scale = p.gate_scale; a.eps = p.eps;
  const int mode = !p.fuse_conv ? chunk::kPlain : (p.phi == 1 ? chunk::kConvElu : chunk::kConvId);
  const chunk::TraceEvents ev{p.ev_start, p.ev_stop};
  return p.d == 64 ? chunk::launch_d64(a, group, mode, stream, ev) : chunk::launch_d128(a, group, mode, stream, ev);
}

}  // namespace lawcat
