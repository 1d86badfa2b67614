// Dispatch layout of the rerouted assignments on gfx950: the send buffer
// groups the assignments by destination rank (ranks ascending) and keeps
// row-major (token, k) order inside one destination, so each destination's
// assignments form one contiguous run that an all-to-all dispatch sends as
// is (the per-destination counts the dispatch consumes, Section 4.3).
//
// One launch; one pass over token_dest for a chunk of one tile per
// workgroup, two passes for longer chunks (at most 512 workgroups):
//   - a one-tile workgroup holds its assignments in registers and ranks
//     them among equal destinations inside each wave (ballots over the
//     destination bits give each lane its peers), then scans the per-wave
//     counts across waves in LDS; a longer chunk is cut into one contiguous
//     part per wave, each wave only counts its part's destinations here
//     (LDS atomics), and once the earlier counts are in ranks its part step by step
//     from its own running base, reading the assignments again, with no
//     workgroup barrier;
//   - it publishes its per-destination counts; workgroups form groups of
//     kLayoutGroup, and the last of a group publishes the group's total in
//     their place (the last of all publishes nothing: nobody would read it).
//     A workgroup then sums the counts of the earlier ones of its group and
//     the totals of the earlier groups, at most kLayoutGroup - 1 rows of each;
//   - slot = send_offsets[dest] + (earlier workgroups) + (earlier waves, or
//     their parts) + (earlier steps of the wave's part) + (rank in the
//     wave).
// A published count is one word, the count + 1, stored and polled with relaxed
// agent-scope atomics: it is valid by itself, so no fence writes back or
// invalidates an L2 under the other workgroups.  (Flags with release and
// acquire cost more than the counting and ranking: R = 64, 4.2 M ids 33.7 us,
// 20.0 now; 0.5 M ids 15.3, 9.3 now; 4 K ids, four workgroups, 5.25 and 5.30.
// Every workgroup summing all earlier rows behind one acquire a wave: 45 us
// for 4.2 M ids.)  The waits are bounded and only on lower workgroup indices,
// which are dispatched first.  The last workgroup of a group to finish (a
// ticket) clears the group's counts, the last of all the totals, so the
// workspace is zero again for the next call: every published word has been
// read by another workgroup before that one's ticket, so no store of it is
// still on its way when it is cleared.
// All arithmetic is integer and no atomic decides an order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "topoep.h"
#include "wave.h"

namespace {

using namespace topoep_dev;

constexpr int kLayoutThreads = 1024;
constexpr int kLayoutMaxRanks = 1024;   // per-wave counts of 16 waves fit 64 KB of LDS
constexpr int kLayoutGroup = 16;        // workgroups whose counts one total stands for
constexpr int kLayoutBlocks = 512;      // workgroups at most (longer chunks take several tiles)
constexpr uint32_t kLayoutSpin = 1u << 24;
constexpr int kLayoutCtrlBytes = 256;
constexpr int kLayoutGroupTickets = 32;   // control words: [0] groups done, [32 + g] workgroups of group g done

struct Layout {
  int R, nbits, nb;
  int64_t n, chunk;
  const int32_t *dest;
  const int32_t *send;
  int32_t *offs_out;   // [R + 1]
  int32_t *slot_out;   // [n]
  int32_t *status;     // [1] or null: TOPOEP_ST_SYNC when a wait gave up
  uint32_t *rows;      // [nb][R] a workgroup's counts + 1, or its group's total + 1
  uint32_t *ctrl;      // finish tickets (kLayoutGroupTickets)
  uint32_t spin_limit;
};

// LDS words: per-wave counts (then offsets, then a long chunk's running
// slot bases) [nw][R], the workgroup's counts [R], the exclusive prefix over
// earlier workgroups [R], send offsets [R + 1], broadcast words, and the
// counting copies of a long chunk's first pass [nw][C][R] (C > 1).
struct LayoutLds {
  int wc, agg, excl, offs, misc, cnt, words;
};

// Copies of each wave's counts in the first pass of a long chunk: lane l
// counts into copy l % C, so equal destinations of one wave instruction
// meet fewer times on one LDS word (at most 64 KB of copies).
__host__ __device__ inline int layout_copies(int R) { return R <= 256 ? 4 : (R <= 512 ? 2 : 1); }

__host__ __device__ inline LayoutLds layout_lds(int R, int nt) {
  LayoutLds l;
  int o = 0;
  l.wc = o; o += (nt / 64) * R;
  l.agg = o; o += R;
  l.excl = o; o += R;
  l.offs = o; o += R + 1;
  l.misc = o; o += 8;
  l.cnt = o; o += layout_copies(R) > 1 ? (nt / 64) * layout_copies(R) * R : 0;
  l.words = o;
  return l;
}

// Rank of each of the wave's IPT x 64 assignments among the wave's earlier
// ones with the same destination (index order: i, then lane) into lr, and
// the wave's count of every destination into its row of wc.
template <int IPT>
__device__ inline void rank_wave(int R, int nbits, const int (&dv)[IPT], int (&lr)[IPT], int *mywc) {
  const int lane = lane_id();
  for (int r = lane; r < R; r += 64) mywc[r] = 0;
  wave_sync();
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    lr[i] = wave_rank(dv[i], (unsigned)dv[i] < (unsigned)R, nbits, mywc);
  }
}

// Per destination: the waves' counts in wc become their offsets (one 16-lane
// scan per rank, lane w holding wave w's count) and tot[r] the row's total.
__device__ inline void scan_waves(int R, int nw, int *wc, int *tot) {
  const int rows = R * 16, span = (rows + 63) & ~63;
  for (int t = threadIdx.x; t < span; t += blockDim.x) {
    const int r = t >> 4, w = t & 15;
    const bool in = t < rows && w < nw;
    const int c = in ? wc[w * R + r] : 0;
    const int incl = row16_incl_scan(c);
    if (in) wc[w * R + r] = incl - c;
    if (t < rows && w == 15) tot[r] = incl;
  }
}

template <int IPT>
__global__ __launch_bounds__(kLayoutThreads) void layout_kernel(Layout L) {
  extern __shared__ int lsm[];
  const int R = L.R, tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;
  const LayoutLds l = layout_lds(R, nt);
  int *wc = lsm + l.wc, *agg = lsm + l.agg, *excl = lsm + l.excl, *offs = lsm + l.offs;
  int *misc = lsm + l.misc;
  const int64_t lo = (int64_t)b * L.chunk;
  const int64_t hi = lo + L.chunk < L.n ? lo + L.chunk : L.n;
  const int64_t tile = (int64_t)nt * IPT;
  // a chunk of one tile keeps its ids and ranks in registers across the
  // wait for the earlier workgroups; a longer chunk counts its tiles first (pass 1) and ranks them
  // after it (pass 2), reading the ids twice
  const bool multi = L.chunk > tile;
  const int64_t wofs = (int64_t)wave * 64 * IPT + lane;
  // a longer chunk: wave w owns the w-th of nw equal contiguous parts, in
  // steps of 64 IPT ids (the chunk is a whole number of tiles)
  const int64_t step = 64 * IPT, sub = L.chunk / nw;
  const int64_t wlo = lo + wave * sub, whi = wlo + sub < hi ? wlo + sub : hi;
  auto load_step = [&](int (&v)[IPT], int64_t base) {
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int64_t idx = base + lane + i * 64;
      v[i] = idx < whi ? L.dest[idx] : -1;
    }
  };
  const int gi = b % kLayoutGroup, grp = b / kLayoutGroup;
  const bool last = b == L.nb - 1;
  auto publish = [&](int r, int count) {
    __hip_atomic_store(L.rows + (int64_t)b * R + r, (uint32_t)count + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  int *mywc = wc + wave * R;

  int dv[IPT], lr[IPT];
  for (int r = tid; r < R; r += nt) {
    offs[r] = L.send[r];
    excl[r] = 0;
  }
  if (tid < 8) misc[tid] = 0;
  if (!multi) {
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int64_t idx = lo + wofs + i * 64;
      dv[i] = idx < hi ? L.dest[idx] : -1;
    }
    rank_wave<IPT>(R, L.nbits, dv, lr, mywc);
  } else {
    // pass 1: each wave's count of every destination over its own part of
    // the chunk, one LDS atomic per assignment into the lane's copy of the
    // wave's counts (the order of the counting does not matter: a lane
    // loads four consecutive ids at once; the next step's loads are in
    // flight meanwhile), then the copies summed into the wave's row
    const int C = layout_copies(R);
    int *rows = C > 1 ? lsm + l.cnt + wave * C * R : mywc;
    for (int r = lane; r < C * R; r += 64) rows[r] = 0;
    wave_sync();
    int *myc = rows + (lane & (C - 1)) * R;
    // V loads of four ids per lane and step (256 V ids; parts start on
    // multiples of 64 ids, so a 16-byte aligned array keeps them aligned)
    constexpr int V = IPT >= 4 ? IPT / 4 : 1;
    const int64_t step1 = 256 * V;
    const bool vec = (reinterpret_cast<uintptr_t>(L.dest) & 15) == 0;
    auto load4 = [&](int4 (&v)[V], int64_t base) {
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const int64_t idx = base + (int64_t)(j * 64 + lane) * 4;
        if (vec && idx + 4 <= whi) {
          v[j] = *reinterpret_cast<const int4 *>(L.dest + idx);
        } else {
          v[j].x = idx < whi ? L.dest[idx] : -1;
          v[j].y = idx + 1 < whi ? L.dest[idx + 1] : -1;
          v[j].z = idx + 2 < whi ? L.dest[idx + 2] : -1;
          v[j].w = idx + 3 < whi ? L.dest[idx + 3] : -1;
        }
      }
    };
    int4 nx[V];
    load4(nx, wlo);
    for (int64_t base = wlo; base < whi; base += step1) {
      int4 cv[V];
#pragma unroll
      for (int j = 0; j < V; ++j) cv[j] = nx[j];
      if (base + step1 < whi) load4(nx, base + step1);
#pragma unroll
      for (int j = 0; j < V; ++j) {
        if ((unsigned)cv[j].x < (unsigned)R) atomicAdd(&myc[cv[j].x], 1);
        if ((unsigned)cv[j].y < (unsigned)R) atomicAdd(&myc[cv[j].y], 1);
        if ((unsigned)cv[j].z < (unsigned)R) atomicAdd(&myc[cv[j].z], 1);
        if ((unsigned)cv[j].w < (unsigned)R) atomicAdd(&myc[cv[j].w], 1);
      }
    }
    if (C > 1) {
      wave_sync();
      for (int r = lane; r < R; r += 64) {
        int sum = 0;
        for (int c = 0; c < C; ++c) sum += rows[c * R + r];
        mywc[r] = sum;
      }
    }
  }
  lds_barrier();
  scan_waves(R, nw, wc, agg);
  lds_barrier();
  if (gi != kLayoutGroup - 1 && !last)
    for (int r = tid; r < R; r += nt) publish(r, agg[r]);
  // send offsets (exclusive prefix of the send counts) by wave 0
  if (wave == 0) {
    const int per = (R + 63) / 64, a0 = imin(R, lane * per), a1 = imin(R, a0 + per);
    int sum = 0;
    for (int r = a0; r < a1; ++r) sum += offs[r];
    int acc = wave_incl_scan(sum) - sum;
    for (int r = a0; r < a1; ++r) {
      const int c = offs[r];
      offs[r] = acc;
      acc += c;
    }
    if (lane == 63) offs[R] = acc;
  }
  lds_barrier();
  if (b == 0 && L.offs_out)
    for (int r = tid; r <= R; r += nt) L.offs_out[r] = offs[r];

  // the earlier workgroups' counts: thread (g0, r0) sums every tr-th row of
  // destination r0, four words in flight
  const int tr = nt / R, g0 = tid / R, r0 = tid - g0 * R;   // (R <= nt)
  bool gave_up = false;
  auto add_rows = [&](int cnt, int first, int stride) {
    int sum = 0;
    for (int q = g0; q < cnt && g0 < tr; q += 4 * tr) {
      uint32_t v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u] = __hip_atomic_load(L.rows + (int64_t)(first + imin(q + u * tr, cnt - 1) * stride) * R + r0,
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (q + u * tr >= cnt) continue;
        for (uint32_t it = 0; v[u] == 0u; ++it) {
          if (it >= L.spin_limit) {
            gave_up = true;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
          v[u] = __hip_atomic_load(L.rows + (int64_t)(first + (q + u * tr) * stride) * R + r0, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        sum += v[u] ? (int)(v[u] - 1u) : 0;
      }
    }
    if (sum) atomicAdd(&excl[r0], sum);
  };
  add_rows(gi, grp * kLayoutGroup, 1);
  if (gi == kLayoutGroup - 1 && !last) {   // (a total short of a word that never came is the waiters' SYNC too)
    lds_barrier();
    for (int r = tid; r < R; r += nt) publish(r, excl[r] + agg[r]);
    lds_barrier();
  }
  add_rows(grp, kLayoutGroup - 1, kLayoutGroup);
  const bool ok = __syncthreads_or(gave_up) == 0;
  // this workgroup has read every word it needs: its ticket is on its way
  // while it writes its slots
  uint32_t *gticket = L.ctrl + kLayoutGroupTickets + grp;
  uint32_t ticket = 0;
  if (tid == 0 && L.nb > 1) ticket = __hip_atomic_fetch_add(gticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!multi) {
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int64_t idx = lo + wofs + i * 64;
      if (idx < hi) {
        const int d = dv[i];
        const bool valid = ok && (unsigned)d < (unsigned)R;
        L.slot_out[idx] = valid ? offs[d] + excl[d] + mywc[d] + lr[i] : -1;
      }
    }
  } else {
    // pass 2: the wave's row becomes its first slot per destination (send
    // offset + earlier workgroups + earlier waves), and each step's slots
    // are that running base plus the rank in the wave, which the rank
    // advances: no workgroup barrier
    for (int r = lane; r < R; r += 64) mywc[r] += offs[r] + excl[r];
    wave_sync();
    int nx[IPT];
    load_step(nx, wlo);
    for (int64_t base = wlo; base < whi; base += step) {
#pragma unroll
      for (int i = 0; i < IPT; ++i) dv[i] = nx[i];
      if (base + step < whi) load_step(nx, base + step);
#pragma unroll
      for (int i = 0; i < IPT; ++i) {
        const int d = dv[i];
        const bool valid = (unsigned)d < (unsigned)R;
        const int slot = wave_rank(d, valid, L.nbits, mywc);
        const int64_t idx = base + lane + i * 64;
        if (idx < whi) L.slot_out[idx] = ok && valid ? slot : -1;
      }
    }
  }
  // the last one of its group to take a ticket clears the group's counts and
  // takes the group's; the last group's clears the totals (atomics on one
  // line take turns: one a workgroup, not two)
  if (tid == 0 && !ok && L.status) atomicOr(reinterpret_cast<unsigned *>(L.status), TOPOEP_ST_SYNC);
  if (L.nb == 1) return;
  const int gsize = imin(kLayoutGroup, L.nb - grp * kLayoutGroup);
  const int groups = (L.nb + kLayoutGroup - 1) / kLayoutGroup;
  if (tid == 0) misc[4] = ticket + 1u == (uint32_t)gsize;
  lds_barrier();
  if (!misc[4]) return;
  if (tid == 0) {
    __hip_atomic_store(gticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    misc[5] = groups > 1 && __hip_atomic_fetch_add(L.ctrl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
                                (uint32_t)groups;
  }
  auto clear = [&](int64_t word) {
    __hip_atomic_store(L.rows + word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // (the group's published counts: not its last workgroup's)
  const int64_t base = (int64_t)grp * kLayoutGroup * R;
  for (int i = tid; i < (gsize - 1) * R; i += nt) clear(base + i);
  if (groups == 1) return;
  lds_barrier();
  if (misc[5]) {
    if (tid == 0) __hip_atomic_store(L.ctrl, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int g = 0; g < groups - 1; ++g)
      for (int r = tid; r < R; r += nt) clear((int64_t)(g * kLayoutGroup + kLayoutGroup - 1) * R + r);
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int ceil_log2(int v) {
  int b = 0;
  while ((1 << b) < v) ++b;
  return b;
}

struct LayoutShape {
  int ipt;
  size_t lds;
};

// Ids per thread of n ids, as layout_setup says, and the most workgroups that
// hold them: 512 where two fit a CU, else 256.
int layout_ipt(int64_t n) {
  if (n > (int64_t)1 << 20) return 8;
  return n <= (int64_t)kLayoutThreads * 64 ? 1 : (n <= (int64_t)kLayoutThreads * 256 ? 2 : 4);
}
int64_t layout_max_blocks(int64_t n, size_t lds) {
  return n > ((int64_t)1 << 21) && lds <= 80 * 1024 ? kLayoutBlocks : kLayoutBlocks / 2;
}

// The most workgroups that n ids or fewer take: a workspace for n serves
// every smaller call.  A range of one number of ids per thread takes most at
// its end, one of longer chunks (from max_blocks tiles on) max_blocks.
int64_t layout_most_blocks(int64_t n, size_t lds) {
  int64_t most = 1;
  for (const int64_t end : {(int64_t)kLayoutThreads * 64, (int64_t)kLayoutThreads * 256, (int64_t)1 << 20,
                            (int64_t)1 << 21, n}) {
    const int64_t m = end < n ? end : n, tile = (int64_t)kLayoutThreads * layout_ipt(m);
    const int64_t tiles = (m + tile - 1) / tile, cap = layout_max_blocks(m, lds);
    const int64_t nb = tiles < cap ? tiles : cap;
    if (nb > most) most = nb;
  }
  return most;
}

// Sizes, launch shape and workspace layout (pointers stay null when ws is).
// *ws_bytes: what these ids need; *ws_most: what they or fewer need.
int layout_setup(const topoep_topology *t, int32_t T, int32_t k, Layout *out, LayoutShape *sh,
                 size_t *ws_bytes, size_t *ws_most, char *ws, size_t max_ws = SIZE_MAX) {
  if (!t) return TOPOEP_EINVAL;
  const int R = t->num_ranks;
  if (R <= 0 || T < 0 || k < 1 || (int64_t)T * k > 0x7FFFFFFF) return TOPOEP_EINVAL;
  if (R > kLayoutMaxRanks) return TOPOEP_ELIMIT;
  Layout L = {};
  L.R = R;
  L.nbits = ceil_log2(R);
  L.n = (int64_t)T * k;
  // ids per thread, then whole tiles per workgroup so that the grid stays
  // within max_blocks: one id while 64 workgroups hold them, two up to 256 (R
  // = 64, 32 K ids: 6.5 us, four ids 7.3; 131 K: 7.4, 8.0), more ids in one
  // tile of each of 256 workgroups up to 2^21 (two tiles of 128 workgroups:
  // 2.1 M ids 16.8 us, one of 256: 13.8); 512 workgroups beyond, where two fit
  // a CU (34 M ids: 256 take 105 us, 512 94; at R = 256, where one fits, 117
  // and 123; those figures without the tickets' about 1 us).  A workspace without room for so
  // many workgroups' counts gets four ids per thread.
  const size_t lds = (size_t)layout_lds(R, kLayoutThreads).words * 4;
  int ipt = layout_ipt(L.n);
  if (ipt < 4 && max_ws < kLayoutCtrlBytes + align256((size_t)((L.n + kLayoutThreads * ipt - 1) / (kLayoutThreads * ipt)) * R * 4))
    ipt = L.n <= (int64_t)kLayoutThreads * 16 ? 1 : 4;
  const int64_t tile = (int64_t)kLayoutThreads * ipt;
  const int64_t tiles = L.n > 0 ? (L.n + tile - 1) / tile : 1;
  const int64_t max_blocks = layout_max_blocks(L.n, lds);
  L.chunk = tile * ((tiles + max_blocks - 1) / max_blocks);
  const int64_t nb = L.n > 0 ? (L.n + L.chunk - 1) / L.chunk : 1;
  if (nb > (1 << 20)) return TOPOEP_ELIMIT;
  L.nb = (int)nb;
  L.spin_limit = kLayoutSpin;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  const size_t o_ctrl = take(kLayoutCtrlBytes);
  const size_t o_rows = take((size_t)L.nb * R * 4);
  *ws_bytes = off;
  *ws_most = o_rows + align256((size_t)layout_most_blocks(L.n, lds) * R * 4);
  if (ws) {
    L.ctrl = reinterpret_cast<uint32_t *>(ws + o_ctrl);
    L.rows = reinterpret_cast<uint32_t *>(ws + o_rows);
  }
  sh->ipt = ipt;
  sh->lds = lds;
  *out = L;
  return TOPOEP_OK;
}

bool g_layout_attrs = false;

void layout_attrs() {
  if (g_layout_attrs) return;
  const void *ks[] = {reinterpret_cast<const void *>(layout_kernel<1>), reinterpret_cast<const void *>(layout_kernel<2>),
                      reinterpret_cast<const void *>(layout_kernel<4>), reinterpret_cast<const void *>(layout_kernel<8>)};
  for (const void *kf : ks) (void)hipFuncSetAttribute(kf, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  g_layout_attrs = true;
}

}  // namespace

extern "C" {

int topoep_layout_workspace_bytes(const topoep_topology *topo, int32_t T, int32_t k, size_t *bytes_out) {
  if (!bytes_out) return TOPOEP_EINVAL;
  Layout L;
  LayoutShape sh;
  size_t need = 0, most = 0;
  const int rc = layout_setup(topo, T, k, &L, &sh, &need, &most, nullptr);
  if (rc == TOPOEP_OK) *bytes_out = most;
  return rc;
}

int topoep_dispatch_layout(const topoep_topology *topo, const int32_t *token_dest, int32_t T, int32_t k,
                           const int32_t *send_counts, int32_t *send_offsets, int32_t *token_slot,
                           int32_t *status, void *workspace, size_t workspace_bytes, void *stream) {
  Layout L;
  LayoutShape sh;
  size_t need = 0, most = 0;
  const int rc = layout_setup(topo, T, k, &L, &sh, &need, &most, static_cast<char *>(workspace), workspace_bytes);
  if (rc != TOPOEP_OK) return rc;
  if (!send_counts || !send_offsets || !workspace || (T > 0 && (!token_dest || !token_slot)))
    return TOPOEP_EINVAL;
  if (workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TOPOEP_EWORKSPACE;
  L.dest = token_dest;
  L.send = send_counts;
  L.offs_out = send_offsets;
  L.slot_out = token_slot;
  L.status = status;
  layout_attrs();
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  const dim3 g(L.nb), bl(kLayoutThreads);
  switch (sh.ipt) {
    case 1: hipLaunchKernelGGL(layout_kernel<1>, g, bl, sh.lds, st, L); break;
    case 2: hipLaunchKernelGGL(layout_kernel<2>, g, bl, sh.lds, st, L); break;
    case 4: hipLaunchKernelGGL(layout_kernel<4>, g, bl, sh.lds, st, L); break;
    default: hipLaunchKernelGGL(layout_kernel<8>, g, bl, sh.lds, st, L); break;
  }
  return hipGetLastError() == hipSuccess ? TOPOEP_OK : TOPOEP_EHIP;
}

}  // extern "C"
