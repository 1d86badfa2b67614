// TopoEP per-layer planner for MI355X (gfx950): HIP kernels and the C ABI
// declared in include/topoep.h.
//
// Three kernels per plan, enqueued back to back on one stream:
//
//   hist     one block per contiguous chunk of the flattened [T, k] ids, one
//            LDS row of counts, one LDS atomic per id.  Writes the
//            block's partial histogram (this rank's row of the routing
//            matrix Omega, Eq. 3, Section 3.1).
//   solve    the placement solver, in one of two shapes:
//            - one workgroup for every domain when the whole state fits in
//              the 160 KB of LDS: Omega, every domain's instances and their
//              q columns live on one CU, and each domain's refinement runs
//              on its own wavefront;
//            - one workgroup per domain (NVLink/xGMI node) otherwise, with a
//              bounded grid barrier that publishes the inter-node placement
//              of every domain and a last-workgroup step that assembles
//              this rank's instance list.
//            (Where that solver is chosen by default and the plan is small
//            enough, the three kernels' work runs as one launch:
//            plan_domains_kernel.)
//            Either way: domain demand D (Eq. 4), inter-node placement by
//            the benefit b = 2 D S - W (Eq. 9), routing construction q, U, L
//            (Section 4.3) and intra-node refinement (Eq. 10) with wave64
//            reductions and no barrier per iteration.  Extra workgroups of
//            the same launch compute each histogram block's exclusive
//            per-expert offsets for the reroute, off the solver's path.
//   reroute  same chunking as hist.  An expert whose occurrences in the chunk
//            all belong to one instance is a table lookup; only an expert
//            whose instance changes inside the chunk has its ids ranked
//            (ballots inside a wave, per-wave counts scanned across waves).
//
// All arithmetic is integer; no atomic decides an order or a placement
// (LDS/global integer atomics only accumulate commutative counts, masks and
// barrier tickets, or pick list slots whose order is re-established by a
// key), so results are bitwise reproducible across runs and launch shapes.
// Divisions by launch-time constants use a multiply and a shift (fastdiv.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <climits>
#include <mutex>
#include <vector>

#include "fastdiv.h"
#include "topoep.h"
#include "wave.h"

namespace {

using namespace topoep_dev;

// ---------------------------------------------------------------- constants

constexpr int kCtrlBytes = 256;
constexpr int kCtrlBar = 0;      // grid-barrier arrivals
constexpr int kCtrlTicket = 1;   // finish tickets of the solver workgroups
constexpr int kCtrlStatus = 2;   // status bits accumulated during the plan
constexpr int kCtrlFinal = 3;    // final status of the plan (read by reroute)
constexpr int kCtrlTotal = 4;    // uint64 at words 4..5: sum of positive loads
constexpr int kCtrlMoves = 6;    // refinement moves of the per-domain solver
constexpr int kCtrlHelpers = 7;  // offset helpers that have published their experts' totals
// one-launch plan.  Every word a wait reads carries the plan's generation g,
// so a word left over by an earlier plan (one whose bounded wait gave up)
// never satisfies a later wait, and no word needs clearing between plans:
//   words 8..9   arrivals of the chunk workgroups, 64-bit, never reset: nb per
//                plan, so the chunk that moves it from g nb + c learns g and
//                whether it is the last (c = nb - 1);
//   word 10      g itself, read by the solver at its start and advanced by it
//                at its end (arrivals = g nb holds between plans);
//   word 11      the last chunk's verdict ((g + 1) << 2) | v (the tag g + 1
//                so that a zero-filled word is no generation's): v =
//                kVerdictSame when the histogram equals row self of Omega and
//                no id is bad, kVerdictRedo otherwise;
//   flags[b]     word 0: g + 1 once the solver's plan is ready; word 1: g + 1
//                once every chunk's counts are written;
//   ghist[g & 1] the histogram of plan g (atomic adds of the chunks), cleared
//                for plan g + 1 by the solver of plan g at its start.
constexpr int kCtrlArrive = 8;
constexpr int kCtrlGen = 10;
constexpr int kCtrlVerdict = 11;
constexpr uint32_t kVerdictSame = 1;
constexpr uint32_t kVerdictRedo = 2;
constexpr int kCtrlCost = 12;    // general cost model: largest cost
constexpr int kCtrlSize = 14;    // uint64 at words 14..15: largest expert size
// words 16..63: phase stamps of the instrumented build (TOPOEP_STAMPS)
constexpr int kCtrlStamps = 16;

constexpr int kMiscGen = 40;    // LDS word of the solvers' misc array: the plan's generation
constexpr uint32_t kNoPlan = TOPOEP_ST_BAD_ID | TOPOEP_ST_NEG_LOAD | TOPOEP_ST_RANGE | TOPOEP_ST_COST;
constexpr int kLdsLimit = 160 * 1024;   // LDS per workgroup on gfx950
constexpr int kMaxSolveGroups = 128;    // co-resident by a wide margin (256 CUs)
constexpr int kMinBlocks = 2048;        // histogram/reroute blocks to aim for, at least
constexpr int kMaxBlocks = 8192;        // and at most
constexpr int64_t kOneTileIds = 1 << 20;   // above: blocks of 1024 threads
constexpr int64_t kStreamIds = 1 << 24;    // above: the histogram reads past the caches
constexpr int kOneThreads = 512;        // threads of plan_domains_kernel
constexpr int kMaxOneGroups = 64;       // its workgroups at most (a quarter of 256 CUs)
constexpr int kLongBlocks = 512;        // and at most this many of them (two per CU)
constexpr int kOffsetExperts = 32;      // experts per offset workgroup
// chunk workgroups the single-launch plan aims for: each chunk reads the
// instance list and up to nb / 2 rows of the other chunks' counts, so 32
// rather than 64 cut the DeepSeek-V3-like plan's HBM traffic from 1.16 to
// 0.97 MB for 0.16 us more latency (two ids per thread)
constexpr int kFusedBlocks = 32;
constexpr int kMaxFusedBlocks = 128;    // and at most (all co-resident: 256 CUs)
constexpr int kFlagStride = 32;         // words between ready flags (one 128-byte line each)
constexpr uint32_t kSpinLimit = 1u << 24;    // polls of a bounded wait before it gives up
constexpr uint32_t kHelperSpin = 1u << 12;   // polls of the offset helpers' counter before summing alone
constexpr int kListRegs = 4;   // instances per thread the instance list keeps in registers
constexpr uint32_t kIterLimit = 1u << 22;    // refinement moves per domain before ITER

// ---------------------------------------------------------------- plan

struct Plan {
  int R, G, M, E, P, N, Neff, PN, I, self, MW, RW, nbits, rbits, cap1, nent_cap, QS;
  int cI, cX;
  int64_t S, W;
  uint64_t tot_max;   // two-level model: the least total load out of the exact range (see out_of_range)
  int64_t n, chunk;
  int nb, n_solvers, n_helpers;
  int rchunks_all, rchunks_dom;   // routing: source-domain chunks (divisors of M)
  int s1_waves;   // stage-1 ranks: solver waves per domain (0: fewer waves than domains)
  uint32_t spin_limit;   // polls of a bounded wait (0: every such wait gives up at once)
  uint32_t iter_limit;   // committed refinement moves per domain before ITER
  FastDiv fE, fG, fGP, fP, fI, fPN, fCap, fN, fMI, fS1;
  const int32_t *gl, *topk;
  int32_t *slots_out, *dest_out, *send_out, *status_out;
  int32_t *recv_out;   // receive counts [R], or null
  const int32_t *Cm;   // general cost matrix [R, R] (with general), else null
  const int64_t *We;   // ||W_e|| per expert [E] (with general), else null
  int general;         // the full model of Section 4.1 (per-domain solver only)
  int lanes;           // the refinement's lane forms: LDS holds position words
  int32_t *slot_out;   // send-buffer slot of every assignment [n], or null
  int32_t *offs_out;   // send offsets [R + 1] (given with slot_out)
  uint32_t *ctrl;
  int32_t *partials, *offsets, *blk_err, *repl1, *seg_e, *seg_q, *csr_ptr, *csr_r, *csr_end;
  int32_t *htot;   // three-kernel plan: each expert's count over the histogram blocks [E]
  // one-launch plan: each chunk's per-expert counts [nb][E] (16 bits: a
  // chunk holds at most 1024 x 8 ids), the histogram of the ids with a
  // bad-id count [2][E + 1] (one buffer per generation parity), one flag
  // line per chunk (kFlagStride words apart)
  uint16_t *pub;
  uint32_t *ghist, *flags;
};


// Phase stamps of the instrumented build (compiled with -DTOPOEP_STAMPS into
// a separate library for measurement; the product library has none):
// thread 0 of the calling workgroup keeps the low word of the 100 MHz
// constant clock (STAMP) or of the core clock (STAMP_CLK) for slot i (0..47)
// in LDS, and STAMP_FLUSH copies slots [lo, hi) to the control words 16..63
// at the end of the role.  Stamps stay out of global memory until then: on
// gfx9 a wait for any load also waits for every earlier store, so a store
// per stamp would delay the phase that follows it.
#ifdef TOPOEP_STAMPS
__shared__ uint32_t stamp_lds[48];
#define STAMP(p, i)                                                          \
  do {                                                                       \
    if (threadIdx.x == 0) stamp_lds[(i)] = (uint32_t)__builtin_readsteadycounter(); \
  } while (0)
#define STAMP_CLK(p, i)                                                      \
  do {                                                                       \
    if (threadIdx.x == 0) stamp_lds[(i)] = (uint32_t)__builtin_amdgcn_s_memtime(); \
  } while (0)
#define STAMP_FLUSH(p, lo, hi)                                               \
  do {                                                                       \
    if (threadIdx.x == 0)                                                    \
      for (int s_ = (lo); s_ < (hi); ++s_) (p).ctrl[kCtrlStamps + s_] = stamp_lds[s_]; \
  } while (0)
#define STAMP_CLEAR(lo, hi)                                       \
  do {                                                            \
    if (threadIdx.x == 0)                                         \
      for (int s_ = (lo); s_ < (hi); ++s_) stamp_lds[s_] = 0;     \
  } while (0)
__device__ inline void stamp_nc(int nc) { stamp_lds[17] = (uint32_t)nc; }
// Core-clock cycles of the refinement loop of domain 0 by section, summed
// over its iterations (slots 32..37, the iteration count in slot 38).
#define RSECT_DECL(d)           \
  const bool rs_on_ = (d) == 0; \
  uint64_t rs_last_ = __builtin_amdgcn_s_memtime();
#define RSECT(k)                                                                     \
  do {                                                                               \
    if (rs_on_) {                                                                    \
      const uint64_t n_ = __builtin_amdgcn_s_memtime();                              \
      if (lane_id() == 0) atomicAdd(&stamp_lds[32 + (k)], (uint32_t)(n_ - rs_last_)); \
      rs_last_ = n_;                                                                 \
    }                                                                                \
  } while (0)
#define RSECT_END(iters)                                           \
  do {                                                             \
    if (rs_on_ && lane_id() == 0) atomicAdd(&stamp_lds[38], (iters)); \
  } while (0)
#else
#define STAMP(p, i) \
  do {              \
  } while (0)
#define STAMP_CLK(p, i) \
  do {                  \
  } while (0)
#define STAMP_FLUSH(p, lo, hi) \
  do {                         \
  } while (0)
#define STAMP_CLEAR(lo, hi) \
  do {                      \
  } while (0)
__device__ inline void stamp_nc(int) {}
#define RSECT_DECL(d)
#define RSECT(k) \
  do {           \
  } while (0)
#define RSECT_END(iters) \
  do {                   \
  } while (0)
#endif

// The solvers hold more uniform values (sizes, divisors, LDS offsets,
// pointers) than the scalar register file takes; the spilled ones come back
// lane by lane (v_readlane) all over the solver.  A value passed through
// vgpr() is kept in a vector register instead (LDS addresses and the
// divisions' multiplies take vector operands anyway).
__device__ inline int vgpr(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The plan with its divisors in vector registers (see vgpr).
__device__ inline Plan solver_plan(Plan q) {
  auto keep = [](FastDiv &f) {
    f.m = (uint32_t)vgpr((int)f.m);
    f.sh = (uint32_t)vgpr((int)f.sh);
  };
  keep(q.fE);
  keep(q.fG);
  keep(q.fGP);
  keep(q.fP);
  keep(q.fI);
  keep(q.fPN);
  keep(q.fCap);
  keep(q.fN);
  keep(q.fMI);
  return q;
}

typedef const __attribute__((address_space(4))) Plan KernargPlan;

// The plan's fields for one role of the one-launch kernel, loaded after the
// role's branch from an opaque pointer to the kernel arguments: otherwise
// the compiler loads every field either role uses at the kernel's entry and
// keeps them all live, and the solver's scalar registers spill.  (The host
// pass only type-checks this function.)
__device__ inline Plan role_plan(const Plan &p) {
#if __HIP_DEVICE_COMPILE__
  (void)p;
  KernargPlan *k = (KernargPlan *)(__builtin_amdgcn_kernarg_segment_ptr());
  asm volatile("" : "+s"(k));
  return *k;
#else
  return p;
#endif
}

// Scratch words of the histogram reduction (hist_from_partials, load_fast)
// for up to 1024 threads: max(E, 4 * threads).
__host__ __device__ inline int hist_scratch_words(const Plan &p) { return imax(p.E, 4 * 1024); }

// LDS layout of the one-workgroup-per-domain solver, in int32 words.
struct DomainLds {
  int ck, fdt, hs, rows, mask, slots, used, L, e_of, U, misc, qcol, ord, ccol, wx, words;
};

// The general cost model's per-domain tables in LDS (see domain_lds).
struct GenCost {
  const uint16_t *ord;
  const int *ccol;
  const int64_t *wx;
};

__host__ __device__ inline DomainLds domain_lds(const Plan &p) {
  DomainLds l;
  int o = 0;
  l.ck = o;    // uint64 stage-1 candidate keys, then the refinement's words per expert or (lane forms) instance
  o += 2 * (p.lanes ? imax(p.E, p.I) : p.E);
  l.fdt = o;   o += 2 * (p.M + 1);           // divisors 1..M
  l.hs = o;    o += p.E;                     // row self of Omega (histogram)
  l.rows = o;  o += p.G * p.E;               // Omega rows of the domain's sources
  l.mask = o;  o += p.E * p.MW;              // per expert: domains hosting it
  l.slots = o; o += p.G * imax(p.Neff, 1);   // replica slots of the domain's ranks
  l.used = o;  o += p.G;
  l.L = o;     o += p.G;                     // rank loads
  l.e_of = o;  o += p.I;                     // expert of each instance (-1 empty)
  l.U = o;     o += p.I;                     // instance loads
  o = (o + 3) & ~3;
  l.misc = o;  o += 64;
  l.qcol = o;                                // q[s][e][r] of the domain's instances
  o += imax(p.I * p.QS, imax(p.E + 2 + p.E * p.RW + 64 + p.nent_cap, hist_scratch_words(p)));
  // general cost model: per (busiest, target) pair of the domain's ranks the
  // sources in (c(s,rt) - c(s,rb), s) order (16-bit), the costs to the
  // domain's ranks, ||W_e||
  l.ord = o;   o += p.general ? (p.G * p.G * p.R + 1) / 2 : 0;
  l.ccol = o;  o += p.general ? p.G * p.R : 0;
  o = (o + 1) & ~1;
  l.wx = o;    o += p.general ? 2 * p.E : 0;
  l.words = o;
  return l;
}

// LDS layout of the single-workgroup solver: every domain's state at once.
struct SingleLds {
  int ck, em, fdt, hs, cnt, dfree, mask, bm, sendl, wt, repl, slots, used, L, e_of, U, misc, om, qcol, words;
};

__host__ __device__ inline SingleLds single_lds(const Plan &p) {
  SingleLds l;
  int o = 0;
  l.ck = o;    o += 2 * p.M * ((p.E + 15) & ~15);   // uint64 stage-1 candidate keys per domain (stride E rounded to 16)
  l.em = o;    // uint64 per domain and expert: local ranks hosting it (LDS form), or per instance its
               // expert's positions (lane forms)
  o += 2 * p.M * (p.lanes ? imax(p.E, p.I) : p.E);
  l.fdt = o;   o += 2 * (p.M + 1);            // divisors 1..M
  l.hs = o;    o += p.E;                      // histogram of local_topk
  l.cnt = o;   o += p.M;                      // candidates per domain
  l.dfree = o; o += p.M;                      // 1: a rank of the domain has a free slot
  l.mask = o;  o += p.E * p.MW;               // per expert: hosting domains
  l.bm = o;    o += p.E * p.RW;               // per expert: ranks in this rank's instance list
  l.sendl = o; o += p.R;                      // send counts being summed
  l.wt = o;    o += imax(32, (p.E + 63) / 64);   // per-wave totals of a scan (and their sum), or per 64 experts
  l.repl = o;  o += p.M * imax(p.cap1, 1);    // stage-1 replicas per domain
  l.slots = o; o += p.R * imax(p.Neff, 1);    // replica slots of every rank
  l.used = o;  o += p.R;
  l.L = o;     o += p.R;                      // rank loads
  l.e_of = o;  o += p.M * p.I;                // expert of each instance
  l.U = o;     o += p.M * p.I;                // instance loads
  o = (o + 3) & ~3;
  l.misc = o;  o += 64;
  l.om = o;                                   // Omega' [R][E], then list scratch
  o += p.R * p.E;
  o = (o + 3) & ~3;
  l.qcol = o;                                 // partial-sum scratch, then q columns
  o += imax(p.M * p.I * p.QS, hist_scratch_words(p));
  l.words = o;
  return l;
}

// LDS layout of a chunk workgroup of the single-launch plan (nt threads).
struct ChunkLds {
  int wc, run, ptr, ent, gs, so, flag, words;
};

__host__ __device__ inline ChunkLds chunk_lds(const Plan &p, int nt) {
  ChunkLds l;
  int o = 0;
  l.wc = o;   o += (nt >> 6) * p.E;          // per-wave counts, then offsets in the block
  l.run = o;  o += p.E;                      // offset of the block per expert
  l.ptr = o;  o += p.E + 1;                  // instance list: first entry per expert
  o = (o + 1) & ~1;
  l.ent = o;  o += 2 * p.nent_cap;           //   (cumulative share, instance rank) per entry
  l.gs = o;   o += imax(nt, p.E);            // partial sums of the chunk's offsets, then counts per rank
  l.so = o;   o += p.R + 1 + (nt >> 6) + 1;  // send offsets and their scan scratch
  l.flag = o; o += 4;
  l.words = o;
  return l;
}

// Global -> LDS copy by the whole workgroup, four 16-byte loads in flight
// per thread when source, destination and length allow.
__device__ __forceinline__ void copy_to_lds(int *dst, const int *src, int n) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0 && (n & 3) == 0) {
    const int n4 = n >> 2;
    const int4 *s4 = reinterpret_cast<const int4 *>(src);
    int4 *d4 = reinterpret_cast<int4 *>(dst);
    int base = tid;
    for (; base + 3 * nt < n4; base += 4 * nt) {
      const int4 a = s4[base], b = s4[base + nt], c = s4[base + 2 * nt], d = s4[base + 3 * nt];
      d4[base] = a;
      d4[base + nt] = b;
      d4[base + 2 * nt] = c;
      d4[base + 3 * nt] = d;
    }
    for (; base < n4; base += nt) d4[base] = s4[base];
  } else {
    int base = tid;
    for (; base + 3 * nt < n; base += 4 * nt) {
      const int a = src[base], b = src[base + nt], c = src[base + 2 * nt], d = src[base + 3 * nt];
      dst[base] = a;
      dst[base + nt] = b;
      dst[base + 2 * nt] = c;
      dst[base + 3 * nt] = d;
    }
    for (; base < n; base += nt) dst[base] = src[base];
  }
}

// make_fastdiv on the device without a 64-bit integer division: for
// d < 2^21 the quotient 2^(31+l) / d is formed in double precision and
// corrected to the exact floor with integer arithmetic.
__device__ inline FastDiv make_fastdiv_dev(uint32_t d) {
  if (d >= (1u << 21)) return make_fastdiv(d);
  const uint32_t l = d <= 1 ? 0u : 32u - (uint32_t)__clz(d - 1);
  const uint64_t x = 1ull << (31 + l);
  uint64_t q = (uint64_t)((double)x / (double)d);
  int64_t r = (int64_t)(x - q * d);
  while (r < 0) {
    --q;
    r += d;
  }
  while (r >= (int64_t)d) {
    ++q;
    r -= d;
  }
  FastDiv f;
  f.m = (uint32_t)(q + (r != 0));
  f.sh = 31 + l;
  return f;
}

// x / d with one high multiply (x < 2^31): m < 2^32 and sh >= 32 except for
// d = 1, where the quotient is x.
__device__ inline uint32_t fdiv_hi(uint32_t x, FastDiv f) {
  const uint32_t hi = __umulhi(x, f.m) >> ((f.sh - 32u) & 31u);   // computed for every lane: a select, no branch
  return f.sh >= 32 ? hi : x;
}

// Histogram of local_topk (row self of Omega) as the sum of the histogram
// blocks' partials: thread (e, g) sums its share of the blocks with eight
// loads in flight; scratch needs hist_scratch_words(p) = max(E, 4 * blockDim)
// words (the int4 path keeps blockDim int4 partial sums).
__device__ __forceinline__ void hist_from_partials(const Plan &p, int *hs, int *scratch) {
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E, nb = p.nb;
  if ((E & 3) == 0) {
    // thread (e4, g): four experts, a share of the blocks, 16-byte loads
    const int E4 = E >> 2;
    const int groups = imax(1, nt / E4);
    const int per = (nb + groups - 1) / groups;
    const int4 *part4 = reinterpret_cast<const int4 *>(p.partials);
    int4 *scr4 = reinterpret_cast<int4 *>(scratch);
    for (int t = tid; t < groups * E4; t += nt) {
      const int g = t / E4, e4 = t - g * E4;
      const int b0 = g * per, b1 = imin(nb, b0 + per);
      int4 run = make_int4(0, 0, 0, 0);
      for (int b = b0; b < b1; b += 8) {
        int4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = b + u < b1 ? part4[(int64_t)(b + u) * E4 + e4] : make_int4(0, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          run.x += v[u].x;
          run.y += v[u].y;
          run.z += v[u].z;
          run.w += v[u].w;
        }
      }
      scr4[t] = run;
    }
    lds_barrier();
    for (int e = tid; e < E; e += nt) {
      int sum = 0;
      for (int g = 0; g < groups; ++g) sum += scratch[g * E + e];
      hs[e] = sum;
    }
    lds_barrier();
    return;
  }
  const int groups = imax(1, nt / E);
  const int per = (nb + groups - 1) / groups;
  for (int t = tid; t < groups * E; t += nt) {
    const int g = (int)fdiv((uint32_t)t, p.fE), e = t - g * E;
    const int b0 = g * per, b1 = imin(nb, b0 + per);
    int run = 0;
    for (int b = b0; b < b1; b += 8) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = b + u < b1 ? p.partials[(int64_t)(b + u) * E + e] : 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) run += v[u];
    }
    scratch[t] = run;
  }
  lds_barrier();
  for (int e = tid; e < E; e += nt) {
    int sum = 0;
    for (int g = 0; g < groups; ++g) sum += scratch[g * E + e];
    hs[e] = sum;
  }
  lds_barrier();
}

// Exclusive per-expert offset of every histogram block, for the reroute
// (offset workgroup h of n_helpers handles kOffsetExperts experts at a time),
// and each expert's count over all blocks (htot, the histogram of
// local_topk), announced by one increment of the helpers' counter as soon
// as the totals are written: the offsets follow in a second pass (only the
// next launch reads them).  A group of kOffsetExperts lanes sums one share
// of the blocks, eight loads in flight.  scratch: one word per thread for
// each expert group of this workgroup (one group when n_helpers covers E, as
// the host sets it).
__device__ __forceinline__ void block_offsets(const Plan &p, int h, int *scratch) {
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E, nb = p.nb;
  const int ng = nt / kOffsetExperts;
  const int el = tid % kOffsetExperts, g = tid / kOffsetExperts;
  const int per = (nb + ng - 1) / ng;
  const int b0 = g * per, b1 = imin(nb, b0 + per);
  const int gstride = p.n_helpers * kOffsetExperts;
  // pass 1: each group's sum over its blocks, per expert
  int grp = 0;
  for (int e0 = h * kOffsetExperts; e0 < E; e0 += gstride, ++grp) {
    const int e = e0 + el;
    int run = 0;
    if (e < E) {
      for (int b = b0; b < b1; b += 8) {
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = b + u < b1 ? p.partials[(int64_t)(b + u) * E + e] : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) run += v[u];
      }
    }
    scratch[grp * nt + tid] = run;
  }
  __syncthreads();
  // the totals (the expert's count over every block), then the announcement
  grp = 0;
  for (int e0 = h * kOffsetExperts; e0 < E; e0 += gstride, ++grp) {
    const int e = e0 + el;
    if (g == ng - 1 && e < E) {
      int tot = 0;
#pragma unroll 8
      for (int g2 = 0; g2 < ng; ++g2) tot += scratch[grp * nt + g2 * kOffsetExperts + el];
      p.htot[e] = tot;
    }
  }
  // publish: every total written before the count of finished helpers
  drain_then_barrier();
  if (tid == 0) __hip_atomic_fetch_add(&p.ctrl[kCtrlHelpers], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  // pass 2: the blocks' exclusive offsets
  grp = 0;
  for (int e0 = h * kOffsetExperts; e0 < E; e0 += gstride, ++grp) {
    const int e = e0 + el;
    if (e >= E) continue;
    int base = 0;
    for (int g2 = 0; g2 < g; ++g2) base += scratch[grp * nt + g2 * kOffsetExperts + el];
    for (int b = b0; b < b1; b += 8) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = b + u < b1 ? p.partials[(int64_t)(b + u) * E + e] : 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (b + u < b1) p.offsets[(int64_t)(b + u) * E + e] = base;
        base += v[u];
      }
    }
  }
}

// The histogram of local_topk (row self of Omega) for the solvers of the
// three-kernel plan: the offset helpers' totals once all of them have published, else
// the sum of the blocks' counts made here.  The helpers normally finish in
// a few microseconds beside the solver workgroups; the wait is bounded by
// kHelperSpin polls (~0.2 ms), not by the hang guard, so a dispatch whose
// helpers start late costs little.  flag: one LDS word.
__device__ __forceinline__ void row_self(const Plan &p, int *hs, int *scratch, int *flag) {
  if (threadIdx.x == 0) {
    uint32_t it = 0;
    int ok = 1;
    while (__hip_atomic_load(&p.ctrl[kCtrlHelpers], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
           (uint32_t)p.n_helpers) {
      if (++it > kHelperSpin) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *flag = ok;
  }
  __syncthreads();
  if (*flag) {
    for (int e = threadIdx.x; e < p.E; e += blockDim.x) hs[e] = p.htot[e];
    lds_barrier();
  } else {
    hist_from_partials(p, hs, scratch);
  }
}

// Exact-range check: the total load fits int32 and 4 S total c + c W < 2^62
// (c = max(c_intra, c_inter, 1)), so every benefit and cost change is exact.
__device__ inline bool out_of_range_cw(const Plan &p, uint64_t total, uint64_t cmax, uint64_t wmax) {
  const uint64_t lim = 1ull << 62;
  const uint64_t cm = cmax > 1 ? cmax : 1;
  if (total > 0x7FFFFFFFull) return true;
  // 4 S total cm and cm W with overflow checks (every factor is nonnegative)
  uint64_t tok = 0, rep = 0;
  if (__builtin_mul_overflow((uint64_t)p.S, 4ull * total, &tok)) return true;
  if (__builtin_mul_overflow(tok, cm, &tok)) return true;
  if (__builtin_mul_overflow(wmax, cm, &rep)) return true;
  if (tok >= lim || rep >= lim) return true;
  return tok + rep >= lim;
}

// The same check for the two-level model, whose c and W the host knows: with
// k = 4 S c, 4 S total c + c W >= 2^62 holds exactly when c W >= 2^62 or
// total >= ceil((2^62 - c W) / k), the threshold the host stores in tot_max
// (0 when c W >= 2^62); two compares instead of overflow-checked products.
__device__ inline bool out_of_range(const Plan &p, uint64_t total) {
  return total > 0x7FFFFFFFull || total >= p.tot_max;
}

// Grid barrier of the per-domain solver workgroups: all of them are
// resident (at most kMaxSolveGroups), and the wait is bounded so the kernel
// always exits.
__device__ __forceinline__ bool grid_barrier(uint32_t *count, uint32_t groups, uint32_t spin_limit, int *flag) {
  drain_then_barrier();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    int ok = 0;
    for (uint32_t it = 0; it < spin_limit; ++it) {
      if (it > 0) __builtin_amdgcn_s_sleep(1);
      if (__hip_atomic_load(count, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) >= groups) {
        ok = 1;
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *flag = ok;
  }
  __syncthreads();
  return *flag != 0;
}

// ---------------------------------------------------------------- histogram

// K ids per lane from base on (64 K ids a wave; base a multiple of 64 ids), -1
// from `end` on: W = min(K, 4) consecutive ids at a time, one load of 4 W
// bytes where the array is 16-byte aligned (vec); element W j + c of lane l is
// id (j * 64 + l) * W + c.  Last: nothing reads the ids after this kernel
// (non-temporal loads; see hist_kernel).
template <int K, bool Last>
__device__ inline void load_ids(const int32_t *ids, int64_t base, int64_t end, bool vec, int (&v)[K]) {
  constexpr int W = K < 4 ? K : 4;
  typedef int words __attribute__((ext_vector_type(W)));
#pragma unroll
  for (int j = 0; j < K / W; ++j) {
    const int64_t idx = base + (int64_t)(j * 64 + lane_id()) * W;
    if (vec && idx + W <= end) {
      const words *at = reinterpret_cast<const words *>(ids + idx);
      const words x = Last ? __builtin_nontemporal_load(at) : *at;
#pragma unroll
      for (int c = 0; c < W; ++c) v[W * j + c] = x[c];
    } else {
#pragma unroll
      for (int c = 0; c < W; ++c) v[W * j + c] = idx + c < end ? ids[idx + c] : -1;
    }
  }
}

// One contiguous chunk per block, in tiles of 64 K ids per wave, counted into
// one LDS row, one atomic per id, the next tile's loads in flight meanwhile.
// Bound: HBM from some 16 M ids on (2^26 ids, E = 128: 43 us on inputs that come
// round alone, 53 on others, 6.2 and 5.1 TB/s), the launch below.  A row per wave, summed at the end, costs more than the atomics
// that meet in one (2^24 ids, E = 128: 19.2 us, 17.0; 2^17 ids, E = 1024: 4.2,
// 3.2).  Plain loads keep the ids in the caches for the reroute, whose own are
// non-temporal (plans of 2^24 ids, inputs that alternate: 53 us, 61 with
// non-temporal loads in both).  Stream (more than kStreamIds ids, 64 MiB):
// non-temporal here too.  Such plans one after another take 176 us for 2^26
// ids, 167 with plain loads, but plain loads suffer where the caches are full
// of other stores: after 268 MB of them the kernel takes 95 us, not 54.
template <int K, bool Stream>
__global__ __launch_bounds__(1024, 8) void hist_kernel(Plan p) {
  extern __shared__ int smem_h[];
  constexpr int W = K < 4 ? K : 4;
  const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, lane = tid & 63, wave = tid >> 6, E = p.E;
  const int b = blockIdx.x;
  int *h = smem_h;
  const int64_t lo = (int64_t)b * p.chunk;
  const int64_t hi = lo + p.chunk < p.n ? lo + p.chunk : p.n;
  const bool vec = (reinterpret_cast<uintptr_t>(p.topk) & 15) == 0;
  const int64_t tile = (int64_t)nw * 64 * K, wofs = (int64_t)wave * 64 * K;
  int nx[K];
  load_ids<K, Stream>(p.topk, lo + wofs, hi, vec, nx);
  for (int e = tid; e < E; e += nt) h[e] = 0;
  __syncthreads();
  int bad = 0;
  for (int64_t base = lo + wofs; base < hi; base += tile) {
    int ev[K];
#pragma unroll
    for (int i = 0; i < K; ++i) ev[i] = nx[i];
    if (base + tile < hi) load_ids<K, Stream>(p.topk, base + tile, hi, vec, nx);
    // ids of the wave's piece that exist
    const int lim = (int)(hi - base < 64 * K ? hi - base : 64 * K);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const bool valid = (unsigned)ev[i] < (unsigned)E;   // (-1 past the end)
      bad |= !valid && (i / W * 64 + lane) * W + i % W < lim ? 1 : 0;
      if (valid) atomicAdd(&h[ev[i]], 1);
    }
  }
  bad = __syncthreads_or(bad);
  for (int e = tid; e < E; e += nt) p.partials[(int64_t)b * E + e] = h[e];
  if (tid == 0) p.blk_err[b] = bad;
}

// ---------------------------------------------------------------- solver steps

// Routing construction (Section 4.3) for NI instances, instance i of domain
// dom_of(i) holding expert e_of[i] (-1 = empty).  The unique instance of e
// inside dom(s) takes all of omega[s][e]; sources of a domain without an
// instance of e split omega[s][e] evenly over every instance of e (one per
// hosting domain, so an instance's position in ascending rank order is the
// number of hosting domains below its own), the lowest positions taking the
// remainder; sources of another domain that hosts e send it nothing.  The
// case is decided once per source domain.  Thread t handles source domains
// [c * M / chunks, (c + 1) * M / chunks) of instance t % NI, c = t / NI
// (chunks divides M); omega[s][e] of instance i is src_of(i, e)[s * stride];
// qcol[i * QS + s] = q[s][e][r_i] (may be the source itself: every value is
// read before it is written); U[i] += sum_s q (U must be zero on entry).
struct RouteCase {
  FastDiv fn;
  int n, below, keep, take;
};

template <int B>
__device__ inline int route_batch(const int *src, int stride, int *dst, const RouteCase &rc) {
  int w[B];
#pragma unroll
  for (int u = 0; u < B; ++u) w[u] = src[u * stride];
  int sum = 0;
#pragma unroll
  for (int u = 0; u < B; ++u) {
    const int qq = (int)fdiv_hi((uint32_t)w[u], rc.fn);
    const int split = qq + (rc.below < w[u] - qq * rc.n ? 1 : 0);
    const int q = (w[u] & rc.keep) + (split & rc.take);   // local: w; hosting domain: 0; else the split
    dst[u] = q;
    sum += q;
  }
  return sum;
}

// q[s][e][r] of an instance of e in domain d for one source s of domain ds,
// w = omega[s][e]: the routing rule of route_instances for a single source
// (the whole load to the instance in the source's own domain, nothing when
// another instance sits there, else the even split over the hosting
// domains, the remainder to the lowest ones).
__device__ inline int route_q(const Plan &p, int d, int e, int w, int ds, const uint32_t *mask, const FastDiv *fdt) {
  if (ds == d) return w;                                   // the instance inside dom(s)
  const uint32_t *me = mask + e * p.MW;
  if ((me[ds >> 5] >> (ds & 31)) & 1u) return 0;           // dom(s) hosts e itself
  int n = 0, below = 0;
  for (int wd = 0; wd < p.MW; ++wd) {
    const uint32_t bits = me[wd];
    n += __popc(bits);
    const int lo = wd * 32;
    if (d >= lo + 32) below += __popc(bits);
    else if (d > lo) below += __popc(bits & ((1u << (d - lo)) - 1u));
  }
  const FastDiv fn = fdt[n];
  const int qq = (int)fdiv_hi((uint32_t)w, fn);
  return qq + (below < w - qq * n ? 1 : 0);
}

__device__ inline int route_self_q(const Plan &p, int d, int e, int w, const uint32_t *mask, const FastDiv *fdt) {
  return route_q(p, d, e, w, (int)fdiv((uint32_t)p.self, p.fG), mask, fdt);
}

// Receive counts: recv[s] = sum over the instances on rank self (instance
// indices i0 .. i0 + PN - 1, expert e_of[i], column qcol + i * QS) of
// q[s][e][self].  With full, every source's q of those instances is in
// qcol (and reflects the refinement); otherwise the routing rule gives it
// from omega(s, e).
// One thread per (source, instance); acc: R words of LDS scratch.
template <class OmegaOf>
__device__ __forceinline__ void write_recv_counts(const Plan &p, int i0, const int *e_of, const int *qcol, bool full,
                                  const uint32_t *mask, const FastDiv *fdt, OmegaOf omega_of, int *acc) {
  const int tid = threadIdx.x, nt = blockDim.x, R = p.R, PN = p.PN;
  const int ds = (int)fdiv((uint32_t)p.self, p.fG);
  for (int s = tid; s < R; s += nt) acc[s] = 0;
  lds_barrier();
  for (int x = tid; x < R * PN; x += nt) {
    const int s = (int)fdiv((uint32_t)x, p.fPN), i = i0 + x - s * PN, e = e_of[i];
    if (e < 0) continue;
    const int q = full ? qcol[i * p.QS + s]
                       : route_q(p, ds, e, omega_of(s, e), (int)fdiv((uint32_t)s, p.fG), mask, fdt);
    if (q) atomicAdd(&acc[s], q);
  }
  lds_barrier();
  for (int s = tid; s < R; s += nt) p.recv_out[s] = acc[s];
}

// full(d): whether every source's q is needed for domain d's instances.  A
// domain whose refinement cannot move anything (no free slot) only needs
// q[self] (send counts and this rank's instance list read nothing else, and
// instance loads feed the refinement only): the chunk holding dom(self)
// writes that one value, then calls on_self(i, d, e, q); the other sources
// of the column are left unset.
template <class SrcOf, class DomOf, class Full, class OnSelf>
__device__ __forceinline__ void route_instances(const Plan &p, int NI, FastDiv fNI, int chunks, const int *e_of,
                                const uint32_t *mask, const FastDiv *fdt, int *qcol, int *U, SrcOf src_of,
                                int stride, DomOf dom_of, Full full, OnSelf on_self) {
  const int tid = threadIdx.x, nt = blockDim.x, G = p.G;
  const int dpc = p.M / chunks;
  const int c_self = (int)fdiv((uint32_t)p.self, p.fG) / dpc;
  for (int t = tid; t < NI * chunks; t += nt) {
    const int c = (int)fdiv((uint32_t)t, fNI), i = t - c * NI;
    const int e = e_of[i];
    const int ds0 = c * dpc, ds1 = ds0 + dpc;
    int *row = qcol + i * p.QS;
    const int d = dom_of(i);
    if (!full(d)) {
      if (c == c_self) {
        const int q = e < 0 ? 0 : route_self_q(p, d, e, src_of(i, e)[p.self * stride], mask, fdt);
        row[p.self] = q;
        on_self(i, d, e, q);
      }
      continue;
    }
    if (e < 0) {
      for (int s = ds0 * G; s < ds1 * G; ++s) row[s] = 0;
      continue;
    }
    const uint32_t *me = mask + e * p.MW;
    RouteCase rc;
    rc.n = 0;
    rc.below = 0;
    for (int wd = 0; wd < p.MW; ++wd) {
      const uint32_t bits = me[wd];
      rc.n += __popc(bits);
      const int lo = wd * 32;
      if (d >= lo + 32) rc.below += __popc(bits);
      else if (d > lo) rc.below += __popc(bits & ((1u << (d - lo)) - 1u));
    }
    rc.fn = fdt[rc.n];
    const int *col = src_of(i, e);
    int usum = 0;
    for (int ds = ds0; ds < ds1; ++ds) {
      const bool local = ds == d;
      const bool zero = !local && ((me[ds >> 5] >> (ds & 31)) & 1u);
      rc.keep = local ? -1 : 0;
      rc.take = (local || zero) ? 0 : -1;
      const int *src = col + ds * G * stride;
      int *dst = row + ds * G;
      int j = 0;
      for (; j + 8 <= G; j += 8) usum += route_batch<8>(src + j * stride, stride, dst + j, rc);
      for (; j + 4 <= G; j += 4) usum += route_batch<4>(src + j * stride, stride, dst + j, rc);
      for (; j < G; ++j) usum += route_batch<1>(src + j * stride, stride, dst + j, rc);
    }
    if (usum) atomicAdd(&U[i], usum);
  }
}

// Divisors 1..M (hosting-domain counts) for the routing's even splits,
// built once per workgroup into fdt[0..M].
__device__ inline void build_divisors(int M, FastDiv *fdt) {
  for (int n = threadIdx.x; n <= M; n += blockDim.x) fdt[n] = make_fastdiv_dev((uint32_t)(n > 0 ? n : 1));
}

// Instance index of expert e on local rank j of domain d, or -1.
__device__ inline int instance_of(const Plan &p, int d, int j, int e, const int *slots,
                                  const int *used) {
  const int rank = d * p.G + j;
  if ((int)fdiv((uint32_t)e, p.fP) == rank) return j * p.PN + (e - rank * p.P);
  const int u = used[j];
  for (int t = 0; t < u; ++t)
    if (slots[j * p.Neff + t] == e) return j * p.PN + p.P + t;
  return -1;
}

// Forms of the refinement loop: the lane forms where an expert's positions
// in the domain fit one 64-bit word (refine_in_lanes), scoring (instance,
// target) pairs (kRefinePairs) or instances (kRefineLanes); else the LDS
// form.  A kernel carries one form's code.
constexpr int kRefinePairs = 1, kRefineLds = 2, kRefineLanes = 3;
__host__ __device__ inline bool refine_in_lanes(int G, int PN) {
  return G >= 2 && ((G <= 8 && PN <= 254) || (G <= 16 && PN <= 14));
}
__host__ __device__ inline bool refine_in_pairs(int G, int PN) { return G <= 8 && PN <= 16; }
// bits of one rank's field in an expert's position word
__host__ __device__ inline int position_bits(int G) { return G <= 8 ? 8 : 4; }

// Maximum / minimum over groups of GM = 8 or 16 lanes, left in every lane of
// the group (DPP: lane pairs, quads, mirrored halves of a row).
template <int GM>
__device__ inline int group_max_i32(int v) {
  v = imax(v, (int)dpp_mov<0xB1>((uint32_t)v));
  v = imax(v, (int)dpp_mov<0x4E>((uint32_t)v));
  v = imax(v, (int)dpp_mov<0x141>((uint32_t)v));
  if (GM == 16) v = imax(v, (int)dpp_mov<0x140>((uint32_t)v));
  return v;
}
template <int GM>
__device__ inline int group_min_i32(int v) {
  v = imin(v, (int)dpp_mov<0xB1>((uint32_t)v));
  v = imin(v, (int)dpp_mov<0x4E>((uint32_t)v));
  v = imin(v, (int)dpp_mov<0x141>((uint32_t)v));
  if (GM == 16) v = imin(v, (int)dpp_mov<0x140>((uint32_t)v));
  return v;
}
// Wave-wide maximum / minimum as a scalar: a row's, then across the rows by
// broadcasts of lanes 15 and 31, read from lane 63.
__device__ inline int wave_max_i32(int v) {
  v = group_max_i32<16>(v);
  v = imax(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x142, 0xA, 0xF, false));
  v = imax(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x143, 0xC, 0xF, false));
  return readlane_i32(v, 63);
}
__device__ inline uint32_t wave_min_u32(uint32_t v) {
  return ~(uint32_t)0 ^ ((uint32_t)wave_max_i32((int)(~v ^ 0x80000000u)) ^ 0x80000000u);
}

// Lane forms of the refinement loop below (two-level cost, refine_in_lanes).
// Lane l keeps the load and used slots of local rank l mod GM (GM = 8 or 16);
// the instances' experts, loads and q columns stay in LDS.  pi[a] (instance
// a of expert e) holds for each local rank a field of position_bits(G) bits:
// e's position on that rank + 1, 0 where the rank does not hold e, so a
// target's instance needs no search.  At the start every expert has one
// instance in the domain at most; the caller sets pi for that.  Same moves in
// the same order as the LDS form.  A move's candidates are scored
//   - Pairs = 1 or 2 (at most 8 or 16 instances per rank with GM = 8, 4 or 8
//     with GM = 16): one lane per (instance of the busiest rank, target rank),
//     one or two each;
//   - else one lane per instance, against its lightest receivers only (its
//     other targets cannot win, see refine_domain): the lightest ranks with
//     a free slot, the same for every instance (usually one), and the ranks
//     hosting its expert that are no heavier.
// Plain: the usual shape, R <= 64 with an intra-domain cost; its move is
// straight-line code.
//
// Bound: one wave's dependent chain.  The next busiest rank is found while
// the q columns are on their way; scores take vector registers only, and the
// scalar unit sees a move's two or more wave-wide minima.  Layers of Mixtral's
// shape (18 moves on one wave) 32.4 -> 23.8 us, DeepSeek-V3's with 4 slots
// (75 over 4 waves) 58.4 -> 45.0, E = 640 on one node (35 moves, 82 instances
// a rank: one lane per instance; pairs took 90 us there, and lanes 62.6 on
// the 12 instances a rank of DeepSeek-V3's) 59.4 -> 45.9.  Pairs with sixteen
// ranks a node matter where loads are small and ties many: EP 64, E = 192, one
// slot, 147 tokens (71 moves) 47.5 us a plan with a lane per instance, 32.5;
// EP 32, E = 128, three slots, 4096 tokens 109 and 83.
template <int GM, int Pairs, bool Plain>
__device__ __forceinline__ uint32_t refine_domain_lanes(const Plan &p, int d, int *e_of, int *U, uint64_t *pi,
                                                        int *qcol, int *slots, int *used, int *Lr, uint32_t *flags) {
  constexpr int IR = 64 / GM;   // Pairs: instances of a round
  constexpr int BW = GM == 8 ? 8 : 4;
  constexpr uint32_t FM = (1u << BW) - 1u;
  const int lane = lane_id();
  const int G = p.G, PN = p.PN, R = p.R, P = p.P, Neff = p.Neff, QS = p.QS;
  {
    const bool free_slot = lane < G && used[lane] < Neff;
    if (__ballot(free_slot) == 0) return 0;   // (no candidate ever: see refine_domain)
  }
  const int r0 = d * G;
  const bool two_level = Plain || p.cI > 0;
  const int64_t tokc = 2 * p.S * (int64_t)p.cI;
  const int64_t repI = (int64_t)p.cI * p.W, repX = (int64_t)p.cX * p.W;
  const int e_lo = d * G * P, e_n = G * P;   // experts whose main lies in the domain
  const int j = vgpr(lane & (GM - 1)), c = vgpr(lane / GM);
  const bool in_rank = j < G;
  const int jq = in_rank ? j : 0;
  const int fsh = (j & (GM / 2 - 1)) * BW;   // this lane's rank's field in its half of a position word
  const bool fhi = j >= GM / 2;
  // rank loads: each group of lanes sums its share of a rank's instances
  int lj = 0;
  if (in_rank)
    for (int pos = c; pos < PN; pos += 64 / GM) lj += U[j * PN + pos];
#pragma unroll
  for (int o = GM; o < 64; o *= 2) lj += __shfl_xor(lj, o);
  if (!in_rank) lj = -1;   // never the busiest, never a receiver
  int uj = in_rank ? used[j] : Neff;
  // the busiest rank: the largest L, lowest index on ties
  int Lrb = group_max_i32<GM>(lj);
  int rbj = group_min_i32<GM>(lj == Lrb ? j : GM);
  auto cost_of = [&](int mx, int pos, int e) {
    const int64_t rep = (unsigned)(e - e_lo) < (unsigned)e_n ? repI : repX;
    return tokc * (int64_t)mx + (pos ? 0 : rep);
  };
  // moved from the busiest rank's own sources less moved from the target's
  // own, of dl assignments (the cost change follows from it)
  auto own_moves = [&](int dl, int u, int qt, int qrb) {
    const int m_rt = imin(dl, qt), rest = dl - m_rt;
    return two_level ? rest - imin(rest, u - qt - qrb) - m_rt : 0;
  };
  uint32_t it = 0;
  RSECT_DECL(d);
  for (;; ++it) {
    const int gap = Lrb - lj;
    const bool low = gap >= 2 && j != rbj, room = uj < Neff;
    const int rbs = readlane_i32(rbj, 0);
    const int a0 = rbs * PN;
    // ---- this lane's best candidate: delta (0: none), target load, what its
    // cost change follows from (own_moves, position on the target, expert);
    // !Pairs: target, instance
    int bd = 0, bl = lj, bx = 0, be = 0, bpos = 0, bt = 0, ba = 0;
    if constexpr (Pairs > 0) {
      // (the words of both instances of a lane are on their way together)
      int es[Pairs], us[Pairs], qb[Pairs], qt[Pairs];
      uint64_t ws[Pairs];
#pragma unroll
      for (int i = 0; i < Pairs; ++i) {
        const int a = a0 + (c + IR * i < PN ? c + IR * i : 0);
        const int *qa = qcol + a * QS + r0;
        es[i] = e_of[a];
        us[i] = U[a];
        ws[i] = pi[a];
        qb[i] = qa[rbs];
        qt[i] = qa[jq];
      }
#pragma unroll
      for (int i = 0; i < Pairs; ++i) {
        const int pos = (int)(((fhi ? (uint32_t)(ws[i] >> 32) : (uint32_t)ws[i]) >> fsh) & FM);
        const bool on = c + IR * i < PN && us[i] > 0 && low && (room || pos != 0);
        const int sd = on ? imin(us[i], gap >> 1) : 0;
        const int sx = own_moves(sd, us[i], qt[i], qb[i]);
        bool lt = i == 0 || sd > bd;
        if (i > 0) {
          // equal delta (and the same target): the lower cost change, then expert
          const bool tie = sd == bd && sd > 0;
          if (__ballot(tie)) {
            const int64_t cn = cost_of(sx, pos, es[i]), cb = cost_of(bx, bpos, be);
            lt = lt || (tie && (cn < cb || (cn == cb && es[i] < be)));
          }
        }
        bd = lt ? sd : bd;
        bx = lt ? sx : bx;
        be = lt ? es[i] : be;
        bpos = lt ? pos : bpos;
        ba = lt ? i : ba;   // (its round)
      }
    } else {
      const int Lb = readlane_i32(Lrb, 0);
      const int lfv = group_min_i32<GM>(low && room ? lj : INT_MAX);
      const int lf = readlane_i32(lfv, 0);
      constexpr uint32_t ranks = (1u << GM) - 1u;
      const uint32_t tf = (uint32_t)__ballot(low && room && lj == lfv) & ranks;   // lightest with a free slot
      // others no heavier (lanes beyond the ranks hold -1 and no room: neither)
      const uint32_t th = (uint32_t)__ballot(low && (uint32_t)lj <= (uint32_t)lfv) & ranks & ~tf;
      const int t1 = tf ? __ffs(tf) - 1 : 0, dfree = tf ? (Lb - lf) >> 1 : 0;
      auto field = [&](uint64_t w, int t) { return (int)(w >> (BW * t)) & (int)FM; };
      // instance a: expert e, load u, position word w, q[rb], q[t1]
      auto score = [&](int a, int e, int u, uint64_t w, int qrb, int q1, bool on) {
        on = on && u > 0;
        int sd = on ? imin(u, dfree) : 0, sl = lf, st = t1, sp = field(w, t1);
        int sx = own_moves(sd, u, q1, qrb);
        const int *qa = qcol + a * QS + r0;
        for (uint32_t m = tf & (tf - 1u); m; m &= m - 1u) {
          // another rank of the same load: the lower cost change, then index
          const int t = __ffs(m) - 1, qt = qa[t], pos = field(w, t);
          const int mx = own_moves(sd, u, qt, qrb);
          if (cost_of(mx, pos, e) < cost_of(sx, sp, e)) {
            st = t;
            sp = pos;
            sx = mx;
          }
        }
        for (uint32_t m = th; m; m &= m - 1u) {
          const int t = __ffs(m) - 1, pos = field(w, t);
          if (__ballot(on && pos != 0) == 0) continue;
          const int Lt = readlane_i32(lj, t), qt = qa[t];
          const int dl = on && pos ? imin(u, (Lb - Lt) >> 1) : 0;
          const int mx = own_moves(dl, u, qt, qrb);
          const int64_t cn = cost_of(mx, pos, e), cb = cost_of(sx, sp, e);
          const bool lt = dl > sd || (dl == sd && dl > 0 &&
                                      (Lt < sl || (Lt == sl && (cn < cb || (cn == cb && t < st)))));
          sd = lt ? dl : sd;
          sl = lt ? Lt : sl;
          st = lt ? t : st;
          sp = lt ? pos : sp;
          sx = lt ? mx : sx;
        }
        // against this lane's earlier instance: delta, load, cost, expert
        bool lt = sd > bd;
        const bool tie = sd == bd && sd > 0;
        if (__ballot(tie)) {
          const int64_t cn = cost_of(sx, sp, e), cb = cost_of(bx, bpos, be);
          lt = lt || (tie && (sl < bl || (sl == bl && (cn < cb || (cn == cb && e < be)))));
        }
        bd = lt ? sd : bd;
        bl = lt ? sl : bl;
        bx = lt ? sx : bx;
        be = lt ? e : be;
        bpos = lt ? sp : bpos;
        bt = lt ? st : bt;
        ba = lt ? a : ba;
      };
      for (int p0 = 0; p0 < PN; p0 += 64) {
        const bool on = p0 + lane < PN;
        const int a = a0 + (on ? p0 + lane : 0);
        const int *qa = qcol + a * QS + r0;
        score(a, e_of[a], U[a], pi[a], qa[rbs], qa[t1], on);
      }
    }
    RSECT(0);
    // ---- the wave's best: delta descending, L[rt], cost change, e, rt
    const int dw = wave_max_i32(bd);
    if (dw == 0 || it >= p.iter_limit) {
      if (dw != 0 && lane == 0) *flags |= TOPOEP_ST_ITER;
      break;
    }
    const uint32_t Lrt = wave_min_u32(bd == dw ? (uint32_t)bl : ~0u);
    const bool in2 = bd == dw && (uint32_t)bl == Lrt;
    uint64_t win = __ballot(in2);
    if (__popcll(win) != 1) {
      const uint64_t kc = (uint64_t)cost_of(bx, bpos, be) ^ (1ull << 63);
      const uint32_t ch = wave_min_u32(in2 ? (uint32_t)(kc >> 32) : ~0u);
      const bool in3 = in2 && (uint32_t)(kc >> 32) == ch;
      const uint32_t cl = wave_min_u32(in3 ? (uint32_t)kc : ~0u);
      const bool in4 = in3 && (uint32_t)kc == cl;
      win = __ballot(in4);
      if (__popcll(win) != 1) {
        // one expert: its lanes (Pairs: one instance against several ranks,
        // ascending) start with the lowest rt
        const uint32_t ew = wave_min_u32(in4 ? (uint32_t)be : ~0u);
        win = __ballot(in4 && (uint32_t)be == ew);
      }
    }
    RSECT(1);
    const int wl = __ffsll((long long)win) - 1;
    const int rtj = Pairs ? wl & (GM - 1) : readlane_i32(bt, wl);
    const int aw = Pairs == 0 ? readlane_i32(ba, wl) : a0 + wl / GM + (Pairs > 1 ? IR * readlane_i32(ba, wl) : 0);
    const int pos = readlane_i32(bpos, wl), ew = readlane_i32(be, wl);
    const uint64_t ww = pi[aw];   // (with the column's words below: one round trip)
    const int at = pos ? pos - 1 : P + readlane_i32(uj, rtj);   // the target's instance: held, or its first free slot
    const int a2 = rtj * PN + at;
    int *qw = qcol + aw * QS, *qb = qcol + a2 * QS;
    const int rt = r0 + rtj, rb = r0 + rbs;
    // ---- the transfer of dw assignments from aw's column to a2's: rt's own
    // first, the other sources ascending, rb's own last (ascending alone
    // when the intra-domain cost is zero); one pass up to 64 sources, lanes
    // >= R on the spare word after them (QS > R)
    const bool one_pass = Plain || R <= 64;
    const int sv = lane < R ? lane : R;
    int av = 0;
    if (one_pass) av = qw[sv];
    const int uw = U[aw];
    // ---- the ranks, and the next busiest one
    lj = j == rbs ? Lrb - dw : (j == rtj ? (int)Lrt + dw : lj);
    uj += j == rtj && pos == 0 ? 1 : 0;
    Lrb = group_max_i32<GM>(lj);
    rbj = group_min_i32<GM>(lj == Lrb ? j : GM);
    RSECT(2);
    if (one_pass) {
      if (lane >= R) av = 0;
      int excl;
      if (two_level) {
        const bool is_rt = lane == rt, is_rb = lane == rb;
        const int other = is_rt || is_rb ? 0 : av, qrt = readlane_i32(av, rt);
        const int incl = wave_incl_scan(other);
        excl = is_rt ? 0 : (is_rb ? qrt + readlane_i32(incl, 63) : qrt + incl - other);
      } else {
        excl = wave_incl_scan(av) - av;
      }
      const int m = imin(imax(dw - excl, 0), av);
      qw[sv] = av - m;
      atomicAdd(&qb[sv], m);
    } else {
      int rest = dw;
      int m_rt = 0;
      if (two_level) {
        m_rt = imin(rest, uniform_i32(qw[rt]));
        rest -= m_rt;
      }
      for (int s0 = 0; s0 < R && rest > 0; s0 += 64) {
        const int s = s0 + lane;
        int v = 0;
        if (s < R && (!two_level || (s != rt && s != rb))) v = qw[s];
        const int incl = wave_incl_scan(v);
        const int m = imin(imax(rest - (incl - v), 0), v);
        if (m) {
          qw[s] = v - m;
          atomicAdd(&qb[s], m);
        }
        const int total = readlane_i32(incl, 63);
        rest -= total < rest ? total : rest;
      }
      if (lane == 0) {
        if (m_rt) {
          atomicSub(&qw[rt], m_rt);
          atomicAdd(&qb[rt], m_rt);
        }
        if (rest > 0) {
          atomicSub(&qw[rb], rest);
          atomicAdd(&qb[rb], rest);
        }
      }
    }
    RSECT(3);
    // ---- the instances: loads; the target's expert and slot (already these
    // where it held the expert), and its position in the words of every
    // instance of that expert
    const uint64_t word = ww | (uint64_t)(uint32_t)(at + 1) << (BW * rtj);
    const int held = (int)(((fhi ? (uint32_t)(word >> 32) : (uint32_t)word) >> fsh) & FM);
    if (lane < GM && held) pi[lane * PN + held - 1] = word;
    if (lane == 0) {
      U[aw] = uw - dw;
      atomicAdd(&U[a2], dw);
      e_of[a2] = ew;
      if (at >= P) slots[rtj * Neff + at - P] = ew;
    }
    wave_sync();
    RSECT(4);
  }
  RSECT_END(it);
  if (lane < G) {
    Lr[lane] = lj;
    used[lane] = uj;
  }
  wave_sync();
  return it;
}

// The lane form for the plan's shape (Form: kRefinePairs or kRefineLanes).
template <int Form>
__device__ __forceinline__ uint32_t refine_domain_in_lanes(const Plan &p, int d, int *e_of, int *U, uint64_t *pi,
                                                           int *qcol, int *slots, int *used, int *Lr,
                                                           uint32_t *flags) {
  const bool plain = p.R <= 64 && p.cI > 0;
  if constexpr (Form == kRefinePairs) {
    if (p.PN <= 8)
      return plain ? refine_domain_lanes<8, 1, true>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags)
                   : refine_domain_lanes<8, 1, false>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags);
    return plain ? refine_domain_lanes<8, 2, true>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags)
                 : refine_domain_lanes<8, 2, false>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags);
  }
  if (p.G <= 8)
    return plain ? refine_domain_lanes<8, 0, true>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags)
                 : refine_domain_lanes<8, 0, false>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags);
  if (p.PN <= 4) return refine_domain_lanes<16, 1, false>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags);
  if (p.PN <= 8) return refine_domain_lanes<16, 2, false>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags);
  return refine_domain_lanes<16, 0, false>(p, d, e_of, U, pi, qcol, slots, used, Lr, flags);
}

// Intra-node refinement of domain d (Section 4.3, Eq. 10), by one wave.
// e_of/U/qcol/slots/used/Lr point at the domain's own state; em (E words of
// 64 bits, scratch) receives, per expert, the mask of the domain's local
// ranks hosting it.  Each iteration picks the busiest rank rb (ties to the
// lowest rank), takes the best (instance of rb, other rank of the domain)
// candidate by key (delta desc, L[rt] asc, cost change asc, e asc, rt asc)
// and commits it: each lane takes an instance of rb and scores only its
// lightest receivers (the others cannot win).  (refine_domain_lanes makes the
// same moves for the domains that fit it.)  The moved assignments come from sources in ascending (c(s,rt) - c(s,rb),
// s) order: with the two-level cost that is rt
// itself, then the other sources ascending, then rb (or plain ascending when
// the intra-domain cost is zero).  The loop ends when no candidate has
// delta >= 1.  Returns the number of moves committed (at once 0 when no rank
// of the domain has a free slot).  With prepared, em already holds the masks
// and the wave sums the rank loads Lr itself; otherwise Lr is given and em is
// scratch filled here.  With General (the full model of Section 4.1) the
// moved assignments come from the sources in the precomputed (c(s,rt) -
// c(s,rb), s) order of gc, and the cost change uses the cost matrix and
// ||W_e||.
template <bool General = false>
__device__ __forceinline__ uint32_t refine_domain(const Plan &p, int d, int *e_of, int *U, int *qcol, int *slots, int *used,
                                  int *Lr, uint64_t *em, uint32_t *flags, bool prepared, GenCost gc = GenCost{}) {
  const int lane = lane_id();
  const int G = p.G, PN = p.PN, R = p.R, P = p.P, Neff = p.Neff, QS = p.QS, E = p.E, I = p.I;
  if (G < 2) return 0;
  const int r0 = d * G;
  // At the start of refinement every expert has at most one instance in the
  // domain (stage 1 places one replica per domain and expert, never in the
  // main's own domain), so a candidate's target must have a free slot:
  // without one anywhere in the domain no candidate ever exists.
  {
    const bool free_slot = lane < G && used[lane] < Neff;
    if (__ballot(free_slot) == 0) return 0;
  }
  if (prepared) {
    // em already holds the hosting masks; the rank loads are summed here
    if (lane < G) {
      int l = 0;
      for (int pos = 0; pos < PN; ++pos) l += U[lane * PN + pos];
      Lr[lane] = l;
    }
  } else {
    // hosting masks per expert
    for (int e = lane; e < E; e += 64) em[e] = 0;
    wave_sync();
    for (int a = lane; a < I; a += 64) {
      const int e = e_of[a];
      if (e >= 0) atomicOr(reinterpret_cast<unsigned long long *>(&em[e]), 1ull << (uint32_t)fdiv((uint32_t)a, p.fPN));
    }
  }
  wave_sync();
  // One lane per instance of rb.  Among the targets an instance may move to
  // (the domain's other ranks with L[rt] <= L[rb] - 2 that host its expert
  // or have a free slot) delta = min(u, (L[rb] - L[rt]) / 2) only grows as
  // L[rt] falls, so the instance's best keys all sit at its lightest
  // targets: the lane scores just those (usually one rank) instead of all
  // G - 1, and the wave keeps the overall minimum of the same key.
  const int rounds = (PN + 63) >> 6;
  // with at most 16 ranks the reductions over ranks stay in the first row
  // of 16 lanes
  const bool rank_row = G <= 16;
  auto min_u32 = [&](uint32_t v) { return rows_min_u32(v, rank_row); };
  const int64_t tokc = 2 * p.S * (int64_t)p.cI;   // cost change per moved assignment and unit of (m_rb - m_rt)
  const int64_t repI = (int64_t)p.cI * p.W, repX = (int64_t)p.cX * p.W;
  // lane j < G keeps rank j's load and used slots in registers (and the
  // LDS copies current for the other lanes' reads)
  int lj = 0, uj = 0;
  if (lane < G) {
    lj = Lr[lane];
    uj = used[lane];
  }
  uint32_t it = 0;
  RSECT_DECL(d);
  for (;; ++it) {
    // busiest rank, lowest index on ties
    const int Lrb = (int)~min_u32(lane < G ? ~(uint32_t)lj : ~0u);
    const int rbj = __ffsll((long long)__ballot(lane < G && lj == Lrb)) - 1;
    const int rb = r0 + rbj;
    // receivers: delta >= 1 needs L[rt] <= L[rb] - 2; those with a free slot
    // take any expert, and the lightest of them form one level (lf, tf)
    const bool low = lane < G && lane != rbj && (int64_t)Lrb - lj >= 2;
    const uint64_t lowm = __ballot(low);
    if (lowm == 0) break;
    const bool fr = low && uj < Neff;
    uint32_t lf = ~0u;
    uint64_t tf = 0;
    if (__ballot(fr)) {
      lf = min_u32(fr ? (uint32_t)lj : ~0u);
      tf = __ballot(fr && (uint32_t)lj == lf);
    }
    // the first rank of the free level: its q is read with the instance's
    // own words (it is usually the one target scored)
    const int jf = tf ? __ffsll((long long)tf) - 1 : 0;
    RSECT(0);
    uint64_t k1 = ~0ull, k2 = ~0ull, k3 = ~0ull, best_hm = 0;
    int best_a = 0, best_u = 0, best_q = 0;
    const bool two_level = !General && p.cI > 0;
    // instance a of rb (expert e, load u, q[rb] and q[r0 + jf] of its
    // column, hosting mask hmf of e) scored against its lightest receivers
    auto score = [&](int a, int e, int u, int qrb, int qf, uint64_t hmf) {
      const int *qa = qcol + a * QS;
      // the lightest receivers already hosting e (no slot needed)
      uint32_t lh = ~0u;
      uint64_t th = 0;
      for (uint64_t h = hmf & lowm; h; h &= h - 1) {
        const int j = __ffsll((long long)h) - 1;
        const uint32_t L = (uint32_t)Lr[j];
        if (L < lh) {
          lh = L;
          th = 0;
        }
        if (L == lh) th |= 1ull << j;
      }
      const uint32_t lm = lf < lh ? lf : lh;
      if (lm == ~0u) return;
      const uint64_t tset = (lf == lm ? tf : 0) | (lh == lm ? th : 0);
      const int delta = imin(u, (Lrb - (int)lm) >> 1);
      // lowest (cost change, rt) among the lightest receivers
      int64_t bc = INT64_MAX;
      int bj = 0, bq = 0;
      for (uint64_t t = tset; t; t &= t - 1) {
        const int rtj = __ffsll((long long)t) - 1;
        const bool hosts = (hmf >> rtj) & 1ull;
        const int rt = r0 + rtj;
        int64_t dcost = 0;
        int qrt = 0;
        if constexpr (General) {
          // fill delta from the sources in (c(s,rt) - c(s,rb), s) order
          const uint16_t *o = gc.ord + (rbj * G + rtj) * R;
          const int *ct = gc.ccol + rtj * R, *cb = gc.ccol + rbj * R;
          int rest = delta;
          int64_t dt = 0;
          // (four sources' words in flight: one at a time, each waits for
          // three dependent LDS reads)
          for (int k0 = 0; k0 < R && rest > 0; k0 += 4) {
            int sx[4], av[4], df[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) sx[i] = o[imin(k0 + i, R - 1)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              av[i] = k0 + i < R ? qa[sx[i]] : 0;
              df[i] = ct[sx[i]] - cb[sx[i]];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int take = imin(rest, av[i]);
              dt += (int64_t)take * df[i];
              rest -= take;
            }
          }
          dcost = 2 * p.S * dt;
          if (!hosts) dcost += (int64_t)gc.ccol[rtj * R + (int)fdiv((uint32_t)e, p.fP)] * gc.wx[e];
        } else {
          if (p.cI > 0) {
            qrt = rtj == jf ? qf : qa[rt];
            const int m_rt = imin(delta, qrt);
            const int rest = delta - m_rt;
            const int m_rb = rest - imin(rest, u - qrt - qrb);
            dcost = tokc * (int64_t)(m_rb - m_rt);
          }
          if (!hosts) dcost += ((int)fdiv((uint32_t)e, p.fGP) == d) ? repI : repX;
        }
        if (dcost < bc) {
          bc = dcost;
          bj = rtj;
          bq = qrt;
        }
      }
      const uint64_t c1 = ((uint64_t)(uint32_t)(0x7FFFFFFF - delta) << 32) | lm;
      const uint64_t c2 = (uint64_t)bc ^ (1ull << 63);
      const uint64_t c3 = ((uint64_t)(uint32_t)e << 32) | (uint32_t)(r0 + bj);
      // (c1, c2, c3) < (k1, k2, k3), with no branches
      const bool lt = (c1 < k1) | ((c1 == k1) & ((c2 < k2) | ((c2 == k2) & (c3 < k3))));
      k1 = lt ? c1 : k1;
      k2 = lt ? c2 : k2;
      k3 = lt ? c3 : k3;
      best_a = lt ? a : best_a;
      best_u = lt ? u : best_u;
      best_hm = lt ? hmf : best_hm;
      best_q = lt ? bq : best_q;
    };
    // one lane per instance, two instances (rounds of 64) at a time: the
    // pair's words and hosting masks are read before either is scored, so
    // their LDS round trips overlap (a lane's instances hold distinct
    // experts, so the order it scores them in does not matter)
    for (int rd = 0; rd < rounds; rd += 2) {
      const int ai0 = lane + rd * 64, ai1 = ai0 + 64;
      const bool v0 = ai0 < PN, v1 = ai1 < PN;
      const int a0 = rbj * PN + (v0 ? ai0 : 0), a1 = rbj * PN + (v1 ? ai1 : 0);
      const int *qa0 = qcol + a0 * QS, *qa1 = qcol + a1 * QS;
      const int e0 = v0 ? e_of[a0] : -1, e1 = v1 ? e_of[a1] : -1;
      const int u0 = v0 ? U[a0] : 0, u1 = v1 ? U[a1] : 0;
      const int qrb0 = two_level ? qa0[rb] : 0, qf0 = two_level ? qa0[r0 + jf] : 0;
      const int qrb1 = two_level && v1 ? qa1[rb] : 0, qf1 = two_level && v1 ? qa1[r0 + jf] : 0;
      const uint64_t hm0 = e0 >= 0 ? em[e0] : 0, hm1 = e1 >= 0 ? em[e1] : 0;
      if (e0 >= 0 && u0 > 0) score(a0, e0, u0, qrb0, qf0, hm0);
      if (e1 >= 0 && u1 > 0) score(a1, e1, u1, qrb1, qf1, hm1);
    }
    RSECT(1);
    const uint64_t m1 = wave_min_u64(k1);
    if (m1 == ~0ull) break;
    // a move is still available after iter_limit of them: stop with ITER
    if (it >= p.iter_limit) {
      if (lane == 0) *flags |= TOPOEP_ST_ITER;
      break;
    }
    uint64_t win = __ballot(k1 == m1);
    if (__popcll(win) != 1) {
      const uint64_t m2 = wave_min_u64(k1 == m1 ? k2 : ~0ull);
      win &= __ballot(k2 == m2);
      if (__popcll(win) != 1) {
        const uint64_t m3 = wave_min_u64((k1 == m1 && k2 == m2) ? k3 : ~0ull);
        win &= __ballot(k3 == m3);
      }
    }
    const int wl = __ffsll((long long)win) - 1;
    const uint64_t kw1 = readlane64(k1, wl);
    const int delta = 0x7FFFFFFF - (int)(kw1 >> 32);
    const int Lrt = (int)(uint32_t)kw1;
    const uint64_t kw = readlane64(k3, wl);
    const int e = (int)(kw >> 32);
    const int rt = (int)(uint32_t)kw;
    const int rtj = rt - r0;
    const int a = readlane_i32(best_a, wl);
    const int ua = readlane_i32(best_u, wl);
    const int qrt = readlane_i32(best_q, wl);
    const bool hosts = (readlane64(best_hm, wl) >> rtj) & 1ull;
    RSECT(2);
    // rt's instance of e: its main expert, the replica slot holding it, or a
    // new replica in rt's first free slot
    int a2 = -1;
    bool fresh = false;
    if (!hosts) {
      a2 = rtj * PN + P + readlane_i32(uj, rtj);
      fresh = true;
    } else if ((int)fdiv((uint32_t)e, p.fP) == rt) {
      a2 = rtj * PN + (e - rt * P);
    } else {
      const int ut = readlane_i32(uj, rtj);
      for (int t0 = 0; t0 < ut && a2 < 0; t0 += 64) {
        const uint64_t hit = __ballot(t0 + lane < ut && slots[rtj * Neff + t0 + lane] == e);
        if (hit) a2 = rtj * PN + P + t0 + __ffsll((long long)hit) - 1;
      }
    }
    RSECT(3);
    int *qa = qcol + a * QS;
    int *qb = qcol + a2 * QS;
    int rest = delta;
    int m_rt = 0;
    if constexpr (General) {
      // the sources in the pair's order, 64 at a time
      const uint16_t *o = gc.ord + (rbj * G + rtj) * R;
      for (int k0 = 0; k0 < R && rest > 0; k0 += 64) {
        const int k = k0 + lane;
        const int s = k < R ? o[k] : 0;
        const int av = k < R ? qa[s] : 0;
        const int incl = wave_incl_scan(av);
        const int excl = incl - av;
        int m = rest - excl;
        m = m < 0 ? 0 : (m > av ? av : m);
        if (m) {
          qa[s] = av - m;
          atomicAdd(&qb[s], m);
        }
        const int total = readlane_i32(incl, 63);
        rest -= total < rest ? total : rest;
      }
    } else {
      // rt's own assignments first, then the other sources ascending (rb's
      // own are taken last, below)
      if (p.cI > 0) {
        m_rt = imin(rest, qrt);
        rest -= m_rt;
      }
      for (int s0 = 0; s0 < R && rest > 0; s0 += 64) {
        const int s = s0 + lane;
        int av = 0;
        if (s < R && (p.cI == 0 || (s != rt && s != rb))) av = qa[s];
        const int incl = wave_incl_scan(av);
        const int excl = incl - av;
        int m = rest - excl;
        m = m < 0 ? 0 : (m > av ? av : m);
        if (m) {
          qa[s] = av - m;
          atomicAdd(&qb[s], m);
        }
        const int total = readlane_i32(incl, 63);
        rest -= total < rest ? total : rest;
      }
    }
    RSECT(4);
    // (the sources above exclude rt and rb, so these words are disjoint
    // from the lanes' updates; LDS atomics without return need no wait)
    if (lane == 0) {
      if (fresh) {
        slots[rtj * Neff + (a2 - rtj * PN - P)] = e;
        used[rtj] = a2 - rtj * PN - P + 1;
        e_of[a2] = e;
        atomicOr(reinterpret_cast<unsigned long long *>(&em[e]), 1ull << rtj);
      }
      if (m_rt) {
        atomicSub(&qa[rt], m_rt);
        atomicAdd(&qb[rt], m_rt);
      }
      if (rest > 0) {   // the rest comes from rb itself (two-level cost, taken last)
        atomicSub(&qa[rb], rest);
        atomicAdd(&qb[rb], rest);
      }
      U[a] = ua - delta;
      atomicAdd(&U[a2], delta);
      Lr[rbj] = Lrb - delta;
      Lr[rtj] = Lrt + delta;
    }
    if (lane == rbj) lj = Lrb - delta;
    if (lane == rtj) {
      lj = Lrt + delta;
      uj += fresh ? 1 : 0;
    }
    wave_sync();
    RSECT(5);
  }
  RSECT_END(it);
  return it;   // one move per completed iteration
}

// Stage-1 candidate key: (D descending, e ascending) as one unsigned
// 64-bit value, smaller first.  This is the order of the benefit
// b = 2 D S - W descending (S > 0), ties to the lower expert id.
__device__ inline uint64_t cand_key(int D, int e) {
  return ((uint64_t)(uint32_t)(0x7FFFFFFF - D) << 32) | (uint32_t)e;
}

// Ranks of a domain's nc candidates by `step` waves, this one the `first` of
// them: 64 candidates at a time, one per lane, against the keys in parts of
// 16, whose reads are broadcasts.  The (64 candidates, part) pairs are dealt
// to the waves in turn across the whole domain, and a wave adds once for its
// parts of one 64.  rk (nc words) starts at zero.  General: keys are benefits
// (descending), ties to the lower expert of es (||W_e|| differs per expert, so
// b does not follow D); else keys ascend (cand_key) and are distinct.
// Padded: the keys go on to a multiple of 16, sorting last.
// One thread per candidate walking all keys took 2.6 us of dependent LDS reads
// for 96 candidates under the general model; pairs dealt with the 64s rounded
// up to a power of two left waves idle, and clamped every key's index (EP 64,
// E = 1024, 1 M ids, some 850 candidates in each of 8 domains: 93.9 us a plan,
// 65.5 now; 79.7 with a thread per candidate).
template <bool General, bool Padded>
__device__ __forceinline__ void rank_keys(int nc, const uint64_t *keys, const int *es, int *rk, int first, int step) {
  const int parts = (nc + 15) >> 4;
  int part = first;
  for (int c0 = 0; c0 < nc; c0 += 64, part -= parts) {
    if (part >= parts) continue;
    const int c = c0 + lane_id(), cc = imin(c, nc - 1);
    const uint64_t kc = keys[cc];
    const int ec = General ? es[cc] : 0;
    int below = 0;
    for (; part < parts; part += step) {
      const int k0 = part * 16;
      uint64_t k[16];
      int e2[16];
      if (Padded || k0 + 16 <= nc) {
        const uint64_t *kp = keys + k0;   // (plain offsets: wide reads)
#pragma unroll
        for (int i = 0; i < 16; ++i) k[i] = kp[i];
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (General) e2[i] = es[k0 + i];
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int at = imin(k0 + i, nc - 1);
          k[i] = k0 + i < nc ? keys[at] : (General ? 0ull : ~0ull);
          if (General) e2[i] = es[at];
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i)
        below += (General ? (k[i] > kc || (k[i] == kc && e2[i] < ec)) : k[i] < kc) ? 1 : 0;
    }
    if (c < nc && below) atomicAdd(&rk[c], below);
  }
}

// Stage 1 (Eq. 9) of every domain by the whole workgroup.  Item (d, e):
// D[d][e] summed over the domain's rows of Omega; an expert whose main lies
// outside d with b = 2 D S - W > 0 is a candidate and takes a slot of
// ck + d E16 (E16 = E rounded up to 16; the keys were set to ~0, which sorts
// after every candidate) from the domain's LDS counter ccnt[d] (the slots'
// order is arbitrary).  Each candidate's rank among its domain's candidates
// by key (D descending, e ascending; keys are distinct) is then counted: the
// waves are split among the domains (one domain after another when there are
// more domains than waves; rank_keys).  (With lanes on different parts the
// reads, 128 bytes apart, met on one LDS bank: a plan of 1.6 M ids with 192
// candidates in each of 4 domains took 111.6 us, 52.2 with broadcast reads.)
// rk[d E + c] = the rank of the domain's candidate in slot c.
// The ranks below cap1 name the domain's stage-1 replicas.  rk: M E words.
__device__ __forceinline__ void stage1_ranks(const Plan &p, const int *om, uint64_t *ck, int *ccnt, int *rk) {
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E, G = p.G, M = p.M, E16 = (E + 15) & ~15;
  // item idx = d E + e, walked with (d, e) kept as the index advances
  const int dstep = (int)fdiv((uint32_t)nt, p.fE), estep = nt - dstep * E;
  int d = (int)fdiv((uint32_t)tid, p.fE), e = tid - d * E;
  for (int idx = tid; idx < M * E; idx += nt, d += dstep, e += estep) {
    if (e >= E) {
      e -= E;
      ++d;
    }
    rk[idx] = 0;
    if ((int)fdiv((uint32_t)e, p.fGP) == d) continue;   // main inside the domain
    const int *col = om + d * G * E + e;
    int D = 0;
#pragma unroll 8
    for (int j = 0; j < G; ++j) D += col[j * E];
    if ((int64_t)2 * D * p.S > p.W) {
      const int pos = atomicAdd(&ccnt[d], 1);
      ck[d * E16 + pos] = cand_key(D, e);
    }
  }
  lds_barrier();
  STAMP(p, 24);
  const int nw = nt >> 6, wave = uniform_i32(tid >> 6);
  const int wpd = p.s1_waves;
  const int d0 = wpd ? (int)fdiv((uint32_t)wave, p.fS1) : 0;
  const int step = wpd ? wpd : nw, first = wpd ? wave - d0 * wpd : wave;
  for (d = d0; d < (wpd ? imin(d0 + 1, M) : M); ++d) {
    const int nc = uniform_i32(ccnt[d]);   // (d is the same in the whole wave)
    rank_keys<false, true>(nc, ck + d * E16, nullptr, rk + d * E, first, step);
  }
  lds_barrier();
  STAMP(p, 26);
}

// The stage-1 replica lists from the ranks: repl[d cap1 + rank] = e for the
// ranks below cap1 (repl holds -1 elsewhere).  Ends with a barrier.
__device__ __forceinline__ void stage1_lists(const Plan &p, const uint64_t *ck, const int *ccnt, const int *rk,
                                             int *repl) {
  for (int idx = threadIdx.x; idx < p.M * p.E; idx += blockDim.x) {
    const int d = (int)fdiv((uint32_t)idx, p.fE), c = idx - d * p.E;
    if (c < ccnt[d] && rk[idx] < p.cap1) repl[d * p.cap1 + rk[idx]] = (int)(uint32_t)ck[d * ((p.E + 15) & ~15) + c];
  }
  lds_barrier();
}

// This rank's per-expert instance list: bm[e * RW ...] marks the ranks
// whose instance of e has a nonzero share q[self][e][r].  Thread t takes
// experts [t * K, (t + 1) * K), K = ceil(E / blockDim): it counts their
// ranks; a wave scan plus the totals of the waves before (one barrier) give
// each expert's first entry; then it walks the ranks in ascending order
// writing (rank, cumulative share).  qcol and e_of address instance (d, a)
// as d * I + a; slots/used are every rank's; tmp holds blockDim / 64 words.
__device__ void emit_instance_list(const Plan &p, const int *qcol, const int *slots, const int *used,
                                   const uint32_t *bm, int *tmp) {
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
  const int E = p.E, RW = p.RW, K = (E + nt - 1) / nt;
  const int e0 = imin(E, tid * K), e1 = imin(E, e0 + K);
  int cnt = 0;
  for (int e = e0; e < e1; ++e)
    for (int w = 0; w < RW; ++w) cnt += __popc(bm[e * RW + w]);
  const int incl = wave_incl_scan(cnt);
  if (lane == 63) tmp[wave] = incl;
  __syncthreads();
  int pos = incl - cnt;
  for (int w = 0; w < wave; ++w) pos += tmp[w];
  if (tid == nt - 1) p.csr_ptr[E] = pos + cnt;
  for (int e = e0; e < e1; ++e) {
    p.csr_ptr[e] = pos;
    int run = 0;
    for (int w = 0; w < RW; ++w) {
      uint32_t bits = bm[e * RW + w];
      while (bits) {
        const int r = w * 32 + __ffs(bits) - 1;
        bits &= bits - 1u;
        const int d = (int)fdiv((uint32_t)r, p.fG), j = r - d * p.G;
        const int a = instance_of(p, d, j, e, slots + d * p.G * p.Neff, used + d * p.G);
        if (a >= 0) run += qcol[(d * p.I + a) * p.QS + p.self];   // a >= 0: bm marks hosts only
        p.csr_r[pos] = r;
        p.csr_end[pos] = run;
        ++pos;
      }
    }
  }
}

// Status bits and the sum of positive loads of Omega' (row self replaced by
// the histogram hs) over rows [r0, r1) held at rows[(s - r0) * E + e];
// wave-reduced, then one LDS atomic per wave into misc[0] (bits) and
// misc[8..9] (total).  Called by every thread of the workgroup.
__device__ __forceinline__ void scan_rows(const Plan &p, int r0, int r1, const int *rows, const int *hs, int *misc) {
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E;
  bool neg = false, diff = false;
  uint64_t tot = 0;
  const int n = (r1 - r0) * E;
  for (int i = tid; i < n; i += nt) {
    const int g = rows[i];
    neg |= g < 0;
    if (g > 0) tot += (uint64_t)g;
  }
  if (p.self >= r0 && p.self < r1) {
    // row self: the plan uses the histogram instead of the gathered row
    for (int e = tid; e < E; e += nt) {
      const int g = rows[(p.self - r0) * E + e];
      if (g > 0) tot -= (uint64_t)g;
      if (hs[e] > 0) tot += (uint64_t)hs[e];
      diff |= g != hs[e];
    }
  }
  tot = wave_sum_u64(tot);
  const uint64_t any_neg = __ballot(neg);
  const uint64_t any_diff = __ballot(diff);
  if (lane_id() == 0) {
    const uint32_t w = (any_neg ? TOPOEP_ST_NEG_LOAD : 0u) | (any_diff ? TOPOEP_ST_SELF_DIFF : 0u);
    if (w) atomicOr(reinterpret_cast<unsigned *>(&misc[0]), w);
    if (tot) atomicAdd(reinterpret_cast<unsigned long long *>(misc + 8), (unsigned long long)tot);
  }
}

// ---------------------------------------------------------------- general cost model

// The full model of Section 4.1 on the device: whether the cost matrix is a
// cost (symmetric, nonnegative, zero diagonal) and every size nonnegative,
// and the largest entry and size for the exact-range bound.  Each workgroup
// looks at its domains' rows of the matrix and a share of the sizes, and the
// control words combine them by the grid barrier (every workgroup used to
// read the whole matrix: 65 536 entries at R = 256, where a plan went from
// 90.0 to 27.6 us with this and the one launch).
struct CostCheck {
  bool bad;
  uint32_t cm;
  uint64_t wm;
};

__device__ __forceinline__ CostCheck general_check(const Plan &p, int wg, int nwg) {
  const int tid = threadIdx.x, nt = blockDim.x, R = p.R, GR = p.G * p.R;
  CostCheck k = {false, 0u, 0ull};
  if (p.Cm) {
    for (int d = wg; d < p.M; d += nwg)
      for (int i = tid; i < GR; i += nt) {
        const int j = i / R, r = i - j * R, s = d * p.G + j;
        const int c = p.Cm[(int64_t)s * R + r], ct = p.Cm[(int64_t)r * R + s];
        k.bad |= c < 0 || (s == r && c != 0) || c != ct;
        if (c > 0 && (uint32_t)c > k.cm) k.cm = (uint32_t)c;
      }
  } else {
    k.cm = (uint32_t)imax(p.cI, p.cX);
  }
  if (p.We) {
    for (int e = wg * nt + tid; e < p.E; e += nwg * nt) {
      const int64_t w = p.We[e];
      k.bad |= w < 0;
      if (w > 0 && (uint64_t)w > k.wm) k.wm = (uint64_t)w;
    }
  } else {
    k.wm = (uint64_t)p.W;
  }
  return k;
}

// Cost tables of domain d for its refinement: ccol[j][s] = c(s, dG + j),
// ||W_e|| and, per ordered pair (jb, jt) of the domain's ranks, the sources
// in ascending (c(s,rt) - c(s,rb), s) order.
__device__ __forceinline__ GenCost general_tables(const Plan &p, int d, int *sm, const DomainLds &lay) {
  const int tid = threadIdx.x, nt = blockDim.x, R = p.R, G = p.G;
  uint16_t *ord = reinterpret_cast<uint16_t *>(sm + lay.ord);
  int *ccol = sm + lay.ccol;
  int64_t *wx = reinterpret_cast<int64_t *>(sm + lay.wx);
  for (int i = tid; i < G * R; i += nt) {
    const int j = i / R, s = i - j * R, r = d * G + j;
    ccol[i] = p.Cm ? p.Cm[(int64_t)s * R + r] : (s == r ? 0 : (s / G == r / G ? p.cI : p.cX));
  }
  for (int e = tid; e < p.E; e += nt) wx[e] = p.We ? p.We[e] : p.W;
  lds_barrier();
  // one wave per pair: lane l ranks source s0 + l among all sources, whose
  // differences come lane by lane from registers
  const int lane = tid & 63, nw = nt >> 6;
  for (int pair = uniform_i32(tid >> 6); pair < G * G; pair += nw) {
    const int jb = pair / G, jt = pair - jb * G;
    if (jb == jt) continue;
    const int *cb = ccol + jb * R, *ct = ccol + jt * R;
    for (int s0 = 0; s0 < R; s0 += 64) {
      const int s = s0 + lane, ds = s < R ? ct[s] - cb[s] : 0;
      int rank = 0;
      for (int t0 = 0; t0 < R; t0 += 64) {
        const int t = t0 + lane, dt = t < R ? ct[t] - cb[t] : 0, nt2 = imin(64, R - t0);
        for (int l = 0; l < nt2; ++l) {
          const int d2 = readlane_i32(dt, l);
          rank += d2 < ds || (d2 == ds && t0 + l < s) ? 1 : 0;
        }
      }
      if (s < R) ord[pair * R + rank] = (uint16_t)s;
    }
  }
  lds_barrier();
  GenCost gc;
  gc.ord = ord;
  gc.ccol = ccol;
  gc.wx = wx;
  return gc;
}

// Send offsets of the one-launch plan (exclusive prefix of the send counts
// sendl, total at [R]) by wave 0, for the caller and for the chunks.
__device__ __forceinline__ void solver_send_offsets(const Plan &p, const int *sendl) {
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x, R = p.R;
  const int per = (R + 63) / 64, lo = imin(R, lane * per), hi = imin(R, lo + per);
  int sum = 0;
  for (int r = lo; r < hi; ++r) sum += sendl[r];
  int run = wave_incl_scan(sum) - sum;
  for (int r = lo; r < hi; ++r) {
    p.offs_out[r] = run;
    run += sendl[r];
  }
  if (lane == 63) p.offs_out[R] = run;
}

// ---------------------------------------------------------------- solver: one workgroup per domain
//
// Workgroups 0 .. n_solvers-1 each take the domains d = wg, wg + n_solvers,
// ...; the n_helpers after them compute the histogram blocks' offsets for
// the reroute and each expert's total (row self of Omega).  Per domain:
// stage 1 (Eq. 9) from the domain's rows of Omega, then a bounded grid
// barrier publishes every domain's replicas; the hosting masks, the
// domain's instances, routing (Section 4.3), refinement (Eq. 10) and the
// domain's outputs follow.  The last solver workgroup to finish (a ticket)
// lists this rank's instances per expert for the reroute and writes the
// final status.
//
// One (plan_domains_kernel, one domain per workgroup): row self and bad ids
// come from the chunk workgroups of the same launch.  The workgroup of the
// domain holding self makes its stage 1 from Omega as gathered, then waits
// for the last chunk's verdict on row self and makes it again when that row
// differs from the histogram; the grid barrier passes the verdict on.  The
// last workgroup to finish releases the chunks.
template <bool One>
__device__ __forceinline__ void domain_solver(const Plan &p0, int *sm) {
  const Plan p = solver_plan(role_plan(p0));
  DomainLds lay = domain_lds(p);
  lay.ck = vgpr(lay.ck);
  lay.fdt = vgpr(lay.fdt);
  lay.hs = vgpr(lay.hs);
  lay.rows = vgpr(lay.rows);
  lay.mask = vgpr(lay.mask);
  lay.slots = vgpr(lay.slots);
  lay.used = vgpr(lay.used);
  lay.L = vgpr(lay.L);
  lay.e_of = vgpr(lay.e_of);
  lay.U = vgpr(lay.U);
  lay.misc = vgpr(lay.misc);
  lay.qcol = vgpr(lay.qcol);
  lay.ord = vgpr(lay.ord);
  lay.ccol = vgpr(lay.ccol);
  lay.wx = vgpr(lay.wx);
  uint64_t *ck = reinterpret_cast<uint64_t *>(sm + lay.ck);
  FastDiv *fdt = reinterpret_cast<FastDiv *>(sm + lay.fdt);
  int *hs = sm + lay.hs;
  int *rows = sm + lay.rows;
  uint32_t *mask = reinterpret_cast<uint32_t *>(sm + lay.mask);
  int *slots = sm + lay.slots;
  int *used = sm + lay.used;
  int *Lr = sm + lay.L;
  int *e_of = sm + lay.e_of;
  int *U = sm + lay.U;
  int *misc = sm + lay.misc;
  int *qcol = sm + lay.qcol;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int wg = blockIdx.x, nwg = p.n_solvers;
  const int E = p.E, G = p.G, R = p.R, M = p.M, I = p.I, P = p.P, PN = p.PN, Neff = p.Neff;
  const int cap = p.cap1;

  STAMP_CLEAR(0, 18);
  if (wg == 0) STAMP(p, 0);
  if (tid < 16) misc[tid] = 0;
  if constexpr (One) {
    // the plan's generation (the last workgroup to finish advances it), the
    // next plan's histogram buffer cleared (see fused_solver), row self as
    // gathered
    if (tid < 64) {
      const uint32_t g = __hip_atomic_load(&p.ctrl[kCtrlGen], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (tid == 0) misc[kMiscGen] = (int)g;
      if (wg == 0) {
        uint32_t *other = p.ghist + ((g + 1u) & 1u) * (E + 1);
        for (int e = tid; e <= E; e += 64)
          __hip_atomic_store(other + e, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tid == 0) p.status_out[0] = 0;   // chunks may OR SYNC into it
      }
    }
    for (int e = tid; e < E; e += nt) hs[e] = p.gl[(int64_t)p.self * E + e];
  }
  build_divisors(M, fdt);
  uint64_t cmax = (uint64_t)imax(p.cI, p.cX), wmax = (uint64_t)p.W;
  CostCheck check = {false, 0u, 0ull};
  if (p.general) check = general_check(p, wg, nwg);
  // ---- row self of Omega: the histogram of local_topk, from the offset
  // helpers; the workgroup of the domain holding self needs it for its
  // stage 1 (it waits once its rows of Omega are loaded), the others only
  // after the grid barrier (by then the helpers are done)
  const int dself = (int)fdiv((uint32_t)p.self, p.fG);
  const bool has_self = dself < M && dself % nwg == wg;
  if (!One && wg == 0)
    for (int b = tid; b < p.nb; b += nt)
      if (p.blk_err[b]) atomicOr(reinterpret_cast<unsigned *>(&misc[0]), TOPOEP_ST_BAD_ID);
  bool waited = true;   // One: the wait for the verdict did not give up
  // domains hosting each expert: the main's here, the stage-1 replicas' after
  // the grid barrier (the words are this workgroup's own until then)
  for (int e = tid; e < E; e += nt) {
    const int dm = (int)fdiv((uint32_t)e, p.fGP);
    for (int w = 0; w < p.MW; ++w) mask[e * p.MW + w] = w == (dm >> 5) ? 1u << (dm & 31) : 0u;
  }

  // ---- inter-node placement (Eq. 9), each domain independently
  for (int d = wg; d < M; d += nwg) {
    const Plan p = solver_plan(role_plan(p0));   // (reloaded: see the domain loop below)
    copy_to_lds(rows, p.gl + (int64_t)d * G * E, G * E);
    if (wg == 0) STAMP(p, 14);
    if (!One && d == dself) row_self(p, hs, qcol, &misc[10]);
    if (wg == 0) STAMP(p, 15);
    for (int pass = 0;; ++pass) {
      if (tid == 0) misc[1] = 0;
      for (int c = tid; c < E; c += nt) qcol[E + c] = 0;   // the candidates' ranks
      lds_barrier();
      scan_rows(p, d * G, (d + 1) * G, rows, hs, misc);
      for (int e = tid; e < E; e += nt) {
        if ((int)fdiv((uint32_t)e, p.fGP) == d) continue;   // main inside the domain
        int D = 0;
#pragma unroll 8
        for (int j = 0; j < G; ++j) {
          const int s = d * G + j;
          D += s == p.self ? hs[e] : rows[j * E + e];
        }
        const int64_t we = p.general && p.We ? p.We[e] : p.W;
        if ((int64_t)2 * D * p.S > we) {
          const int pos = atomicAdd(&misc[1], 1);
          if (p.general) {
            // sizes differ per expert: rank by the benefit itself (qcol is
            // free until the routing and holds the experts)
            ck[pos] = (uint64_t)((int64_t)2 * D * p.S - we);
            qcol[pos] = e;
          } else {
            ck[pos] = cand_key(D, e);
          }
        }
      }
      lds_barrier();
      if (wg == 0) STAMP(p, 16);
      const int nc = misc[1];
      if (wg == 0 && tid == 0) stamp_nc(nc);
      const int wave = uniform_i32(tid >> 6), nw = nt >> 6;
      if (p.general) rank_keys<true, false>(nc, ck, qcol, qcol + E, wave, nw);
      else rank_keys<false, false>(nc, ck, nullptr, qcol + E, wave, nw);
      lds_barrier();
      // the first cap ranks name the domain's stage-1 replicas
      for (int c = tid; c < nc; c += nt) {
        const int rank = qcol[E + c];
        if (rank < cap) p.repl1[(int64_t)d * cap + rank] = p.general ? qcol[c] : (int)(uint32_t)ck[c];
      }
      for (int i = imin(nc, cap) + tid; i < cap; i += nt) p.repl1[(int64_t)d * cap + i] = -1;
      lds_barrier();
      if (!One || d != dself || pass > 0) break;
      if (tid == 0) {
        const uint32_t want = ((uint32_t)misc[kMiscGen] + 1u) & 0x3FFFFFFFu;
        uint32_t v = 0;
        int ok = 0;
        for (uint32_t it = 0; it < p.spin_limit; ++it) {
          if (it > 0) __builtin_amdgcn_s_sleep(1);
          v = __hip_atomic_load(&p.ctrl[kCtrlVerdict], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if ((v >> 2) == want) {
            ok = 1;
            break;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        misc[2] = ok;
        misc[3] = (int)(v & 3u);
      }
      __syncthreads();
      waited = misc[2] != 0;
      if (!waited || (uint32_t)misc[3] == kVerdictSame) break;
      // row self := the histogram, and the stage again (its replicas' stores
      // above complete before they are stored again)
      drain_then_barrier();
      const uint32_t *gh = p.ghist + (misc[kMiscGen] & 1) * (E + 1);
      for (int e = tid; e < E; e += nt) hs[e] = (int)gh[e];
      if (tid == 0) {
        misc[0] = (int)(gh[E] ? TOPOEP_ST_BAD_ID : 0u);
        misc[8] = misc[9] = 0;
      }
    }
  }
  if (p.general) {
    // (one atomic per wave)
    const uint32_t cm = ~rows_min_u32(~check.cm, false);
    const uint64_t wm = ~wave_min_u64(~check.wm), any_bad = __ballot(check.bad);
    if (lane_id() == 0) {
      if (any_bad) atomicOr(&p.ctrl[kCtrlStatus], TOPOEP_ST_COST);
      atomicMax(&p.ctrl[kCtrlCost], cm);
      atomicMax(reinterpret_cast<unsigned long long *>(p.ctrl + kCtrlSize), (unsigned long long)wm);
    }
  }
  if (tid == 0) {
    const uint32_t st = (uint32_t)misc[0] | (waited ? 0u : TOPOEP_ST_SYNC);
    if (st) atomicOr(&p.ctrl[kCtrlStatus], st);
    const unsigned long long t = *reinterpret_cast<unsigned long long *>(misc + 8);
    if (t) atomicAdd(reinterpret_cast<unsigned long long *>(p.ctrl + kCtrlTotal), t);
  }

  // ---- every domain's replicas are needed by every routing construction
  if (wg == 0) STAMP(p, 1);
  const bool synced = grid_barrier(&p.ctrl[kCtrlBar], (uint32_t)nwg, p.spin_limit, &misc[2]);
  if (wg == 0) STAMP(p, 2);
  // every domain's replicas on their way with the status words
  int rv[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) rv[u] = tid + u * nt < M * cap ? p.repl1[tid + u * nt] : 0;
  uint32_t gst = __hip_atomic_load(&p.ctrl[kCtrlStatus], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t total = __hip_atomic_load(reinterpret_cast<unsigned long long *>(p.ctrl + kCtrlTotal),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (p.general) {
    cmax = __hip_atomic_load(&p.ctrl[kCtrlCost], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wmax = __hip_atomic_load(reinterpret_cast<unsigned long long *>(p.ctrl + kCtrlSize), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  }
  if (out_of_range_cw(p, total, cmax, wmax)) gst |= TOPOEP_ST_RANGE;
  if (!synced) gst |= TOPOEP_ST_SYNC;
  const bool noplan = (gst & (kNoPlan | TOPOEP_ST_SYNC)) != 0;

  if constexpr (One) {
    const uint32_t v = __hip_atomic_load(&p.ctrl[kCtrlVerdict], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!has_self && !noplan && (v & 3u) == kVerdictRedo) {
      const uint32_t *gh = p.ghist + (misc[kMiscGen] & 1) * (E + 1);
      for (int e = tid; e < E; e += nt) hs[e] = (int)gh[e];   // (a barrier follows before any is read)
    }
  } else {
    if (!has_self && !noplan) row_self(p, hs, qcol, &misc[10]);
  }

  // ---- domains hosting each expert: the main's domain plus stage-1 replicas
  const bool one_domain = M <= nwg;
  bool empty = false;   // an empty entry: a rank of that domain has a free slot
  if (!noplan) {
    auto host = [&](int i, int e) {
      const int dd = (int)fdiv((uint32_t)i, p.fCap);
      // a workgroup of one domain keeps that domain's list (rows is free
      // after stage 1: cap = G Neff <= G E words)
      if (one_domain && dd == wg) rows[i - dd * cap] = e;
      if ((unsigned)e < (unsigned)E) atomicOr(&mask[e * p.MW + (dd >> 5)], 1u << (dd & 31));
      else empty = true;
    };
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (tid + u * nt < M * cap) host(tid + u * nt, rv[u]);
    for (int i = tid + 2 * nt; i < M * cap; i += nt) host(i, p.repl1[i]);
  }
  // No domain can refine (every slot taken by stage 1, or one rank per
  // domain): the routing rule alone gives this rank's shares (see
  // fast_finish), and every workgroup writes its own domains' part of the
  // instance list, which otherwise waits for the last one.
  // (One only: the three-kernel solver has no registers left for it.)
  bool lean = false;
  if constexpr (One) lean = __syncthreads_or(empty) == 0 || G < 2;
  else __syncthreads();
  if (wg == 0) STAMP(p, 3);

  uint32_t flags = 0;
  if (lean && !noplan) {
    const int ds = dself;
    int *first = qcol;   // E + 1: each expert's first entry
    for (int e = tid; e < E; e += nt) {
      const uint32_t *me = mask + e * p.MW;
      const int w = hs[e];
      int n = 0;
      for (int wd = 0; wd < p.MW; ++wd) n += __popc(me[wd]);
      first[e] = w <= 0 ? 0 : (((me[ds >> 5] >> (ds & 31)) & 1u) ? 1 : imin(n, w));
    }
    lds_barrier();
    const int all = block_excl_scan(first, E, qcol + E + 2);
    if (wg == 0) {
      for (int e = tid; e < E; e += nt) p.csr_ptr[e] = first[e];
      if (tid == 0) p.csr_ptr[E] = all;
    }
    for (int d = wg; d < M; d += nwg) {
      for (int j = tid; j < G; j += nt) Lr[j] = 0;   // the ranks' send counts
      lds_barrier();
      for (int a = tid; a < I; a += nt) {
        const int j = (int)fdiv((uint32_t)a, p.fPN), pos = a - j * PN, r = d * G + j;
        int e = r * P + pos;
        if (pos >= P) {
          // stage-1 entry t G + j sits in slot t of local rank j
          const int c = (pos - P) * G + j;
          e = one_domain ? rows[c] : p.repl1[(int64_t)d * cap + c];
          p.slots_out[(int64_t)r * p.N + pos - P] = e;
        }
        e_of[a] = e;
        const int w = e >= 0 ? hs[e] : 0;
        if (w <= 0) continue;
        const uint32_t *me = mask + e * p.MW;
        int i = 0, q = w, end = w;
        if ((me[ds >> 5] >> (ds & 31)) & 1u) {
          if (d != ds) continue;   // all of w to the instance in dom(self)
        } else {
          int n = 0;
          for (int wd = 0; wd < p.MW; ++wd) {
            const uint32_t bits = me[wd];
            n += __popc(bits);
            const int lo = wd * 32;
            if (d >= lo + 32) i += __popc(bits);
            else if (d > lo) i += __popc(bits & ((1u << (d - lo)) - 1u));
          }
          const FastDiv fn = fdt[n];
          const int qq = (int)fdiv_hi((uint32_t)w, fn), rem = w - qq * n;
          q = qq + (i < rem ? 1 : 0);
          if (q <= 0) continue;
          end = (i + 1) * qq + imin(i + 1, rem);
        }
        p.csr_r[first[e] + i] = r;
        p.csr_end[first[e] + i] = end;
        atomicAdd(&Lr[j], q);
      }
      // slots beyond the experts a rank does not hold stay empty
      for (int i = tid; i < G * (p.N - Neff); i += nt) {
        const int j = i % G, t = Neff + i / G;
        p.slots_out[(int64_t)(d * G + j) * p.N + t] = -1;
      }
      lds_barrier();
      for (int j = tid; j < G; j += nt) p.send_out[d * G + j] = Lr[j];
      if (p.recv_out && d == ds)
        write_recv_counts(p, (p.self - d * G) * PN, e_of, nullptr, false, mask, fdt,
                          [&](int s, int e) { return s == p.self ? hs[e] : p.gl[(int64_t)s * E + e]; },
                          reinterpret_cast<int *>(ck));
      lds_barrier();
    }
  }
  for (int d = wg; d < M && !(lean && !noplan); d += nwg) {
    // the plan's fields load again in every iteration (see role_plan): the
    // loop usually runs once, and invariants hoisted out of it would only
    // crowd the scalar registers
    const Plan p = solver_plan(role_plan(p0));
    if (noplan) {
      for (int i = tid; i < G * p.N; i += nt) p.slots_out[(int64_t)d * G * p.N + i] = -1;
      for (int j = tid; j < G; j += nt) p.send_out[d * G + j] = 0;
      if (p.recv_out && d == (int)fdiv((uint32_t)p.self, p.fG))
        for (int r = tid; r < R; r += nt) p.recv_out[r] = 0;
      for (int a = tid; a < I; a += nt) {
        p.seg_e[(int64_t)d * I + a] = -1;
        p.seg_q[(int64_t)d * I + a] = 0;
      }
      continue;
    }
    // stage-1 slots of the domain's ranks: candidate i sits on local rank
    // i mod G, slot i / G; the chosen ones are a prefix of the list, in
    // rows (kept there by the mask loop when the workgroup holds one domain)
    int *sel = rows;
    if (!one_domain) {
      for (int c = tid; c < cap; c += nt) sel[c] = p.repl1[(int64_t)d * cap + c];
      lds_barrier();
    }
    if (tid < 64) {
      // the chosen ones: the prefix before the first empty entry
      int nsel = cap;
      for (int c0 = 0; c0 < cap; c0 += 64) {
        const int c = c0 + tid;
        const uint64_t m = __ballot(c < cap && (unsigned)sel[c] >= (unsigned)E);
        if (m) {
          nsel = c0 + __ffsll((long long)m) - 1;
          break;
        }
      }
      if (tid == 0) misc[3] = nsel;
    }
    lds_barrier();
    const int nsel = misc[3];
    for (int j = tid; j < G; j += nt) {
      const int u = nsel > j ? (int)fdiv((uint32_t)(nsel - j + G - 1), p.fG) : 0;
      used[j] = u;
      for (int t = 0; t < Neff; ++t) slots[j * Neff + t] = t < u ? sel[t * G + j] : -1;
    }
    lds_barrier();
    for (int a = tid; a < I; a += nt) {
      const int j = (int)fdiv((uint32_t)a, p.fPN), pos = a - j * PN;
      int e;
      if (pos < P) e = (d * G + j) * P + pos;
      else e = (pos - P) < used[j] ? slots[j * Neff + pos - P] : -1;
      e_of[a] = e;
      U[a] = 0;
      if (p.lanes) ck[a] = e >= 0 ? (uint64_t)(uint32_t)(pos + 1) << (position_bits(G) * j) : 0;
    }
    lds_barrier();
    if (wg == 0) STAMP(p, 4);
    // whether the domain can refine at all (a rank with a free slot); if not,
    // only the q[self] column is needed, else the columns omega[s][e] of the
    // domain's instances, then q in place
    if (tid < 64) {
      const bool fr = __ballot(tid < G && used[tid] < Neff) != 0;   // G <= 64
      if (tid == 0) misc[5] = fr ? 1 : 0;
    }
    lds_barrier();
    const bool full = misc[5] != 0;
    if (full) {
      for (int t = tid; t < I * R; t += nt) {
        const int s = (int)fdiv((uint32_t)t, p.fI), a = t - s * I;
        const int e = e_of[a];
        qcol[a * p.QS + s] = e < 0 ? 0 : (s == p.self ? hs[e] : p.gl[(int64_t)s * E + e]);
      }
    } else {
      for (int a = tid; a < I; a += nt) {
        const int e = e_of[a];
        qcol[a * p.QS + p.self] = e < 0 ? 0 : hs[e];
      }
    }
    lds_barrier();
    if (wg == 0) STAMP(p, 5);
    route_instances(
        p, I, p.fI, p.rchunks_dom, e_of, mask, fdt, qcol, U, [&](int i, int) { return qcol + i * p.QS; }, 1,
        [&](int) { return d; }, [&](int) { return full; }, [](int, int, int, int) {});
    lds_barrier();
    for (int j = tid; j < G; j += nt) {
      int l = 0;
      for (int pos = 0; pos < PN; ++pos) l += U[j * PN + pos];
      Lr[j] = l;
    }
    lds_barrier();
    if (wg == 0) STAMP(p, 6);
    if (p.general && full) {
      const GenCost gc = general_tables(p, d, sm, lay);
      if (tid < 64) {
        const uint32_t mv = refine_domain<true>(p, d, e_of, U, qcol, slots, used, Lr, ck, &flags, false, gc);
        if (tid == 0 && mv) atomicAdd(&p.ctrl[kCtrlMoves], mv);
      }
    } else if (tid < 64) {
      const uint32_t mv = p.lanes && refine_in_pairs(G, PN)
                              ? refine_domain_in_lanes<kRefinePairs>(p, d, e_of, U, ck, qcol, slots, used, Lr, &flags)
                          : p.lanes ? refine_domain_in_lanes<kRefineLanes>(p, d, e_of, U, ck, qcol, slots, used, Lr, &flags)
                                 : refine_domain<>(p, d, e_of, U, qcol, slots, used, Lr, ck, &flags, false);
      if (tid == 0 && mv) atomicAdd(&p.ctrl[kCtrlMoves], mv);
    }
    lds_barrier();
    if (wg == 0) STAMP(p, 7);
    // outputs of the domain's ranks
    for (int i = tid; i < G * p.N; i += nt) {
      const int j = (int)fdiv((uint32_t)i, p.fN), t = i - j * p.N;
      p.slots_out[(int64_t)(d * G + j) * p.N + t] = (t < used[j]) ? slots[j * Neff + t] : -1;
    }
    for (int j = tid; j < G; j += nt) {
      int sc = 0;
      for (int pos = 0; pos < PN; ++pos) sc += qcol[(j * PN + pos) * p.QS + p.self];
      p.send_out[d * G + j] = sc;
    }
    for (int a = tid; a < I; a += nt) {
      p.seg_e[(int64_t)d * I + a] = e_of[a];
      p.seg_q[(int64_t)d * I + a] = e_of[a] >= 0 ? qcol[a * p.QS + p.self] : 0;
    }
    if (p.recv_out && d == (int)fdiv((uint32_t)p.self, p.fG))
      write_recv_counts(p, (p.self - d * G) * PN, e_of, qcol, full, mask, fdt,
                        [&](int s, int e) { return s == p.self ? hs[e] : p.gl[(int64_t)s * E + e]; },
                        reinterpret_cast<int *>(ck));
    lds_barrier();
  }
  if (tid == 0 && (flags || !synced)) atomicOr(&p.ctrl[kCtrlStatus], flags | (synced ? 0u : TOPOEP_ST_SYNC));

  // ---- the last workgroup to finish lists this rank's instances per expert
  if (wg == 0) STAMP(p, 8);
  drain_then_barrier();
  if (wg == 0) STAMP(p, 9);
  if (wg == 0) STAMP_FLUSH(p, 0, 10);
  if (wg == 0) STAMP_FLUSH(p, 14, 18);
  if (tid == 0) {
    const uint32_t t = __hip_atomic_fetch_add(&p.ctrl[kCtrlTicket], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    misc[4] = t == (uint32_t)nwg - 1;
  }
  __syncthreads();
  if (!misc[4]) return;
  STAMP(p, 10);
  if (!lean || noplan) {
  int *cnt = qcol;                                            // E + 1
  uint32_t *bm = reinterpret_cast<uint32_t *>(qcol + E + 2);  // E * RW
  int *tmp = qcol + E + 2 + E * p.RW;                         // scan scratch (64)
  int *cv = tmp + 64;                                         // nent_cap: shares, then their prefix
  for (int e = tid; e <= E; e += nt) cnt[e] = 0;
  for (int i = tid; i < E * p.RW; i += nt) bm[i] = 0;
  __syncthreads();
  // the domains' instances (expert, share of self): the first kListRegs per
  // thread are read once and kept in registers for the second pass
  auto count = [&](int idx, int e, int q) {
    if ((unsigned)e < (unsigned)E && q > 0) {
      const int d = (int)fdiv((uint32_t)idx, p.fI), a = idx - d * I;
      const int r = d * G + (int)fdiv((uint32_t)a, p.fPN);
      atomicAdd(&cnt[e], 1);
      atomicOr(&bm[e * p.RW + (r >> 5)], 1u << (r & 31));
    }
  };
  auto place = [&](int idx, int e, int q) {
    if ((unsigned)e < (unsigned)E && q > 0) {
      const int d = (int)fdiv((uint32_t)idx, p.fI), a = idx - d * I;
      const int r = d * G + (int)fdiv((uint32_t)a, p.fPN);
      const uint32_t *row = bm + e * p.RW;
      int pos = 0;
      for (int w = 0; w < (r >> 5); ++w) pos += __popc(row[w]);
      pos += __popc(row[r >> 5] & ((1u << (r & 31)) - 1u));
      const int j = cnt[e] + pos;
      p.csr_r[j] = r;
      cv[j] = q;
    }
  };
  int se[kListRegs], sq[kListRegs];
#pragma unroll
  for (int u = 0; u < kListRegs; ++u) {
    const int idx = tid + u * nt;
    se[u] = idx < M * I ? p.seg_e[idx] : -1;
    sq[u] = idx < M * I ? p.seg_q[idx] : 0;
  }
#pragma unroll
  for (int u = 0; u < kListRegs; ++u) count(tid + u * nt, se[u], sq[u]);
  for (int idx = tid + kListRegs * nt; idx < M * I; idx += nt) count(idx, p.seg_e[idx], p.seg_q[idx]);
  __syncthreads();
  STAMP(p, 11);
  block_excl_scan(cnt, E + 1, tmp);
  for (int e = tid; e <= E; e += nt) p.csr_ptr[e] = cnt[e];
#pragma unroll
  for (int u = 0; u < kListRegs; ++u) place(tid + u * nt, se[u], sq[u]);
  for (int idx = tid + kListRegs * nt; idx < M * I; idx += nt) place(idx, p.seg_e[idx], p.seg_q[idx]);
  __syncthreads();
  // cumulative shares per expert, in LDS, then out
  for (int e = tid; e < E; e += nt) {
    int run = 0;
    for (int j = cnt[e]; j < cnt[e + 1]; ++j) {
      run += cv[j];
      cv[j] = run;
    }
  }
  __syncthreads();
  STAMP(p, 12);
  for (int j = tid; j < cnt[E]; j += nt) p.csr_end[j] = cv[j];
  __syncthreads();
  }
  STAMP(p, 13);
  STAMP_FLUSH(p, 10, 14);
  if (tid == 0) {
    uint32_t fin = __hip_atomic_load(&p.ctrl[kCtrlStatus], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    fin |= gst & TOPOEP_ST_RANGE;
    p.ctrl[kCtrlFinal] = fin;
    if (One) atomicOr(reinterpret_cast<unsigned *>(p.status_out), fin);
    else p.status_out[0] = (int32_t)fin;
    p.status_out[1] = (fin & (kNoPlan | TOPOEP_ST_SYNC))
                          ? 0
                          : (int32_t)__hip_atomic_load(&p.ctrl[kCtrlMoves], __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
    // every solver workgroup has taken its ticket, so the words it
    // accumulated are final: restore them for the next solve (which may be
    // this stage again, without a histogram kernel before it); the helpers'
    // count goes back by their number (one still running adds its own last)
    p.ctrl[kCtrlBar] = 0;
    p.ctrl[kCtrlTicket] = 0;
    p.ctrl[kCtrlStatus] = 0;
    p.ctrl[kCtrlMoves] = 0;
    p.ctrl[kCtrlCost] = 0;
    *reinterpret_cast<unsigned long long *>(p.ctrl + kCtrlTotal) = 0ull;
    *reinterpret_cast<unsigned long long *>(p.ctrl + kCtrlSize) = 0ull;
    if (!One)
      __hip_atomic_fetch_sub(&p.ctrl[kCtrlHelpers], (uint32_t)p.n_helpers, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  }
  if constexpr (One) {
    if (p.offs_out && !noplan) {
      for (int r = tid; r < R; r += nt) hs[r] = p.send_out[r];   // (hs: E >= R words, no longer needed)
      lds_barrier();
      solver_send_offsets(p, hs);
    }
    // the instance list, the final status and the send offsets, then the
    // chunks' flags and the next generation
    drain_then_barrier();
    if (tid < 64) {
      const uint32_t next = (uint32_t)misc[kMiscGen] + 1u;
      for (int b = tid; b < p.nb; b += 64)
        __hip_atomic_store(p.flags + (int64_t)b * kFlagStride, next, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      STAMP(p, 46);
      STAMP_FLUSH(p, 46, 47);
      if (tid == 0) __hip_atomic_store(&p.ctrl[kCtrlGen], next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// NT: the most threads per workgroup (launch bounds): the usual 512-thread
// launch gets twice the registers a 1024-thread one may use.
template <int NT>
__global__ __launch_bounds__(NT) void solve_kernel(Plan p0) {
  extern __shared__ int64_t smem_s[];
  int *sm = reinterpret_cast<int *>(smem_s);
  if ((int)blockIdx.x >= p0.n_solvers) {
    block_offsets(p0, blockIdx.x - p0.n_solvers, sm);
    return;
  }
  domain_solver<false>(p0, sm);
}

// ---------------------------------------------------------------- solver: one workgroup for every domain

// LDS state of the single-workgroup solver.
struct SingleState {
  uint64_t *ck, *em;
  FastDiv *fdt;
  int *hs, *ccnt, *dfree, *repl, *slots, *used, *Lr, *e_of, *U, *misc, *om, *qcol;
  uint32_t *mask, *bm;
  int *sendl, *wt;
};

__device__ inline SingleState single_state(const Plan &p, int *sm) {
  SingleLds lay = single_lds(p);
  lay.ck = vgpr(lay.ck);
  lay.em = vgpr(lay.em);
  lay.fdt = vgpr(lay.fdt);
  lay.hs = vgpr(lay.hs);
  lay.cnt = vgpr(lay.cnt);
  lay.dfree = vgpr(lay.dfree);
  lay.mask = vgpr(lay.mask);
  lay.bm = vgpr(lay.bm);
  lay.sendl = vgpr(lay.sendl);
  lay.wt = vgpr(lay.wt);
  lay.repl = vgpr(lay.repl);
  lay.slots = vgpr(lay.slots);
  lay.used = vgpr(lay.used);
  lay.L = vgpr(lay.L);
  lay.e_of = vgpr(lay.e_of);
  lay.U = vgpr(lay.U);
  lay.misc = vgpr(lay.misc);
  lay.om = vgpr(lay.om);
  lay.qcol = vgpr(lay.qcol);
  SingleState t;
  t.ck = reinterpret_cast<uint64_t *>(sm + lay.ck);
  t.em = reinterpret_cast<uint64_t *>(sm + lay.em);
  t.fdt = reinterpret_cast<FastDiv *>(sm + lay.fdt);
  t.hs = sm + lay.hs;
  t.ccnt = sm + lay.cnt;
  t.dfree = sm + lay.dfree;
  t.mask = reinterpret_cast<uint32_t *>(sm + lay.mask);
  t.bm = reinterpret_cast<uint32_t *>(sm + lay.bm);
  t.sendl = sm + lay.sendl;
  t.wt = sm + lay.wt;
  t.repl = sm + lay.repl;
  t.slots = sm + lay.slots;
  t.used = sm + lay.used;
  t.Lr = sm + lay.L;
  t.e_of = sm + lay.e_of;
  t.U = sm + lay.U;
  t.misc = sm + lay.misc;
  t.om = sm + lay.om;
  t.qcol = sm + lay.qcol;
  return t;
}

// misc[0] status bits, misc[2] wait flag, misc[8..9] total load, misc[12]
// refinement moves, misc[14] a domain with a free slot; candidate counts,
// hosting-domain masks, local hosting masks, instance-list bitmaps and send
// counts zero; stage-1 replica lists empty; the divisor table.
__device__ inline void single_init(const Plan &p, const SingleState &t) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (tid < 16) t.misc[tid] = 0;
  for (int d = tid; d < p.M; d += nt) {
    t.ccnt[d] = 0;
    t.dfree[d] = 0;
  }
  for (int i = tid; i < p.E * p.MW; i += nt) t.mask[i] = 0;
  for (int i = tid; i < p.E * p.RW; i += nt) t.bm[i] = 0;
  for (int i = tid; i < p.R; i += nt) t.sendl[i] = 0;
  for (int i = tid; i < p.M * p.cap1; i += nt) t.repl[i] = -1;
  if (!p.lanes)
    for (int i = tid; i < p.M * p.E; i += nt) t.em[i] = 0;
  // candidate keys: ~0 sorts after every candidate (stage1_ranks reads
  // whole parts of 16)
  for (int i = tid; i < p.M * ((p.E + 15) & ~15); i += nt) t.ck[i] = ~0ull;
  build_divisors(p.M, t.fdt);
}

// The rest of the plan when no domain can refine: every domain's replica
// slots are all taken by stage 1 (or a domain holds one rank).  Every expert
// then has at most one instance per domain (stage 1 places one replica per
// domain and expert, never in the main's own domain), a refinement move
// needs a free slot on its target, so none is committed; and this rank's
// share of expert e follows from the routing rule of Section 4.3 alone: all
// of w = omega[self][e] to the instance in dom(self) if there is one, else
// the even split over the n instances, one per hosting domain in ascending
// order: the i-th takes floor(w / n) + [i < w mod n].  The instances with a
// nonzero share are then the first min(n, w), and the i-th of them ends at
// the cumulative share (i + 1) floor(w / n) + min(i + 1, w mod n).
// Phases: the stage-1 lists with the hosting domains and instance ranks;
// per expert its number of entries, scanned within each wave; per (expert,
// domain) the entry of that domain's instance, the send counts and the
// replica slots.  rr: M E words (rank of e's instance in domain d); ex:
// E words (each expert's first entry inside its wave).  Sets misc[15].
__device__ __forceinline__ void fast_finish(const Plan &p, const SingleState &t, const uint64_t *ck, const int *rk,
                                            int *rr, int *ex) {
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E, G = p.G, M = p.M, R = p.R, cap = p.cap1;
  const int E16 = (E + 15) & ~15, lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  const int *om = t.om, *ccnt = t.ccnt;
  int *repl = t.repl;
  uint32_t *mask = t.mask;
  int *sendl = t.sendl, *misc = t.misc, *wt = t.wt;
  const int ds = (int)fdiv((uint32_t)p.self, p.fG);
  if (tid == 0) misc[15] = 1;   // (single_recv_counts: the plan came from here; barriers follow)
  // the stage-1 lists, hosting domains and the rank of each instance
  for (int e = tid; e < E; e += nt) {
    const int dm = (int)fdiv((uint32_t)e, p.fGP);
    atomicOr(&mask[e * p.MW + (dm >> 5)], 1u << (dm & 31));
    rr[dm * E + e] = (int)fdiv((uint32_t)e, p.fP);
  }
  // items idx = d E + c, walked with (d, c) kept as the index advances
  const int dstep = (int)fdiv((uint32_t)nt, p.fE), estep = nt - dstep * E;
  const int dfirst = (int)fdiv((uint32_t)tid, p.fE), efirst = tid - dfirst * E;
  int d = dfirst, c = efirst;
  for (int idx = tid; idx < M * E; idx += nt, d += dstep, c += estep) {
    if (c >= E) {
      c -= E;
      ++d;
    }
    const int rank = rk[idx];
    if (c >= ccnt[d] || rank >= cap) continue;
    const int e = (int)(uint32_t)ck[d * E16 + c];
    repl[d * cap + rank] = e;
    atomicOr(&mask[e * p.MW + (d >> 5)], 1u << (d & 31));
    rr[d * E + e] = d * G + (rank - (int)fdiv_hi((uint32_t)rank, p.fG) * G);
  }
  lds_barrier();
  STAMP(p, 27);
  // per expert: its entries, scanned inside the wave; the waves' totals
  // (experts e and e + blockDim ... take rounds; wt holds 16 totals a round)
  const int rounds = (E + nt - 1) / nt;
  for (int r0 = 0; r0 < rounds; ++r0) {
    const int e = r0 * nt + tid;
    int c = 0;
    if (e < E) {
      const int w = om[p.self * E + e];
      const uint32_t *me = mask + e * p.MW;
      int n = 0;
      for (int wd = 0; wd < p.MW; ++wd) n += __popc(me[wd]);
      c = w <= 0 ? 0 : (((me[ds >> 5] >> (ds & 31)) & 1u) ? 1 : imin(n, w));
    }
    const int incl = wave_incl_scan(c);
    if (e < E) ex[e] = incl - c;
    if (lane == 63 && r0 * nt + wave * 64 < E) wt[r0 * nw + wave] = incl;   // per block of 64 experts
  }
  lds_barrier();
  STAMP(p, 28);
  // per (expert, domain): the entry of the domain's instance
  d = dfirst;
  int e = efirst;
  for (int idx = tid; idx < M * E; idx += nt, d += dstep, e += estep) {
    if (e >= E) {
      e -= E;
      ++d;
    }
    const uint32_t *me = mask + e * p.MW;
    const int w = om[p.self * E + e];
    // the expert's first entry: its place in its wave plus the totals of the
    // waves (and rounds) before it
    int first = ex[e];
    for (int b = 0; b < (e >> 6); ++b) first += wt[b];
    if (d == 0) p.csr_ptr[e] = first;
    if (w <= 0 || !((me[d >> 5] >> (d & 31)) & 1u)) continue;
    const bool local = (me[ds >> 5] >> (ds & 31)) & 1u;
    int i = 0, q = w, end = w;
    if (local) {
      if (d != ds) continue;   // all of w to the instance in dom(self)
    } else {
      int n = 0;
      for (int wd = 0; wd < p.MW; ++wd) {
        n += __popc(me[wd]);
        const int lo = wd * 32;
        if (d >= lo + 32) i += __popc(me[wd]);
        else if (d > lo) i += __popc(me[wd] & ((1u << (d - lo)) - 1u));
      }
      const FastDiv fn = t.fdt[n];
      const int qq = (int)fdiv_hi((uint32_t)w, fn), rem = w - qq * n;
      q = qq + (i < rem ? 1 : 0);
      if (q <= 0) continue;
      end = (i + 1) * qq + imin(i + 1, rem);
    }
    const int r = rr[d * E + e];
    p.csr_r[first + i] = r;
    p.csr_end[first + i] = end;
    atomicAdd(&sendl[r], q);
  }
  if (tid == 0) {
    int all = 0;
    for (int b = 0; b < (E + 63) >> 6; ++b) all += wt[b];
    p.csr_ptr[E] = all;
  }
  lds_barrier();
  STAMP(p, 30);
}

// The lean finish's replica slots and send counts, for the caller alone (no
// chunk reads them, so they go out after the flags): slot t of local rank j
// of domain d holds stage-1 entry t G + j (entries are a prefix of the
// domain's list).
__device__ __forceinline__ void fast_outputs(const Plan &p, const SingleState &t) {
  const int tid = threadIdx.x, nt = blockDim.x, G = p.G, R = p.R, cap = p.cap1;
  for (int i = tid; i < R * p.N; i += nt) {
    const int r = (int)fdiv((uint32_t)i, p.fN), s2 = i - r * p.N;
    const int d = (int)fdiv((uint32_t)r, p.fG), j = r - d * G;
    p.slots_out[i] = s2 < p.Neff ? t.repl[d * cap + s2 * G + j] : -1;
  }
  for (int r = tid; r < R; r += nt) p.send_out[r] = t.sendl[r];
}

// Every step after the load: with Omega' in om (row self = the histogram hs)
// and the status bits gst, plans all domains (Eq. 9 placement, routing,
// Eq. 10 refinement) and writes replica_slots, send_counts, this rank's
// instance list and the final status (ctrl word and status_out).  With
// BAD_ID, NEG_LOAD, RANGE or SYNC in gst only the blank outputs are written.
struct NoHook {
  __device__ void operator()() const {}
};
template <class H> struct IsNoHook { static constexpr bool value = false; };
template <> struct IsNoHook<NoHook> { static constexpr bool value = true; };

template <int Form, class Published = NoHook>
__device__ __forceinline__ void single_plan(const Plan &p, const SingleState &t, uint32_t gst, bool or_status,
                                            Published published = NoHook{}) {
  uint64_t *ck = t.ck, *em = t.em;
  FastDiv *fdt = t.fdt;
  int *hs = t.hs, *ccnt = t.ccnt, *dfree = t.dfree, *repl = t.repl, *slots = t.slots, *used = t.used;
  int *Lr = t.Lr, *e_of = t.e_of, *U = t.U, *misc = t.misc, *om = t.om, *qcol = t.qcol;
  uint32_t *mask = t.mask;
  (void)hs;
  const int tid = threadIdx.x, nt = blockDim.x, wave = tid >> 6, nw = nt >> 6;
  const int E = p.E, G = p.G, R = p.R, M = p.M, I = p.I, P = p.P, PN = p.PN, Neff = p.Neff;
  const int cap = p.cap1;
  if (gst & (kNoPlan | TOPOEP_ST_SYNC)) {
    for (int i = tid; i < R * p.N; i += nt) p.slots_out[i] = -1;
    for (int r = tid; r < R; r += nt) p.send_out[r] = 0;
    if (p.recv_out)
      for (int r = tid; r < R; r += nt) p.recv_out[r] = 0;
    if (tid == 0) {
      p.ctrl[kCtrlFinal] = gst;
      if (or_status) atomicOr(reinterpret_cast<unsigned *>(p.status_out), gst);
      else p.status_out[0] = (int32_t)gst;
      p.status_out[1] = 0;
    }
    return;
  }
  lds_barrier();
  STAMP(p, 23);

  // ---- inter-node placement (Eq. 9), every domain by the whole workgroup
  // (qcol is free until the routing)
  stage1_ranks(p, om, ck, ccnt, qcol);

  // ---- no domain can refine (all slots taken, or one rank per domain):
  // the routing rule alone gives this rank's shares
  {
    bool full = true;
    for (int d = 0; d < M && full; ++d) full = uniform_i32(ccnt[d]) >= cap;
    if (full || G < 2) {
      fast_finish(p, t, ck, qcol, reinterpret_cast<int *>(em), U);
      STAMP(p, 7);
      if (tid == 0) {
        const uint32_t fin = (uint32_t)misc[0] | (gst & TOPOEP_ST_RANGE);
        p.ctrl[kCtrlFinal] = fin;
        misc[45] = (int)fin;   // (kept in LDS past the hook)
      }
      published();
      // the caller's outputs (no chunk reads them)
      fast_outputs(p, t);
      if (tid == 0) {
        const uint32_t fin = (uint32_t)misc[45];
        if (or_status) atomicOr(reinterpret_cast<unsigned *>(p.status_out), fin);
        else p.status_out[0] = (int32_t)fin;
        p.status_out[1] = 0;
      }
      return;
    }
  }
  stage1_lists(p, ck, ccnt, qcol, repl);
  STAMP(p, 2);

  // ---- hosting domains per expert; every rank's slots and instances, and
  // the local ranks hosting each expert in its domain (one pass: stage-1
  // replica i of domain d sits on local rank i mod G, slot i / G, so rank j
  // uses ceil((n_sel - j) / G) slots)
  // (four independent loops over one index space, so each thread runs one
  // loop body instead of one of each)
  {
    const int n1 = M * I, n2 = n1 + E, n3 = n2 + M * cap, n4 = n3 + R;
    for (int v = tid; v < n4; v += nt) {
      if (v < n1) {
        const int idx = v;
        const int d = (int)fdiv((uint32_t)idx, p.fI), a = idx - d * I;
        const int j = (int)fdiv((uint32_t)a, p.fPN), pos = a - j * PN;
        int e;
        if (pos < P) {
          e = (d * G + j) * P + pos;
        } else {
          const int ns = imin(ccnt[d], cap);
          const int u = ns > j ? (int)fdiv((uint32_t)(ns - j + G - 1), p.fG) : 0;
          e = (pos - P) < u ? repl[d * cap + (pos - P) * G + j] : -1;
        }
        e_of[idx] = e;
        U[idx] = 0;
        if constexpr (Form != kRefineLds) {
          em[idx] = e >= 0 ? (uint64_t)(uint32_t)(pos + 1) << (position_bits(G) * j) : 0;
        } else {
          if (e >= 0) atomicOr(reinterpret_cast<unsigned long long *>(&em[d * E + e]), 1ull << (uint32_t)j);
        }
      } else if (v < n2) {
        const int e = v - n1;
        const int dm = (int)fdiv((uint32_t)e, p.fGP);
        atomicOr(&mask[e * p.MW + (dm >> 5)], 1u << (dm & 31));
      } else if (v < n3) {
        const int i = v - n2;
        const int e = repl[i];
        if (e >= 0) {
          const int dd = (int)fdiv((uint32_t)i, p.fCap);
          atomicOr(&mask[e * p.MW + (dd >> 5)], 1u << (dd & 31));
        }
      } else {
        const int r = v - n3;
        const int d = (int)fdiv((uint32_t)r, p.fG), j = r - d * G;
        const int ns = imin(ccnt[d], cap);
        const int u = ns > j ? (int)fdiv((uint32_t)(ns - j + G - 1), p.fG) : 0;
        used[r] = u;
        for (int t = 0; t < Neff; ++t) slots[r * Neff + t] = t < u ? repl[d * cap + t * G + j] : -1;
        if (u < Neff) {
          dfree[d] = 1;
          misc[14] = 1;
        }
      }
    }
  }
  lds_barrier();

  STAMP(p, 3);
  // ---- routing construction (Section 4.3) for every domain's instances;
  // instances of domains that cannot refine enter this rank's instance-list
  // bitmaps and send counts at once
  uint32_t *bm = t.bm;
  int *sendl = t.sendl;
  auto mark = [&](int i, int d, int e, int q) {
    if (q > 0) {
      const int r = d * G + (int)fdiv((uint32_t)(i - d * I), p.fPN);
      atomicOr(&bm[e * p.RW + (r >> 5)], 1u << (r & 31));
      atomicAdd(&sendl[r], q);
    }
  };
  route_instances(
      p, M * I, p.fMI, p.rchunks_all, e_of, mask, fdt, qcol, U, [&](int, int e) { return om + e; }, E,
      [&](int i) { return (int)fdiv((uint32_t)i, p.fI); }, [&](int d) { return dfree[d] != 0; }, mark);
  lds_barrier();
  STAMP(p, 4);

  if (misc[14]) {
    // ---- intra-node refinement (Eq. 10): one wave per domain (it sums its
    // ranks' loads first; a domain without a free slot returns at once)
    uint32_t flags = 0, moves = 0;
    for (int d = wave; d < M; d += nw) {
      if constexpr (Form != kRefineLds)
        moves += refine_domain_in_lanes<Form>(p, d, e_of + d * I, U + d * I, em + d * I, qcol + d * I * p.QS,
                                       slots + d * G * Neff, used + d * G, Lr + d * G, &flags);
      else
        moves += refine_domain<>(p, d, e_of + d * I, U + d * I, qcol + d * I * p.QS, slots + d * G * Neff,
                                 used + d * G, Lr + d * G, em + (int64_t)d * E, &flags, true);
    }
    if (lane_id() == 0) {
      if (flags) atomicOr(reinterpret_cast<unsigned *>(&misc[0]), flags);
      if (moves) atomicAdd(reinterpret_cast<unsigned *>(&misc[12]), moves);
    }
    lds_barrier();
  }
  // (the plan's fields load again: kept across the refinement they would take
  // the registers of its loop)
  const Plan pr = solver_plan(role_plan(p));
  if (misc[14]) {
    // ---- the refined domains' instances enter the bitmaps and send counts
    for (int idx = tid; idx < M * I; idx += nt) {
      const int d = (int)fdiv((uint32_t)idx, pr.fI);
      const int e = e_of[idx], q = qcol[idx * pr.QS + pr.self];
      if (dfree[d] && e >= 0 && q > 0) {
        const int r = d * G + (int)fdiv((uint32_t)(idx - d * I), pr.fPN);
        atomicOr(&bm[e * pr.RW + (r >> 5)], 1u << (r & 31));
        atomicAdd(&sendl[r], q);
      }
    }
    lds_barrier();
  }

  STAMP(p, 5);
  // ---- outputs: replica slots, send counts, this rank's instance list and
  // the final status.  With a hook (the one-launch plan, whose chunks read
  // only the list and the final status word) the caller's outputs wait
  // until the hook has released the chunks.
  constexpr bool defer = !IsNoHook<Published>::value;
  auto caller_outputs = [&]() {
    for (int i = tid; i < R * pr.N; i += nt) {
      const int r = (int)fdiv((uint32_t)i, pr.fN), t2 = i - r * pr.N;
      pr.slots_out[i] = t2 < used[r] ? slots[r * Neff + t2] : -1;
    }
    for (int r = tid; r < R; r += nt) pr.send_out[r] = sendl[r];
    if (tid == 0) {
      const uint32_t fin = (uint32_t)misc[45];
      if (or_status) atomicOr(reinterpret_cast<unsigned *>(pr.status_out), fin);
      else pr.status_out[0] = (int32_t)fin;
      pr.status_out[1] = misc[12];
    }
  };
  if constexpr (!defer) {
    for (int i = tid; i < R * pr.N; i += nt) {
      const int r = (int)fdiv((uint32_t)i, pr.fN), t2 = i - r * pr.N;
      pr.slots_out[i] = t2 < used[r] ? slots[r * Neff + t2] : -1;
    }
    for (int r = tid; r < R; r += nt) pr.send_out[r] = sendl[r];
  }
  STAMP(p, 6);
  emit_instance_list(pr, qcol, slots, used, bm, t.wt);
  STAMP(p, 7);
  if (tid == 0) {
    const uint32_t fin = (uint32_t)misc[0] | (gst & TOPOEP_ST_RANGE);
    pr.ctrl[kCtrlFinal] = fin;
    misc[45] = (int)fin;   // (kept in LDS past the hook)
    if constexpr (!defer) {
      if (or_status) atomicOr(reinterpret_cast<unsigned *>(pr.status_out), fin);
      else pr.status_out[0] = (int32_t)fin;
      pr.status_out[1] = misc[12];
    }
  }
  published();
  if constexpr (defer) caller_outputs();
}

// Receive counts from the single-workgroup solver's final LDS state (after
// single_plan made a plan): the instances on rank self, full columns when
// its domain was routed for every source.  A plan of fast_finish (misc[15])
// kept no instance state: rank self's instances are its mains and its
// stage-1 replicas (slot t = entry t G + j of its domain's list), and the
// routing rule gives every source's share.
__device__ __forceinline__ void single_recv_counts(const Plan &p, const SingleState &t) {
  const int ds = (int)fdiv((uint32_t)p.self, p.fG), E = p.E;
  const int *om = t.om;
  if (t.misc[15]) {
    int *selfe = t.U;
    const int js = p.self - ds * p.G;
    for (int a = threadIdx.x; a < p.PN; a += blockDim.x)
      selfe[a] = a < p.P ? p.self * p.P + a : t.repl[ds * p.cap1 + (a - p.P) * p.G + js];
    lds_barrier();
    write_recv_counts(p, 0, selfe, nullptr, false, t.mask, t.fdt, [&](int s, int e) { return om[s * E + e]; },
                      t.hs);
    return;
  }
  // (hs, the histogram, is no longer needed: it is the scratch)
  write_recv_counts(p, ds * p.I + (p.self - ds * p.G) * p.PN, t.e_of, t.qcol, t.dfree[ds] != 0, t.mask, t.fdt,
                    [&](int s, int e) { return om[s * E + e]; }, t.hs);
}

// Omega to LDS with its status bits and total load (row self included as
// gathered; the caller swaps in the histogram later).  `between` runs on
// every thread once the first loads are issued (LDS set-up that overlaps
// their latency); the status words are written after a barrier behind it.
template <typename Between>
__device__ __forceinline__ void load_omega(const Plan &p, int *om, int *misc, Between between) {
  const int tid = threadIdx.x, nt = blockDim.x, n = p.R * p.E;
  bool neg = false;
  uint64_t tot = 0;
  if ((p.E & 3) == 0 && (reinterpret_cast<uintptr_t>(p.gl) & 15) == 0) {
    const int n4 = n >> 2;
    const int4 *g4 = reinterpret_cast<const int4 *>(p.gl);
    int4 *o4 = reinterpret_cast<int4 *>(om);
    int4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = g4[imin(tid + u * nt, n4 - 1)];
    between();
    for (int i = tid; i < n4; i += 4 * nt) {
      if (i != tid) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = g4[imin(i + u * nt, n4 - 1)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i + u * nt < n4) {
          o4[i + u * nt] = v[u];
          neg |= (v[u].x | v[u].y | v[u].z | v[u].w) < 0;
          tot += (uint64_t)(v[u].x > 0 ? v[u].x : 0) + (uint64_t)(v[u].y > 0 ? v[u].y : 0) +
                 (uint64_t)(v[u].z > 0 ? v[u].z : 0) + (uint64_t)(v[u].w > 0 ? v[u].w : 0);
        }
      }
    }
  } else {
    between();
    for (int i = tid; i < n; i += nt) {
      const int g = p.gl[i];
      om[i] = g;
      neg |= g < 0;
      if (g > 0) tot += (uint64_t)g;
    }
  }
  tot = wave_sum_u64(tot);
  const uint64_t any_neg = __ballot(neg);
  lds_barrier();
  if (lane_id() == 0) {
    if (any_neg) atomicOr(reinterpret_cast<unsigned *>(&misc[0]), TOPOEP_ST_NEG_LOAD);
    if (tot) atomicAdd(reinterpret_cast<unsigned long long *>(misc + 8), (unsigned long long)tot);
  }
}

// Row self of Omega' in om := the histogram hs; SELF_DIFF in misc[0] when the
// gathered row differs, and the total load of misc[8..9] follows.  Ends with
// a barrier.
__device__ __forceinline__ void swap_self_row(const Plan &p, const SingleState &t) {
  bool diff = false;
  int64_t adj = 0;
  for (int e = threadIdx.x; e < p.E; e += blockDim.x) {
    const int h = t.hs[e], g = t.om[p.self * p.E + e];
    diff |= g != h;
    adj += (int64_t)(h > 0 ? h : 0) - (int64_t)(g > 0 ? g : 0);
    t.om[p.self * p.E + e] = h;
  }
  adj = (int64_t)wave_sum_u64((uint64_t)adj);
  const uint64_t any_diff = __ballot(diff);
  if (lane_id() == 0) {
    if (any_diff) atomicOr(reinterpret_cast<unsigned *>(&t.misc[0]), TOPOEP_ST_SELF_DIFF);
    if (adj) atomicAdd(reinterpret_cast<unsigned long long *>(t.misc + 8), (unsigned long long)adj);
  }
  lds_barrier();
}

// The same steps with every domain's state in the LDS of one CU; each
// domain's refinement runs on its own wave.  Used when Omega and all q
// columns fit in LDS.  Workgroups beyond the first compute the histogram
// blocks' offsets for the reroute.  Form: the refinement's form for the shape
// (refine_form), one a kernel: two together spilled registers.
template <int Form>
__global__ __launch_bounds__(1024) void solve_single_kernel(Plan p0) {
  extern __shared__ int64_t smem_1[];
  int *sm = reinterpret_cast<int *>(smem_1);
  if (blockIdx.x > 0) {
    block_offsets(p0, blockIdx.x - 1, sm);
    return;
  }
  {
    // the blocks' bad-id flags and Omega on their way together; row self of
    // Omega := the histogram once the helpers have its totals
    const Plan p = solver_plan(role_plan(p0));
    const SingleState t = single_state(p, sm);
    int bad = 0;
    for (int b = threadIdx.x; b < p.nb; b += blockDim.x) bad |= p.blk_err[b];
    load_omega(p, t.om, t.misc, [&] { single_init(p, t); });
    const uint64_t any_bad = __ballot(bad != 0);
    if (lane_id() == 0 && any_bad) atomicOr(reinterpret_cast<unsigned *>(&t.misc[0]), TOPOEP_ST_BAD_ID);
    row_self(p, t.hs, t.qcol, &t.misc[10]);
    swap_self_row(p, t);
  }
  // (the plan's fields load again: see role_plan)
  const Plan p = solver_plan(role_plan(p0));
  const SingleState t = single_state(p, sm);
  uint32_t gst = (uint32_t)t.misc[0];
  if (out_of_range(p, *reinterpret_cast<const unsigned long long *>(t.misc + 8))) gst |= TOPOEP_ST_RANGE;
  single_plan<Form>(p, t, gst, false);
  if (threadIdx.x == 0)   // (a helper still running adds its own last)
    __hip_atomic_fetch_sub(&p.ctrl[kCtrlHelpers], (uint32_t)p.n_helpers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (p.recv_out && !(gst & kNoPlan)) single_recv_counts(p, t);
}

// ---------------------------------------------------------------- send-buffer slots
//
// The send buffer groups the assignments by destination (ranks ascending,
// row-major order inside one destination).  An assignment's slot is
// offs[d] + (assignments to d before its tile) + (those of earlier waves of
// the tile) + (its rank among its wave's earlier assignments to d).  The
// count before a tile follows from the per-expert counts before it, with no
// pass over earlier ids: expert e's occurrences are dealt to its instances
// in occurrence order, instance j taking [end(j-1), end(j)), so
// clamp(run[e] - end(j-1), 0, end(j) - end(j-1)) of them went to j's rank.

// offs[0..R) holds the send counts: it becomes their exclusive prefix with
// the total at offs[R] (tmp: blockDim/64 + 1 words); `first` writes it out.
__device__ void slot_offsets(const Plan &p, int *offs, int *tmp, bool first) {
  lds_barrier();
  offs[p.R] = block_excl_scan(offs, p.R, tmp);
  if (first && p.offs_out)
    for (int r = threadIdx.x; r <= p.R; r += blockDim.x) p.offs_out[r] = offs[r];
}

// Per-wave counts to offsets, one column per key: wc[(w * ws + k) * S] (w <
// nw <= 16 waves, k < n keys, ws > n odd so a column's words sit in distinct
// banks; S: words per element) becomes base[k] + the counts of waves
// 0..w-1, and base[k] grows by the column's total (base may be null:
// offsets from 0).  Beyond four waves a group of g lanes (g = nw rounded up
// to a power of two) per key scans the column in registers instead of
// walking it with nw dependent LDS round trips.
template <int S = 1>
__device__ inline void scan_wave_columns(int *wc, int ws, int n, int nw, int *base) {
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
  if (nw <= 4) {
    // short columns: one thread walks each
    for (int k = tid; k < n; k += nt) {
      int run = base ? base[k] : 0;
      for (int w = 0; w < nw; ++w) {
        const int t = wc[(w * ws + k) * S];
        wc[(w * ws + k) * S] = run;
        run += t;
      }
      if (base) base[k] = run;
    }
    return;
  }
  const int lg = nw <= 1 ? 0 : 32 - __clz(nw - 1);   // log2 of the group size
  const int g = 1 << lg, w = lane & (g - 1);
  for (int k = tid >> lg; k < n; k += nt >> lg) {
    const int v = w < nw ? wc[(w * ws + k) * S] : 0;
    int x = v;
    // inclusive scan inside the group (row shifts; a group never crosses a row)
    int y;
    y = (int)dpp_mov<0x111>((uint32_t)x); x += w >= 1 ? y : 0;
    y = (int)dpp_mov<0x112>((uint32_t)x); x += w >= 2 ? y : 0;
    y = (int)dpp_mov<0x114>((uint32_t)x); x += w >= 4 ? y : 0;
    y = (int)dpp_mov<0x118>((uint32_t)x); x += w >= 8 ? y : 0;
    const int tot = __shfl(x, lane | (g - 1));
    const int b0 = base ? base[k] : 0;
    if (w < nw) wc[(w * ws + k) * S] = b0 + x - v;
    if (base && w == 0) base[k] = b0 + tot;
  }
}

// ---------------------------------------------------------------- reroute

// The workgroup holds the chunk of the same histogram block.  An expert's
// occurrences go to its instances in order, so when the chunk's occurrences
// of e all lie inside one instance's share they need no rank: one
// destination, looked up by id.  Only an expert whose occurrences run past a
// share's end in this chunk ("crossing") has its ids ranked, tile by tile,
// and there is at most one such (chunk, expert) pair per share end in the
// whole plan, so most chunks stream with no barrier.
//
// td[e]: the destination of e's occurrences in the chunk, or ~j where they
// start in entry j and run past its end; tx[e] is then the index of e's next
// occurrence.
//
// Bound: HBM (4 B read and 4 B written per id): 101 to 122 us for 2^26 ids, E =
// 128, by the inputs, 5.3 to 4.4 TB/s.  Ranking every id (a ballot per id bit) in
// 256-thread blocks, 4096 of them, took 147 us, and the solver summed 4096 rows
// of counts (42 us, now 512 rows, 10): plan 278 -> 151 us.
//
// Slots: also the send-buffer slots.  A wave's piece of a tile is then read
// in 4-byte order (element i of lane l is id i * 64 + l), else as load_ids
// does.
template <int K, bool Slots>
__global__ __launch_bounds__(1024, 8) void reroute_kernel(Plan p) {
  extern __shared__ int smem_r[];
  constexpr int W = K < 4 ? K : 4;   // consecutive ids of a lane (load_ids)
  const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, lane = tid & 63, wave = tid >> 6;
  const int E = p.E, es = E | 1, rs = p.R | 1;
  int2 *ent = reinterpret_cast<int2 *>(smem_r);   // nent_cap: (cumulative share, rank) per entry
  int *td = reinterpret_cast<int *>(ent + p.nent_cap);   // E
  int *tx = td + E;                  // E
  int *ptr = tx + E;                 // E + 1
  int *wc = ptr + E + 1;             // nw * es: per wave a crossing expert's count in the tile, then its next occurrence
  int *wcd = wc + nw * es;           // nw * rs: per wave and rank the count in the tile, then the next slot
  int *so = wcd + nw * rs;           // R + 1 + nw + 1: next slot per rank, scan scratch
  int *flag = so + p.R + nw + 2;     // 1: an expert crosses in this chunk
  const int b = blockIdx.x;
  const int64_t lo = (int64_t)b * p.chunk;
  const int64_t hi = lo + p.chunk < p.n ? lo + p.chunk : p.n;
  const uint32_t fin = p.ctrl[kCtrlFinal];
  if (fin & (kNoPlan | TOPOEP_ST_SYNC)) {
    for (int64_t i = lo + tid; i < hi; i += nt) p.dest_out[i] = -1;
    if (Slots) {
      for (int64_t i = lo + tid; i < hi; i += nt) p.slot_out[i] = -1;
    }
    if (b == 0 && p.offs_out)
      for (int r = tid; r <= p.R; r += nt) p.offs_out[r] = 0;
    return;
  }
  const bool vec = (reinterpret_cast<uintptr_t>(p.topk) & 15) == 0;
  const bool vec_out = (reinterpret_cast<uintptr_t>(p.dest_out) & 15) == 0;
  const int64_t tile = (int64_t)nw * 64 * K, wofs = (int64_t)wave * 64 * K;
  int nx[K];
  auto load_piece = [&](int64_t base) {
    if constexpr (Slots) {
#pragma unroll
      for (int i = 0; i < K; ++i) nx[i] = base + i * 64 + lane < hi ? p.topk[base + i * 64 + lane] : -1;
    } else {
      load_ids<K, true>(p.topk, base, hi, vec, nx);
    }
  };
  // the first tile's ids are on their way while the tables are made
  load_piece(lo + wofs);
  if (p.offs_out) {
    for (int r = tid; r < p.R; r += nt) so[r] = p.send_out[r];
    slot_offsets(p, so, so + p.R + 1, b == 0);
  }
  if (tid == 0) *flag = 0;
  for (int e = tid; e <= E; e += nt) {
    const int v = p.csr_ptr[e];
    ptr[e] = v < 0 ? 0 : (v > p.nent_cap ? p.nent_cap : v);
    if (e < E) {
      tx[e] = p.offsets[(int64_t)b * E + e];
      td[e] = p.partials[(int64_t)b * E + e];
    }
  }
  for (int j = tid; j < p.nent_cap; j += nt) ent[j] = make_int2(p.csr_end[j], p.csr_r[j]);
  __syncthreads();
  bool any = false;
  for (int e = tid; e < E; e += nt) {
    const int start = tx[e], end = start + td[e], j1 = ptr[e + 1];
    // the entry holding occurrence `start`: the first whose cumulative share
    // exceeds it (shares ascend)
    int j = ptr[e];
    if constexpr (Slots) {
      // assignments of earlier chunks per rank: entry j holds occurrences
      // [end(j - 1), end(j))
      int from = 0;
      for (int i = j; i < j1 && from < start; ++i) {
        const int2 en = ent[i];
        const int c = imin(start, en.x) - from;
        if (c > 0 && (unsigned)en.y < (unsigned)p.R) atomicAdd(&so[en.y], c);
        from = en.x;
      }
    }
    for (int top = j1; j < top;) {
      const int mid = (j + top) >> 1;
      if (ent[mid].x <= start) j = mid + 1;
      else top = mid;
    }
    const int2 en = j < j1 ? ent[j] : make_int2(INT_MIN, -1);
    const bool inside = end <= en.x;
    td[e] = inside ? en.y : ~j;
    any |= !inside && end > start;
  }
  if (__ballot(any) && lane == 0) *flag = 1;
  __syncthreads();
  const bool crossing = *flag != 0;
  int *mywc = wc + wave * es, *mywcd = wcd + wave * rs;
  for (int64_t tb = lo; tb < hi; tb += tile) {
    const int64_t base = tb + wofs;
    int ev[K], dv[K];
#pragma unroll
    for (int i = 0; i < K; ++i) ev[i] = nx[i];
    // the next tile's ids load while this one is placed (the barriers below
    // order LDS only, so they do not wait for these loads)
    if (tb + tile < hi) load_piece(base + tile);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const bool valid = (unsigned)ev[i] < (unsigned)E;   // (-1 past the end)
      const int d = td[valid ? ev[i] : 0];
      if (!valid) ev[i] = -1;
      dv[i] = valid ? d : -1;
    }
    if (crossing) {
      // the wave's crossing experts one at a time: each of their ids' rank in
      // the wave's piece (into dv, below the sign bit), the wave's count into
      // its row
      for (int e = lane; e < E; e += 64) mywc[e] = 0;
      wave_sync();
      uint32_t todo = 0;   // this lane's elements not yet ranked
#pragma unroll
      for (int i = 0; i < K; ++i) todo |= (ev[i] >= 0 && dv[i] < 0 ? 1u : 0u) << i;
      uint64_t pend;
      while ((pend = __ballot(todo != 0u)) != 0) {
        int e1 = 0;
#pragma unroll
        for (int i = K - 1; i >= 0; --i) e1 = (todo >> i) & 1u ? ev[i] : e1;
        const int ec = readlane_i32(e1, __ffsll((long long)pend) - 1);
        int seen = 0;
        if constexpr (Slots) {
#pragma unroll
          for (int i = 0; i < K; ++i) {
            const uint64_t m = __ballot(ev[i] == ec);
            if (ev[i] == ec) dv[i] = INT_MIN | count_below(m, seen);
            seen += __popcll(m);
          }
        } else {
#pragma unroll
          for (int j = 0; j < K; j += W) {
            int below = seen;
#pragma unroll
            for (int c = 0; c < W; ++c) {
              const uint64_t m = __ballot(ev[j + c] == ec);
              below = count_below(m, below);
              seen += __popcll(m);
            }
#pragma unroll
            for (int c = 0; c < W; ++c)
              if (ev[j + c] == ec) dv[j + c] = INT_MIN | below++;
          }
        }
        if (lane == 0) mywc[ec] = seen;
#pragma unroll
        for (int i = 0; i < K; ++i)
          if (ev[i] == ec) todo &= ~(1u << i);
      }
      lds_barrier();
      // each wave's first occurrence index of a crossing expert
      for (int e = tid; e < E; e += nt) {
        if (td[e] >= 0) continue;
        int r = tx[e];
        for (int w = 0; w < nw; ++w) {
          const int t = wc[w * es + e];
          wc[w * es + e] = r;
          r += t;
        }
        tx[e] = r;
      }
      lds_barrier();
#pragma unroll
      for (int i = 0; i < K; ++i) {
        if (ev[i] < 0 || dv[i] >= 0) continue;
        const int rho = mywc[ev[i]] + (dv[i] & INT_MAX), j1 = ptr[ev[i] + 1];
        int j = ~td[ev[i]];
        while (j < j1 && ent[j].x <= rho) ++j;
        dv[i] = j < j1 ? ent[j].y : -1;
      }
    }
    if constexpr (Slots) {
      for (int r = lane; r < p.R; r += 64) mywcd[r] = 0;
      wave_sync();
      int lr[K];
#pragma unroll
      for (int i = 0; i < K; ++i) lr[i] = wave_rank(dv[i], (unsigned)dv[i] < (unsigned)p.R, p.rbits, mywcd);
      lds_barrier();
      scan_wave_columns(wcd, rs, p.R, nw, so);
      lds_barrier();
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int64_t idx = base + i * 64 + lane;
        if (idx < hi) {
          const bool valid = (unsigned)dv[i] < (unsigned)p.R;
          p.dest_out[idx] = dv[i];
          p.slot_out[idx] = valid ? mywcd[dv[i]] + lr[i] : -1;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < K; j += W) {
        typedef int words __attribute__((ext_vector_type(W)));
        const int64_t idx = base + (int64_t)(j * 64 + lane * W);
        if (vec_out && idx + W <= hi) {
          words x;
#pragma unroll
          for (int c = 0; c < W; ++c) x[c] = dv[j + c];
          __builtin_nontemporal_store(x, reinterpret_cast<words *>(p.dest_out + idx));
        } else {
#pragma unroll
          for (int c = 0; c < W; ++c)
            if (idx + c < hi) p.dest_out[idx + c] = dv[j + c];
        }
      }
    }
  }
}

// ---------------------------------------------------------------- single-launch plan
//
// Workgroup 0 solves; workgroups 1..nb each hold one chunk of ids.  The
// plan's generation g orders the hand-overs (control words 8..11 above):
//   chunk -> everyone: chunk b writes its count of every expert to
//     pub[b][e] and adds it to the histogram ghist[g & 1][e] with an
//     agent-scope atomic (integer adds commute: the sum does not depend on
//     their order; word E counts bad ids), then makes one release increment
//     of the 64-bit arrival counter; the value it moves the counter from,
//     g nb + c, gives g and tells the last arrival (c = nb - 1).  A chunk
//     reads g from word 10 to pick the histogram buffer before it arrives;
//     that read can only be stale when the solver has already given up on
//     this plan, and the chunk then takes its adds back.
//   last chunk -> chunks: word 1 of every chunk's flag line = g + 1
//     (release): every count is written.  Chunk b then sums its first
//     occurrence index of each expert from the counts of the chunks before
//     it, or from the histogram less the counts of the chunks from b on,
//     whichever reads fewer rows (at most nb / 2).
//   last chunk -> solver: the histogram against row self of Omega, released
//     as the verdict ((g + 1) << 2) | v.  Only the solver polls that word.
//   solver -> chunk b: word 0 of chunk b's flag line = g + 1 (release) once
//     the outputs, this rank's instance list and the final status are
//     written.  Chunk b polls only its own 128-byte flag line, acquires, and
//     reads the instance list in one round trip.
// No word is cleared between plans except the other histogram buffer (by
// the solver, before any chunk of the next plan can use it): a workspace is
// zero-filled before its first plan, and a plan whose bounded wait gave up
// (SYNC) leaves nothing that a later plan's waits could mistake for its own.

// Solver side of a redo: hs[e] = the histogram of local_topk, gh[e] (every
// chunk's adds, acquired with the last chunk's verdict), BAD_ID from gh[E].
__device__ __forceinline__ void read_histogram(const Plan &p, const uint32_t *gh, int *hs, int *misc) {
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E;
  bool bad = false;
  for (int e = tid; e <= E; e += nt) {
    const uint32_t v = gh[e];
    if (e < E) hs[e] = (int)v;
    else bad = v != 0;
  }
  const uint64_t any_bad = __ballot(bad);
  if (lane_id() == 0 && any_bad) atomicOr(reinterpret_cast<unsigned *>(&misc[0]), TOPOEP_ST_BAD_ID);
  __syncthreads();
}

// Solver role (workgroup 0): Omega goes to LDS and the whole plan is made
// from it while the chunks count; once the last chunk has compared the
// histogram with row self of Omega, that plan stands (equal rows, so Omega'
// = Omega) or is made again from Omega' on fresh state; then every chunk's
// flag is set to g + 1 and the generation advances.
template <int Form>
__device__ __forceinline__ void fused_solver(const Plan &p, int *sm) {
  const SingleState t = single_state(p, sm);
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E;
  // this plan's generation (stored by the previous plan's solver); wave 0
  // waits for the verdict and sets the flags
  uint32_t gen = 0;
  if (tid < 64) {
    gen = __hip_atomic_load(&p.ctrl[kCtrlGen], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the next plan's histogram buffer starts from zero (stored long before
    // this plan ends, which is when that plan's chunks may start)
    uint32_t *other = p.ghist + ((gen + 1u) & 1u) * (p.E + 1);
    for (int e = tid; e <= p.E; e += 64) __hip_atomic_store(other + e, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  STAMP_CLEAR(0, 39);
  STAMP(p, 0);
  STAMP_CLK(p, 20);
  if (tid == 0) p.status_out[0] = 0;   // chunks may OR SYNC into it
  load_omega(p, t.om, t.misc, [&] { single_init(p, t); });
  if (tid == 0) {
    t.misc[40] = (int)gen;   // (single_init clears words 0..15 only)
    t.misc[44] = 0;          // the speculative plan went out early
  }
  lds_barrier();
  STAMP(p, 1);
  // Omega's status (single_plan starts with a barrier before any thread
  // writes these words again)
  const uint64_t total0 = uniform_u64(*reinterpret_cast<const unsigned long long *>(t.misc + 8));
  const uint32_t gst0 = ((uint32_t)uniform_i32(t.misc[0]) & TOPOEP_ST_NEG_LOAD) |
                        (out_of_range(p, total0) ? TOPOEP_ST_RANGE : 0u);
  const uint32_t neg0 = gst0 & TOPOEP_ST_NEG_LOAD;
  // Speculative plan from Omega as gathered while the chunks count: it is
  // the plan whenever the histogram equals row self (the gathered row is
  // this rank's own count), else it is redone below; nothing reads the
  // outputs before the flags say the plan is ready.
  const bool spec = !(gst0 & kNoPlan);
  // the flags: every output the chunks read (the instance list, the final
  // status, the send offsets) drained first, then released
  auto release_flags = [&]() {
    STAMP(p, 10);
    STAMP_CLK(p, 21);
    if (tid < 64)
      for (int b = tid; b < p.nb; b += 64)
        __hip_atomic_store(p.flags + (int64_t)b * kFlagStride, gen + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto set_flags = [&]() {
    drain_then_barrier();
    release_flags();
  };
  // as soon as the speculative plan's list and status are written: when the
  // verdict is already in and says the plan stands (the usual case), the
  // flags go out at once
  auto publish_early = [&]() {
    if (tid == 0) {
      const uint32_t v = __hip_atomic_load(&p.ctrl[kCtrlVerdict], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      t.misc[44] = ((v >> 2) == ((gen + 1u) & 0x3FFFFFFFu) && (v & 3u) == kVerdictSame) ? 1 : 0;
    }
    lds_barrier();
    if (t.misc[44]) {
      if (p.offs_out) solver_send_offsets(p, t.sendl);
      set_flags();
    }
  };
  if (spec) single_plan<Form>(p, t, gst0, true, publish_early);   // (with its status: it usually stands)
  STAMP(p, 8);
  const bool early = t.misc[44] != 0;
  // the last chunk's verdict on this generation: its first read overlaps
  // the drain of the speculative outputs
  uint32_t w = 0;
  if (!early && tid == 0) w = __hip_atomic_load(&p.ctrl[kCtrlVerdict], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!early) drain_then_barrier();
  if (early) {
    if (tid == 0) {
      t.misc[2] = 1;
      t.misc[3] = (int)kVerdictSame;
    }
  } else if (tid == 0) {
    const uint32_t want = (gen + 1u) & 0x3FFFFFFFu;
    bool ok = false;
    for (uint32_t it = 0; it < p.spin_limit; ++it) {
      if (it > 0) {
        __builtin_amdgcn_s_sleep(1);
        w = __hip_atomic_load(&p.ctrl[kCtrlVerdict], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if ((w >> 2) == want) {
        ok = true;
        break;
      }
    }
    // acquire: the histogram of a redo, and (passed on by the flags' release)
    // the chunks' counts
    if (ok) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    t.misc[2] = ok;
    t.misc[3] = (int)(w & 3u);
  }
  __syncthreads();
  STAMP(p, 9);
  const bool synced = t.misc[2] != 0;
  const uint32_t verdict = (uint32_t)t.misc[3];
  const bool stands = synced && verdict == kVerdictSame && spec;
  bool planned = stands;
  // a plan that does not stand: its status bits go (a chunk's SYNC stays)
  if (spec && !stands && tid == 0) atomicAnd(reinterpret_cast<unsigned *>(p.status_out), TOPOEP_ST_SYNC);
  // the speculative plan stands (Omega' = Omega) with its status, or: Omega
  // itself refused or a wait given up (blank outputs); or row self differs
  // from the histogram, or a bad id: plan again from Omega' (row self = the
  // histogram) on fresh state
  if (!stands) {
    uint32_t gst = synced ? gst0 : TOPOEP_ST_SYNC;
    if (synced && verdict != kVerdictSame) {
      single_init(p, t);
      lds_barrier();
      read_histogram(p, p.ghist + (int64_t)(t.misc[40] & 1) * (E + 1), t.hs, t.misc);
      if (tid == 0 && neg0) atomicOr(reinterpret_cast<unsigned *>(&t.misc[0]), neg0);
      swap_self_row(p, t);
      gst = (uint32_t)t.misc[0];
      if (out_of_range(p, total0 + *reinterpret_cast<const unsigned long long *>(t.misc + 8))) gst |= TOPOEP_ST_RANGE;
      planned = !(gst & kNoPlan);
    }
    single_plan<Form>(p, t, gst, true);
  }
  if (!early) {
    if (planned && p.offs_out) solver_send_offsets(p, t.sendl);
    set_flags();
  }
  // the next generation
  if (tid == 0) __hip_atomic_store(&p.ctrl[kCtrlGen], gen + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  STAMP_FLUSH(p, 0, 12);
  STAMP_FLUSH(p, 20, 39);
  // receive counts of a plan that was made (a refused one wrote zeros):
  // for the caller only, so they are summed while the chunks route
  if (planned && p.recv_out) single_recv_counts(p, t);
}

// x / d for x < 2^52 and 0 < d < 2^31: the quotient formed in double
// precision (within one of the exact one there), then corrected to the floor.
__device__ inline uint64_t div_u64_small(uint64_t x, uint32_t d) {
  uint64_t q = (uint64_t)((double)x / (double)d);
  int64_t r = (int64_t)(x - q * d);
  while (r < 0) {
    --q;
    r += d;
  }
  while (r >= (int64_t)d) {
    ++q;
    r -= d;
  }
  return q;
}

// The last chunk to arrive (every chunk's counts are in pub and in
// ghist[g & 1]): word 1 of every chunk's flag line (the chunks start summing
// their offsets), then the histogram against row self of Omega and the
// bad-id count, released as the verdict of generation g.
__device__ __forceinline__ void last_arrival(const Plan &p, uint32_t g) {
  const int tid = threadIdx.x, E = p.E;
  if (tid < 64)
    for (int c = tid; c < p.nb; c += 64)
      __hip_atomic_store(p.flags + (int64_t)c * kFlagStride + 1, g + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t *gh = p.ghist + (g & 1u) * (E + 1);
  bool diff = false;
  for (int e = tid; e <= E; e += blockDim.x) {
    const uint32_t v = gh[e];
    diff |= e < E ? (int)v != p.gl[(int64_t)p.self * E + e] : v != 0u;
  }
  const bool redo = __syncthreads_or(diff) != 0;
  if (tid == 0)
    __hip_atomic_store(&p.ctrl[kCtrlVerdict], (((g + 1u) & 0x3FFFFFFFu) << 2) | (redo ? kVerdictRedo : kVerdictSame),
                       __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Bounded wait of chunk b's workgroup until word w of its flag line holds
// `target` (the plan's generation + 1), at most spin_limit polls.  Thread 0
// polls (more pollers per chunk slow every agent-coherent load down), then
// acquires (the L1 and L2 invalidations cover the whole CU).  Returns false
// (on every thread) if the wait gave up.
__device__ __forceinline__ bool wait_flag(const Plan &p, int b, int w, uint32_t target, int *flag) {
  if (threadIdx.x == 0) {
    uint32_t *f = p.flags + (int64_t)b * kFlagStride + w;
    int ok = 0;
    for (uint32_t it = 0; it < p.spin_limit; ++it) {
      if (it > 0) __builtin_amdgcn_s_sleep(2);
      if (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == target) {
        ok = 1;
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *flag = ok;
  }
  __syncthreads();
  return *flag != 0;
}

// Chunk b's first occurrence index of every expert (run[e]) once every
// count is written: the sum of the counts of chunks 0 .. b - 1, or the
// histogram gh less the counts of chunks b .. nb - 1 when that reads fewer
// rows.  Thread (grp, e) sums its share of the rows with eight loads in
// flight; gs: blockDim words of partial sums.
__device__ __forceinline__ void chunk_offsets(const Plan &p, int b, const uint32_t *gh, int *run, int *gs) {
  const int tid = threadIdx.x, nt = blockDim.x, E = p.E, nb = p.nb;
  const bool from_start = 2 * b <= nb;
  const int r0 = from_start ? 0 : b, cnt = from_start ? b : nb - b;
  const int groups = imax(1, nt / E);
  const int per = (cnt + groups - 1) / groups;
  for (int t = tid; t < groups * E; t += nt) {
    const int g = (int)fdiv((uint32_t)t, p.fE), e = t - g * E;
    const int b0 = r0 + g * per, n = imax(0, imin(r0 + cnt, b0 + per) - b0);
    int sum = 0;
    for (int j0 = 0; j0 < n; j0 += 8) {
      uint32_t w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = p.pub[(int64_t)(b0 + imin(j0 + u, n - 1)) * E + e];   // (16-bit loads)
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += j0 + u < n ? (int)w[u] : 0;
    }
    gs[t] = sum;
  }
  __syncthreads();
  for (int e = tid; e < E; e += nt) {
    int sum = 0;
    for (int g = 0; g < groups; ++g) sum += gs[g * E + e];
    run[e] = from_start ? sum : (int)gh[e] - sum;
  }
}

// Send-buffer slots of a chunk of the one-launch plan, with three barriers:
// the counts per rank before the chunk (from run[e] and the instance list,
// into excl, zeroed with the instance-list load) and each wave's ranks by
// destination (its own row of wc, stride E, which only it read before) are
// made together; the wave offsets per rank come from one 16-lane scan per
// rank (lane w of a row holds wave w's count); then the slots.  offs: the
// send offsets.
template <int IPT>
__device__ __forceinline__ void chunk_slots(const Plan &p, const int (&dv)[IPT], int64_t wbase, int64_t hi,
                                            const int *run, const int *ptr, const int2 *ent,
                                            const int *offs, int *excl, int *wc) {
  const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, lane = tid & 63, wave = tid >> 6;
  const int R = p.R, E = p.E;
  for (int e = tid; e < E; e += nt) {
    const int re = run[e], j1 = ptr[e + 1];
    int start = 0;
    for (int j = ptr[e]; j < j1; ++j) {
      const int end = ent[j].x, rk = ent[j].y;
      const int c = imin(imax(re - start, 0), end - start);
      if (c > 0 && (unsigned)rk < (unsigned)R) atomicAdd(&excl[rk], c);
      start = end;
    }
  }
  int *mw = wc + wave * E;
  wave_sync();
  for (int r = lane; r < R; r += 64) mw[r] = 0;
  wave_sync();
  int lr[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    // (dv is -1 past the end)
    lr[i] = wave_rank(dv[i], (unsigned)dv[i] < (unsigned)R, p.rbits, mw);
  }
  lds_barrier();
  // lane w of the row of rank r: wave w's count, scanned across the row
  const int rows = R * 16, span = (rows + 63) & ~63;
  for (int t = tid; t < span; t += nt) {
    const int r = t >> 4, w = t & 15;
    const bool in = t < rows && w < nw;
    const int c = in ? wc[w * E + r] : 0;
    const int incl = row16_incl_scan(c);
    if (in) wc[w * E + r] = incl - c;
  }
  lds_barrier();
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int64_t idx = wbase + i * 64;
    if (idx < hi) {
      const int d = dv[i];
      p.slot_out[idx] = (unsigned)d < (unsigned)R ? offs[d] + excl[d] + mw[d] + lr[i] : -1;
    }
  }
}

// Chunk role (workgroup 1 + b): ids [b * chunk, (b + 1) * chunk) stay in
// registers for the whole plan.  Each wave ranks its ids among equal ids
// (row-major order); the workgroup writes its counts, adds them to the
// histogram and arrives (the last to arrive announces that every count is
// written and sends the verdict); it then sums its first occurrence index
// per expert; once the plan is ready each id's occurrence index rho =
// (offset of the chunk) + (offset of the wave in the chunk) + (rank in the
// wave) picks the instance from this rank's instance list.  A bounded wait
// that gives up writes -1 and SYNC.
template <int IPT, bool One>
__device__ __forceinline__ void fused_chunk(const Plan &p, int b, int *sm) {
  const ChunkLds l = chunk_lds(p, blockDim.x);
  int *wc = sm + l.wc, *run = sm + l.run, *ptr = sm + l.ptr;
  int2 *ent = reinterpret_cast<int2 *>(sm + l.ent);
  int *gs = sm + l.gs, *so = sm + l.so, *flag = sm + l.flag;
  const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, lane = tid & 63, wave = tid >> 6;
  const int E = p.E;
  const int64_t lo = (int64_t)b * p.chunk;
  const int64_t hi = lo + p.chunk < p.n ? lo + p.chunk : p.n;
  const int64_t wbase = lo + (int64_t)wave * 64 * IPT + lane;
  int ev[IPT], lr[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int64_t idx = wbase + i * 64;
    ev[i] = idx < hi ? p.topk[idx] : -1;
  }
  // the generation as the solver left it: the histogram buffer to add to
  const uint32_t gread = __hip_atomic_load(&p.ctrl[kCtrlGen], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // Counting by LDS atomics lets the chunk arrive before its ids are ranked
  // (One, Stress-like, eight ids per thread: 2.6 us after the start, 5.1
  // ranked first); up to 32 experts they meet on too few words, and the short
  // ranks come first.  With the single-workgroup solver, which plans meanwhile,
  // the ranks of the last chunk to arrive are on the path: four or eight ids
  // per thread are ranked first there (EP 64, E = 128, 692 368 ids: 17.8 us,
  // ranked first 16.9; Qwen3-like with dispatch, one id: 11.0 and 11.2).
  constexpr bool count = One || IPT <= 2;
  const bool rank_first = !count || p.nbits <= 5;
  int *mywc = wc + wave * E;
  for (int e = lane; e < E; e += 64) mywc[e] = 0;
  wave_sync();
  int bad = 0;
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int64_t idx = wbase + i * 64;
    const bool inr = idx < hi;
    const bool valid = (unsigned)ev[i] < (unsigned)E;   // (ev is -1 past the end)
    bad |= (inr && !valid) ? 1 : 0;
    if (rank_first) lr[i] = wave_rank(ev[i], valid, p.nbits, mywc);
    else if (valid) atomicAdd(&mywc[ev[i]], 1);
  }
  bad = __syncthreads_or(bad);
  // publish the chunk's counts; wc becomes each wave's offset in the chunk
  uint32_t *gh = p.ghist + (gread & 1u) * (E + 1);
  for (int e = tid; e < E; e += nt) {
    int sum = 0;
    for (int w = 0; w < nw; ++w) {
      const int c = wc[w * E + e];
      wc[w * E + e] = sum;
      sum += c;
    }
    p.pub[(int64_t)b * E + e] = (uint16_t)sum;
    if (sum) atomicAdd(gh + e, (uint32_t)sum);
  }
  if (tid == 0 && bad) atomicAdd(gh + E, 1u);
  drain_then_barrier();
  if (tid == 0) {
    const uint64_t before = __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(p.ctrl + kCtrlArrive), 1ull,
                                                   __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t g = div_u64_small(before, (uint32_t)p.nb);
    const bool last = before - g * (uint64_t)p.nb == (uint64_t)(p.nb - 1);
    // the last arrival acquires every other chunk's counts
    if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    flag[1] = last;
    flag[2] = (int)(uint32_t)g;
  }
  __syncthreads();
  if (b == 0) STAMP(p, 40);
  const uint32_t gen = (uint32_t)flag[2];
  if (gen != gread) {
    // the solver has already given up on this plan and moved on: take the
    // adds back out of the next plan's buffer (it starts after this kernel)
    for (int e = tid; e < E; e += nt) {
      const uint32_t c = p.pub[(int64_t)b * E + e];
      if (c) atomicSub(gh + e, c);
    }
    if (tid == 0 && bad) atomicSub(gh + E, 1u);
  }
  if (flag[1]) {
    STAMP(p, 45);
    last_arrival(p, gen);
    STAMP(p, 41);
    STAMP_FLUSH(p, 41, 42);
    STAMP_FLUSH(p, 45, 46);
  }
  // the ids' occurrence indices in the chunk (each wave counts on from its
  // offset, in its own row), while the other chunks arrive
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const bool valid = (unsigned)ev[i] < (unsigned)E;
    if (!rank_first) lr[i] = wave_rank(ev[i], valid, p.nbits, mywc);
    else if (count) lr[i] += mywc[valid ? ev[i] : 0];
  }
  // every count is written: this chunk's first occurrence index per expert
  bool ok = wait_flag(p, b, 1, gen + 1u, flag);
  if (ok) chunk_offsets(p, b, p.ghist + (gen & 1u) * (E + 1), run, gs);
  if (b == 0) STAMP(p, 44);
  // each id's occurrence index rho = chunk offset + index in the chunk,
  // while the plan is still being made
  __syncthreads();
  int rho[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int e = (unsigned)ev[i] < (unsigned)E ? ev[i] : 0;
    rho[i] = run[e] + lr[i] + (count ? 0 : mywc[e]);
  }
  // the plan is ready
  ok = ok && wait_flag(p, b, 0, gen + 1u, flag);
  if (b == 0) STAMP(p, 42);
  uint32_t fin = 0;
  if (ok) {
    // the instance list and the final status in one round trip: every load
    // of a pass issued before any is used
    fin = __hip_atomic_load(&p.ctrl[kCtrlFinal], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int n_ld = imax(E + 1, p.nent_cap);
    for (int i = tid; i < n_ld; i += nt) {
      const int pv = p.csr_ptr[imin(i, E)];
      const int rv = p.csr_r[imin(i, p.nent_cap - 1)];
      const int xv = p.csr_end[imin(i, p.nent_cap - 1)];
      if (i <= E) ptr[i] = pv < 0 ? 0 : (pv > p.nent_cap ? p.nent_cap : pv);
      if (i < p.nent_cap) ent[i] = make_int2(xv, rv);
    }
    if (p.slot_out) {
      // the send offsets (the solver wrote them) in the same round trip;
      // the per-rank counts before this chunk start from zero
      for (int r = tid; r < p.R; r += nt) {
        so[r] = p.offs_out[r];
        gs[r] = 0;
      }
    }
  }
  if (!ok || (fin & (kNoPlan | TOPOEP_ST_SYNC))) {
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int64_t idx = wbase + i * 64;
      if (idx < hi) {
        p.dest_out[idx] = -1;
        if (p.slot_out) p.slot_out[idx] = -1;
      }
    }
    if (b == 0 && p.offs_out)
      for (int r = tid; r <= p.R; r += nt) p.offs_out[r] = 0;
    if (!ok && tid == 0) atomicOr(reinterpret_cast<unsigned *>(p.status_out), TOPOEP_ST_SYNC);
    return;
  }
  __syncthreads();
  // the destination of each id: the entry of its expert's list that holds its
  // occurrence (shares ascend).  With many domains a list may be long, and is
  // halved down to four entries first (EP 48 over 24 nodes, 800 000 ids: 31.0
  // us walked, 30.1; with four or eight ids per thread and three nodes the
  // halving inside the loop costs 0.3 us, hence the loop of its own)
  const bool long_lists = p.M > (One ? 4 : 8);
  int dv[IPT];
  if (One || long_lists) {
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int64_t idx = wbase + i * 64;
      int dest = -1;
      if (idx < hi) {
        if ((unsigned)ev[i] < (unsigned)E) {
          const int j1 = ptr[ev[i] + 1];
          int j = ptr[ev[i]];
          for (int len = long_lists ? j1 - j : 0; len > 4;) {
            const int half = len >> 1;
            if (ent[j + half - 1].x <= rho[i]) {
              j += half;
              len -= half;
            } else {
              len = half;
            }
          }
          for (; j < j1; ++j) {
            const int2 en = ent[j];
            if (rho[i] < en.x) {
              dest = en.y;
              break;
            }
          }
        }
        p.dest_out[idx] = dest;
      }
      dv[i] = dest;
    }
  } else {
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int64_t idx = wbase + i * 64;
      int dest = -1;
      if (idx < hi) {
        if ((unsigned)ev[i] < (unsigned)E) {
          const int j1 = ptr[ev[i] + 1];
          for (int j = ptr[ev[i]]; j < j1; ++j) {
            const int2 en = ent[j];
            if (rho[i] < en.x) {
              dest = en.y;
              break;
            }
          }
        }
        p.dest_out[idx] = dest;
      }
      dv[i] = dest;
    }
  }
  if (p.slot_out) chunk_slots<IPT>(p, dv, wbase, hi, run, ptr, ent, so, gs, wc);
  if (b == 0) {
    STAMP(p, 43);
    STAMP_FLUSH(p, 40, 41);
    STAMP_FLUSH(p, 42, 45);
  }
}

// The whole plan in one launch: workgroup 0 solves, workgroups 1..nb hold
// the ids; all are resident at once (nb <= kMaxFusedBlocks) and every wait
// is bounded.
// Form: the refinement's form for the shape (refine_form: (instance, target)
// pairs in lanes, instances in lanes, or LDS); one instantiation each keeps
// the others' registers out.
template <int IPT, int Form>
__global__ __launch_bounds__(1024) void plan_fused_kernel(Plan p) {
  extern __shared__ int64_t smem_f[];
  int *sm = reinterpret_cast<int *>(smem_f);
  (void)p;
  if (blockIdx.x == 0) {
    const Plan q = solver_plan(role_plan(p));
    fused_solver<Form>(q, sm);
  } else {
    const Plan q = role_plan(p);
    fused_chunk<IPT, false>(q, blockIdx.x - 1, sm);
  }
}

// The per-domain solver and the chunks in one launch: workgroups 0 ..
// n_solvers - 1 solve one domain each, the nb after them hold the ids.  All
// are resident at once (kMaxOneGroups) and every wait is bounded.  Bound:
// latency.  A Stress-like layer (R = 256, E = 512, 131 072 ids) takes 21 us,
// three kernels 32 (4.8 + 19.3 + 8.2 and their boundaries); a Qwen3-like one
// under a general cost model 23, three kernels 33.
template <int IPT>
__global__ __launch_bounds__(512) void plan_domains_kernel(Plan p) {
  extern __shared__ int64_t smem_d[];
  int *sm = reinterpret_cast<int *>(smem_d);
  if ((int)blockIdx.x < p.n_solvers) {
    domain_solver<true>(p, sm);
  } else {
    const Plan q = role_plan(p);
    fused_chunk<IPT, true>(q, blockIdx.x - q.n_solvers, sm);
  }
}

// Same launch shape, empty body: the launch floor of a plan's kernel.
__global__ __launch_bounds__(1024) void empty_kernel(Plan p) { (void)p; }

// ---------------------------------------------------------------- host side

struct Shape {
  int ipt, bt, st;
  // workspace words beside the control words that must be zero before a
  // first plan (one launch: the ready flags and histogram buffers)
  size_t zero_off, zero_bytes;
  int mode;       // 1 single-workgroup solver, 2 per-domain solver (three kernels each), 3 one launch
  size_t lds_hist, lds_solve, lds_reroute, lds_fused;
  int solve_groups;
  // a plan with the per-domain solver that runs as one launch
  // (plan_domains_kernel): chunk workgroups (0: three kernels), ids per
  // thread, LDS
  int one_nb, one_ipt;
  size_t lds_one;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int ceil_log2(int v) {
  int b = 0;
  while ((1 << b) < v) ++b;
  return b;
}

template <typename K>
void allow_lds(K kernel) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
}

void set_attrs();

// Workgroups of one kernel shape that the current device keeps resident at
// once: its compute units times the shape's occupancy per unit.  Kernels
// whose workgroups wait on each other (the one-launch plan, the per-domain
// solver's grid barrier) are only chosen when every workgroup fits.  A
// device that cannot be queried (no GPU: sizes only) counts as gfx950's
// 256 compute units with one workgroup each, which every shape within the
// LDS and thread limits checked here reaches.  Results are cached.
int resident_capacity(const void *fn, int threads, size_t lds) {
  struct Entry {
    int dev;
    const void *fn;
    int threads;
    size_t lds;
    int cap;
  };
  static std::mutex mu;
  static std::vector<Entry> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return 256;
  }
  {
    std::lock_guard<std::mutex> lock(mu);
    for (const Entry &e : cache)
      if (e.dev == dev && e.fn == fn && e.threads == threads && e.lds == lds) return e.cap;
  }
  set_attrs();
  int cus = 0, occ = 0;
  int cap = 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0 &&
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, threads, lds) == hipSuccess)
    cap = cus * occ;
  (void)hipGetLastError();   // a failed query is not the caller's error
  std::lock_guard<std::mutex> lock(mu);
  cache.push_back(Entry{dev, fn, threads, lds, cap});
  return cap;
}

const void *fused_fn(int ipt, int form);

int refine_form(const Plan &p) {
  return !p.lanes ? kRefineLds : (refine_in_pairs(p.G, p.PN) ? kRefinePairs : kRefineLanes);
}
const void *domains_fn(int ipt);

// Validate the arguments and fill the plan's sizes, launch shape and
// workspace layout (pointers are offsets when ws == nullptr).
int setup(const topoep_topology *t, int32_t T, int32_t k, int32_t N, const topoep_launch *lc, Plan *p,
          Shape *sh, size_t *ws_bytes, char *ws, bool general = false, size_t max_ws = SIZE_MAX) {
  if (!t) return TOPOEP_EINVAL;
  const int R = t->num_ranks, G = t->ranks_per_node, E = t->num_experts;
  if (R <= 0 || G <= 0 || E <= 0 || R % G != 0 || E % R != 0) return TOPOEP_EINVAL;
  if (k < 1 || k > E || T < 0 || (int64_t)T * k > 0x7FFFFFFF || N < 0) return TOPOEP_EINVAL;
  if (t->self_rank < 0 || t->self_rank >= R) return TOPOEP_EINVAL;
  if (t->cost_intra < 0 || t->cost_inter < 0 || t->tok_bytes <= 0 || t->expert_bytes < 0) return TOPOEP_EINVAL;
  if (G > 64) return TOPOEP_ELIMIT;
  Plan q = {};
  q.R = R;
  q.G = G;
  q.M = R / G;
  q.E = E;
  q.P = E / R;
  q.N = N;
  q.Neff = imin(N, E - q.P);
  q.PN = q.P + q.Neff;
  q.I = G * q.PN;
  q.self = t->self_rank;
  q.MW = (q.M + 31) / 32;
  q.RW = (R + 31) / 32;
  q.nbits = ceil_log2(E);
  q.rbits = ceil_log2(R);
  q.cap1 = G * q.Neff;
  q.nent_cap = E + R * q.Neff;
  // odd row stride of the q columns (no LDS bank conflicts) with at least
  // one spare word after the R sources
  q.QS = (R + 1) | 1;
  q.cI = t->cost_intra;
  q.cX = t->cost_inter;
  q.S = t->tok_bytes;
  q.W = t->expert_bytes;
  {
    // the two-level model's range threshold (out_of_range): exact in 128 bits
    const unsigned __int128 lim = (unsigned __int128)1 << 62;
    const uint64_t cm = (uint64_t)imax(imax(q.cI, q.cX), 1);
    const unsigned __int128 rep = (unsigned __int128)(uint64_t)q.W * cm;
    const unsigned __int128 kk = (unsigned __int128)4 * (uint64_t)q.S * cm;
    q.tot_max = rep >= lim ? 0 : (uint64_t)((lim - rep + kk - 1) / kk);
  }
  q.n = (int64_t)T * k;
  q.spin_limit = kSpinLimit;
  q.iter_limit = kIterLimit;
  if (lc) {
    if (lc->spin_limit < -1 || lc->iter_limit < 0) return TOPOEP_EINVAL;
    if (lc->spin_limit == -1) q.spin_limit = 0;   // every bounded wait gives up at once
    else if (lc->spin_limit > 0) q.spin_limit = (uint32_t)lc->spin_limit;
    if (lc->iter_limit > 0) q.iter_limit = (uint32_t)lc->iter_limit;
  }
  q.general = general ? 1 : 0;
  if (general && R > 65535) return TOPOEP_ELIMIT;
  if ((int64_t)q.M * q.I * q.QS >= (1 << 30) || (int64_t)R * E >= (1 << 30)) return TOPOEP_ELIMIT;
  q.fE = make_fastdiv((uint32_t)E);
  q.fG = make_fastdiv((uint32_t)G);
  q.fGP = make_fastdiv((uint32_t)(G * q.P));
  q.fP = make_fastdiv((uint32_t)q.P);
  q.fI = make_fastdiv((uint32_t)q.I);
  q.fPN = make_fastdiv((uint32_t)q.PN);
  q.fCap = make_fastdiv((uint32_t)imax(q.cap1, 1));
  q.fN = make_fastdiv((uint32_t)imax(N, 1));
  q.fMI = make_fastdiv((uint32_t)(q.M * q.I));

  Shape s;
  s.one_nb = s.one_ipt = 0;
  s.lds_one = 0;
  const int ipt_req = lc ? lc->items_per_thread : 0;
  s.ipt = ipt_req ? ipt_req : (q.n >= ((int64_t)1 << 24) ? 8 : 4);
  s.bt = lc && lc->block_threads ? lc->block_threads : 256;
  s.st = lc && lc->solve_threads ? lc->solve_threads : 0;
  const int solver = lc ? lc->solver : 0;
  if (solver < 0 || solver > 3) return TOPOEP_EINVAL;
  if (!(s.ipt == 1 || s.ipt == 2 || s.ipt == 4 || s.ipt == 8)) return TOPOEP_EINVAL;
  if (s.bt < 64 || s.bt > 1024 || s.bt % 64) return TOPOEP_EINVAL;
  if (s.st != 0 && (s.st < 64 || s.st > 1024 || s.st % 64)) return TOPOEP_EINVAL;
  if (lc && lc->tiles_per_block < 0) return TOPOEP_EINVAL;

  // the single-workgroup solver when its whole state fits in LDS
  const int64_t single_words = (int64_t)single_lds(q).words;
  const int64_t multi_words = (int64_t)domain_lds(q).words;
  const bool single_fits = single_words * 4 <= kLdsLimit;
  const bool multi_fits = multi_words * 4 <= kLdsLimit;
  // the lane forms where LDS has room for its words (they take the place of
  // the other form's unless a domain has more instances than experts) beside
  // all that decides which solver runs (1 KiB for the one-launch kernel's
  // static LDS)
  int64_t single_lds_words = single_words, multi_lds_words = multi_words;
  bool single_lanes = false, multi_lanes = false;
  if (refine_in_lanes(q.G, q.PN) && !general) {
    q.lanes = 1;
    const int64_t sw = (int64_t)single_lds(q).words, mw = (int64_t)domain_lds(q).words;
    q.lanes = 0;
    single_lanes = sw * 4 + 1024 <= kLdsLimit;
    multi_lanes = mw * 4 + 1024 <= kLdsLimit;
    if (single_lanes) single_lds_words = sw;
    if (multi_lanes) multi_lds_words = mw;
  }
  q.lanes = single_lanes ? 1 : 0;   // (of the single-workgroup solver until the per-domain one is chosen)

  // one launch: the single-workgroup solver plus at most kMaxFusedBlocks
  // chunk workgroups of st threads holding ipt ids per thread
  {
    const int st = s.st ? s.st : 1024;
    int ipt = 0;
    int64_t nbf = 0;
    for (int c = 1; c <= 8; c *= 2) {
      if (ipt_req && c != ipt_req) continue;
      const int64_t nbc = q.n > 0 ? (q.n + (int64_t)st * c - 1) / ((int64_t)st * c) : 1;
      if (nbc <= kMaxFusedBlocks && (ipt == 0 || nbf > kFusedBlocks)) {
        ipt = c;
        nbf = nbc;
      }
    }
    const int64_t chunk_words = (int64_t)chunk_lds(q, st).words;
    // (1 KiB left for the kernel's static LDS, which __syncthreads_or uses)
    const int64_t fused_words = single_lds_words > chunk_words ? single_lds_words : chunk_words;
    bool fused_ok = single_fits && ipt > 0 && fused_words * 4 + 1024 <= kLdsLimit;
    // every workgroup of the launch resident at once (they wait on each other)
    if (fused_ok)
      fused_ok = nbf + 1 <= resident_capacity(fused_fn(ipt, refine_form(q)), st, (size_t)fused_words * 4);
    if (solver == 3 && !fused_ok) return TOPOEP_ELIMIT;
    if (general && solver == 3) return TOPOEP_EINVAL;   // the general model runs the per-domain solver
    if (fused_ok && !general && (solver == 3 || solver == 0)) {
      s.mode = 3;
      s.ipt = ipt;
      s.st = st;
      q.chunk = (int64_t)st * ipt;
      q.nb = (int)nbf;
      q.n_solvers = 1;
      q.n_helpers = 0;
      s.solve_groups = 1;
      s.lds_hist = s.lds_solve = s.lds_reroute = 0;
      s.lds_fused = (size_t)fused_words * 4;
    } else {
      s.mode = 0;
    }
  }

  int64_t ws_rows = 0;   // rows of the blocks' counts and offsets in the workspace
  if (s.mode != 3) {
  // instance entries, the chunk's table (destination, next occurrence), ptr,
  // per-wave counts of crossing experts, per-wave slots, next slots and scan
  // scratch, a flag
  // (the largest E and R taken come from the layout with (offset, entry)
  // pairs per wave and expert that the reroute had room for)
  const size_t w0 = s.bt / 64;
  const size_t lds_bound = (2 * ((size_t)q.nent_cap + 1) + 2 * (size_t)E + 2 * (size_t)(E | 1) * w0 + (size_t)E +
                            (size_t)E + 1 + (size_t)(R | 1) * w0 + (size_t)R + (size_t)R + 1 + w0 + 1) * 4;
  auto lds_reroute = [&](int bt) {
    const size_t nw = bt / 64;
    return (2 * (size_t)q.nent_cap + 2 * (size_t)E + (size_t)E + 1 + (size_t)(E | 1) * nw + (size_t)(R | 1) * nw +
            (size_t)R + 1 + nw + 1 + 1) * 4;
  };
  const bool given = lc && (lc->items_per_thread || lc->block_threads || lc->tiles_per_block > 0);
  const int64_t tile = (int64_t)s.bt * s.ipt;
  const int64_t tiles = (q.n + tile - 1) / tile;
  // about 16 K ids per block of a small-block launch, 2048..8192 blocks
  const int64_t want = q.n / 16384;
  const int64_t small_blocks = want < kMinBlocks ? kMinBlocks : (want > kMaxBlocks ? kMaxBlocks : want);
  int64_t tpb = lc && lc->tiles_per_block > 0 ? lc->tiles_per_block : (tiles + small_blocks - 1) / small_blocks;
  if (tpb < 1) tpb = 1;
  q.chunk = tpb * tile;
  ws_rows = q.n > 0 ? (q.n + q.chunk - 1) / q.chunk : 1;
  if (ws_rows > (1 << 24)) return TOPOEP_ELIMIT;
  if (!given && q.n > kOneTileIds) {
    // Large blocks of 1024 threads, two per CU: the solver and its helpers
    // read every block's counts (1.6 M ids, E = 256: 1563 blocks of 256
    // threads 52 us a plan, 196 of these 28).  The workspace
    // keeps its rows, more than these blocks need: its size, and with it
    // which plans the no-allocation array takes, is not the launch's.
    s.ipt = 8;
    s.bt = 1024;
    while (s.bt > 256 && lds_reroute(s.bt) > (size_t)kLdsLimit) s.bt >>= 1;
    const int64_t big = (int64_t)s.bt * s.ipt;
    q.chunk = big;
    if (q.n > big * kLongBlocks) q.chunk = (q.n + (int64_t)kLongBlocks * 64 - 1) / ((int64_t)kLongBlocks * 64) * 64;
  }
  q.nb = q.n > 0 ? (int)((q.n + q.chunk - 1) / q.chunk) : 1;
  q.n_helpers = (E + kOffsetExperts - 1) / kOffsetExperts;
  if (general) {
    if (solver == 1) return TOPOEP_EINVAL;
    if (!multi_fits) return TOPOEP_ELIMIT;
    s.mode = 2;
  } else if (solver == 1) {
    if (!single_fits) return TOPOEP_ELIMIT;
    s.mode = 1;
  } else if (solver == 2) {
    if (!multi_fits) return TOPOEP_ELIMIT;
    s.mode = 2;
  } else {
    if (!single_fits && !multi_fits) return TOPOEP_ELIMIT;
    s.mode = single_fits ? 1 : 2;
  }
  if (s.st == 0) s.st = s.mode == 1 ? 1024 : 512;
  if (s.mode == 2) q.lanes = multi_lanes ? 1 : 0;
  s.lds_solve = (size_t)(s.mode == 1 ? single_lds_words : multi_lds_words) * 4;
  q.n_solvers = s.mode == 1 ? 1 : imin(q.M, kMaxSolveGroups);
  // the per-domain solver's workgroups meet at a grid barrier: all resident
  if (s.mode == 2 && q.n_solvers > resident_capacity(s.st <= 512 ? reinterpret_cast<const void *>(solve_kernel<512>)
                                                                  : reinterpret_cast<const void *>(solve_kernel<1024>),
                                                     s.st, s.lds_solve))
    return TOPOEP_ELIMIT;
  s.solve_groups = q.n_solvers + q.n_helpers;
  // The whole plan in one launch when one workgroup per domain and the
  // chunks' workgroups together fill at most a quarter of the device: they
  // wait on each other, and so up to four such plans on four hardware queues
  // are resident together.  Two ids per thread while that keeps to 32
  // chunks, else eight.
  if (s.mode == 2 && solver == 0 && !given && !(lc && lc->solve_threads) && q.n_solvers == q.M) {
    for (int ipt = 2; ipt <= 8 && s.one_nb == 0; ipt *= 4) {
      const int64_t per = (int64_t)kOneThreads * ipt;
      const int64_t nbo = q.n > 0 ? (q.n + per - 1) / per : 1;
      const int64_t chunk_words = (int64_t)chunk_lds(q, kOneThreads).words;
      const int64_t words = multi_lds_words > chunk_words ? multi_lds_words : chunk_words;
      if (nbo > kFusedBlocks && ipt < 8) continue;
      if (words * 4 + 1024 > kLdsLimit || q.n_solvers + nbo > kMaxOneGroups) continue;
      if (4 * (q.n_solvers + nbo) > resident_capacity(domains_fn(ipt), kOneThreads, (size_t)words * 4)) continue;
      s.one_nb = (int)nbo;
      s.one_ipt = ipt;
      s.lds_one = (size_t)words * 4;
    }
  }
  s.lds_hist = (size_t)E * 4;
  s.lds_reroute = lds_reroute(s.bt);
  s.lds_fused = 0;
  if (lds_bound > (size_t)kLdsLimit) return TOPOEP_ELIMIT;
  }

  // routing: the largest divisor c of M with (instances routed at once) * c
  // <= solver threads, so every thread routes whole source domains
  auto chunks_for = [&](int64_t ni) {
    int best = 1;
    for (int c = 1; c <= q.M; ++c)
      if (q.M % c == 0 && ni * c <= s.st) best = c;
    return best;
  };
  q.rchunks_all = chunks_for((int64_t)q.M * q.I);
  q.rchunks_dom = chunks_for(q.I);
  q.s1_waves = (s.st / 64) / q.M;
  q.fS1 = make_fastdiv((uint32_t)imax(q.s1_waves, 1));

  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  // The control words, the three-kernel plan's buffers, then the one-launch
  // plan's: a plan with the per-domain solver that runs as one launch keeps
  // both (its stages run alone too), and its own words lie behind everything
  // a three-kernel plan of the same shape writes, so launches of one shape
  // share a workspace in any order, and one without room for both (max_ws)
  // runs the plan as three kernels.  Large batches take fewer rows of counts
  // than the workspace has room for (ws_rows); the room lies behind the rows,
  // so the layout follows from the shape alone.
  const bool one = s.mode == 3;
  const bool three = !one;
  const size_t o_ctrl = take(kCtrlBytes);
  const size_t o_repl = take(s.mode == 2 ? (size_t)q.M * imax(q.cap1, 1) * 4 : 0);
  const size_t o_sege = take(s.mode == 2 ? (size_t)q.M * q.I * 4 : 0);
  const size_t o_segq = take(s.mode == 2 ? (size_t)q.M * q.I * 4 : 0);
  const size_t o_cptr = take((size_t)(E + 1) * 4);
  const size_t o_cr = take((size_t)q.nent_cap * 4);
  const size_t o_ce = take((size_t)q.nent_cap * 4);
  const size_t o_ht = take(three ? (size_t)E * 4 : 0);
  const size_t o_rows = off;
  const size_t o_part = take(three ? (size_t)q.nb * E * 4 : 0);
  const size_t o_offs = take(three ? (size_t)q.nb * E * 4 : 0);
  const size_t o_berr = take(three ? (size_t)q.nb * 4 : 0);
  if (three) off = o_rows + 2 * align256((size_t)ws_rows * E * 4) + align256((size_t)ws_rows * 4);
  const size_t three_bytes = off;
  int chunks = one ? q.nb : s.one_nb;   // one launch: chunk workgroups
  const size_t o_flg = take((size_t)chunks * kFlagStride * 4);
  const size_t o_gh = take(chunks ? (size_t)2 * (E + 1) * 4 : 0);
  s.zero_off = o_flg;
  s.zero_bytes = off - o_flg;
  const size_t o_pub = take((size_t)chunks * E * 2);
  if (s.one_nb > 0 && off > max_ws) {   // no room for one launch: three kernels
    chunks = s.one_nb = 0;
    s.zero_bytes = 0;
    off = three_bytes;
  }
  *ws_bytes = off;
  if (ws) {
    auto at = [&](size_t o, bool have) { return have ? reinterpret_cast<int32_t *>(ws + o) : nullptr; };
    auto atu = [&](size_t o, bool have) { return have ? reinterpret_cast<uint32_t *>(ws + o) : nullptr; };
    q.ctrl = atu(o_ctrl, true);
    q.partials = at(o_part, three);
    q.offsets = at(o_offs, three);
    q.blk_err = at(o_berr, three);
    q.repl1 = at(o_repl, s.mode == 2);
    q.seg_e = at(o_sege, s.mode == 2);
    q.seg_q = at(o_segq, s.mode == 2);
    q.csr_ptr = at(o_cptr, true);
    q.csr_r = at(o_cr, true);
    q.csr_end = at(o_ce, true);
    q.htot = at(o_ht, three);
    q.flags = atu(o_flg, chunks > 0);
    q.pub = chunks > 0 ? reinterpret_cast<uint16_t *>(ws + o_pub) : nullptr;
    q.ghist = atu(o_gh, chunks > 0);
  }
  *p = q;
  *sh = s;
  return TOPOEP_OK;
}

std::atomic<bool> g_attrs_set{false};

template <int IPT>
const void *fused_fn_ipt(int form) {
  return form == kRefineLanes ? reinterpret_cast<const void *>(plan_fused_kernel<IPT, kRefineLanes>)
         : form == kRefinePairs ? reinterpret_cast<const void *>(plan_fused_kernel<IPT, kRefinePairs>)
                              : reinterpret_cast<const void *>(plan_fused_kernel<IPT, kRefineLds>);
}

const void *fused_fn(int ipt, int form) {
  switch (ipt) {
    case 1: return fused_fn_ipt<1>(form);
    case 2: return fused_fn_ipt<2>(form);
    case 4: return fused_fn_ipt<4>(form);
    default: return fused_fn_ipt<8>(form);
  }
}

const void *domains_fn(int ipt) {
  return ipt == 2 ? reinterpret_cast<const void *>(plan_domains_kernel<2>)
                  : reinterpret_cast<const void *>(plan_domains_kernel<8>);
}

void set_attrs() {
  if (g_attrs_set) return;
  allow_lds(plan_domains_kernel<2>);
  allow_lds(plan_domains_kernel<8>);
  allow_lds(hist_kernel<1, false>);
  allow_lds(hist_kernel<2, false>);
  allow_lds(hist_kernel<4, false>);
  allow_lds(hist_kernel<8, false>);
  allow_lds(hist_kernel<8, true>);
  allow_lds(reroute_kernel<1, false>);
  allow_lds(reroute_kernel<2, false>);
  allow_lds(reroute_kernel<4, false>);
  allow_lds(reroute_kernel<4, true>);
  allow_lds(reroute_kernel<8, false>);
  allow_lds(solve_kernel<512>);
  allow_lds(solve_kernel<1024>);
  allow_lds(solve_single_kernel<kRefineLanes>);
  allow_lds(solve_single_kernel<kRefinePairs>);
  allow_lds(solve_single_kernel<kRefineLds>);
  allow_lds(plan_fused_kernel<1, kRefineLds>);
  allow_lds(plan_fused_kernel<1, kRefinePairs>);
  allow_lds(plan_fused_kernel<1, kRefineLanes>);
  allow_lds(plan_fused_kernel<2, kRefineLds>);
  allow_lds(plan_fused_kernel<2, kRefinePairs>);
  allow_lds(plan_fused_kernel<2, kRefineLanes>);
  allow_lds(plan_fused_kernel<4, kRefineLds>);
  allow_lds(plan_fused_kernel<4, kRefinePairs>);
  allow_lds(plan_fused_kernel<4, kRefineLanes>);
  allow_lds(plan_fused_kernel<8, kRefineLds>);
  allow_lds(plan_fused_kernel<8, kRefinePairs>);
  allow_lds(plan_fused_kernel<8, kRefineLanes>);
  allow_lds(empty_kernel);
  // (an attribute a kernel refuses must not linger as the caller's error)
  (void)hipGetLastError();
  g_attrs_set = true;
}

void launch_hist(const Plan &p, const Shape &s, hipStream_t st) {
  const dim3 g(p.nb), b(s.bt);
  switch (s.ipt) {
    case 1: hipLaunchKernelGGL((hist_kernel<1, false>), g, b, s.lds_hist, st, p); break;
    case 2: hipLaunchKernelGGL((hist_kernel<2, false>), g, b, s.lds_hist, st, p); break;
    case 4: hipLaunchKernelGGL((hist_kernel<4, false>), g, b, s.lds_hist, st, p); break;
    default:
      if (p.n > kStreamIds) hipLaunchKernelGGL((hist_kernel<8, true>), g, b, s.lds_hist, st, p);
      else hipLaunchKernelGGL((hist_kernel<8, false>), g, b, s.lds_hist, st, p);
  }
}

// (with slots four ids a tile: eight spill the 64 registers of two blocks a CU)
void launch_reroute(const Plan &p, const Shape &s, hipStream_t st) {
  const dim3 g(p.nb), b(s.bt);
  if (p.slot_out) hipLaunchKernelGGL((reroute_kernel<4, true>), g, b, s.lds_reroute, st, p);
  else if (s.ipt == 1) hipLaunchKernelGGL((reroute_kernel<1, false>), g, b, s.lds_reroute, st, p);
  else if (s.ipt == 2) hipLaunchKernelGGL((reroute_kernel<2, false>), g, b, s.lds_reroute, st, p);
  else if (s.ipt == 4) hipLaunchKernelGGL((reroute_kernel<4, false>), g, b, s.lds_reroute, st, p);
  else hipLaunchKernelGGL((reroute_kernel<8, false>), g, b, s.lds_reroute, st, p);
}

void launch_solve(const Plan &p, const Shape &s, hipStream_t st) {
  const dim3 g(s.solve_groups), b(s.st);
  const int form = refine_form(p);
  if (s.mode == 1 && form == kRefineLanes)
    hipLaunchKernelGGL((solve_single_kernel<kRefineLanes>), g, b, s.lds_solve, st, p);
  else if (s.mode == 1 && form == kRefinePairs)
    hipLaunchKernelGGL((solve_single_kernel<kRefinePairs>), g, b, s.lds_solve, st, p);
  else if (s.mode == 1)
    hipLaunchKernelGGL((solve_single_kernel<kRefineLds>), g, b, s.lds_solve, st, p);
  else if (s.st <= 512) hipLaunchKernelGGL(solve_kernel<512>, g, b, s.lds_solve, st, p);
  else hipLaunchKernelGGL(solve_kernel<1024>, g, b, s.lds_solve, st, p);
}

template <int IPT>
void launch_fused_ipt(int form, dim3 g, dim3 b, size_t lds, hipStream_t st, const Plan &p) {
  if (form == kRefineLanes) hipLaunchKernelGGL((plan_fused_kernel<IPT, kRefineLanes>), g, b, lds, st, p);
  else if (form == kRefinePairs) hipLaunchKernelGGL((plan_fused_kernel<IPT, kRefinePairs>), g, b, lds, st, p);
  else hipLaunchKernelGGL((plan_fused_kernel<IPT, kRefineLds>), g, b, lds, st, p);
}

void launch_fused(const Plan &p, const Shape &s, hipStream_t st) {
  const dim3 g(p.nb + 1), b(s.st);
  const int form = refine_form(p);
  switch (s.ipt) {
    case 1: launch_fused_ipt<1>(form, g, b, s.lds_fused, st, p); break;
    case 2: launch_fused_ipt<2>(form, g, b, s.lds_fused, st, p); break;
    case 4: launch_fused_ipt<4>(form, g, b, s.lds_fused, st, p); break;
    default: launch_fused_ipt<8>(form, g, b, s.lds_fused, st, p); break;
  }
}

// The one-launch plan with the per-domain solver: p's chunks are this
// launch's.
void launch_domains(Plan p, const Shape &s, hipStream_t st) {
  p.nb = s.one_nb;
  p.chunk = (int64_t)kOneThreads * s.one_ipt;
  const dim3 g(p.n_solvers + p.nb), b(kOneThreads);
  if (s.one_ipt == 2) hipLaunchKernelGGL(plan_domains_kernel<2>, g, b, s.lds_one, st, p);
  else hipLaunchKernelGGL(plan_domains_kernel<8>, g, b, s.lds_one, st, p);
}

// Kernels of one plan in launch order: grid, threads, dynamic LDS (with the
// per-domain solver its three stages', also where the plan is one launch).
int plan_kernels(const Plan &p, const Shape &s, int grid[3], int block[3], size_t lds[3]) {
  if (s.mode == 3) {
    grid[0] = p.nb + 1;
    block[0] = s.st;
    lds[0] = s.lds_fused;
    return 1;
  }
  grid[0] = p.nb;
  block[0] = s.bt;
  lds[0] = s.lds_hist;
  grid[1] = s.solve_groups;
  block[1] = s.st;
  lds[1] = s.lds_solve;
  grid[2] = p.nb;
  block[2] = s.bt;
  lds[2] = s.lds_reroute;
  return 3;
}

constexpr int kFloorMask = 8;

int enqueue(int stage_mask, const topoep_topology *topo, const int32_t *global_load,
            const int32_t *local_topk, int32_t T, int32_t k, int32_t N, int32_t *replica_slots,
            int32_t *token_dest, int32_t *send_counts, int32_t *status, void *workspace,
            size_t workspace_bytes, void *stream, const topoep_launch *launch,
            int32_t *recv_counts = nullptr, int32_t *send_offsets = nullptr, int32_t *token_slot = nullptr,
            const topoep_costs *costs = nullptr) {
  Plan p;
  Shape s;
  size_t need = 0;
  const bool general = costs != nullptr;
  const int rc = setup(topo, T, k, N, launch, &p, &s, &need, static_cast<char *>(workspace), general, workspace_bytes);
  if (rc != TOPOEP_OK) return rc;
  if (!global_load || !send_counts || !status || !workspace) return TOPOEP_EINVAL;
  if ((int64_t)topo->num_ranks * N > 0 && !replica_slots) return TOPOEP_EINVAL;
  if (T > 0 && (!local_topk || !token_dest)) return TOPOEP_EINVAL;
  if (workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TOPOEP_EWORKSPACE;
  p.Cm = general ? costs->cost : nullptr;
  p.We = general ? costs->expert_bytes : nullptr;
  p.gl = global_load;
  p.topk = local_topk;
  p.slots_out = replica_slots;
  p.dest_out = token_dest;
  p.send_out = send_counts;
  p.status_out = status;
  p.recv_out = recv_counts;
  p.offs_out = send_offsets;
  p.slot_out = send_offsets ? token_slot : nullptr;   // (null when T == 0: offsets only)
  set_attrs();
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  if (stage_mask == kFloorMask) {
    int grid[3], block[3];
    size_t lds[3];
    int nk = plan_kernels(p, s, grid, block, lds);
    if (s.one_nb > 0) {   // the one kernel of the plan, not its stages
      nk = 1;
      grid[0] = p.n_solvers + s.one_nb;
      block[0] = kOneThreads;
      lds[0] = s.lds_one;
    }
    for (int i = 0; i < nk; ++i) hipLaunchKernelGGL(empty_kernel, dim3(grid[i]), dim3(block[i]), lds[i], st, p);
  } else if (s.mode == 3) {
    if (stage_mask != 7 && stage_mask != 1) return TOPOEP_EINVAL;   // one kernel: the plan, or stage 0
    launch_fused(p, s, st);
  } else if (s.one_nb > 0 && stage_mask == 7) {
    launch_domains(p, s, st);
  } else {
    // a plan that ran as one launch has left no counts or offsets of the
    // blocks: a later stage alone brings the stages before it
    const int mask = s.one_nb > 0 ? (stage_mask << 1) - 1 : stage_mask;
    if (mask & 1) launch_hist(p, s, st);
    if (mask & 2) launch_solve(p, s, st);
    if (mask & 4) launch_reroute(p, s, st);
  }
  return hipGetLastError() == hipSuccess ? TOPOEP_OK : TOPOEP_EHIP;
}

// ---------------------------------------------------------------- no-allocation entry point
//
// topoep_plan_noalloc plans into `scratch`, a device array of fixed size in
// place of a caller's workspace: one copy per GPU the library runs on, held
// until the process ends.  In host code the array's name is only a
// host-side stand-in; kernels and the clearing launch get the device
// address hipGetSymbolAddress returns for the current device, looked up
// once per device and kept.

constexpr size_t kScratchBytes = TOPOEP_NOALLOC_SCRATCH_BYTES;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];

int scratch_address(void **out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return TOPOEP_EHIP;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
      (void)hipGetLastError();
      return TOPOEP_EHIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return TOPOEP_OK;
}

// Zero the control words at w and n more words at w2 (what a first plan needs
// zero): a kernel, so that the clearing can be captured in a HIP graph like
// the plan itself.
__global__ __launch_bounds__(256) void zero_words(uint32_t *w, uint32_t *w2, int64_t n) {
  constexpr int kCtrlWords = kCtrlBytes / 4;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kCtrlWords) w[i] = 0u;
  else if (i - kCtrlWords < n) w2[i - kCtrlWords] = 0u;
}

}  // namespace

extern "C" {

int topoep_plan_noalloc(const topoep_topology *topo, const int32_t *global_load, const int32_t *local_topk,
                        int32_t T, int32_t k, int32_t replica_budget, int32_t *replica_slots, int32_t *token_dest,
                        int32_t *send_counts, int32_t *status, void *stream) {
  Plan p;
  Shape s;
  size_t need = 0;
  int rc = setup(topo, T, k, replica_budget, nullptr, &p, &s, &need, nullptr, false, kScratchBytes);
  if (rc != TOPOEP_OK) return rc;
  // the argument checks of topoep_plan, before anything is enqueued
  if (!global_load || !send_counts || !status) return TOPOEP_EINVAL;
  if ((int64_t)topo->num_ranks * replica_budget > 0 && !replica_slots) return TOPOEP_EINVAL;
  if (T > 0 && (!local_topk || !token_dest)) return TOPOEP_EINVAL;
  if (need > kScratchBytes) return TOPOEP_EWORKSPACE;
  void *ws = nullptr;
  rc = scratch_address(&ws);
  if (rc != TOPOEP_OK) return rc;
  // the previous call may have been another shape: clear what this plan
  // needs zero (control words, flags, histogram buffers)
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  const int64_t words = (int64_t)(s.zero_bytes / 4);
  hipLaunchKernelGGL(zero_words, dim3((unsigned)((kCtrlBytes / 4 + words + 255) / 256)), dim3(256), 0, st,
                     static_cast<uint32_t *>(ws), reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + s.zero_off),
                     words);
  if (hipGetLastError() != hipSuccess) return TOPOEP_EHIP;
  return enqueue(7, topo, global_load, local_topk, T, k, replica_budget, replica_slots, token_dest, send_counts,
                 status, ws, kScratchBytes, stream, nullptr);
}

int topoep_workspace_bytes_ex(const topoep_topology *topo, int32_t T, int32_t k, int32_t replica_budget,
                              const topoep_launch *launch, size_t *bytes_out) {
  if (!bytes_out) return TOPOEP_EINVAL;
  Plan p;
  Shape s;
  size_t need = 0;
  const int rc = setup(topo, T, k, replica_budget, launch, &p, &s, &need, nullptr);
  if (rc == TOPOEP_OK) *bytes_out = need;
  return rc;
}

int topoep_workspace_bytes(const topoep_topology *topo, int32_t T, int32_t k, int32_t replica_budget,
                           size_t *bytes_out) {
  return topoep_workspace_bytes_ex(topo, T, k, replica_budget, nullptr, bytes_out);
}

int topoep_plan_ex(const topoep_topology *topo, const int32_t *global_load, const int32_t *local_topk,
                   int32_t T, int32_t k, int32_t replica_budget, int32_t *replica_slots,
                   int32_t *token_dest, int32_t *send_counts, int32_t *status, void *workspace,
                   size_t workspace_bytes, void *stream, const topoep_launch *launch) {
  return enqueue(7, topo, global_load, local_topk, T, k, replica_budget, replica_slots, token_dest,
                 send_counts, status, workspace, workspace_bytes, stream, launch);
}

int topoep_plan_shape(const topoep_topology *topo, int32_t T, int32_t k, int32_t replica_budget,
                      const topoep_launch *launch, topoep_shape *out) {
  if (!out) return TOPOEP_EINVAL;
  Plan p;
  Shape s;
  size_t need = 0;
  const int rc = setup(topo, T, k, replica_budget, launch, &p, &s, &need, nullptr);
  if (rc != TOPOEP_OK) return rc;
  int grid[3] = {0, 0, 0}, block[3] = {0, 0, 0};
  size_t lds[3] = {0, 0, 0};
  topoep_shape o = {};
  o.kernels = plan_kernels(p, s, grid, block, lds);
  o.solver = s.mode;
  o.items_per_thread = s.ipt;
  o.chunk_blocks = p.nb;
  for (int i = 0; i < 3; ++i) {
    o.grid[i] = grid[i];
    o.block[i] = block[i];
    o.lds_bytes[i] = (int32_t)lds[i];
  }
  *out = o;
  return TOPOEP_OK;
}

int topoep_plan(const topoep_topology *topo, const int32_t *global_load, const int32_t *local_topk,
                int32_t T, int32_t k, int32_t replica_budget, int32_t *replica_slots, int32_t *token_dest,
                int32_t *send_counts, int32_t *status, void *workspace, size_t workspace_bytes,
                void *stream) {
  return enqueue(7, topo, global_load, local_topk, T, k, replica_budget, replica_slots, token_dest,
                 send_counts, status, workspace, workspace_bytes, stream, nullptr);
}

int topoep_dispatch_workspace_bytes(const topoep_topology *topo, int32_t T, int32_t k, int32_t replica_budget,
                                    size_t *bytes_out) {
  return topoep_workspace_bytes_ex(topo, T, k, replica_budget, nullptr, bytes_out);
}

int topoep_plan_dispatch(const topoep_topology *topo, const int32_t *global_load, const int32_t *local_topk,
                         int32_t T, int32_t k, int32_t replica_budget, int32_t *replica_slots,
                         int32_t *token_dest, int32_t *send_counts, int32_t *recv_counts, int32_t *send_offsets,
                         int32_t *token_slot, int32_t *status, void *workspace, size_t workspace_bytes,
                         void *stream) {
  const bool layout = send_offsets != nullptr || token_slot != nullptr;
  if (layout && (!send_offsets || (T > 0 && !token_slot))) return TOPOEP_EINVAL;
  if (!recv_counts && !layout) return TOPOEP_EINVAL;
  return enqueue(7, topo, global_load, local_topk, T, k, replica_budget, replica_slots, token_dest, send_counts,
                 status, workspace, workspace_bytes, stream, nullptr, recv_counts, send_offsets, token_slot);
}

int topoep_costs_workspace_bytes(const topoep_topology *topo, int32_t T, int32_t k, int32_t replica_budget,
                                 size_t *bytes_out) {
  if (!bytes_out) return TOPOEP_EINVAL;
  Plan p;
  Shape s;
  size_t need = 0;
  const int rc = setup(topo, T, k, replica_budget, nullptr, &p, &s, &need, nullptr, true);
  if (rc == TOPOEP_OK) *bytes_out = need;
  return rc;
}

int topoep_plan_costs(const topoep_topology *topo, const topoep_costs *costs, const int32_t *global_load,
                      const int32_t *local_topk, int32_t T, int32_t k, int32_t replica_budget,
                      int32_t *replica_slots, int32_t *token_dest, int32_t *send_counts, int32_t *status,
                      void *workspace, size_t workspace_bytes, void *stream) {
  const topoep_costs none = {nullptr, nullptr};
  return enqueue(7, topo, global_load, local_topk, T, k, replica_budget, replica_slots, token_dest, send_counts,
                 status, workspace, workspace_bytes, stream, nullptr, nullptr, nullptr, nullptr,
                 costs ? costs : &none);
}

int topoep_plan_stage(int32_t stage, const topoep_topology *topo, const int32_t *global_load,
                      const int32_t *local_topk, int32_t T, int32_t k, int32_t replica_budget,
                      int32_t *replica_slots, int32_t *token_dest, int32_t *send_counts, int32_t *status,
                      void *workspace, size_t workspace_bytes, void *stream, const topoep_launch *launch) {
  if (stage < 0 || stage > TOPOEP_STAGE_FLOOR) return TOPOEP_EINVAL;
  return enqueue(1 << stage, topo, global_load, local_topk, T, k, replica_budget, replica_slots,
                 token_dest, send_counts, status, workspace, workspace_bytes, stream, launch);
}

}  // extern "C"
