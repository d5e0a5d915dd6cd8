// Multi-source BFS: up to 64 traversals share every sweep over the graph (the
// paper's future-work "higher-level task parallelism", Sec. 8: several BFS at
// once).  Per vertex, 64-bit masks hold one bit per source: `visit` (reached),
// `front` (in the current frontier of that source) and `next` (reached at this
// level).  One level:
//   expand   push: every active vertex u ORs front[u] & ~visit[v] into next[v]
//                  (atomic OR; the first setter appends v to the touched list);
//            pull: every vertex with unreached bits ORs front[u] over its
//                  neighbours (early exit once all its unreached bits appear);
//   finalize for every touched v: visit |= next, front' = next, and the depth
//            d + 1 for each new source bit.
// The parent of a (source, vertex) pair is the first neighbour u (ascending)
// with the source's bit in front[u], the smallest-id parent of the single-source
// definition: the pull meets it as it scans, a push level takes the minimum of
// the frontier neighbours' ids with an atomic.
//
// The caller's arrays are [source][vertex], so writing a pair's depth and
// parent as it is found costs two scattered 4-byte stores.  While the depth
// fits kMsPlanes bits they are kept per vertex instead: depths as bit planes
// (plane j of a vertex holds bit j of its depth for all sources: one 32-byte
// row, touched once per level), parents in one row of `kp` words; one pass at
// the end (k_ms_output) transposes both, in caller order, and writes every
// entry of the outputs once, so they need no fill before.  A traversal that gets
// deeper writes out what it has and goes on in the caller's arrays.
#include "k_advance.h"
#include "k_dloop.h"

namespace gr {

namespace {

using u64 = unsigned long long;

// Where parent values go: word s * ps + pv of the array for source s, with pv
// from the vertex (rows: v << kp_log; the caller's array: its caller id).
struct MsParents {
  uint32_t* p;   // nullable: no parents wanted
  int64_t ps;
  int kp_log;    // >= 0: rows of 1 << kp_log words; < 0: the caller's array
  const int32_t* perm;
  __device__ __forceinline__ int64_t at(int64_t v) const {
    return kp_log >= 0 ? v << kp_log : (int64_t)(perm ? perm[v] : v);
  }
  __device__ __forceinline__ uint32_t id(int32_t u) const { return (uint32_t)(perm ? perm[u] : u); }
};

// Push expansion.  PARENT: each edge also takes the minimum of its new pairs'
// parents (no returning atomic; a pair's word starts at 0xffffffff).  A search by
// the finalize pass instead scanned every touched vertex's row up to the last of
// its new parents: 109 K hubs reached by 204 K edges took 1.58 ms of an R-MAT 20
// batch.  Where a level pushes much of the graph the atomics are the larger cost (25 M
// and 31 M edges: 5.9 and 8.2 ms with them, 1.1 and 0.8 without); there the pull
// kernels find the parents afterwards (0.9 and 0.4 ms; kMsSearchDivisor).
template <bool PARENT>
struct MsPush {
  const u64* __restrict__ visit;
  u64* __restrict__ next;
  const u64* __restrict__ front;
  MsParents par;

  using pay_t = u64;
  static constexpr bool kFar = false;
  static constexpr bool kBatchCommit = true;
  __device__ __forceinline__ u64 seg_payload(int32_t u) const { return front[u]; }
  __device__ __forceinline__ uint32_t edge_value(int64_t) const { return 0u; }
  __device__ __forceinline__ bool probe(int32_t, u64 fm, int32_t v, uint32_t) const {
    return (fm & ~visit[v]) != 0ull;
  }
  __device__ __forceinline__ bool commit(int32_t, u64, int32_t, uint32_t) const { return false; }
  // the returning ORs of a lane's B edges are in flight together, then the
  // parent minima, whose results nobody waits for
  template <int B>
  __device__ __forceinline__ void commit_batch(const int32_t (&u)[B], const u64 (&fm)[B],
                                               const int32_t (&v)[B], const uint32_t (&)[B],
                                               const bool (&ok)[B], int (&code)[B]) const {
    u64 m[B], old[B];
    uint32_t uo[B];
    int64_t pv[B];
#pragma unroll
    for (int r = 0; r < B; ++r) {
      m[r] = ok[r] ? fm[r] & ~visit[v[r]] : 0ull;
      uo[r] = PARENT && ok[r] ? par.id(u[r]) : 0u;
      pv[r] = PARENT && ok[r] ? par.at(v[r]) : 0;
    }
#pragma unroll
    for (int r = 0; r < B; ++r) old[r] = m[r] ? atomicOr(&next[v[r]], m[r]) : ~0ull;
    if constexpr (PARENT) {
#pragma unroll
      for (int r = 0; r < B; ++r)
        for (u64 b = m[r]; b; b &= b - 1)
          atomicMin(&par.p[(int64_t)(__ffsll(b) - 1) * par.ps + pv[r]], uo[r]);
    }
#pragma unroll
    for (int r = 0; r < B; ++r) code[r] = old[r] == 0ull;  // first setter lists v once
  }
  // hooks of a device-predicated level (k_dstep): nothing to prepare or carry
  __device__ __forceinline__ void frontier_vertex(int32_t) const {}
  __device__ __forceinline__ MsPush prepare(const Ctrl*, int) const { return *this; }
  __device__ __forceinline__ void advance(Ctrl*, int, bool) const {}
};

__device__ __forceinline__ u64 wave_or(u64 x) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) x |= __shfl_xor(x, o);
  return x;
}

constexpr int kMsU = 8;                    // neighbours in flight per lane
constexpr int kMsLaneMax = 64;             // rows up to this long: one lane
constexpr int kMsWaveMax = 2048;           // ... up to this long: one wavefront
constexpr int kMsHubBlock = 1024;          // longer: a workgroup of this many threads
// Vertices per thread of the lane tier; one in graphs of up to kMsPullSmall vertices, which
// have too few workgroups otherwise (R-MAT 10, 64 sources: a level's lane and wavefront
// tiers 50 + 38 us with four vertices and eight rows at a time, 18 + 8 with one).
constexpr int kMsPullRuns = 4;
constexpr int64_t kMsPullSmall = 1 << 18;
constexpr int kMsWaveBatch = 8;            // most rows a wavefront takes at a time

// Neighbours base + r * 64 + lane of a row ending at re, and the bits of nd in
// their frontier masks.
// (Positions as unsigned: a row may end right below 2^31.)
__device__ __forceinline__ void ms_load(const int32_t* __restrict__ C,
                                        const u64* __restrict__ front, uint32_t base, uint32_t re,
                                        u64 nd, int32_t (&u)[kMsU], u64 (&f)[kMsU]) {
#pragma unroll
  for (int r = 0; r < kMsU; ++r) {
    const uint32_t j = base + r * kWave + lane();
    u[r] = j < re ? C[j] : -1;
  }
#pragma unroll
  for (int r = 0; r < kMsU; ++r) f[r] = u[r] >= 0 ? (front[u[r]] & nd) : 0ull;
}

// The first neighbour (r-major, then lane: ascending) whose mask holds bit sb.
__device__ __forceinline__ int32_t ms_first(const int32_t (&u)[kMsU], const u64 (&f)[kMsU], int sb) {
  int32_t pu = -1;
#pragma unroll
  for (int r = kMsU - 1; r >= 0; --r) {
    const uint64_t b = __ballot((f[r] >> sb) & 1ull);
    if (b) pu = __shfl(u[r], __ffsll((unsigned long long)b) - 1);
  }
  return pu;
}

// Pull expansion, three tiers by row length.  Every vertex with unreached bits
// scans its ascending row with an early exit once all of them appeared, so the
// neighbour where a bit first appears is that source's smallest-id parent.  As
// some source's frontier is small on most levels, most rows are scanned to
// their end, so the split has to balance edges: with every long row left to the
// wavefront that owns the vertex, the first 64 vertices of a degree-ordered
// graph shared one wavefront (R-MAT 20, 64 sources: 10.2 ms of a level's
// 10.3 ms).  With touched null the level was pushed without parents: the rows are
// scanned for the bits in next, only their parents are written.  This kernel scans
// the rows of up to kMsLaneMax neighbours, one lane each, and lists the longer ones
// for the two kernels below.
template <int K>
__global__ __launch_bounds__(256) void k_ms_pull(int64_t V, const int32_t* __restrict__ R,
                                                 const int32_t* __restrict__ C,
                                                 const u64* __restrict__ front,
                                                 const u64* __restrict__ visit, u64 full,
                                                 u64* __restrict__ next, int32_t* __restrict__ touched,
                                                 uint32_t* __restrict__ n_touched, MsParents par,
                                                 int32_t* __restrict__ mid_q,
                                                 int32_t* __restrict__ hub_q,
                                                 uint32_t* __restrict__ n_big) {
  const int64_t v0 = (int64_t)blockIdx.x * (256 * K) + threadIdx.x;
  u64 need[K];
  int32_t rb[K], re[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t v = v0 + k * 256;
    need[k] = v < V ? (touched ? full & ~visit[v] : next[v]) : 0ull;
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t v = v0 + k * 256;
    rb[k] = need[k] ? R[v] : 0;
    re[k] = need[k] ? R[v + 1] : 0;
  }
  uint32_t hits = 0, mids = 0, hubs = 0;  // bit k: vertex v0 + k * 256
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t v = v0 + k * 256;
    const int32_t len = re[k] - rb[k];
    if (len <= 0) continue;
    if (len > kMsLaneMax) {
      if (len > kMsWaveMax) hubs |= 1u << k;
      else mids |= 1u << k;
      continue;
    }
    const int64_t pv = par.p ? par.at(v) : 0;
    u64 acc = 0;
    const uint32_t end = (uint32_t)re[k];
    for (uint32_t j0 = (uint32_t)rb[k]; j0 < end && acc != need[k]; j0 += kMsU) {
      int32_t u[kMsU];
      u64 f[kMsU];
#pragma unroll
      for (int r = 0; r < kMsU; ++r) u[r] = j0 + r < end ? C[j0 + r] : -1;
#pragma unroll
      for (int r = 0; r < kMsU; ++r) f[r] = u[r] >= 0 ? front[u[r]] & need[k] : 0ull;
#pragma unroll
      for (int r = 0; r < kMsU; ++r) {
        u64 g = f[r] & ~acc;
        acc |= g;
        if (par.p && g) {
          const uint32_t uo = par.id(u[r]);
          for (; g; g &= g - 1) par.p[(int64_t)(__ffsll(g) - 1) * par.ps + pv] = uo;
        }
      }
    }
    if (acc && touched) {
      next[v] = acc;
      hits |= 1u << k;
    }
  }
  uint32_t slot;
  if (touched) {
    slot = block_append<256>(__popc(hits), n_touched);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if ((hits >> k) & 1u) touched[slot++] = (int32_t)(v0 + k * 256);
  }
  if (mid_q) {
    slot = block_append<256>(__popc(mids), &n_big[0]);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if ((mids >> k) & 1u) mid_q[slot++] = (int32_t)(v0 + k * 256);
  }
  if (hub_q) {
    slot = block_append<256>(__popc(hubs), &n_big[1]);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if ((hubs >> k) & 1u) hub_q[slot++] = (int32_t)(v0 + k * 256);
  }
}

// Rows of kMsLaneMax + 1 .. kMsWaveMax neighbours: one wavefront each, 512
// neighbours per step; lane s keeps source s's parent, so a row's parents leave
// in one store.  Up to kMsWaveBatch rows per turn (their bounds loaded together, one
// append), as many as leave every wavefront some; wavefronts in a grid-stride loop over
// the listed rows.
__global__ __launch_bounds__(256) void k_ms_pull_mid(
    const int32_t* __restrict__ list, const uint32_t* __restrict__ n_list,
    const int32_t* __restrict__ R, const int32_t* __restrict__ C, const u64* __restrict__ front,
    const u64* __restrict__ visit, u64 full, u64* __restrict__ next, int32_t* __restrict__ touched,
    uint32_t* __restrict__ n_touched, MsParents par) {
  constexpr int NW = 256 / kWave;
  const int64_t n = *n_list;
  const int64_t waves = (int64_t)gridDim.x * NW;
  const int batch = n <= waves ? 1 : n < waves * kMsWaveBatch ? (int)((n + waves - 1) / waves) : kMsWaveBatch;
  for (int64_t i0 = ((int64_t)blockIdx.x * NW + threadIdx.x / kWave) * batch; i0 < n;
       i0 += waves * batch) {
    const int cnt = n - i0 < batch ? (int)(n - i0) : batch;
    int32_t lv = 0, lrb = 0, lre = 0;
    u64 lneed = 0;
    if (lane() < cnt) {
      lv = list[i0 + lane()];
      lneed = touched ? full & ~visit[lv] : next[lv];
      lrb = R[lv];
      lre = R[lv + 1];
    }
    uint32_t hits = 0;
    for (int k = 0; k < cnt; ++k) {
      const int32_t v = __shfl(lv, k);
      const uint32_t rb = (uint32_t)__shfl(lrb, k), re = (uint32_t)__shfl(lre, k);
      const u64 nd = __shfl(lneed, k);
      u64 fnd = 0;
      int32_t pu = -1;
      for (uint32_t base = rb; base < re && fnd != nd; base += kMsU * kWave) {
        int32_t u[kMsU];
        u64 f[kMsU];
        ms_load(C, front, base, re, nd, u, f);
        u64 any = 0;
#pragma unroll
        for (int r = 0; r < kMsU; ++r) any |= f[r];
        if (!__ballot((any & ~fnd) != 0ull)) continue;
        const u64 nw = wave_or(any) & ~fnd;
        if (par.p)
          for (u64 g = nw; g; g &= g - 1) {
            const int sb = __ffsll(g) - 1;
            const int32_t x = ms_first(u, f, sb);
            if (lane() == sb) pu = x;
          }
        fnd |= nw;
      }
      if (fnd) {
        if (par.p && pu >= 0) par.p[(int64_t)lane() * par.ps + par.at(v)] = par.id(pu);
        if (lane() == 0 && touched) next[v] = fnd;
        hits |= 1u << k;
      }
    }
    if (hits && touched) {
      uint32_t base = 0;
      if (lane() == 0) base = atomicAdd(n_touched, (uint32_t)__popc(hits));
      base = __shfl(base, 0);
      if (lane() < cnt && ((hits >> lane()) & 1u))
        touched[base + __popc(hits & ((1u << lane()) - 1u))] = lv;
    }
  }
}

// Longer rows: one workgroup each, its wavefronts taking consecutive pieces of
// a window of 8192 neighbours.  A bit found by several wavefronts belongs to the
// first of them; the pieces' found bits are exchanged through LDS (two buffers,
// so one barrier per window).
__global__ __launch_bounds__(kMsHubBlock) void k_ms_pull_hub(
    const int32_t* __restrict__ list, const uint32_t* __restrict__ n_list,
    const int32_t* __restrict__ R, const int32_t* __restrict__ C, const u64* __restrict__ front,
    const u64* __restrict__ visit, u64 full, u64* __restrict__ next, int32_t* __restrict__ touched,
    uint32_t* __restrict__ n_touched, MsParents par) {
  constexpr int NW = kMsHubBlock / kWave;
  __shared__ u64 s_or[2][NW];
  const int w = threadIdx.x / kWave;
  const int64_t n = *n_list;
  int buf = 0;
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int32_t v = list[i];
    const u64 nd = touched ? full & ~visit[v] : next[v];
    const uint32_t rb = (uint32_t)R[v], re = (uint32_t)R[v + 1];
    const int64_t pv = par.p ? par.at(v) : 0;
    u64 fnd = 0;
    for (uint32_t base = rb; base < re && fnd != nd; base += kMsU * kMsHubBlock) {
      int32_t u[kMsU];
      u64 f[kMsU];
      ms_load(C, front, base + (uint32_t)w * (kMsU * kWave), re, nd & ~fnd, u, f);
      u64 any = 0;
#pragma unroll
      for (int r = 0; r < kMsU; ++r) any |= f[r];
      const u64 mine = __ballot(any != 0ull) ? wave_or(any) : 0ull;
      if (lane() == 0) s_or[buf][w] = mine;
      __syncthreads();
      u64 before = 0, all = 0;
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const u64 x = s_or[buf][k];
        if (k < w) before |= x;
        all |= x;
      }
      if (par.p)
        for (u64 g = mine & ~before; g; g &= g - 1) {
          const int sb = __ffsll(g) - 1;
          const int32_t x = ms_first(u, f, sb);
          if (lane() == 0) par.p[(int64_t)sb * par.ps + pv] = par.id(x);
        }
      fnd |= all;
      buf ^= 1;
    }
    if (threadIdx.x == 0 && fnd && touched) {
      next[v] = fnd;
      touched[atomicAdd(n_touched, 1u)] = v;
    }
  }
}

// Finalise the touched vertices: masks and depths (bit planes, or with planes
// null the caller's array).  The level's frontier has been read: its masks are
// cleared on the way, and the pull's row lists start empty again.
__global__ __launch_bounds__(256) void k_ms_finalize(
    const int32_t* __restrict__ touched, const uint32_t* __restrict__ n_touched,
    const int32_t* __restrict__ cur_q, const uint32_t* __restrict__ n_cur,
    const int32_t* __restrict__ R, u64* __restrict__ front_cur, u64* __restrict__ front_next,
    u64* __restrict__ visit,
    u64* __restrict__ next, u64* __restrict__ planes, int32_t* __restrict__ depth,
    const int32_t* __restrict__ perm, int64_t V, int32_t next_depth, Ctrl* __restrict__ ctrl,
    bool predicated, int64_t* __restrict__ m_next) {
  __shared__ int64_t s_pairs[256 / kWave], s_pe[256 / kWave], s_m[256 / kWave];
  if (predicated && ctrl->dl_stop) return;  // a level of the block declined
  const int64_t n = *n_touched;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)*n_cur) front_cur[cur_q[i]] = 0ull;
  if (!predicated && i == 0) ctrl->ms_big[0] = ctrl->ms_big[1] = 0;
  if ((int64_t)blockIdx.x * blockDim.x >= n) return;
  int64_t deg = 0;
  u64 nw = 0;
  if (i < n) {
    const int32_t v = touched[i];
    nw = next[v];
    const u64 vis = visit[v];
    deg = (int64_t)R[v + 1] - R[v];
    next[v] = 0;
    visit[v] = vis | nw;
    front_next[v] = nw;
    if (planes) {
#pragma unroll
      for (int j = 0; j < kMsPlanes; ++j)
        if ((next_depth >> j) & 1) planes[(int64_t)v * kMsPlanes + j] |= nw;
    } else {
      const int64_t vo = perm ? perm[v] : v;
      for (u64 b = nw; b; b &= b - 1) depth[(int64_t)(__ffsll(b) - 1) * V + vo] = next_depth;
    }
  }
  // the pairs reached at this level and their degrees (selector features), and
  // (nullable) the next frontier's edges
  const int64_t pc = __popcll(nw);
  const int64_t wp = wave_sum(pc), we = wave_sum(pc * deg), wm = m_next ? wave_sum(deg) : 0;
  if (lane() == 0) {
    s_pairs[threadIdx.x / kWave] = wp;
    s_pe[threadIdx.x / kWave] = we;
    s_m[threadIdx.x / kWave] = wm;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t tp = 0, te = 0, tm = 0;
    for (int k = 0; k < 256 / kWave; ++k) {
      tp += s_pairs[k];
      te += s_pe[k];
      tm += s_m[k];
    }
    if (tm) atomicAdd((unsigned long long*)m_next, (unsigned long long)tm);
    if (tp) atomicAdd((unsigned long long*)&ctrl->ms_pairs, (unsigned long long)tp);
    if (te) atomicAdd((unsigned long long*)&ctrl->ms_pair_edges, (unsigned long long)te);
  }
}

// The outputs of a pass from the bit planes and parent rows: a workgroup takes
// 64 consecutive caller ids, reads their rows (each row contiguous), turns the
// tile round in LDS and writes, per source, 64 consecutive depths and parents.
// A pair not reached gets depth -1; parents of depth 0 or none are -1.  Bound by
// the memory traffic of the rows and outputs.
__global__ __launch_bounds__(256) void k_ms_output(const u64* __restrict__ visit,
                                                   const u64* __restrict__ planes,
                                                   const uint32_t* __restrict__ prow, int kp_log,
                                                   int k, const int32_t* __restrict__ inv, int64_t V,
                                                   int32_t* __restrict__ depth,
                                                   int32_t* __restrict__ parent) {
  __shared__ int32_t s_v[kWave];
  __shared__ uint32_t s_p[kWave][kWave + 1];  // [source][vertex]
  const int64_t c0 = (int64_t)blockIdx.x * kWave;
  const int w = threadIdx.x / kWave;
  const int64_t c = c0 + lane();
  const int32_t v = c < V ? (inv ? inv[c] : (int32_t)c) : -1;
  u64 vis = 0, pl[kMsPlanes];
#pragma unroll
  for (int j = 0; j < kMsPlanes; ++j) pl[j] = 0;
  if (v >= 0) {
    vis = visit[v];
    const ulonglong2* row = reinterpret_cast<const ulonglong2*>(planes + (int64_t)v * kMsPlanes);
#pragma unroll
    for (int j = 0; j < kMsPlanes / 2; ++j) {
      const ulonglong2 x = row[j];
      pl[2 * j] = x.x;
      pl[2 * j + 1] = x.y;
    }
  }
  if (parent) {
    if (w == 0) s_v[lane()] = v;
    __syncthreads();
    const int kp = 1 << kp_log;
    for (int t = threadIdx.x; t < (kWave << kp_log); t += 256) {
      const int i = t >> kp_log, s = t & (kp - 1);
      const int32_t x = s_v[i];
      if (x >= 0) s_p[s][i] = prow[((int64_t)x << kp_log) + s];
    }
    __syncthreads();
  }
  if (v < 0) return;
  for (int s = w; s < k; s += 256 / kWave) {
    int32_t d = 0;
#pragma unroll
    for (int j = 0; j < kMsPlanes; ++j) d |= (int32_t)((pl[j] >> s) & 1ull) << j;
    const bool reached = (vis >> s) & 1ull;
    depth[(int64_t)s * V + c] = reached ? d : -1;
    if (parent) parent[(int64_t)s * V + c] = reached && d > 0 ? (int32_t)s_p[s][lane()] : -1;
  }
}

// Masks, planes and (nullable) parent rows of a pass cleared, the frontier
// counters set (n_src distinct sources).
__global__ __launch_bounds__(256) void k_ms_init(u64* __restrict__ visit, u64* __restrict__ f0,
                                                 u64* __restrict__ f1, u64* __restrict__ next,
                                                 u64* __restrict__ planes,
                                                 uint32_t* __restrict__ prow, int kp_log, int64_t V,
                                                 uint32_t n_src, Ctrl* __restrict__ ctrl) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t v = i0; v < V; v += stride) {
    visit[v] = f0[v] = f1[v] = next[v] = 0ull;
    if (planes) {
      ulonglong2* row = reinterpret_cast<ulonglong2*>(planes + v * kMsPlanes);
#pragma unroll
      for (int j = 0; j < kMsPlanes / 2; ++j) row[j] = make_ulonglong2(0ull, 0ull);
    }
  }
  if (prow)
    for (int64_t i = i0; i < V << kp_log; i += stride) prow[i] = 0xffffffffu;
  if (i0 == 0) {
    ctrl->q_count[0] = n_src;
    ctrl->ms_big[0] = ctrl->ms_big[1] = 0;
    ctrl->ms_pairs = 0;
    ctrl->ms_pair_edges = 0;
  }
}

// Sources: their bits in visit / front, depth 0 (when the caller's array is
// written directly), and the reached-pair counters start at the k source pairs.
__global__ __launch_bounds__(64) void k_ms_seed(SourceArgs a, int32_t n_uniq,
                                                u64* __restrict__ visit, u64* __restrict__ front,
                                                int32_t* __restrict__ depth, int64_t V,
                                                const int32_t* __restrict__ R,
                                                int32_t* __restrict__ queue,
                                                Ctrl* __restrict__ ctrl) {
  const int s = threadIdx.x;
  if (s < n_uniq) queue[s] = a.v[2 * a.n + s];
  if (s < a.n) {
    const int32_t v = a.v[s];
    atomicOr(&visit[v], 1ull << s);
    atomicOr(&front[v], 1ull << s);
    if (depth) depth[(int64_t)s * V + a.v[a.n + s]] = 0;
    atomicAdd((unsigned long long*)&ctrl->ms_pair_edges, (unsigned long long)(R[v + 1] - R[v]));
  }
  if (s == 0) atomicAdd((unsigned long long*)&ctrl->ms_pairs, (unsigned long long)a.n);
}

// sum over v of popcount(visit[v]) * degree(v)
__global__ __launch_bounds__(256) void k_ms_teps(const u64* __restrict__ visit,
                                                 const int32_t* __restrict__ R, int64_t V,
                                                 int64_t* __restrict__ out) {
  __shared__ int64_t s[256 / kWave];
  // four vertices per thread and round, all loaded before any is used
  constexpr int K = 4;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t acc = 0;
  for (int64_t v0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v0 < V; v0 += stride * K) {
    u64 m[K];
    int32_t a[K], b[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
      const int64_t v = v0 + r * stride < V ? v0 + r * stride : V - 1;
      m[r] = visit[v];
      a[r] = R[v];
      b[r] = R[v + 1];
    }
#pragma unroll
    for (int r = 0; r < K; ++r)
      if (v0 + r * stride < V) acc += (int64_t)__popcll(m[r]) * ((int64_t)b[r] - a[r]);
  }
  acc = wave_sum(acc);
  if (lane() == 0) s[threadIdx.x / kWave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int i = 0; i < 256 / kWave; ++i) t += s[i];
    atomicAdd((unsigned long long*)out, (unsigned long long)t);
  }
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

hipError_t launch_ms_seed(const SourceArgs& src, int32_t n_uniq, u64* visit, u64* front,
                          int32_t* depth, int64_t V, const int32_t* R, int32_t* queue, Ctrl* ctrl,
                          hipStream_t st) {
  k_ms_seed<<<1, 64, 0, st>>>(src, n_uniq, visit, front, depth, V, R, queue, ctrl);
  return hipGetLastError();
}

namespace {
MsParents parents_of(const MsOut& o, int64_t V, const int32_t* perm) {
  if (o.planes) return MsParents{o.prow, 1, o.kp_log, perm};
  return MsParents{reinterpret_cast<uint32_t*>(o.parent), V, -1, perm};
}
}  // namespace

hipError_t launch_ms_init(u64* visit, u64* f0, u64* f1, u64* next, const MsOut& o, int64_t V,
                          int32_t n_src, Ctrl* ctrl, hipStream_t st) {
  int64_t g = blocks_for(V, 256);
  if (g > 4096) g = 4096;
  k_ms_init<<<(unsigned)g, 256, 0, st>>>(visit, f0, f1, next, o.planes,
                                         o.planes ? o.prow : nullptr, o.kp_log, V,
                                         (uint32_t)n_src, ctrl);
  return hipGetLastError();
}

hipError_t launch_ms_push(int mode, const int32_t* active, const int32_t* offsets,
                          const int32_t* rstart, const int32_t* chunk_start, int64_t n_a,
                          int64_t m_a, const int32_t* R, const int32_t* C, const u64* front,
                          const u64* visit, u64* next, const MsOut& o, int64_t V,
                          const int32_t* perm, bool parents, int32_t* touched,
                          uint32_t* n_touched, const AdvCfg& cfg, hipStream_t st) {
  const MsParents par = parents_of(o, V, perm);
  if (par.p && parents)
    return push_dispatch(mode, active, offsets, rstart, chunk_start, n_a, m_a, R, C,
                         MsPush<true>{visit, next, front, par}, touched, n_touched, cfg, st);
  return push_dispatch(mode, active, offsets, rstart, chunk_start, n_a, m_a, R, C,
                       MsPush<false>{visit, next, front, par}, touched, n_touched, cfg, st);
}

hipError_t launch_ms_pull(int64_t V, int64_t E, int64_t max_degree, const int32_t* R,
                          const int32_t* C, const u64* front, const u64* visit, u64 full, u64* next,
                          int32_t* touched, uint32_t* n_touched, const MsOut& o,
                          const int32_t* perm, int32_t* mid_q, int32_t* hub_q, uint32_t* n_big,
                          hipStream_t st) {
  const MsParents par = parents_of(o, V, perm);
  const bool mid = max_degree > kMsLaneMax, hub = max_degree > kMsWaveMax;
  const bool small = V <= kMsPullSmall;
  const auto lane_tier = small ? k_ms_pull<1> : k_ms_pull<kMsPullRuns>;
  lane_tier<<<blocks_for(V, small ? 256 : 256 * kMsPullRuns), 256, 0, st>>>(
      V, R, C, front, visit, full, next, touched, n_touched, par, mid ? mid_q : nullptr,
      hub ? hub_q : nullptr, n_big);
  // the hubs first: the longest rows of the level start earliest
  if (hub) {
    const int64_t most = E / kMsWaveMax + 1;  // rows this long
    k_ms_pull_hub<<<(unsigned)(most < 512 ? most : 512), kMsHubBlock, 0, st>>>(
        hub_q, &n_big[1], R, C, front, visit, full, next, touched, n_touched, par);
  }
  if (mid) {
    const int64_t most = E / kMsLaneMax + 1;
    const int64_t g = blocks_for(most < V ? most : V, 4);
    k_ms_pull_mid<<<(unsigned)(g < 2048 ? g : 2048), 256, 0, st>>>(
        mid_q, &n_big[0], R, C, front, visit, full, next, touched, n_touched, par);
  }
  return hipGetLastError();
}

hipError_t launch_ms_finalize(const int32_t* touched, const uint32_t* n_touched, int64_t max_n,
                              const int32_t* cur_q, const uint32_t* n_cur, int64_t max_cur,
                              const int32_t* R, u64* front_cur, u64* front_next, u64* visit,
                              u64* next, const MsOut& o, const int32_t* perm, int64_t V,
                              int32_t next_depth, Ctrl* ctrl, hipStream_t st) {
  const int64_t most = max_n > max_cur ? max_n : max_cur;
  if (most <= 0) return hipSuccess;
  k_ms_finalize<<<blocks_for(most, 256), 256, 0, st>>>(touched, n_touched, cur_q, n_cur, R,
                                                       front_cur, front_next, visit, next, o.planes,
                                                       o.depth, perm, V, next_depth, ctrl, false,
                                                       nullptr);
  return hipGetLastError();
}

namespace {
template <bool PARENT>
void ms_dlevel_push(const DlArgs& a, const MsPush<PARENT>& f, bool short_rows, int n_blocks,
                    hipStream_t st) {
  if (short_rows) k_dpush<MsPush<PARENT>><<<n_blocks, kAdvBlock, 0, st>>>(a, f);
  else k_dstep<MsPush<PARENT>><<<n_blocks, kAdvBlock, 0, st>>>(a, f);
}
}  // namespace

hipError_t launch_ms_dlevel(const DlArgs& a, const MsLevel& m, bool short_rows, int n_blocks,
                            int64_t max_touched, hipStream_t st) {
  const MsParents par = parents_of(m.out, m.V, m.perm);
  if (par.p)
    ms_dlevel_push(a, MsPush<true>{m.visit, m.next, m.front_cur, par}, short_rows, n_blocks, st);
  else
    ms_dlevel_push(a, MsPush<false>{m.visit, m.next, m.front_cur, par}, short_rows, n_blocks, st);
  const int64_t most = max_touched > a.max_n ? max_touched : a.max_n;
  k_ms_finalize<<<blocks_for(most, 256), 256, 0, st>>>(
      a.q_next, &a.ctrl->q_count[(a.cur + 1) % 3], a.q_cur, &a.ctrl->q_count[a.cur], m.R,
      const_cast<u64*>(m.front_cur), m.front_next, m.visit, m.next, m.out.planes, m.out.depth,
      m.perm, m.V, m.next_depth, a.ctrl, true,
      short_rows ? &a.ctrl->dl_mf[(a.step + 1) & 1] : nullptr);
  return hipGetLastError();
}

hipError_t launch_ms_output(const u64* visit, const MsOut& o, int32_t k, const int32_t* inv,
                            int64_t V, hipStream_t st) {
  if (V <= 0) return hipSuccess;
  k_ms_output<<<blocks_for(V, kWave), 256, 0, st>>>(visit, o.planes, o.prow, o.kp_log, k, inv, V,
                                                    o.depth, o.parent);
  return hipGetLastError();
}

hipError_t launch_ms_teps(const u64* visit, const int32_t* R, int64_t V, int64_t* out,
                          hipStream_t st) {
  unsigned g = blocks_for(V, 256);
  if (g > 1024) g = 1024;  // one atomic per workgroup, all on one address
  k_ms_teps<<<g, 256, 0, st>>>(visit, R, V, out);
  return hipGetLastError();
}

}  // namespace gr
