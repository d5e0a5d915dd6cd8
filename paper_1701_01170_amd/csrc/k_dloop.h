// Device-predicated level step: one push level of BFS or SSSP for a small
// frontier, written so that many levels can be enqueued back to back with no
// host round trip in between (the per-iteration termination check of the
// bulk-synchronous loop, Sec. 4 and Sec. 5.2, moved onto the device).
//
// Every workgroup reads the same control values, all written by earlier
// kernels, and stages the same frontier, so all take the same decision: the
// level runs only if no earlier level of the block declined, the frontier is
// non-empty, it fits the LDS staging (kDlMaxN vertices) and the caller's edge
// bound, and (batched BFS) the direction heuristic of Sec. 5.1 would still push.
// A declining level sets dl_stop, so the rest of the block does nothing.
//
// A running level is output-balanced like LB (Sec. 5.1): each workgroup stages
// the whole frontier in LDS, scans its degrees (which gives the level its m_f
// without a statistics pass), and expands one equal slice of the edges.
//
// A block is a fixed sequence of kernels on a device-chosen number of levels:
// k_team runs as many small levels as it can on the workgroups of one XCD, k_dstep
// one level on the whole chip, and both take up where the kernel before left off
// (ctrl->dl_step[seq & 1], the levels of the block that ran; the next kernel's slot
// is the other one, so nothing is read and written by the same kernel).
//
// Functors used here also provide prepare(ctrl, step) (the functor of this
// step from the one of the block's first level, e.g. SSSP's priority-queue threshold
// read from the control block), next() (the functor of the level after, with the
// same queue state), advance(ctrl, step, refill) (the state of the next step,
// written once) and store(ctrl, step) (the functor's own state as that of `step`).
// With the SSSP priority queue (kFar), a step whose frontier is empty but
// whose far pile is not becomes a refill step instead of stopping the block.
#pragma once

#include "k_advance.h"
#include "team_join.h"

namespace gr {

constexpr int kDlPerThread = kDlMaxN / kAdvBlock;
static_assert(kDlMaxN % kAdvBlock == 0, "frontier staging assumes whole rows");

template <class F>
__global__ __launch_bounds__(kAdvBlock) void k_dstep(DlArgs a, F f) {
  using pay_t = typename F::pay_t;
  constexpr int B = 4;
  __shared__ int32_t s_u[kDlMaxN];
  __shared__ int32_t s_rb[kDlMaxN];
  __shared__ int32_t s_off[kDlMaxN + 1];
  __shared__ pay_t s_pay[kDlMaxN];
  __shared__ int64_t s_tot[kAdvBlock / kWave + 1];
  __shared__ int64_t s_max[kAdvBlock / kWave];
  Ctrl* ctrl = a.ctrl;
  if (ctrl->dl_stop) return;
  const int step = ctrl->dl_step[a.seq & 1];
  const F fs = f.prepare(ctrl, step);
  const int cur = (a.cur0 + step) % 3, next = (cur + 1) % 3, prev = (cur + 2) % 3;
  const int32_t* __restrict__ q_cur = a.qs.q[cur];
  int32_t* __restrict__ q_next = a.qs.q[next];
  const int64_t n_f = ctrl->q_count[cur];
  const int64_t vm = ctrl->dl_vm[step & 1];
  const int64_t vn = ctrl->dl_vn[step & 1];
  const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
  bool refill = false;
  if constexpr (F::kFar) refill = n_f == 0 && fs.far_pending(ctrl);
  if (step >= a.max_steps || (!refill && !(n_f > 0 && n_f <= a.max_n && n_f <= kDlMaxN))) {
    if (lead) ctrl->dl_stop = 1;
    return;
  }
  if constexpr (F::kFar) {
    if (refill) {
      if (lead) {
        // none of these is read by this kernel
        ctrl->dl_levels = step + 1;
        ctrl->dl_step[(a.seq + 1) & 1] = step + 1;
        ctrl->q_count[prev] = 0;
        ctrl->dl_vm[(step + 1) & 1] = vm;
        ctrl->dl_vn[(step + 1) & 1] = vn;
        fs.advance(ctrl, step, true);
        if (a.log) {
          a.log[3 * step + 0] = 0;
          a.log[3 * step + 1] = 0;
          a.log[3 * step + 2] = 0;
        }
      }
      fs.refill(ctrl, q_next, &ctrl->q_count[next], blockIdx.x, gridDim.x);
      return;
    }
  }
  // every workgroup stages the whole frontier and scans its degrees
  // (kDlPerThread consecutive entries per thread); the scan total is the
  // level's frontier edge count m_f
  const int nf = (int)n_f;
  for (int j = threadIdx.x; j < nf; j += kAdvBlock) s_u[j] = q_cur[j];
  __syncthreads();
  const int j0 = threadIdx.x * kDlPerThread;
  int32_t d[kDlPerThread];
  int64_t sum = 0, mx = 0;
#pragma unroll
  for (int r = 0; r < kDlPerThread; ++r) {
    const int j = j0 + r;
    d[r] = 0;
    if (j < nf) {
      const int32_t u = s_u[j];
      const int32_t rb = a.R[u];
      d[r] = a.R[u + 1] - rb;
      s_rb[j] = rb;
      s_pay[j] = fs.seg_payload(u);
      sum += d[r];
      mx = d[r] > mx ? d[r] : mx;
    }
  }
  int64_t total;
  int64_t ex = block_excl_scan<kAdvBlock>(sum, s_tot, &total);
#pragma unroll
  for (int r = 0; r < kDlPerThread; ++r) {
    const int j = j0 + r;
    if (j < nf) {
      s_off[j] = (int32_t)ex;
      ex += d[r];
    }
  }
  if (threadIdx.x == 0) s_off[nf] = (int32_t)total;
  mx = wave_max(mx);
  if (lane() == 0) s_max[threadIdx.x / kWave] = mx;
  __syncthreads();
  // the level runs only within the caller's edge bound and (batched BFS) while
  // the push test of Sec. 5.1 holds; every workgroup computes the same total, so
  // all take the same decision
  bool run = total <= a.max_m;
  if (run && a.do_a >= 0.0 && (double)total > (double)a.E * a.do_a) run = false;
  if (!run) {
    if (lead) ctrl->dl_stop = 1;
    return;
  }
  if (lead) {
    // none of these is read by this kernel: the counter of the previous
    // frontier becomes the append target of the next level
    ctrl->dl_levels = step + 1;
    ctrl->dl_step[(a.seq + 1) & 1] = step + 1;
    ctrl->q_count[prev] = 0;
    ctrl->dl_vm[(step + 1) & 1] = vm + total;
    ctrl->dl_vn[(step + 1) & 1] = vn + n_f;
    fs.advance(ctrl, step, false);
    if (a.log) {
      int64_t m = 0;
      for (int i = 0; i < kAdvBlock / kWave; ++i) m = s_max[i] > m ? s_max[i] : m;
      a.log[3 * step + 0] = n_f;
      a.log[3 * step + 1] = total;
      a.log[3 * step + 2] = m;
    }
  }
  for (int j = blockIdx.x * kAdvBlock + threadIdx.x; j < nf; j += gridDim.x * kAdvBlock)
    fs.frontier_vertex(s_u[j]);
  // equal edge slices (at least one row of the workgroup each); workgroups
  // past the last slice have nothing more to do
  const int64_t G = gridDim.x;
  int64_t per = (total + G - 1) / G;
  if (per < kAdvBlock) per = kAdvBlock;
  const int64_t lo = (int64_t)blockIdx.x * per;
  if (lo >= total) return;
  const int64_t hi = lo + per < total ? lo + per : total;
  for (int64_t base = lo; base < hi; base += (int64_t)kAdvBlock * B) {
    bool ok[B];
    int32_t u[B];
    pay_t pay[B];
    int32_t ce[B];
#pragma unroll
    for (int r = 0; r < B; ++r) {
      const int64_t e = base + r * kAdvBlock + threadIdx.x;
      ok[r] = e < hi;
      const int k = ok[r] ? upper_index(s_off, 0, nf - 1, (int32_t)e) : 0;
      u[r] = s_u[k];
      pay[r] = s_pay[k];
      ce[r] = s_rb[k] + (int32_t)(e - s_off[k]);
    }
    edge_batch<F, B, true>(fs, a.C, ok, u, pay, ce, q_next, &ctrl->q_count[next]);
  }
}

// ---- levels on a team of workgroups -----------------------------------------
//
// Small levels, up to a.max_steps of the block in one launch.  A small level is a
// chain of dependent memory trips (queue, row bounds, columns, probe, atomic,
// append); as a kernel of its own it also pays the launch, the control block's
// trip and caches that the kernel boundary emptied: 14.5 us a level of a 2048 x 2048
// grid BFS as k_dstep launches, 5.6 us here (1.7 K vertices on average).
//
// The team are the workgroups that run on one XCD: their L2 is one cache, so a level
// ends with every wavefront's stores and atomics acknowledged by it and a barrier on
// a counter in it, and the next level reads what changes past the L1s; nothing has
// to be written back to memory in between, which the caches of different XCDs would
// need (and which made a barrier over the whole chip slower than a kernel boundary).
// Whoever runs elsewhere leaves at once.  Members register in one word together with
// the total of workgroups seen (team_join.h); when all have been seen, all members run
// at the same time and know their number.  If that takes too long (the chip is full of
// other work) the first to give up calls the run off for all of them, the block's other
// kernels do the levels, and the rest of the call runs without teams.  One workgroup
// alone has the same latency per trip, but its CU's throughput bounds levels of more
// than some 2 K edges (6.7 K edges: 32 us).
//
// Rows of at most 8 (a.log_w >= 0): a workgroup takes an equal slice of the
// frontier with 1 << log_w edge slots per vertex.  Other graphs: every workgroup
// stages the frontier, scans its degrees and takes an equal share of the edges, as
// k_dstep.  Either way the arrival word of the level's barrier also adds up the new
// frontier's vertices and (sliced) edges.
struct TeamWord {       // one per kernel of a block, zero at its start
  uint32_t reg;         // registration word (team_join.h)
  uint32_t pad;
  uint32_t q_count[3];  // append counters, rotating by level
  uint32_t pad1;
  unsigned long long arrive[3];  // arrivals | vertices << 8 | edges << 32, rotating by level
  uint32_t max_deg[3];  // traced calls: largest degree of the frontier, rotating by level
  uint32_t pad2;
};
static_assert(sizeof(TeamWord) == 64, "word size");
static_assert(kTeamWords * sizeof(TeamWord) <= kStatsGrid * sizeof(int64_t),
              "the team words use the statistics' block results");

__device__ __forceinline__ uint32_t xcc_id() {
  // hardware register XCC_ID (20), bits 3:0
  return __builtin_amdgcn_s_getreg((4 - 1) << 11 | 0 << 6 | 20) & 0xfu;
}

constexpr int kTeamWaitPolls = 1 << 22;   // polls of a level's barrier: far beyond any level

struct TeamRegWord {  // the registration word in memory (team_join.h)
  uint32_t* p;
  __device__ __forceinline__ uint32_t add(uint32_t x) { return atomicAdd(p, x); }
  __device__ __forceinline__ uint32_t load() {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ uint32_t cas(uint32_t e, uint32_t x) { return atomicCAS(p, e, x); }
};

// Joins the team of kernel word t: the member's index and the team's size, or -1 to
// leave; whoever calls the team off counts it in the control block.  Called by every
// thread.
__device__ __forceinline__ int team_join(TeamWord* t, int polls, Ctrl* ctrl, int* size) {
  __shared__ int s_idx, s_size;
  if (threadIdx.x == 0) {
    TeamRegWord w{&t->reg};
    // (polls 0: a count that is never complete, so that no team forms)
    TeamJoin j(gridDim.x + (polls == 0 ? 1u : 0u), xcc_id() == 0, polls);
#pragma unroll 1
    while (j.next != TeamJoin::kDone) {
      if (j.next == TeamJoin::kPoll) __builtin_amdgcn_s_sleep(1);
      j.step(w);
    }
    if (j.called_off) atomicAdd(&ctrl->dl_team_off, 1u);
    s_idx = j.index;
    s_size = j.size;
  }
  __syncthreads();
  *size = s_size;
  return s_idx;
}

// End of a level: everything this workgroup stored is in the XCD's L2, and so is
// everybody else's after it.  (The L1s still hold old lines: what changes during the
// kernel is read with load_shared<true>, past them.  Invalidating them at agent scope
// instead took 6 us a level.)  Returns the arrival word of the whole team (~0 when
// the wait ran out).  Called by every thread.
__device__ __forceinline__ unsigned long long team_barrier(unsigned long long* w, int size,
                                                           uint32_t n, uint32_t m) {
  __shared__ unsigned long long s_x;
  // this wavefront's stores and atomics are acknowledged.  (As the builtin, the wait
  // would not be declared to touch memory: the compiler could place a store after it, and
  // the workgroup fence of __syncthreads does not wait for one.)
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long add = 1ull | (unsigned long long)n << 8 | (unsigned long long)m << 32;
    unsigned long long x = atomicAdd(w, add) + add;
#pragma unroll 1
    for (int i = 0; (int)(x & 0xffull) < size; ++i) {
      if (i >= kTeamWaitPolls) {
        x = ~0ull;
        break;
      }
      x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    s_x = x;
  }
  __syncthreads();
  return s_x;
}

template <class F>
__global__ __launch_bounds__(kAdvBlock) void k_team(DlArgs a, F f) {
  using pay_t = typename F::pay_t;
  constexpr int B = 4;
  constexpr int NW = kAdvBlock / kWave;
  __shared__ int32_t s_u[kTeamMaxStaged];
  __shared__ int32_t s_rb[kTeamMaxStaged];
  __shared__ int32_t s_off[kTeamMaxStaged + 1];  // degrees (sliced) or their scan
  __shared__ pay_t s_pay[kTeamMaxStaged];
  __shared__ int64_t s_tot[NW + 1];
  __shared__ int32_t s_max[NW];
  __shared__ uint32_t s_n[NW], s_m[NW], s_base;
  Ctrl* ctrl = a.ctrl;
  if (ctrl->dl_stop) return;
  TeamWord* tw = reinterpret_cast<TeamWord*>(a.team) + a.seq;
  const int step0 = ctrl->dl_step[a.seq & 1];
  const uint32_t n0 = ctrl->q_count[(a.cur0 + step0) % 3];
  // the levels so far, in case nobody runs any here (they only grow)
  if (blockIdx.x == 0 && threadIdx.x == 0) atomicMax(&ctrl->dl_step[(a.seq + 1) & 1], step0);
  // a team that could not form waited in vain: the block's later ones are not tried (a
  // workgroup that reads this late, in the kernel whose team was called off, would find
  // that in the word)
  if (ctrl->dl_team_off) return;
  const bool sliced = a.log_w >= 0;
  if (!sliced && n0 > (uint32_t)kTeamMaxStaged) return;  // nothing to run here
  int size;
  const int me = team_join(tw, a.team_polls, ctrl, &size);
  if (me < 0) return;
  const int w = threadIdx.x / kWave;
  int step = step0;
  int64_t vm = ctrl->dl_vm[step & 1], vn = ctrl->dl_vn[step & 1];
  int64_t n = n0;
  F fs = f.prepare(ctrl, step);
  // sliced: a slice is at most one vertex per thread
  const int64_t max_n = sliced ? (int64_t)size * kAdvBlock : kTeamMaxStaged;
  int it = 0;         // barriers so far: picks the rotating words
  int64_t m = -1;     // sliced: the frontier's edges (-1: to be counted)
  bool failed = false;
  // clears the words of the next barrier, which are those of the barrier before the
  // last one: every member has left that one (it arrived at the last), while the last
  // one's may still be polled
  auto rotate = [&]() {
    if (me == 0 && threadIdx.x == 0) {
      __hip_atomic_store(&tw->arrive[(it + 1) % 3], 0ull, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&tw->q_count[(it + 1) % 3], 0u, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      if (a.log)
        __hip_atomic_store(&tw->max_deg[(it + 1) % 3], 0u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  while (step < a.max_steps) {
    if (n == 0) {
      if constexpr (F::kFar) {
        // priority queue: split the far pile into the next frontier
        if (!fs.far_pending(ctrl)) break;
        if (me == 0 && threadIdx.x == 0) {
          fs.clear_far(ctrl);
          if (a.log) a.log[3 * step] = a.log[3 * step + 1] = a.log[3 * step + 2] = 0;
        }
        uint32_t* cnt = &tw->q_count[it % 3];
        fs.refill(ctrl, a.qs.q[(a.cur0 + step + 1) % 3], cnt, me, size);
        rotate();
        if (team_barrier(&tw->arrive[it % 3], size, 0, 0) == ~0ull) {
          failed = true;
          break;
        }
        n = load_shared<true>(cnt);
        m = -1;
        ++it;
        ++step;
        fs = fs.after_refill();
        continue;
      }
      break;
    }
    if (n > max_n || n > a.max_n) break;
    const int32_t* __restrict__ q = a.qs.q[(a.cur0 + step) % 3];
    int64_t total;
    int nf, slots, e0, e1, mx = 0;  // staged vertices, the workgroup's edge (slot) range
    int64_t lo_v = 0;
    if (sliced) {
      const int64_t per = (n + size - 1) / size;
      lo_v = me * per;
      nf = (int)(lo_v >= n ? 0 : (n - lo_v < per ? n - lo_v : per));
      int32_t u = 0, rb = 0, d = 0;
      if ((int)threadIdx.x < nf) {
        u = load_shared<true>(&q[lo_v + threadIdx.x]);
        rb = a.R[u];
        d = a.R[u + 1] - rb;
        s_u[threadIdx.x] = u;
        s_rb[threadIdx.x] = rb;
        s_off[threadIdx.x] = d;
        s_pay[threadIdx.x] = fs.seg_payload(u);
      }
      if (m < 0) {  // a frontier from outside: count its edges first
        const uint32_t ws = wave_sum((uint32_t)d);
        if (lane() == 0) s_m[w] = ws;
        __syncthreads();
        uint32_t mine = 0;
        for (int i = 0; i < NW; ++i) mine += s_m[i];
        rotate();
        const unsigned long long x = team_barrier(&tw->arrive[it % 3], size, 0, mine);
        if (x == ~0ull) {
          failed = true;
          break;
        }
        m = (int64_t)(x >> 32);
        ++it;
      }
      total = m;
      if (a.log) {  // traced: the largest degree over the team
        mx = wave_max(d);
        if (lane() == 0 && mx > 0) atomicMax(&tw->max_deg[it % 3], (uint32_t)mx);
      }
      slots = nf << a.log_w;
      e0 = 0;
      e1 = slots;
      __syncthreads();
    } else {
      nf = (int)n;
      for (int j = threadIdx.x; j < nf; j += kAdvBlock) s_u[j] = load_shared<true>(&q[j]);
      __syncthreads();
      constexpr int KMAX = kTeamMaxStaged / kAdvBlock;
      const int K = (nf + kAdvBlock - 1) / kAdvBlock;  // consecutive vertices per thread
      const int j0 = (int)threadIdx.x * K;
      int64_t sum = 0;
      int32_t rb[KMAX], d[KMAX];
      pay_t pay[KMAX];
#pragma unroll
      for (int r = 0; r < KMAX; ++r) {
        const int32_t u = r < K && j0 + r < nf ? s_u[j0 + r] : -1;
        rb[r] = u >= 0 ? a.R[u] : 0;
        d[r] = u >= 0 ? a.R[u + 1] - rb[r] : 0;
        pay[r] = u >= 0 ? fs.seg_payload(u) : (pay_t)0;
      }
#pragma unroll
      for (int r = 0; r < KMAX; ++r) {
        sum += d[r];
        mx = d[r] > mx ? d[r] : mx;
      }
      int64_t ex = block_excl_scan<kAdvBlock>(sum, s_tot, &total);
#pragma unroll
      for (int r = 0; r < KMAX; ++r)
        if (r < K && j0 + r < nf) {
          s_rb[j0 + r] = rb[r];
          s_pay[j0 + r] = pay[r];
          s_off[j0 + r] = (int32_t)ex;
          ex += d[r];
        }
      if (threadIdx.x == 0) s_off[nf] = (int32_t)total;
      mx = wave_max(mx);
      if (lane() == 0) s_max[w] = mx;
      __syncthreads();
      for (int i = 0; i < NW; ++i) mx = s_max[i] > mx ? s_max[i] : mx;
      int64_t per = (total + size - 1) / size;
      if (per < kAdvBlock) per = kAdvBlock;
      e0 = (int)(me * per < total ? me * per : total);
      e1 = (int)(e0 + per < total ? e0 + per : total);
      slots = e1 - e0;
    }
    if (total > kTeamMaxM || total > a.max_m) break;
    // each frontier vertex once over the team
    if (sliced) {
      if ((int)threadIdx.x < nf) fs.frontier_vertex(s_u[threadIdx.x]);
    } else {
      for (int j = me * kAdvBlock + threadIdx.x; j < nf; j += size * kAdvBlock)
        fs.frontier_vertex(s_u[j]);
    }
    int32_t* __restrict__ q_next = a.qs.q[(a.cur0 + step + 1) % 3];
    uint32_t* cnt = &tw->q_count[it % 3];
    uint32_t n_new = 0, m_new = 0;  // this workgroup's new vertices and their edges
    for (int base = e0; base < e1; base += kAdvBlock * B) {
      bool ok[B];
      int32_t u[B], ce[B], v[B];
      pay_t pay[B];
#pragma unroll
      for (int r = 0; r < B; ++r) {
        const int e = base + r * kAdvBlock + (int)threadIdx.x;
        int k = 0, x = 0;
        ok[r] = e < e1;
        if (sliced) {
          k = ok[r] ? e >> a.log_w : 0;
          x = e & ((1 << a.log_w) - 1);
          ok[r] = ok[r] && x < s_off[k];
        } else if (ok[r]) {
          k = upper_index(s_off, 0, nf - 1, e);
          x = e - s_off[k];
        }
        u[r] = s_u[k];
        pay[r] = s_pay[k];
        ce[r] = s_rb[k] + x;
      }
      const uint32_t n_app = edge_commit<F, B>(fs, a.C, ok, u, pay, ce, v);
      // (the new vertices' degrees are on their way while the slots are reserved)
      int32_t dg[B];
#pragma unroll
      for (int r = 0; r < B; ++r) dg[r] = sliced && ok[r] ? a.R[v[r] + 1] - a.R[v[r]] : 0;
      const uint32_t inc = wave_incl_scan(n_app);
      if (lane() == kWave - 1) s_n[w] = inc;
      __syncthreads();
      uint32_t before = 0, all = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        if (i < w) before += s_n[i];
        all += s_n[i];
      }
      n_new += all;
      if (threadIdx.x == 0) s_base = all ? atomicAdd(cnt, all) : 0u;
      __syncthreads();
      uint32_t at = s_base + before + inc - n_app;
#pragma unroll
      for (int r = 0; r < B; ++r) {
        if (ok[r]) q_next[at++] = v[r];
        m_new += (uint32_t)dg[r];
      }
    }
    if (sliced) {
      m_new = wave_sum(m_new);
      if (lane() == 0) s_m[w] = m_new;
      __syncthreads();
      m_new = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) m_new += s_m[i];
    }
    rotate();
    const unsigned long long x = team_barrier(&tw->arrive[it % 3], size, n_new, m_new);
    if (x == ~0ull) {
      failed = true;
      break;
    }
    if (a.log && me == 0 && threadIdx.x == 0) {
      a.log[3 * step + 0] = n;
      a.log[3 * step + 1] = total;
      a.log[3 * step + 2] = sliced ? (int64_t)load_shared<true>(&tw->max_deg[it % 3]) : mx;
    }
    vm += total;
    vn += n;
    n = (int64_t)((x >> 8) & 0xffffffull);
    m = (int64_t)(x >> 32);
    ++it;
    ++step;
    fs = fs.next();
  }
  if (me == 0 && threadIdx.x == 0) {
    const int cur = (a.cur0 + step) % 3;
    atomicMax(&ctrl->dl_step[(a.seq + 1) & 1], step);
    if (step != step0) {
      ctrl->dl_levels = step;
      ctrl->dl_team += step - step0;
      ctrl->q_count[cur] = (uint32_t)n;
      ctrl->q_count[(cur + 1) % 3] = 0;
      ctrl->q_count[(cur + 2) % 3] = 0;
      ctrl->dl_vm[step & 1] = vm;
      ctrl->dl_vn[step & 1] = vn;
      fs.store(ctrl, step);
    }
  }
  if (failed && threadIdx.x == 0) atomicOr(&ctrl->dl_fail, 1u);
}

// A level like those of k_dstep on graphs without long rows (every row at most kDpMaxDegree
// neighbours): the frontier needs no balancing across workgroups, so each one
// takes slices of kAdvBlock vertices of it, scans their degrees and strip-mines
// their edges.  No workgroup stages the whole frontier, which lifts the bound on
// its size to kDpMaxN; the level's edge count m_f, which the decision needs
// first, comes from the pass that finalised the previous level
// (ctrl->dl_mf[step & 1]; that pass adds up the other slot, cleared here).
// Bound by the chain of dependent loads (queue, row bounds, columns, probe,
// atomic, append); against a level with its own host round trip it saves the
// statistics, the publication and the wait (64-source batch on a 384 x 384 grid,
// pushed throughout: 35 -> 21 us a level).
template <class F>
__global__ __launch_bounds__(kAdvBlock) void k_dpush(DlArgs a, F f) {
  constexpr int B = 4;
  __shared__ int32_t s_off[kAdvBlock];
  __shared__ int32_t s_u[kAdvBlock];
  __shared__ int32_t s_rb[kAdvBlock];
  __shared__ typename F::pay_t s_pay[kAdvBlock];
  __shared__ int32_t s_tot[kAdvBlock / kWave + 1];
  Ctrl* ctrl = a.ctrl;
  if (ctrl->dl_stop) return;
  const int64_t n_f = ctrl->q_count[a.cur];
  const int64_t m_f = ctrl->dl_mf[a.step & 1];
  const int64_t vm = ctrl->dl_vm[a.step & 1];
  const int64_t vn = ctrl->dl_vn[a.step & 1];
  const int next = (a.cur + 1) % 3, prev = (a.cur + 2) % 3;
  const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
  if (!(n_f > 0 && n_f <= a.max_n && m_f <= a.max_m) ||
      (a.do_a >= 0.0 && (double)m_f > (double)a.E * a.do_a)) {
    if (lead) ctrl->dl_stop = 1;
    return;
  }
  if (lead) {
    // none of these is read by this kernel
    ctrl->dl_levels = a.step + 1;
    ctrl->q_count[prev] = 0;
    ctrl->dl_vm[(a.step + 1) & 1] = vm + m_f;
    ctrl->dl_vn[(a.step + 1) & 1] = vn + n_f;
    ctrl->dl_mf[(a.step + 1) & 1] = 0;
  }
  for (int64_t b0 = (int64_t)blockIdx.x * kAdvBlock; b0 < n_f; b0 += (int64_t)gridDim.x * kAdvBlock) {
    const int64_t i = b0 + threadIdx.x;
    int32_t u0 = 0, rb = 0, d = 0;
    typename F::pay_t pay0 = 0;
    if (i < n_f) {
      u0 = a.q_cur[i];
      rb = a.R[u0];
      d = a.R[u0 + 1] - rb;
      pay0 = f.seg_payload(u0);
    }
    int32_t total;
    s_off[threadIdx.x] = block_excl_scan<kAdvBlock>(d, s_tot, &total);
    s_u[threadIdx.x] = u0;
    s_rb[threadIdx.x] = rb;
    s_pay[threadIdx.x] = pay0;
    __syncthreads();
    for (int base = 0; base < total; base += kAdvBlock * B) {
      bool ok[B];
      int32_t u[B];
      typename F::pay_t pay[B];
      int32_t ce[B];
#pragma unroll
      for (int r = 0; r < B; ++r) {
        const int e = base + r * kAdvBlock + threadIdx.x;
        ok[r] = e < total;
        const int k = ok[r] ? upper_index(s_off, 0, kAdvBlock - 1, e) : 0;
        u[r] = s_u[k];
        pay[r] = s_pay[k];
        ce[r] = s_rb[k] + (e - s_off[k]);
      }
      edge_batch<F, B, true>(f, a.C, ok, u, pay, ce, a.q_next, &ctrl->q_count[next]);
    }
    __syncthreads();
  }
}

}  // namespace gr
