// Batched shortest paths: up to 16 single-source SSSP runs share each sweep
// over the graph (the paper's future-work task parallelism, Sec. 8, applied to
// Alg. 1).  Every vertex holds KS packed keys (dist << 32 | pred, one per
// source, as in the single-source relaxation) in one 8 * KS byte row, so the
// keys of a target vertex for all sources sit in one or two cache lines.  The
// frontier is the union of the sources' frontiers; amask[v] says for which
// sources v is active (its distance dropped in the previous iteration).
//
// One iteration:
//   relax  output-balanced like LB: each workgroup takes a chunk of the
//          frontier's edges, a lane an edge.  One load brings the target's row
//          of one-byte distance bounds (the mirror) and screens all sources of
//          the edge; the (edge, source) pairs that pass are listed in LDS and
//          relaxed with a plain read of the target's key and a no-return
//          atomic minimum (Update_Label).  An edge that lowered distances ORs
//          their sources into nmask[v] once.  Few edges (LIST): the first
//          setter appends v to the candidates of the next frontier
//          (Remove_Redundant for the union);
//   clear  amask of the current frontier = 0 (LIST);
//   move   for the candidates, or after many edges for every vertex:
//          amask = nmask, nmask = 0, listing the vertices with an active
//          source left.
// With `relaxed` (nullable, KS words per vertex like the keys), each chunk
// raises relaxed[u][s] to 1 + the distance of (u, s) as it stages u, for every
// active source s of u (the distance that the chunk's edges of u are relaxed
// with), and move resets it when the pair joins the next
// frontier.  A pair whose relaxed value equals 1 + its distance at move time
// was active and had every edge relaxed with that final distance, so move
// drops it (the single-source cull of vertices already relaxed with their
// final distance, per source); a value from an earlier iteration is larger
// than 1 + a distance that has dropped since, and 0 never matches.
// Keys only decrease, so a source's bit is set exactly when the vertex's
// distance for that source dropped in the iteration; every vertex then
// relaxes its edges with its final distance for every source at least once,
// and the key ends as the smallest (distance, predecessor) pair: the same
// canonical result as the single-source runs.
//
// Optional near / far split (Sec. 5.1 priority queue; one threshold T for all
// sources): an improvement to a distance >= T sets the pair's bit in fmask[v]
// instead of nmask[v] (the first setter puts v on the far pile).  When the
// frontier runs dry, T grows by delta and the far pile is split: pairs now
// below T join the frontier, pairs still above stay, pairs whose distance fell
// below the old threshold meanwhile were expanded with it already and are
// dropped.  Results are unchanged.
#include "edge_range.h"
#include "k_advance.h"

namespace gr {

namespace {

using u64 = unsigned long long;

// Orders a wavefront's LDS stores before its later loads of them by other lanes.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A wavefront's entries for a list in memory, collected in LDS and appended with one
// counter atomic per kCap - 64 or more of them: the counter is one address for the whole
// grid and takes some 6.4 ns per atomic.  (A star's 1 M edges into the far pile: 82 us
// with an atomic per 64 edges, 41 with these.)
struct WaveList {
  static constexpr int kCap = 256;
  int32_t* buf;  // LDS [kCap], the wavefront's own
  int n = 0;     // the same in all lanes
  __device__ __forceinline__ void flush(int32_t* __restrict__ q, uint32_t* __restrict__ count) {
    if (n == 0) return;
    wave_lds_fence();
    uint32_t base = 0;
    if (lane() == 0) base = atomicAdd(count, (uint32_t)n);
    base = __shfl(base, 0);
    for (int i = lane(); i < n; i += kWave) q[base + i] = buf[i];
    wave_lds_fence();
    n = 0;
  }
  // v of the lanes with `first`; called by all lanes
  __device__ __forceinline__ void put(bool first, int32_t v, int32_t* __restrict__ q,
                                      uint32_t* __restrict__ count) {
    const uint64_t m = __ballot(first);
    if (!m) return;
    if (first) buf[n + __popcll(m & ((1ull << lane()) - 1ull))] = v;
    n += __popcll(m);
    if (n > kCap - kWave) flush(q, count);
  }
};

// A vertex's mirror row: one byte per source.
template <int KS>
using MirrorRow = std::conditional_t<KS == 16, uint4, std::conditional_t<KS == 8, uint2, uint32_t>>;

__device__ __forceinline__ uint32_t row_word(const uint4& r, int i) {
  return i == 0 ? r.x : (i == 1 ? r.y : (i == 2 ? r.z : r.w));
}
__device__ __forceinline__ uint32_t row_word(const uint2& r, int i) { return i == 0 ? r.x : r.y; }
__device__ __forceinline__ uint32_t row_word(uint32_t r, int) { return r; }

constexpr int kMsSegs = 256;   // frontier segments staged per pass
constexpr int kMsItems = 512;  // listed (edge, source) pairs a wavefront relaxes at a time

// What bounds it: the rows of keys are 128 bytes, one cache line per edge that only
// the memory behind the L2s holds (R-MAT 20, 16 sources: 134 MB), and the pairs are
// KS times the edges.  A pair per lane spent some 120 instructions on finding its
// edge and source and a line per edge on the keys.  Screened with the mirror a pair
// costs 9 instructions, and an edge 16 bytes of a table an eighth of the size; the
// mirror is sharpened inside the launch (a byte store per relaxed pair that is lower
// than the entry; entries stay upper bounds whatever the order of the stores), so
// that after the first few edges into a vertex only improvements read its keys.
// The sources' distances of 256 segments are staged in LDS (16 KB, so that 7
// workgroups share a CU).
// LIST costs atomics on one counter, some 6.4 ns each (WaveList): with one per wavefront
// and 64 edges, 420 K of them held an iteration of 27 M edges at 2.7 ms.  Without, nmask
// itself is the list.  R-MAT 20, 16 sources, the four large iterations: 14.3 ms as a
// pair per lane, 12.0 with LIST (one per 64 edges), 2.4 without.
template <int KS, bool PQ, bool LIST>
__global__ __launch_bounds__(256) void k_msssp_relax(
    const int32_t* __restrict__ frontier, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ rstart, const int32_t* __restrict__ chunk_start, int32_t n_f,
    int32_t m_f, int32_t chunk, const int32_t* __restrict__ C, const uint32_t* __restrict__ W,
    u64* __restrict__ keys, DistMirror mirror, const uint32_t* __restrict__ amask,
    uint32_t* __restrict__ nmask, uint32_t* __restrict__ fmask, int32_t* __restrict__ far_q,
    uint32_t* __restrict__ far_count, uint32_t T, const int32_t* __restrict__ perm,
    uint32_t* __restrict__ relaxed, int32_t* __restrict__ out_q,
    uint32_t* __restrict__ out_count) {
  constexpr int BLOCK = 256;
  constexpr int WAVES = BLOCK / kWave;
  constexpr int B = 2;  // edges per lane in flight
  constexpr int J = 2;  // pairs per lane in flight
  using Row = MirrorRow<KS>;
  __shared__ int32_t s_off[kMsSegs + 1];
  __shared__ int32_t s_rb[kMsSegs];
  __shared__ uint32_t s_id[kMsSegs];
  __shared__ int32_t s_u[kMsSegs];
  __shared__ uint16_t s_am[kMsSegs];
  __shared__ __align__(16) uint32_t s_du[kMsSegs * KS];  // ~0: source not active
  __shared__ uint16_t s_item[WAVES][kMsItems];           // source << 6 | lane
  __shared__ uint32_t s_near[WAVES][kWave], s_far[WAVES][kWave];
  __shared__ int32_t s_list[LIST ? WAVES * WaveList::kCap : 1];
  __shared__ int32_t s_pile[PQ ? WAVES * WaveList::kCap : 1];
  const int wv = threadIdx.x / kWave;
  WaveList near_l{LIST ? &s_list[wv * WaveList::kCap] : nullptr};
  WaveList far_l{PQ ? &s_pile[wv * WaveList::kCap] : nullptr};
  const int c = blockIdx.x;
  const int64_t e0 = (int64_t)c * chunk;
  const int64_t e1 = e0 + chunk < m_f ? e0 + chunk : m_f;
  const int nchunks = (int)(((int64_t)m_f + chunk - 1) / chunk);
  const int sb = chunk_start[c];
  const int se = c + 1 < nchunks ? chunk_start[c + 1] : n_f - 1;
  for (int pb = sb; pb <= se; pb += kMsSegs) {
    const int cnt = (se - pb + 1) < kMsSegs ? (se - pb + 1) : kMsSegs;
    for (int i = threadIdx.x; i < cnt; i += BLOCK) {
      const int s = pb + i;
      s_off[i] = offsets[s];
      s_rb[i] = rstart[s];
      const int32_t u = frontier[s];
      s_u[i] = u;
      s_am[i] = (uint16_t)amask[u];
      s_id[i] = (uint32_t)(perm ? perm[u] : u);
    }
    if (threadIdx.x == 0) s_off[cnt] = offsets[pb + cnt];
    __syncthreads();
    // a thread per (segment, source), so that the rows are read and raised in whole
    // lines; kRows of them in flight
    constexpr int kRows = 4;
    for (int x0 = threadIdx.x; x0 < cnt * KS; x0 += BLOCK * kRows) {
      uint32_t d[kRows];
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        const int x = x0 + j * BLOCK;
        d[j] = ~0u;
        if (x < cnt * KS && (s_am[x / KS] >> (x % KS) & 1u))
          d[j] = (uint32_t)(keys[(int64_t)s_u[x / KS] * KS + x % KS] >> 32);
      }
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        const int x = x0 + j * BLOCK;
        if (x >= cnt * KS) continue;
        if (relaxed && d[j] != ~0u)
          atomicMax(&relaxed[(int64_t)s_u[x / KS] * KS + x % KS], d[j] + 1u);
        s_du[x] = d[j];
      }
    }
    __syncthreads();
    const int32_t lo = (int32_t)(e0 > s_off[0] ? e0 : s_off[0]);
    const int32_t hi = (int32_t)(e1 < s_off[cnt] ? e1 : s_off[cnt]);
    for (int64_t b0 = wave_first_edge(lo, wv); b0 < hi; b0 += BLOCK * B) {
      int32_t v[B], k[B];
      uint32_t w[B];
      Row row[B];
#pragma unroll
      for (int r = 0; r < B; ++r) {
        const int64_t e = b0 + r * BLOCK + lane();
        k[r] = -1;
        v[r] = 0;
        w[r] = 0;
        if (e < hi) {
          k[r] = upper_index(s_off, 0, cnt - 1, e);
          const int64_t ce = (int64_t)s_rb[k[r]] + (e - s_off[k[r]]);
          v[r] = C[ce];
          w[r] = W[ce];
        }
      }
#pragma unroll
      for (int r = 0; r < B; ++r)
        if (mirror.p && k[r] >= 0) row[r] = reinterpret_cast<const Row*>(mirror.p)[v[r]];
#pragma unroll
      for (int r = 0; r < B; ++r) {
        // the sources whose candidate may reach or beat the target's distance
        uint32_t pm = 0;
        if (k[r] >= 0) {
          const uint32_t* du = &s_du[k[r] * KS];
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            const uint32_t d = du[s];
            const uint32_t cand = d + w[r];
            // ceil(cand / 2^shift) <= the entry, or no entry; no sum past 2^32 - 2
            const uint32_t q = (cand > 0u ? cand - 1u : 0u) >> mirror.shift;
            const uint32_t m =
                mirror.p && cand ? (row_word(row[r], s / 4) >> (8 * (s % 4)) & 0xffu) : kMirrorNone;
            const bool ok = cand >= d && cand != ~0u &&
                            (q < kMirrorNone - 1u ? q : kMirrorNone - 1u) < m;
            pm |= ok ? 1u << s : 0u;
          }
        }
        s_near[wv][lane()] = 0;
        if constexpr (PQ) s_far[wv][lane()] = 0;
        const uint32_t n = (uint32_t)__popc(pm);
        const uint32_t inc = wave_incl_scan(n);
        const uint32_t total = __builtin_amdgcn_readfirstlane(__shfl(inc, kWave - 1));
        uint32_t at = inc - n;  // of this lane's next pair
        for (uint32_t t0 = 0; t0 < total; t0 += kMsItems) {
          for (; pm && at < t0 + kMsItems; pm &= pm - 1, ++at)
            s_item[wv][at - t0] = (uint16_t)((__ffs(pm) - 1) << 6 | lane());
          wave_lds_fence();
          const uint32_t end = total < t0 + kMsItems ? total : t0 + kMsItems;
          for (uint32_t t = t0; t < end; t += J * kWave) {
            u64 key[J], nk[J];
            int64_t y[J];
            uint32_t it[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
              const uint32_t x = t + j * kWave + lane();
              it[j] = x < end ? (uint32_t)s_item[wv][x - t0] : ~0u;
              const int l = (int)(it[j] & 63u);
              const int s = (int)(it[j] >> 6) & (KS - 1);
              const int32_t vl = __shfl(v[r], l);
              const int32_t kl = __shfl(k[r], l);
              const uint32_t wl = __shfl(w[r], l);
              key[j] = 0;
              if (it[j] != ~0u) {
                y[j] = (int64_t)vl * KS + s;
                nk[j] = (u64)(s_du[kl * KS + s] + wl) << 32 | s_id[kl];
                key[j] = keys[y[j]];
              }
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
              if (it[j] == ~0u) continue;
              const bool lower = nk[j] < key[j];
              if (lower) atomicMin(&keys[y[j]], nk[j]);
              if (mirror.p) {
                const uint8_t qn = mirror_of(nk[j], mirror.shift);
                const uint8_t q = lower ? qn : mirror_of(key[j], mirror.shift);
                if (lower ? q != kMirrorNone : q < qn) mirror.p[y[j]] = q;
              }
              if ((uint32_t)(nk[j] >> 32) < (uint32_t)(key[j] >> 32)) {
                const uint32_t bit = 1u << (it[j] >> 6);
                if (!PQ || (uint32_t)(nk[j] >> 32) < T) atomicOr(&s_near[wv][it[j] & 63u], bit);
                else atomicOr(&s_far[wv][it[j] & 63u], bit);
              }
            }
          }
          wave_lds_fence();  // the list is rewritten
        }
        if (total == 0) continue;
        const uint32_t nb = s_near[wv][lane()];
        if constexpr (LIST)
          near_l.put(nb != 0 && atomicOr(&nmask[v[r]], nb) == 0u, v[r], out_q, out_count);
        else if (nb) atomicOr(&nmask[v[r]], nb);
        if constexpr (PQ) {
          const uint32_t fb = s_far[wv][lane()];
          far_l.put(fb != 0 && atomicOr(&fmask[v[r]], fb) == 0u, v[r], far_q, far_count);
        }
        wave_lds_fence();
      }
    }
    __syncthreads();
  }
  if constexpr (LIST) near_l.flush(out_q, out_count);
  if constexpr (PQ) far_l.flush(far_q, far_count);
}

// Far-pile split (priority queue): for every pile entry and every source bit
// of its fmask, distance >= T1 stays (next pile), T0 <= distance < T1 joins
// the frontier, distance < T0 was expanded already (dropped).
__global__ __launch_bounds__(256) void k_msssp_refill(
    const int32_t* __restrict__ pile, const uint32_t* __restrict__ n_pile,
    int32_t* __restrict__ pile_next, uint32_t* __restrict__ n_pile_next,
    const u64* __restrict__ keys, int KS, uint32_t* __restrict__ fmask,
    uint32_t* __restrict__ amask, uint32_t T0, uint32_t T1, int32_t* __restrict__ out_q,
    uint32_t* __restrict__ out_count) {
  const int64_t n = *n_pile;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t b0 = (int64_t)blockIdx.x * 256; b0 < n; b0 += stride) {
    const int64_t i = b0 + threadIdx.x;
    int32_t v = 0;
    uint32_t act = 0, keep = 0;
    if (i < n) {
      v = pile[i];
      const uint32_t m = fmask[v];
      for (uint32_t b = m; b; b &= b - 1) {
        const int sI = __ffs(b) - 1;
        const uint32_t d = (uint32_t)(keys[(int64_t)v * KS + sI] >> 32);
        if (d >= T1) keep |= 1u << sI;
        else if (d >= T0) act |= 1u << sI;
      }
      fmask[v] = keep;
      if (act) amask[v] = act;
    }
    const uint32_t a = block_append<256>(act ? 1u : 0u, out_count);
    if (act) out_q[a] = v;
    const uint32_t k = block_append<256>(keep ? 1u : 0u, n_pile_next);
    if (keep) pile_next[k] = v;
  }
}

// keys = no path (~0), mirror = no entry, masks = 0, then the sources: key (0, -1) and the
// source's bit in amask; the distinct source vertices form frontier 0.
__global__ __launch_bounds__(256) void k_msssp_init(u64* __restrict__ keys, int KS,
                                                    uint32_t* __restrict__ amask,
                                                    uint32_t* __restrict__ nmask,
                                                    uint32_t* __restrict__ fmask,
                                                    uint32_t* __restrict__ relaxed,
                                                    uint8_t* __restrict__ mirror, int64_t V) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t n = V * KS;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    keys[i] = ~0ull;
    if (relaxed) relaxed[i] = 0u;
    if (mirror && i < n / 4) reinterpret_cast<uint32_t*>(mirror)[i] = ~0u;
    if (i < V) {
      amask[i] = 0u;
      nmask[i] = 0u;
      fmask[i] = 0u;
    }
  }
}

__global__ __launch_bounds__(64) void k_msssp_seed(const int32_t* __restrict__ src, int32_t k,
                                                   int KS, u64* __restrict__ keys,
                                                   uint32_t* __restrict__ amask) {
  const int s = threadIdx.x;
  if (s < k) {
    const int32_t v = src[s];
    keys[(int64_t)v * KS + s] = 0xffffffffull;  // distance 0, predecessor -1
    atomicOr(&amask[v], 1u << s);
  }
}

__global__ __launch_bounds__(256) void k_msssp_clear(const int32_t* __restrict__ q,
                                                     const uint32_t* __restrict__ n,
                                                     uint32_t* __restrict__ amask) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)*n) amask[q[i]] = 0u;
}

// LIST: over the *n vertices of q; otherwise over all V, which also clears amask.
// KS lanes per vertex, so that the rows are read in whole lines, four rows in flight
// per lane.  The appends share one counter (6.4 ns each): many vertices go in tiles
// of 1024, a list or a small graph, which need workgroups more than fewer appends, in
// tiles of 64 (16 K vertices: 15 us in tiles of 1024, 5 in tiles of 64), graphs between
// in tiles of 256 (90 K vertices, 16 sources: 28 us in tiles of 1024, 11 in tiles of 256).
template <int KS, bool LIST, int kMoveTile>
__global__ __launch_bounds__(256) void k_msssp_move(const int32_t* __restrict__ q,
                                                    const uint32_t* __restrict__ n, int64_t V,
                                                    uint32_t* __restrict__ amask,
                                                    uint32_t* __restrict__ nmask,
                                                    const u64* __restrict__ keys,
                                                    uint32_t* __restrict__ relaxed,
                                                    int32_t* __restrict__ out_q,
                                                    uint32_t* __restrict__ out_count) {
  constexpr int VPT = (kMoveTile + 255) / 256;
  constexpr int STEP = 256 / KS;                // vertices per turn
  constexpr int U = kMoveTile / STEP < 4 ? 1 : 4;
  static_assert(kMoveTile % (STEP * U) == 0);
  __shared__ int32_t s_v[kMoveTile];
  __shared__ uint16_t s_nm[kMoveTile];
  const int64_t count = LIST ? (int64_t)*n : V;
  const int sI = threadIdx.x % KS;
  for (int64_t b0 = (int64_t)blockIdx.x * kMoveTile; b0 < count;
       b0 += (int64_t)gridDim.x * kMoveTile) {
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int j = r * 256 + threadIdx.x;
      if (j >= kMoveTile) continue;
      int32_t v = 0;
      uint32_t nm = 0;
      if (b0 + j < count) {
        v = LIST ? q[b0 + j] : (int32_t)(b0 + j);
        nm = nmask[v];
      }
      s_v[j] = v;
      s_nm[j] = (uint16_t)nm;
    }
    __syncthreads();
    if (relaxed) {
      for (int j0 = threadIdx.x / KS; j0 < kMoveTile; j0 += STEP * U) {
        bool on[U];
        uint32_t rel[U], d[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int64_t x = (int64_t)s_v[j0 + j * STEP] * KS + sI;
          on[j] = s_nm[j0 + j * STEP] >> sI & 1u;
          rel[j] = on[j] ? relaxed[x] : 0u;
          d[j] = on[j] ? (uint32_t)(keys[x] >> 32) : 0u;
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          if (on[j] && rel[j] == d[j] + 1u) on[j] = false;
          else if (rel[j]) relaxed[(int64_t)s_v[j0 + j * STEP] * KS + sI] = 0u;
          const uint32_t nm = (uint32_t)(__ballot(on[j]) >> (lane() - sI)) & ((1u << KS) - 1u);
          if (sI == 0) s_nm[j0 + j * STEP] = (uint16_t)nm;
        }
      }
      __syncthreads();
    }
    uint32_t listed = 0;
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int j = r * 256 + threadIdx.x;
      if (j >= kMoveTile || b0 + j >= count) continue;
      nmask[s_v[j]] = 0u;
      amask[s_v[j]] = s_nm[j];
      listed += s_nm[j] ? 1u : 0u;
    }
    uint32_t a = block_append<256>(listed, out_count);
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int j = r * 256 + threadIdx.x;
      if (j < kMoveTile && b0 + j < count && s_nm[j]) out_q[a++] = s_v[j];
    }
    __syncthreads();  // the tile is rewritten
  }
}

// dist[s][o] / pred[s][o] at caller ids for the k sources of the pass, and the sum
// over sources of the degrees of their reached vertices (R: the caller's row
// offsets).  Threads run over caller ids: a row of keys is read wherever it lies as
// whole lines, and the outputs are written in order (the other way round, each of 32
// arrays is written 4 bytes at a time: 383 us, now 54, for R-MAT 20 and 16 sources).
template <int KS>
__global__ __launch_bounds__(256) void k_msssp_finalize(const u64* __restrict__ keys, int32_t k,
                                                        const int32_t* __restrict__ R,
                                                        int64_t V, uint32_t* __restrict__ dist,
                                                        int32_t* __restrict__ pred,
                                                        const int32_t* __restrict__ inv,
                                                        int64_t* __restrict__ reached_edges) {
  __shared__ int64_t s[256 / kWave];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t acc = 0;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < V; o += stride) {
    const int64_t v = inv ? inv[o] : o;
    const int64_t deg = (int64_t)R[o + 1] - R[o];
    u64 key[KS];
    const ulonglong2* row = reinterpret_cast<const ulonglong2*>(keys + v * KS);
#pragma unroll
    for (int j = 0; j < KS / 2; ++j) {
      if (2 * j >= k) break;
      const ulonglong2 x = row[j];
      key[2 * j] = x.x;
      key[2 * j + 1] = x.y;
    }
#pragma unroll
    for (int sI = 0; sI < KS; ++sI) {
      if (sI >= k) break;
      const uint32_t d = (uint32_t)(key[sI] >> 32);
      dist[(int64_t)sI * V + o] = d;
      if (pred) pred[(int64_t)sI * V + o] = (int32_t)(uint32_t)(key[sI] & 0xffffffffull);
      if (d != 0xffffffffu) acc += deg;
    }
  }
  acc = wave_sum(acc);
  if (lane() == 0) s[threadIdx.x / kWave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int i = 0; i < 256 / kWave; ++i) t += s[i];
    if (t) atomicAdd((unsigned long long*)reached_edges, (unsigned long long)t);
  }
}

// A source has no predecessor; a zero-weight edge into it may have tied its
// distance 0 with a smaller (distance, predecessor) key.
__global__ __launch_bounds__(64) void k_msssp_source_pred(const int32_t* __restrict__ src_orig,
                                                          int32_t k, int64_t V,
                                                          int32_t* __restrict__ pred) {
  const int s = threadIdx.x;
  if (s < k) pred[(int64_t)s * V + src_orig[s]] = -1;
}

constexpr int64_t kMsMidVertices = 1 << 19;  // k_msssp_move: tiles of 256 up to here

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

int msssp_row(int k) { return k <= 4 ? 4 : (k <= 8 ? 8 : 16); }

int msssp_chunk(int chunk) { return chunk == 512 || chunk == 2048 ? chunk : 1024; }

hipError_t launch_msssp_init(u64* keys, int KS, uint32_t* amask, uint32_t* nmask, uint32_t* fmask,
                             uint32_t* relaxed, uint8_t* mirror, int64_t V,
                             const int32_t* src_dev, int32_t k, hipStream_t st) {
  int64_t g = blocks_for(V * KS, 256);
  if (g > 8192) g = 8192;
  k_msssp_init<<<(unsigned)g, 256, 0, st>>>(keys, KS, amask, nmask, fmask, relaxed, mirror,
                                            V);
  k_msssp_seed<<<1, 64, 0, st>>>(src_dev, k, KS, keys, amask);
  return hipGetLastError();
}

#define GR_MS_ROW(KS, CALL)          \
  switch (KS) {                       \
    case 4: { constexpr int R_ = 4; CALL; break; }   \
    case 8: { constexpr int R_ = 8; CALL; break; }   \
    default: { constexpr int R_ = 16; CALL; break; } \
  }

hipError_t launch_msssp_relax(int KS, int chunk, const int32_t* frontier, const int32_t* offsets,
                              const int32_t* rstart, const int32_t* chunk_start, int64_t n_f,
                              int64_t m_f, const int32_t* C, const uint32_t* W, u64* keys,
                              DistMirror mirror, const uint32_t* amask, uint32_t* nmask,
                              const MsFar* far, const int32_t* perm, uint32_t* relaxed,
                              int32_t* out_q, uint32_t* out_count, hipStream_t st) {
  if (n_f <= 0 || m_f <= 0) return hipSuccess;
  const unsigned g = blocks_for(m_f, chunk);
#define GR_MS_RELAX(FAR, LIST, FM, FQ, FN, FT)                                              \
  GR_MS_ROW(KS, (k_msssp_relax<R_, FAR, LIST><<<g, 256, 0, st>>>(                           \
                    frontier, offsets, rstart, chunk_start, (int32_t)n_f, (int32_t)m_f,     \
                    chunk, C, W, keys, mirror, amask, nmask, FM, FQ, FN, FT, perm, relaxed, \
                    out_q, out_count)))
  if (far) {
    if (out_q) GR_MS_RELAX(true, true, far->fmask, far->pile, far->pile_count, far->T)
    else GR_MS_RELAX(true, false, far->fmask, far->pile, far->pile_count, far->T)
  } else {
    if (out_q) GR_MS_RELAX(false, true, nullptr, nullptr, nullptr, 0u)
    else GR_MS_RELAX(false, false, nullptr, nullptr, nullptr, 0u)
  }
#undef GR_MS_RELAX
  return hipGetLastError();
}

hipError_t launch_msssp_refill(const int32_t* pile, const uint32_t* n_pile, int64_t max_pile,
                               int32_t* pile_next, uint32_t* n_pile_next, const u64* keys, int KS,
                               uint32_t* fmask, uint32_t* amask, uint32_t T0, uint32_t T1,
                               int32_t* out_q, uint32_t* out_count, hipStream_t st) {
  if (max_pile <= 0) return hipSuccess;
  int64_t g = blocks_for(max_pile, 256);
  if (g > 2048) g = 2048;
  k_msssp_refill<<<(unsigned)g, 256, 0, st>>>(pile, n_pile, pile_next, n_pile_next, keys, KS,
                                              fmask, amask, T0, T1, out_q, out_count);
  return hipGetLastError();
}

hipError_t launch_msssp_rotate(const int32_t* cur_q, const uint32_t* cur_n, int64_t max_cur,
                               const int32_t* next_q, const uint32_t* next_n, int64_t max_next,
                               int64_t V, uint32_t* amask, uint32_t* nmask, const u64* keys, int KS,
                               uint32_t* relaxed, int32_t* out_q, uint32_t* out_count,
                               hipStream_t st) {
  if (next_q && max_cur > 0)
    k_msssp_clear<<<blocks_for(max_cur, 256), 256, 0, st>>>(cur_q, cur_n, amask);
  const int64_t n = next_q ? max_next : V;
  if (n <= 0) return hipGetLastError();
  const int tile = next_q || n <= kMsScanVertices ? 64 : n <= kMsMidVertices ? 256 : 1024;
  unsigned g = blocks_for(n, tile);
  if (g > 4096) g = 4096;
#define GR_MS_MOVE(LIST, TILE)                                                                  \
  GR_MS_ROW(KS, (k_msssp_move<R_, LIST, TILE><<<g, 256, 0, st>>>(next_q, next_n, V, amask, nmask, \
                                                                 keys, relaxed, out_q, out_count)))
  if (next_q) GR_MS_MOVE(true, 64)
  else if (tile == 64) GR_MS_MOVE(false, 64)
  else if (tile == 256) GR_MS_MOVE(false, 256)
  else GR_MS_MOVE(false, 1024)
#undef GR_MS_MOVE
  return hipGetLastError();
}

hipError_t launch_msssp_finalize(const u64* keys, int KS, int32_t k, const int32_t* R, int64_t V,
                                 uint32_t* dist, int32_t* pred, const int32_t* inv,
                                 const int32_t* src_orig_dev, int64_t* reached_edges,
                                 hipStream_t st) {
  unsigned g = blocks_for(V, 256);
  if (g > 1024) g = 1024;  // one atomic per workgroup, all on one address
  GR_MS_ROW(KS, (k_msssp_finalize<R_><<<g, 256, 0, st>>>(keys, k, R, V, dist, pred, inv,
                                                         reached_edges)))
  if (pred) k_msssp_source_pred<<<1, 64, 0, st>>>(src_orig_dev, k, V, pred);
  return hipGetLastError();
}

}  // namespace gr
