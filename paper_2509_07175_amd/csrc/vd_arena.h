// vd_arena.h -- per-wave output allocation and the work queue of the
// persistent clip kernels.
//
// A persistent wave processes many sites (or triangles).  Its output records
// go to arenas shared by all waves; instead of one global atomic per record
// (which serialises every wave on a handful of addresses), a wave reserves a
// chunk of C.chunk[r] slots with one atomic and hands out slots from it.  The
// unused tail of the last piece chunk is marked piece_site = -1 when the wave
// ends; face/vertex/neighbour/face-moment records are reached through offsets
// only, so their holes need no marking.
//
// Work items come from VD_QUEUES queues, queue k owning the k-th eighth of the
// items in order; workgroup b starts on queue b % 8 (the XCD it runs on when
// workgroups are dealt round-robin over the 8 XCDs), so an XCD works through a
// contiguous block of grid-ordered sites and keeps their neighbourhoods in its
// L2.  A wave whose queue is exhausted moves on to the next queue.  A batch
// can instead give each queue a list of positions (C.order), so that every
// queue starts with its most expensive diagrams.
#pragma once
#include "vd_internal.h"

// A wave's totals for the counters of one kind, lane l of the close adding entry
// l (one atomic instruction: counters of one line travel together).
struct WaveArena {
  long long cur[AR_N], end[AR_N];
  union {
    unsigned long long stat[CNT_STATS];
    struct {  // in the order of the counters from CNT_QUERIES on
      unsigned long long queries, clips, cands, gridq;
      unsigned long long pieces, faces, verts, nbrs;  // records written (real counts)
      unsigned long long dropped;                     // records that did not fit their arena
      // work counters of the clips (lane 0 updates them in LDS, so they cost no
      // registers across the carve)
      unsigned long long lowmargin, rounds, classified, newc, wasted, fantets;
    };
  };
  double minmargin;                               // smallest relative classification margin
  int qi;                                         // queues tried so far
};
static_assert(offsetof(WaveArena, fantets) - offsetof(WaveArena, queries) == 8 * (CNT_STATS - 1), "stat[] = the counters");

__device__ __forceinline__ void arena_init(WaveArena &A) {
  const int l = vd_lane();
  if (l < AR_N) A.cur[l] = A.end[l] = 0;
  if (l < CNT_STATS) A.stat[l] = 0;
  if (l == 0) {
    A.minmargin = 1.0;
    A.qi = 0;
  }
}

// k slots of each arena (lane r < AR_N: of arena r, 0 for none) for this wave;
// returns the first slot in the same lanes.  The range may reach past the
// arena's capacity: callers check.  All arenas that run short are refilled by
// one atomic instruction: their counters share a line, and a small clip waits
// for little else (thousands of waves, one site each).
__device__ __forceinline__ long long arena_take_all(WaveArena &A, const CellsDev &C, long long k) {
  const int l = vd_lane();
  long long cur = 0;
  if (l < AR_N) {
    cur = A.cur[l];
    if (k > 0 && cur + k > A.end[l]) {
      const long long c = C.chunk[l], t = k > c ? k : c;
      cur = (long long)__hip_atomic_fetch_add(GL(C.cnt) + l, (unsigned long long)t, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
      A.end[l] = cur + t;
    }
    A.cur[l] = cur + k;
  }
  return cur;
}

// (uniform counts -> lanes)
__device__ __forceinline__ int arena_counts(int piece, int face, int vert, int fint) {
  const int l = vd_lane();
  return l == AR_PIECE ? piece : l == AR_FACE ? face : l == AR_VERT ? vert : l == AR_FINT ? fint : 0;
}

// k slots of arena r (k and r uniform); returns the first slot.
__device__ __forceinline__ long long arena_take(WaveArena &A, const CellsDev &C, int r, long long k) {
  return readlane_ll(arena_take_all(A, C, vd_lane() == r ? k : 0), r);
}

// The piece slots that a chunk has left when it is too short for the next k at
// once become unused ones.
__device__ __forceinline__ void arena_skip_pieces(WaveArena &A, const CellsDev &C, int k) {
  const long long cur = readlane_ll(A.cur[AR_PIECE], 0), end = readlane_ll(A.end[AR_PIECE], 0);
  if (cur + k > end) {
    const long long p = cur + vd_lane();
    if (p < end && p < C.cap_piece) GL(C.piece_site)[p] = -1;
  }
}

// Next work item in [0, n), or -1 when every queue is exhausted.
__device__ __forceinline__ int queue_next(WaveArena &A, const CellsDev &C, long long n) {
  int r = -1;
  if (vd_lane() == 0) {
    const long long q8 = (n + VD_QUEUES - 1) / VD_QUEUES;
    const int x = (int)(blockIdx.x % VD_QUEUES);
    for (; A.qi < VD_QUEUES; A.qi++) {
      const int k = (x + A.qi) % VD_QUEUES;
      const long long beg = C.order ? C.qoff[k] : k * q8;
      const long long end = C.order ? C.qoff[k + 1] : ((k + 1) * q8 < n ? (k + 1) * q8 : n);
      if (beg >= end) continue;
      const int v = __hip_atomic_fetch_add(GL(C.queue) + k * VD_QSTRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (v < end) { r = C.order ? GL(C.order)[v] : v; break; }
    }
  }
  return __builtin_amdgcn_readlane(r, 0);
}

// Next item of the list that the sweep kernel left (complete when this runs), or
// -1.  A wave's first one is its own number, the others follow by atomics: waves
// beyond the list's end, usually all of them, read its length and are done.
__device__ __forceinline__ int redo_next(WaveArena &A, const CellsDev &C) {
  int r = -1;
  if (vd_lane() == 0) {
    const int n = (int)GL(C.cnt)[CNT_REDO];
    int v = blockIdx.x;
    if (A.qi && v < n)
      v = gridDim.x + __hip_atomic_fetch_add(GL(C.queue) + VD_QREDO * VD_QSTRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    A.qi = 1;
    if (v < n) r = GL(C.redo)[v];
  }
  return __builtin_amdgcn_readlane(r, 0);
}

// End of a persistent wave: mark the unused tail of its piece chunk and add
// its statistics to the global counters.
__device__ __forceinline__ void arena_close(WaveArena &A, const CellsDev &C) {
  const int l = vd_lane();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (written by other lanes)
  __builtin_amdgcn_wave_barrier();
  const long long a = A.cur[AR_PIECE], b = A.end[AR_PIECE] < C.cap_piece ? A.end[AR_PIECE] : C.cap_piece;
  for (long long p = a + l; p < b; p += 64) GL(C.piece_site)[p] = -1;
  if (l < CNT_STATS && A.stat[l]) atomicAdd(&C.cnt[CNT_QUERIES + l], A.stat[l]);
  if (l == 0 && A.minmargin < 1.0)
    atomicMin(&C.cnt[CNT_MINMARGIN], (unsigned long long)__double_as_longlong(A.minmargin));
}

// Adds v to a work counter of the wave's LDS totals: an LDS atomic from lane 0
// whose result is unused, so nothing waits for it and no register stays live.
__device__ __forceinline__ void count_add(unsigned long long &ctr, unsigned long long v) {
  if (vd_lane() == 0) __hip_atomic_fetch_add(&ctr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Relative margin of the classification of corners y against the plane
// n.y = c: |n.y - c| / (|n0 y0| + |n1 y1| + |n2 y2| + |c|), the signed distance
// over the magnitude its rounding error scales with.  Each lane brings up to two
// corners (valid flag, signed distance, scale).  Lane 0 keeps the wave's minimum
// and the count of margins below 1e-12 (near-degenerate decisions); the
// division is only taken when some corner is within 1e-3 of its plane.
__device__ __forceinline__ void margin_track(WaveArena &A, bool v0, double sd0, double sc0, bool v1, double sd1,
                                             double sc1) {
  const bool n0 = v0 && fabs(sd0) < 1e-3 * sc0, n1 = v1 && fabs(sd1) < 1e-3 * sc1;
  if (__ballot(n0 || n1)) {
    const int nlow = __popcll(__ballot(v0 && fabs(sd0) < 1e-12 * sc0)) + __popcll(__ballot(v1 && fabs(sd1) < 1e-12 * sc1));
    double r = n0 ? fabs(sd0) / sc0 : 1.0;
    if (n1) r = fmin(r, fabs(sd1) / sc1);
    r = wave_min(r);
    if (vd_lane() == 0) {
      A.lowmargin += nlow;
      if (r < A.minmargin) A.minmargin = r;
    }
  }
}
