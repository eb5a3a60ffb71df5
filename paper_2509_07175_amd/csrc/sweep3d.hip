// sweep3d.hip -- the default clip of a tetrahedral domain, one wavefront per
// site: the cell is cut from the padded box of the domain by the bisectors of
// the nearby sites in order of distance, and each piece is the cell cut by
// the four planes of a tetrahedron.
//
// The point-in-cell test (Sec. 4.1, Eq. 2) of all corners at once: lane l
// owns corner l, and one step tests every corner against one site (is the
// corner nearer to that site than to v_i?), so a site that fails no test is
// discarded for three FMAs and a ballot, and a site that some corner fails is
// a clip.  Sites come from the LDS copy of the neighbourhood in bucket order
// of distance; the sweep ends at the first site farther than twice the
// farthest corner, which no corner can be nearer to.  In distance order few
// clips are wasted: 16.6 cuts for the 15.5 faces of a uniform cell after 52
// sites, where the searched carve of clip3d.hip spends 13 rounds of queries to
// clip by the faces alone.  A corner whose ball may hold sites that are not in
// the copy is certified by grid queries, four at a time (ask_grid).
//
// The polytope stays in registers: a lane holds its corner's coordinates, its
// three planes and the corners across its three edges.  A cut removes the
// outside corners (the polytope is convex, so they are connected) and gives
// the new corners their free lanes, so survivors never move.  Planes and
// the tables that link the fan of a new face are in LDS.
//
// What bounds it: waits for LDS round trips (two fifths of a wave's time) and VALU
// issue (three fifths of the cycles), at four waves per SIMD (128 VGPRs).  1M clustered
// sites in 750,000 tetrahedra take 22 ms, 5M uniform sites 50 (searched carve: 64.7 and
// 168.6).  Figures for a choice, here and below, are of the two sides in one tree at the
// time: five waves at 96 VGPRs spill, 26.0 against 24.6 ms on the clustered sites and
// 58.8 against 57.7 on the uniform ones.  Reads that do not depend on each other are
// issued together: the planes of four sites before their tests, the planes of a new
// corner before the tables that link it, those of up to seven tetrahedra for one chain
// of mesh reads; and rows of LDS are 16-byte aligned (57.7 -> 53.5 ms uniform, 24.6 ->
// 23.3 clustered).  Two pieces at once, one in each half of the wave, or corners placed
// along the cut edge instead of solved for, gained nothing.
// All control flow is on scalar values (ballots, readlane): where the compiler
// cannot see that a value is uniform it is passed through readlane, or every
// branch behind it would save and restore the exec mask (36 -> 28 ms clustered).
//
// A cell that does not fit (more than 64 corners or 36 planes at a time), whose cut
// is degenerate or that has a corner which its planes hardly fix is put on a list that
// clip3d.hip's kernel works through afterwards; options other than the defaults of the
// search go there as a whole.
#include "vd_site.h"
#include "vd_sweep.h"

namespace {

constexpr int kPC = 36;      // plane slots of the cell (64 corners have at most 34 faces)
constexpr int kTB = 7;       // tetrahedra whose planes are computed at a time
constexpr int kP = kPC + 4 * kTB;  // ... and theirs: a plane to a lane
static_assert(kP == 64, "masks of planes");
constexpr int kT = 64;       // simplices of a site held in LDS
constexpr int kRounds = 3;   // rounds of grid queries for a cell before its pieces are certified instead

struct __align__(16) SweepLds {
  union {
    struct {
      double pn[kP][4];          // planes: outward normal (relative coordinates), offset
      int plab[kP];              // plane flag: sorted site >= 0, -(b+1), boundary / box code
      int clab[kP];              // the same with the caller's site index
      unsigned char first[kP], second[kP];  // the new corner whose first / second plane is this one
      unsigned char mark[kP];    // planes in use
    };
    struct {
      unsigned short row[kCand];         // the row that starts at a candidate
      int base[kRows];                   // sorted position minus candidate number
    } R;
    unsigned short pre[kBatch][kNB];     // entries of a bucket before a batch
  };
  unsigned rec[64];          // new corners: planes u, w and the surviving end of the cut edge
  int tq[kT];                // simplices of the site, breadth-first
  union alignas(16) {  // (whole sites and corners are read 16 bytes at a time)
    struct {
      double s[kK][4];       // sites relative to v_i, and the offset of their bisector
      int p[kK];             // sorted position
      unsigned char kb[kK];  // distance bucket (non-decreasing)
    } K;
    struct {
      unsigned long long bits[kBatch][kNB];  // the candidates of each bucket
    } B;
    struct {
      double y[64][4];       // corners of a piece
      unsigned tri[128];     // triangles of its faces: three corners
      int pfirst[kP];        // lowest corner of each plane
      int cp[64], nb[64];    // topology (face moments)
    } F;
  };
  double step, keep;         // bucket width (squared distance); radius within which every block site is held
  double blk[6];             // the block's sides relative to v_i (far away where the grid ends)
  double acc[5];             // per-site volume, first moment, energy
  WaveArena ar;
};

// ---------------------------------------------------------------------------
// The polytope: this lane's corner (coordinates relative to v_i, planes
// a | b << 8 | c << 16 counter-clockwise from outside, and 63 minus the lane of
// the corner across a->b | b->c << 8 | c->a << 16: a mask shifted left by that
// has the corner's bit as its sign) and the mask of the lanes that hold one.
// ---------------------------------------------------------------------------
struct Poly {
  double y0, y1, y2;
  int cp, nb;
  uint64_t M;
};

__device__ __forceinline__ uint64_t outside_of(const Poly &Q, const double *n, double c) {
  return lanes(n[0] * Q.y0 + n[1] * Q.y1 + n[2] * Q.y2 > c) & Q.M;
}
// the lane of the corner across edge e
__device__ __forceinline__ int across(const Poly &Q, int e) { return ~(Q.nb >> (8 * e)) & 63; }

// Vertex of the planes n0, n1 (offset last) and n.y = c, by Cramer's rule.
__device__ __forceinline__ void vertex_of(const double *n0, const double *n1, const double *n, double c, double &y0,
                                          double &y1, double &y2) {
  const double c12[3] = {n1[1] * n[2] - n1[2] * n[1], n1[2] * n[0] - n1[0] * n[2], n1[0] * n[1] - n1[1] * n[0]};
  const double c20[3] = {n[1] * n0[2] - n[2] * n0[1], n[2] * n0[0] - n[0] * n0[2], n[0] * n0[1] - n[1] * n0[0]};
  const double c01[3] = {n0[1] * n1[2] - n0[2] * n1[1], n0[2] * n1[0] - n0[0] * n1[2], n0[0] * n1[1] - n0[1] * n1[0]};
  const double det = n0[0] * c12[0] + n0[1] * c12[1] + n0[2] * c12[2];
  const double id = 1.0 / det;
  y0 = (n0[3] * c12[0] + n1[3] * c20[0] + c * c01[0]) * id;
  y1 = (n0[3] * c12[1] + n1[3] * c20[1] + c * c01[1]) * id;
  y2 = (n0[3] * c12[2] + n1[3] * c20[2] + c * c01[2]) * id;
}

// Cuts the polytope by plane slot P (n.y = c), whose outside corners are O (not
// empty, and not all).  One new corner on every edge that leaves O, in a free
// lane; a corner of the fan of the new face has planes u, w, P where u is its
// first and w its second plane, so its neighbours in the fan are the corners
// whose first plane is w and whose second is u.  Returns false, the polytope
// unchanged, when there are too few edges for a face or too many for the free
// lanes.  `bad` collects the lanes whose new corner is degenerate (the edges do
// not form one loop) or hardly fixed by its planes: on regular lattices of sites it
// can lie past the ends of its edge, out of order with the planes before, and clip3d.hip
// takes the site.  (Done here as well, the corner's place on the edge takes registers
// that every cut pays for: 2 % of the kernel, 6 with face moments.  Cuts of sites in
// general position have no such corner; cells of a cubic lattice with noise of 1e-9
// all have, and take 5.6 ms per 64,000 instead of 4.6 in that kernel alone.)
__device__ __forceinline__ bool cut(SweepLds &S, Poly &Q, uint64_t O, int P, const double *n, double c, uint64_t &bad) {
  const int l = vd_lane();
  auto beyond = [&](int e) { return lanes((int)((O << ((Q.nb >> (8 * e)) & 63)) >> 32) < 0); };
  const uint64_t x0 = beyond(0), x1 = beyond(1), x2 = beyond(2);  // the corner across edge e is outside
  const uint64_t b0 = O & ~x0, b1 = O & ~x1, b2 = O & ~x2;
  const int k0 = __popcll(b0), k1 = k0 + __popcll(b1), nnew = k1 + __popcll(b2);
  const uint64_t keep = Q.M & ~O, F = ~keep;
  if (nnew < 3 || __popcll(F) < nnew) return false;
  // planes u | w << 8 and the surviving corner << 16 of each cut edge
  if (in_mask(b0)) S.rec[mbcnt64(b0)] = __builtin_amdgcn_perm(Q.nb, Q.cp, 0x0c040100u);
  if (in_mask(b1)) S.rec[k0 + mbcnt64(b1)] = __builtin_amdgcn_perm(Q.nb, Q.cp, 0x0c050201u);
  if (in_mask(b2)) S.rec[k1 + mbcnt64(b2)] = __builtin_amdgcn_perm(Q.nb, Q.cp, 0x0c060002u);
  lds_order();
  const int rank = mbcnt64(F);
  const uint64_t N = lanes(rank < nnew) & F;
  const unsigned rec = S.rec[rank & 63];
  const int u = in_mask(N) ? rec & 255 : 0, w = in_mask(N) ? (rec >> 8) & 255 : 0;
  if (in_mask(N)) {
    S.first[u] = (unsigned char)(63 - l);
    S.second[w] = (unsigned char)(63 - l);
  }
  const double g0[4] = {S.pn[u][0], S.pn[u][1], S.pn[u][2], S.pn[u][3]};
  const double g1[4] = {S.pn[w][0], S.pn[w][1], S.pn[w][2], S.pn[w][3]};
  lds_order();
  // a surviving end: the edge's new corner has as first plane the edge's second plane seen from here
  const int f0 = S.first[p8(Q.cp, 1)], f1 = S.first[p8(Q.cp, 2)], f2 = S.first[p8(Q.cp, 0)];
  const int fw = S.first[w], su = S.second[u], fu = S.first[u], sw = S.second[w];
  int nb = Q.nb;
  nb = in_mask(keep & x0) ? (int)__builtin_amdgcn_perm(f0, nb, 0x03020104u) : nb;
  nb = in_mask(keep & x1) ? (int)__builtin_amdgcn_perm(f1, nb, 0x03020400u) : nb;
  nb = in_mask(keep & x2) ? (int)__builtin_amdgcn_perm(f2, nb, 0x03040100u) : nb;
  Q.nb = nb;
  const double c12[3] = {g1[1] * n[2] - g1[2] * n[1], g1[2] * n[0] - g1[0] * n[2], g1[0] * n[1] - g1[1] * n[0]};
  const double det = g0[0] * c12[0] + g0[1] * c12[1] + g0[2] * c12[2];
  const uint64_t fixed = lanes(fixed_to(kSure, det, g0, g1, n));
  bad |= N & ~fixed;
  if (in_mask(N)) {
    vertex_of(g0, g1, n, c, Q.y0, Q.y1, Q.y2);
  }
  bool wrong = false;
  if (in_mask(N)) {
    Q.nb = (int)(rec >> 16) | fw << 8 | su << 16;
    Q.cp = (int)(rec & 0xffff) | P << 16;
    // two corners with the same first (second) plane: not a simple loop
    wrong = (fu != 63 - l) | (sw != 63 - l);
  }
  bad |= lanes(wrong);
  Q.M = keep | N;
  return true;
}

// the planes of the polytope's corners
__device__ __forceinline__ uint64_t planes_in_use(SweepLds &S, const Poly &Q) {
  const int l = vd_lane();
  if (l < kP / 4) reinterpret_cast<int *>(S.mark)[l] = 0;
  lds_order();
  if (in_mask(Q.M)) {
    S.mark[p8(Q.cp, 0)] = 1;
    S.mark[p8(Q.cp, 1)] = 1;
    S.mark[p8(Q.cp, 2)] = 1;
  }
  lds_order();
  return lanes(S.mark[l] != 0);
}

// a free plane slot of the cell, or -1
__device__ __forceinline__ int take_plane(SweepLds &S, const Poly &Q, uint64_t &free_planes) {
  if (!free_planes) {
    free_planes = ~planes_in_use(S, Q) & ((1ull << kPC) - 1ull);
    if (!free_planes) return -1;
  }
  const int P = __ffsll((unsigned long long)free_planes) - 1;
  free_planes &= free_planes - 1;
  return P;
}

__device__ __forceinline__ void set_plane(SweepLds &S, int P, const double *n, double c, int lab) {
  if (vd_lane() == 0) {
    S.pn[P][0] = n[0]; S.pn[P][1] = n[1]; S.pn[P][2] = n[2]; S.pn[P][3] = c;
    S.plab[P] = lab;
  }
  lds_order();
}

constexpr int kBoxFlag = VD_BND_BASE + 16;  // flags of the box planes (never emitted)

// P <- box [lo, hi] (planes x-,x+,y-,y+,z-,z+; corner (bx,by,bz) = 4bx+2by+bz)
__device__ __forceinline__ void start_box(SweepLds &S, Poly &Q, const SiteCtx &X, const double *lo, const double *hi) {
  const int l = vd_lane();
  if (l < 6) {
    const int ax = l >> 1, side = l & 1;
    const double vc = ax == 0 ? X.vx : (ax == 1 ? X.vy : X.vz);
    const double lov = ax == 0 ? lo[0] : (ax == 1 ? lo[1] : lo[2]);
    const double hiv = ax == 0 ? hi[0] : (ax == 1 ? hi[1] : hi[2]);
    S.pn[l][0] = ax == 0 ? (side ? 1.0 : -1.0) : 0.0;
    S.pn[l][1] = ax == 1 ? (side ? 1.0 : -1.0) : 0.0;
    S.pn[l][2] = ax == 2 ? (side ? 1.0 : -1.0) : 0.0;
    S.pn[l][3] = side ? hiv - vc : vc - lov;
    S.plab[l] = kBoxFlag + l;
  }
  // planes / neighbours of corner l, 4 bits per entry (12 bits per corner)
  const unsigned long long CP = 0x240ull | 0x520ull << 12 | 0x430ull << 24 | 0x350ull << 36 | 0x421ull << 48;
  const unsigned long long CP2 = 0x251ull | 0x341ull << 12 | 0x531ull << 24;
  const unsigned long long CN = 0x142ull | 0x350ull << 12 | 0x063ull << 24 | 0x271ull << 36 | 0x605ull << 48;
  const unsigned long long CN2 = 0x417ull | 0x724ull << 12 | 0x536ull << 24;
  const int q = l & 7;
  const unsigned cp = q < 5 ? (unsigned)((CP >> (12 * q)) & 0xfff) : (unsigned)((CP2 >> (12 * (q - 5))) & 0xfff);
  const unsigned nb = q < 5 ? (unsigned)((CN >> (12 * q)) & 0xfff) : (unsigned)((CN2 >> (12 * (q - 5))) & 0xfff);
  Q.cp = pack3(cp & 15, (cp >> 4) & 15, (cp >> 8) & 15);
  Q.nb = pack3(63 - (nb & 15), 63 - ((nb >> 4) & 15), 63 - ((nb >> 8) & 15));
  Q.y0 = ((l >> 2) & 1 ? hi[0] : lo[0]) - X.vx;
  Q.y1 = ((l >> 1) & 1 ? hi[1] : lo[1]) - X.vy;
  Q.y2 = (l & 1 ? hi[2] : lo[2]) - X.vz;
  Q.M = 0xffull;
  lds_order();
}

// Is this lane's corner certified by the LDS copy alone: does the copy hold
// every site that could be nearer to it than v_i?  (Those lie in the ball of
// its distance d to v_i, so within |y| + d of v_i; h2: the squared lifted
// coordinate of a power site.)
__device__ __forceinline__ bool covered(const SweepLds &S, const Poly &Q, double h2) {
  const double s2 = Q.y0 * Q.y0 + Q.y1 * Q.y1 + Q.y2 * Q.y2;
  const double d = sqrt_bound(s2 + h2) * (1.0 + 1e-9), s = sqrt_bound(s2) * (1.0 + 1e-9);
  return (s + d < S.keep) & (d - Q.y0 < S.blk[0]) & (d + Q.y0 < S.blk[1]) & (d - Q.y1 < S.blk[2]) &
         (d + Q.y1 < S.blk[3]) & (d - Q.y2 < S.blk[4]) & (d + Q.y2 < S.blk[5]);
}

struct SweepStats {
  long long queries = 0, cands = 0, clips = 0, grid = 0;
};

// Cuts the box down to Omega_i (intersected with it).  Returns 0 done, 1 empty
// (a power cell), 2 too large, 3 degenerate.
template <bool POW>
__device__ __forceinline__ int sweep(SweepLds &S, const GridView &G, const SiteCtx &X, int held, Poly &Q,
                                     uint64_t &free_planes, SweepStats &st) {
  const int l = vd_lane();
  const double h2 = POW ? X.h * X.h : 0.0;
  uint64_t bad = 0;
  int k = 0, check = 0;
  for (;;) {
    // the next site that some corner is nearer to, four at a time: their planes
    // are read together, for one wait
    uint64_t any = 0;
    while (k < held) {
      if (k >= check) {
        check = k + 8;
        // no site beyond twice the farthest corner is nearer to any corner than v_i
        const double R2 = wave_bound(in_mask(Q.M) ? Q.y0 * Q.y0 + Q.y1 * Q.y1 + Q.y2 * Q.y2 : 0.0);
        double lim = 4.0 * R2;
        if (POW) {
          const double reach = sqrt_bound(R2) + sqrt_bound(R2 + h2);
          lim = reach * reach;
        }
        if (uni((double)S.K.kb[k] * S.step > lim * (1.0 + 1e-6))) break;
      }
      if (k + 4 <= held) {
        double g[4][4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const double2 *e = reinterpret_cast<const double2 *>(S.K.s[k + j]);
          const double2 e0 = e[0], e1 = e[1];
          g[j][0] = e0.x; g[j][1] = e0.y; g[j][2] = e1.x; g[j][3] = e1.y;
        }
        __builtin_amdgcn_sched_barrier(0);
        const uint64_t o0 = outside_of(Q, g[0], g[0][3]), o1 = outside_of(Q, g[1], g[1][3]),
                       o2 = outside_of(Q, g[2], g[2][3]), o3 = outside_of(Q, g[3], g[3][3]);
        any = o0 | o1 | o2 | o3;
        if (any) {
          k += o0 ? 0 : (o1 ? 1 : (o2 ? 2 : 3));
          break;
        }
        k += 4;
      } else {
        any = outside_of(Q, S.K.s[k], S.K.s[k][3]);
        if (any) break;
        k++;
      }
    }
    if (!any) break;
    const double n[3] = {S.K.s[k][0], S.K.s[k][1], S.K.s[k][2]}, c = S.K.s[k][3];
    const uint64_t O = outside_of(Q, n, c);
    if (O == Q.M) return 1;
    const int P = take_plane(S, Q, free_planes);
    if (P < 0) return 2;
    set_plane(S, P, n, c, S.K.p[k]);
    if (!cut(S, Q, O, P, n, c, bad)) return 2;
    if (bad) return 3;
    st.clips++;
    k++;
  }
  st.cands += k;
  st.queries += __popcll(Q.M);
  return 0;
}

// Asks the grid for the nearest sites of four corners of Q among `ask` (the
// farthest ones: their clips remove most) and clips the cell by every site
// found that is nearer than v_i.  `ask` loses the corners found inside
// Omega_i; `kept` loses the cell's corners that were removed.  Returns 0, 1
// when nothing of the cell is left (a power cell), 2 too large, 3 degenerate.
template <bool POW>
__device__ __forceinline__ int ask_grid(SweepLds &S, const GridView &G, const SiteCtx &X, const Poly &Q, uint64_t &ask,
                                        Poly &cell, uint64_t &free_planes, uint64_t &kept, uint64_t &cellpos, SweepStats &st) {
  const int l = vd_lane(), grp = l >> 4;
  const double h2 = POW ? X.h * X.h : 0.0;
  int slot = -1;
  {
    int f = in_mask(ask) ? __double2hiint(Q.y0 * Q.y0 + Q.y1 * Q.y1 + Q.y2 * Q.y2) : -1;
#pragma unroll 1
    for (int g = 0; g < 4; g++) {
      const int top = wave_imax(f);
      if (top < 0) break;
      const uint64_t at = lanes(f == top);
      const int s = __ffsll((unsigned long long)at) - 1;
      slot = grp == g ? s : slot;
      f = l == s ? -1 : f;
    }
  }
  const int src = slot >= 0 ? slot : __ffsll((unsigned long long)ask) - 1;
  const double q0 = __shfl(Q.y0, src, 64), q1 = __shfl(Q.y1, src, 64), q2 = __shfl(Q.y2, src, 64);
  const int cp = __shfl(Q.cp, src, 64);
  const double qx = X.vx + q0, qy = X.vy + q1, qz = X.vz + q2;
  const double dx = qx - X.vx, dy = qy - X.vy, dz = qz - X.vz;
  const int kq = nn_query<POW>(G, 16, qx, qy, qz, dx * dx + dy * dy + dz * dz + h2, X.si, st.cands, 0.0);
  const bool lead = slot >= 0 && (l & 15) == 0;
  const bool in = (kq == X.si) | (kq == S.plab[p8(cp, 0)]) | (kq == S.plab[p8(cp, 1)]) | (kq == S.plab[p8(cp, 2)]);
  const uint64_t asked = lanes(lead);
  st.queries += __popcll(asked);
  st.grid += __popcll(asked);
  const uint64_t inside = lanes(in);
  uint64_t fresh = 0;  // planes of this round
  for (uint64_t m = asked; m; m = uni64(m & (m - 1))) {
    cell.M = uni64(cell.M);
    free_planes = uni64(free_planes);
    ask = uni64(ask);
    kept = uni64(kept);
    cellpos = uni64(cellpos);
    const int g = __ffsll((unsigned long long)m) - 1;
    const int j = __builtin_amdgcn_readlane(kq, g);
    const uint64_t at = 1ull << __builtin_amdgcn_readlane(slot, g);
    if ((inside >> g) & 1ull) { ask &= ~at; continue; }
    const double n[3] = {GL(G.sx)[j] - X.vx, GL(G.sy)[j] - X.vy, GL(G.sz)[j] - X.vz};
    const double nn = n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
    const double c = POW ? 0.5 * (nn + X.w - GL(G.sw)[j]) : 0.5 * nn;
    // a site that has clipped already is nearer by rounding only, and the corner
    // is inside (cells are closed); or the site clipped for another corner of
    // this round, and this one is gone as well or asked again
    const uint64_t has = lanes(l < kPC && S.plab[l < kPC ? l : 0] == j) & ~free_planes;
    if (has) {
      if ((has & ~fresh) && (outside_of(Q, n, c + 1e-9 * nn) & at)) return 3;
      ask &= ~at;
      continue;
    }
    const uint64_t O = outside_of(cell, n, c);
    if (!O) { ask &= ~at; continue; }
    if (O == cell.M) return 1;
    const int P = take_plane(S, cell, free_planes);
    if (P < 0) return 2;
    set_plane(S, P, n, c, j);
    S.clab[P] = GL(G.perm)[j];
    cellpos |= 1ull << P;
    fresh |= 1ull << P;
    uint64_t bad = 0;
    if (!cut(S, cell, O, P, n, c, bad)) return 2;
    if (bad) return 3;
    st.clips++;
    kept &= ~O;
  }
  return 0;
}

// planes_in_use for a piece, and the lowest corner of each plane to F.pfirst
__device__ __forceinline__ uint64_t faces_of(SweepLds &S, const Poly &Q) {
  const int l = vd_lane();
  S.F.pfirst[l] = 64;
  lds_order();
  if (in_mask(Q.M)) {
    atomicMin(&S.F.pfirst[p8(Q.cp, 0)], l);
    atomicMin(&S.F.pfirst[p8(Q.cp, 1)], l);
    atomicMin(&S.F.pfirst[p8(Q.cp, 2)], l);
  }
  lds_order();
  return lanes(S.F.pfirst[l] < 64);
}

// Lists the triangles (lowest corner, corner, next corner) of the faces that do
// not hold corner `apex` (LOW: it is the lowest one); returns their number (124 at
// most).
template <bool LOW>
__device__ __forceinline__ int list_triangles(SweepLds &S, const Poly &Q, int apex) {
  const int l = vd_lane(), at = __builtin_amdgcn_readlane(Q.cp, apex);
  int T = 0;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    // plane e of the corner continues around its face to the corner across edge e + 2
    const int p = p8(Q.cp, e), nx = across(Q, e == 0 ? 2 : e - 1), s = S.F.pfirst[p];
    const bool apart = LOW ? s != apex : (p != p8(at, 0)) & (p != p8(at, 1)) & (p != p8(at, 2));
    const uint64_t act = lanes(apart & (s != l) & (s != nx)) & Q.M;
    if (in_mask(act)) S.F.tri[T + mbcnt64(act)] = (unsigned)(s | l << 8 | nx << 16);
    T += __popcll(act);
  }
  lds_order();
  return T;
}

// Sums over the wave by the matrix cores: a product with ones adds the four
// lanes 16 apart, a second one the four of a quad.  The four blocks of lanes
// that are left (bits 2 and 3) are added for four sums at once, sum r in the
// lanes of r = l & 3: 8 MFMA and 12 VALU instructions where the butterfly of
// four sums takes 92.
__device__ __forceinline__ double block_sum(double v) {
  const double rows = __builtin_amdgcn_mfma_f64_4x4x4f64(v, 1.0, 0.0, 0, 0, 0);
  return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, rows, 0.0, 0, 0, 0);
}
__device__ __forceinline__ double blocks_sum(double v) {
  v += perm_d<0x128>(v);  // row_ror:8
  v += perm_d<0x124>(v);  // row_ror:4
  return v;
}
__device__ __forceinline__ void wave_sum4(double &a, double &b, double &c, double &d) {
  const int r = vd_lane() & 3;
  const double A = block_sum(a), B = block_sum(b), C = block_sum(c), E = block_sum(d);
  const double t = blocks_sum(r == 0 ? A : r == 1 ? B : r == 2 ? C : E);
  a = readlane_d(t, 0); b = readlane_d(t, 1); c = readlane_d(t, 2); d = readlane_d(t, 3);
}

// Face moments of the bisector faces of the piece, for the adjoint: for face x
// on B_ik, I0 = int y dA/d, I1 = int y y^T dA/d, I2 = int |y|^2 y dA/d with
// y = x - v_i and d = |v_k - v_i|.  Lane x walks around face x from its lowest
// corner (a fixed order, so the sums are reproducible) and integrates the fan
// of triangles (foot of the plane, corner, next corner): linear and quadratic
// terms in closed form, the cubic term with the degree-3 rule of Strang and Fix
// (centroid -27/48, points (3/5,1/5,1/5) 25/48); with a density every integrand
// carries it and one degree-5 rule takes all twelve.
template <bool DENS>
__device__ __forceinline__ void face_moments(SweepLds &S, const Poly &Q, const CellsDev &C,
                                             const SiteCtx &X, long long pidx, uint64_t pos, long long base) {
  const int l = vd_lane();
  if (in_mask(Q.M)) {
    S.F.cp[l] = Q.cp;
    S.F.nb[l] = Q.nb;
    S.F.y[l][0] = Q.y0; S.F.y[l][1] = Q.y1; S.F.y[l][2] = Q.y2;
  }
  lds_order();
  const bool mine = in_mask(pos);
  const int npos = __popcll(pos);
  const bool fits = base + npos <= C.cap_fint;
  if (l == 0 && pidx < C.cap_piece) {
    GL(C.piece_fint_start)[pidx] = base;
    GL(C.piece_nfint)[pidx] = fits ? npos : 0;
    if (!fits) S.ar.dropped++;
  }
  if (mine) {
    const int x = l;
    const double n0 = S.pn[x][0], n1 = S.pn[x][1], n2 = S.pn[x][2], cc = S.pn[x][3];
    const double nn = n0 * n0 + n1 * n1 + n2 * n2;
    const double d = sqrt(nn), f = cc / nn;
    const double h0 = n0 / d, h1 = n1 / d, h2 = n2 / d;
    const double r0 = n0 * f, r1 = n1 * f, r2 = n2 * f;
    double I[12];
#pragma unroll
    for (int k = 0; k < 12; k++) I[k] = 0.0;
    const int start = S.F.pfirst[x];
    int T = start;
    double a0 = S.F.y[T][0], a1 = S.F.y[T][1], a2 = S.F.y[T][2];
#pragma unroll 1
    for (int s = 0; s < 64; s++) {
      const int pl = S.F.cp[T];
      const int e = p8(pl, 0) == x ? 0 : (p8(pl, 1) == x ? 1 : 2);
      const int nx = ~p8(S.F.nb[T], e == 0 ? 2 : e - 1) & 63;
      const double b0 = S.F.y[nx][0], b1 = S.F.y[nx][1], b2 = S.F.y[nx][2];
      const double u0 = a0 - r0, u1 = a1 - r1, u2 = a2 - r2, w0 = b0 - r0, w1 = b1 - r1, w2 = b2 - r2;
      const double A = 0.5 * ((u1 * w2 - u2 * w1) * h0 + (u2 * w0 - u0 * w2) * h1 + (u0 * w1 - u1 * w0) * h2);
      if (DENS) {
        // weighted by the density: one degree-5 rule for all twelve integrals
        const double P0[3] = {r0, r1, r2}, P1[3] = {a0, a1, a2}, P2[3] = {b0, b1, b2};
        tri_density_face(C.dens, X.vx, X.vy, X.vz, P0, P1, P2, A, I);
      } else {
        const double s0 = r0 + a0 + b0, s1 = r1 + a1 + b1, s2 = r2 + a2 + b2;
        I[0] += A * s0 / 3.0; I[1] += A * s1 / 3.0; I[2] += A * s2 / 3.0;
        const double q = A / 12.0;
        I[3] += q * (r0 * r0 + a0 * a0 + b0 * b0 + s0 * s0);
        I[4] += q * (r0 * r1 + a0 * a1 + b0 * b1 + s0 * s1);
        I[5] += q * (r0 * r2 + a0 * a2 + b0 * b2 + s0 * s2);
        I[6] += q * (r1 * r1 + a1 * a1 + b1 * b1 + s1 * s1);
        I[7] += q * (r1 * r2 + a1 * a2 + b1 * b2 + s1 * s2);
        I[8] += q * (r2 * r2 + a2 * a2 + b2 * b2 + s2 * s2);
        // cubic |y|^2 y: degree-3 rule on (r, a, b)
        const double c0 = s0 / 3.0, c1 = s1 / 3.0, c2 = s2 / 3.0;
        const double t0 = -27.0 / 48.0 * (c0 * c0 + c1 * c1 + c2 * c2);
        double acc0 = t0 * c0, acc1 = t0 * c1, acc2 = t0 * c2;
#pragma unroll
        for (int v = 0; v < 3; v++) {
          // point 3/5 at vertex v, 1/5 at the other two
          const double p0 = 0.2 * s0 + 0.4 * (v == 0 ? r0 : (v == 1 ? a0 : b0));
          const double p1 = 0.2 * s1 + 0.4 * (v == 0 ? r1 : (v == 1 ? a1 : b1));
          const double p2 = 0.2 * s2 + 0.4 * (v == 0 ? r2 : (v == 1 ? a2 : b2));
          const double w = 25.0 / 48.0 * (p0 * p0 + p1 * p1 + p2 * p2);
          acc0 += w * p0; acc1 += w * p1; acc2 += w * p2;
        }
        I[9] += A * acc0; I[10] += A * acc1; I[11] += A * acc2;
      }
      a0 = b0; a1 = b1; a2 = b2;
      T = nx;
      if (T == start) break;
    }
    const long long r = base + __popcll(pos & low_mask_lt(l));
    if (r < C.cap_fint) {
      const double id = 1.0 / d;
#pragma unroll
      for (int k = 0; k < 12; k++) GL(C.fint)[12 * r + k] = I[k] * id;
      GL(C.fint_lab)[r] = S.clab[x];
    }
  }
  lds_order();
}

// ---------------------------------------------------------------------------
// One site.  The simplices of the cell are visited breadth-first through
// negative face flags from the tetrahedron that holds v_i (and, with boundary
// seeds, those behind the boundary triangles its cell meets): Alg. 5.
// Returns false when the site has to go to the general kernel (pcount is
// negative if some of its pieces have been written).
// ---------------------------------------------------------------------------
template <bool DENS, bool POW, bool CORNERS, bool LOOSE, bool GRAD>
__device__ __forceinline__ bool do_cell(SweepLds &S, const GridView &G, const DomainView &D, const CellsDev &C, int si) {
  const int l = vd_lane();
  SiteCtx X;
  // (through readlane: uniform values belong in scalar registers)
  X.vx = readlane_d(GL(G.sx)[si], 0); X.vy = readlane_d(GL(G.sy)[si], 0); X.vz = readlane_d(GL(G.sz)[si], 0);
  X.h = POW ? readlane_d(GL(G.sh)[si], 0) : 0.0;
  X.w = POW ? readlane_d(GL(G.sw)[si], 0) : 0.0;
  X.si = si;
  const int orig = uni(GL(G.perm)[si]);
  const long long spill = (long long)blockIdx.x * (C.q_spill + VD_Q_MAX);
  SweepStats st;
  int err = 0, where = 0;  // 2 capacity, 4 outside M without boundary seeds; failing stage (VD_STAGE_*)
  int nt = 0, head = 0, npieces = 0;
  long long nbseed = 0;  // boundary triangles the cell meets (when computed)
  const int held = uni(fill_sites<POW>(S, G, X.vx, X.vy, X.vz, X.w, 0.0));
  if (l < 5) S.acc[l] = 0.0;

  // simplices b0 (lane l: the l-th of `m` new ones, all distinct) join the queue unless listed
  auto push = [&](int b) {
    bool have = false;
    const int nl = nt < kT ? nt : kT;
    if (l < nl) have = S.tq[l] == b;
    for (int e = kT + l; e < nt; e += 64) have = have || GL(C.tq_spill)[spill + e - kT] == b;
    if (lanes(have)) return true;
    if (nt >= VD_Q_MAX + C.q_spill) return false;
    if (l == 0) {
      if (nt < kT) S.tq[nt] = b;
      else GL(C.tq_spill)[spill + nt - kT] = b;
    }
    if (nt >= kT) __threadfence_block();  // read back by the other lanes
    nt++;
    lds_order();
    return true;
  };
  {
    const int seed = GL(C.seed)[si];
    if (seed >= 0 && seed < D.m) push(seed);
    if (C.bseed_off) {
      const long long q0 = GL(C.bseed_off)[orig], q1 = GL(C.bseed_off)[orig + 1];
      nbseed = q1 - q0;
      for (long long q = q0; q < q1; q++)
        if (!push(GL(C.btet)[GL(C.bseed_tri)[GL(C.bseed_pid)[q]]])) { err = 2; where = VD_STAGE_SIMPLICES; break; }
    } else if (!nt && !POW) {
      err = 4;
    }
  }
  uint64_t nbmask = 0, cellpos = 0;
  // face moments (want_grad): the faces of a cell inside M are taken whole, once,
  // so a piece's wait until a piece has met the boundary (touched); lane k keeps
  // the slot and the tetrahedron of the k-th piece that waits
  int nwait = 0, wait_a = 0, nlate = 0;
  int pl0 = 0, pl1 = 0;  // the queue entries whose planes are in LDS
  long long wait_p = 0;
  bool touched = false;
  unsigned sum_faces = 0, sum_verts = 0, dropped = 0;
  Poly cell;
  bool whole = false, loose = false;  // loose: some corners of the cell are not certified
  uint64_t free_planes = 0;
  if ((nt || POW) && !err) {
    free_planes = ((1ull << kPC) - 1ull) & ~63ull;
    start_box(S, cell, X, D.box_lo, D.box_hi);
    int rc = sweep<POW>(S, G, X, held, cell, free_planes, st);
    if (!rc) {
      const uint64_t used = planes_in_use(S, cell);
      int lab = -1;
      if (in_mask(used)) {
        lab = S.plab[l];
        S.clab[l] = convert_label(G, lab);
      }
      cellpos = lanes(in_mask(used) && lab >= 0);
      // corners that the copy does not certify: their nearest site from the
      // grid.  Most cells need a round or two.  A cell that needs more often
      // reaches far out of M (around a re-entrant edge), where its shape does
      // not matter: its pieces are certified instead, corner by corner.  (The
      // seed of a power cell and the interior tests need the whole cell.)
      uint64_t kept = 0;
#pragma unroll 1
      for (int it = 0;; it++) {
        cell.M = uni64(cell.M);
        kept = uni64(kept);
        uint64_t ask = (held < 0 ? ~0ull : lanes(!covered(S, cell, POW ? X.h * X.h : 0.0))) & cell.M & ~kept;
        if (!ask) break;
        if (it >= (LOOSE && !C.whole ? kRounds : 1024)) {
          if (!LOOSE || C.whole) rc = 3;
          loose = true;
          break;
        }
        const uint64_t before = ask;
        uint64_t same = ~0ull;
        rc = uni(ask_grid<POW>(S, G, X, cell, ask, cell, free_planes, same, cellpos, st));
        if (rc) break;
        kept = (kept | (before & ~ask)) & same;
      }
    }
    if (POW && rc == 1) {
      head = nt;  // an empty power cell
    } else if (rc) {
      if (l == 0) GL(C.pcount)[orig] = 0;
      return false;
    } else {
      double c0 = 0, c1 = 0, c2 = 0;
      if (POW) {
        // the mean of the corners, a point of the cell
        const bool live = in_mask(cell.M);
        const double in = 1.0 / __popcll(cell.M);
        c0 = wave_sum(live ? cell.y0 : 0.0) * in;
        c1 = wave_sum(live ? cell.y1 : 0.0) * in;
        c2 = wave_sum(live ? cell.y2 : 0.0) * in;
      }
      // Alg. 5's interior sites: a cell that meets no boundary triangle lies
      // inside M or outside it as a whole; of a convex M that holds every site,
      // a cell whose corners all lie in M.  Such a cell is one piece.
      if (C.whole && nbseed == 0 &&
          (!CORNERS || !lanes(in_mask(cell.M) && !in_domain(D, X.vx + cell.y0, X.vy + cell.y1, X.vz + cell.y2)))) {
        whole = !POW || locate_wave(D, X.vx + c0, X.vy + c1, X.vz + c2) >= 0;
        head = nt;
      } else if (POW) {
        const int t = locate_wave(D, X.vx + c0, X.vy + c1, X.vz + c2);
        if (t >= 0 && !push(t)) { err = 2; where = VD_STAGE_SIMPLICES; }
      }
    }
  } else {
    head = nt;
  }
#pragma unroll 1
  while (uni((whole || head < nt || (GRAD && nlate < nwait)) && !err)) {
    int a = -1;
    cell.M = uni64(cell.M);
    free_planes = uni64(free_planes);
    cellpos = uni64(cellpos);
    nbmask = uni64(nbmask);
    nt = uni(nt);
    head = uni(head);
    npieces = uni(npieces);
    pl0 = uni(pl0);
    pl1 = uni(pl1);
    sum_faces = uni(sum_faces);
    sum_verts = uni(sum_verts);
    dropped = uni(dropped);
    whole = uni(whole);
    if (LOOSE) loose = uni(loose);
    if (GRAD) {
      nwait = uni(nwait);
      nlate = uni(nlate);
      touched = uni(touched);
    }
    const bool late = GRAD && uni(!whole && head >= nt);  // the face moments of what waits
    long long pidx = -1, fb = 0;
    Poly Q = cell;
    if (late) {
      pidx = readlane_ll(wait_p, nlate);
      a = touched ? __builtin_amdgcn_readlane(wait_a, nlate) : -1;
      nlate = touched ? nlate + 1 : nwait;
    } else if (!whole) {
      a = head < kT ? S.tq[head] : GL(C.tq_spill)[spill + head - kT];
      a = uni(a);
      head++;
    }
    int P = kPC;  // the tetrahedron's planes
    if (a >= 0) {
      // planes of the tetrahedra from `head` on in the queue, for one chain of
      // reads (mesh, vertices) instead of one for each
      if (late || head > pl1) {
        pl0 = head - 1;
        pl1 = late ? head : min(nt, pl0 + kTB);
        const int e = pl0 + (l >> 2);
        if (l < (late ? 4 : 4 * (pl1 - pl0))) {
          const int b = late ? a : (e < kT ? S.tq[e] : GL(C.tq_spill)[spill + e - kT]);
          double pl[4];
          int lab;
          tet_plane(D, X, b, l & 3, pl, lab);
          S.pn[kPC + l][0] = pl[0]; S.pn[kPC + l][1] = pl[1]; S.pn[kPC + l][2] = pl[2]; S.pn[kPC + l][3] = pl[3];
          S.plab[kPC + l] = lab;
          S.clab[kPC + l] = lab;
        }
        lds_order();
      }
      P = kPC + (late ? 0 : 4 * (head - 1 - pl0));
      uint64_t bad = 0;
      bool empty = false;
      // (a plane that no corner of the cell is behind cuts nothing of it later)
      unsigned todo = 0;
      {
        double g[4][4];
#pragma unroll
        for (int f = 0; f < 4; f++) {
          const double2 *e = reinterpret_cast<const double2 *>(S.pn[P + f]);
          const double2 e0 = e[0], e1 = e[1];
          g[f][0] = e0.x; g[f][1] = e0.y; g[f][2] = e1.x; g[f][3] = e1.y;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < 4; f++) {
          const uint64_t O = outside_of(Q, g[f], g[f][3]);
          todo |= O ? 1u << f : 0u;
          empty = empty | (O == Q.M);
        }
      }
      if (empty) continue;
#pragma unroll 1
      for (; todo; todo &= todo - 1) {
        const int f = P + __ffs(todo) - 1;
        const double n[3] = {S.pn[f][0], S.pn[f][1], S.pn[f][2]}, c = S.pn[f][3];
        const uint64_t O = outside_of(Q, n, c);
        if (!O) continue;
        if (O == Q.M) { empty = true; break; }
        if (!cut(S, Q, O, f, n, c, bad)) { bad = 1; break; }
        st.clips += late ? 0 : 1;
      }
      if (bad) { err = 9; break; }
      if (empty) continue;
      if (LOOSE && loose) {
        // certify the piece; a clip of the cell starts the piece again
        uint64_t ask = (held < 0 ? ~0ull : lanes(!covered(S, Q, 0.0))) & Q.M, all = ~0ull;
        int rc = 0;
#pragma unroll 1
        while (ask && !rc && !~all) rc = uni(ask_grid<POW>(S, G, X, Q, ask, cell, free_planes, all, cellpos, st));
        if (rc) { err = 9; break; }
        if (~all) { head--; continue; }
      }
    }
    // ---- moments of the piece: tetrahedra of a corner o and the triangles of
    // the faces that do not hold it (about 40, one to a lane), in coordinates
    // relative to o, so that the rounding error scales with the piece and not
    // with its distance to v_i.  Only the volume's, that is: first moments and energy
    // are summed about v_i, or with a density about o and moved there by terms that
    // cancel where |o| is large, so o is the corner nearest to v_i then (errors of the
    // energy of uniform cells' pieces 3.7e-16 on average, with a density 3.2e-16 and
    // 6.6e-16 from any corner).  With a density, four Lloyd steps of 60,000
    // sites: 15.1 ms with 15 points in three tetrahedra per corner (the planes'
    // feet and three edges, 26 lanes at work), 8.7 ms here; without one the
    // chain of LDS round trips is what it costs either way (25.7 against 26.3 ms
    // on the 1M clustered workload) ----
    const uint64_t fmask = faces_of(S, Q);
    uint64_t bis = GRAD ? fmask & cellpos : 0ull;  // its bisector faces
    const bool live = in_mask(Q.M);
    double pv = 0, pmx = 0, pmy = 0, pmz = 0, pe = 0;
    const int nc = __popcll(Q.M), nface = __popcll(fmask);
    long long fo = 0, vo = 0;
    bool now = late;  // its face moments
    if (late) {
      fb = arena_take(S.ar, C, AR_FINT, __popcll(bis));
    } else {
      int apex = __ffsll((unsigned long long)Q.M) - 1;
      if (DENS) {
        const int far = live ? __double2hiint(Q.y0 * Q.y0 + Q.y1 * Q.y1 + Q.y2 * Q.y2) : 0x7fffffff;
        apex = __ffsll((unsigned long long)lanes(far == -wave_imax(-far))) - 1;
      }
      const double o0 = readlane_d(Q.y0, apex), o1 = readlane_d(Q.y1, apex), o2 = readlane_d(Q.y2, apex);
      if (live) {
        S.F.y[l][0] = DENS ? Q.y0 - o0 : Q.y0;
        S.F.y[l][1] = DENS ? Q.y1 - o1 : Q.y1;
        S.F.y[l][2] = DENS ? Q.y2 - o2 : Q.y2;
      }
      const int T = list_triangles<!DENS>(S, Q, apex);
      const double oo = o0 * o0 + o1 * o1 + o2 * o2;
      double dm = 0;  // (DENS: the moments are weighted, pv is the volume)
      ConeDensity cd;
      if (DENS) cd = cone_density(C.dens, X.vx + o0, X.vy + o1, X.vz + o2);
#pragma unroll 1
      for (int t0 = 0; t0 < T; t0 += 64) {
        if (t0 + l < T) {
          const unsigned tri = S.F.tri[t0 + l];
          const double *P = S.F.y[tri & 255], *Y = S.F.y[(tri >> 8) & 255], *Z = S.F.y[tri >> 16];
          const double P0 = P[0], P1 = P[1], P2 = P[2], Y0 = Y[0], Y1 = Y[1], Y2 = Y[2], Z0 = Z[0], Z1 = Z[1], Z2 = Z[2];
          const double p[3] = {DENS ? P0 : P0 - o0, DENS ? P1 : P1 - o1, DENS ? P2 : P2 - o2};
          const double y[3] = {DENS ? Y0 : Y0 - o0, DENS ? Y1 : Y1 - o1, DENS ? Y2 : Y2 - o2};
          const double z[3] = {DENS ? Z0 : Z0 - o0, DENS ? Z1 : Z1 - o1, DENS ? Z2 : Z2 - o2};
          // 6 vol of (0, p, y, z)
          const double det = p[0] * (y[1] * z[2] - y[2] * z[1]) - p[1] * (y[0] * z[2] - y[2] * z[0]) +
                             p[2] * (y[0] * z[1] - y[1] * z[0]);
          pv += det;
          if (DENS) {
            cone_density_moments(cd, p, y, z, det, dm, pmx, pmy, pmz, pe);
          } else {
            const double s0 = o0 + P0 + Y0 + Z0, s1 = o1 + P1 + Y1 + Z1, s2 = o2 + P2 + Y2 + Z2;
            pmx += det * s0; pmy += det * s1; pmz += det * s2;
            pe += det * (oo + P0 * P0 + P1 * P1 + P2 * P2 + Y0 * Y0 + Y1 * Y1 + Y2 * Y2 + Z0 * Z0 + Z1 * Z1 + Z2 * Z2 +
                         s0 * s0 + s1 * s1 + s2 * s2);
          }
        }
      }
      if (DENS) {
        pv = readlane_d(blocks_sum(block_sum(pv)), 0);
      } else {
        dm = pv;
      }
      wave_sum4(dm, pmx, pmy, pmz);
      pe = readlane_d(blocks_sum(block_sum(pe)), 0);
      if (!DENS) pv = dm;
      // a piece exists when its volume is positive; with a density its moments
      // are the weighted ones
      if (!(pv > 0.0)) {
        if (whole) break;
        continue;
      }
      pv = dm * (1.0 / 6.0);
      pmx *= DENS ? 1.0 / 6.0 : 1.0 / 24.0; pmy *= DENS ? 1.0 / 6.0 : 1.0 / 24.0; pmz *= DENS ? 1.0 / 6.0 : 1.0 / 24.0;
      pe *= DENS ? 1.0 / 6.0 : 1.0 / 120.0;
      if (DENS) {  // from o to v_i
        pe += 2.0 * (o0 * pmx + o1 * pmy + o2 * pmz) + oo * pv;
        pmx += o0 * pv; pmy += o1 * pv; pmz += o2 * pv;
      }
      if (l == 0) { S.acc[0] += pv; S.acc[1] += pmx; S.acc[2] += pmy; S.acc[3] += pmz; S.acc[4] += pe; }
      // ---- emit the piece ----
      if (GRAD) {
        touched = touched | (LOOSE && loose) | (nwait == 64) |
                  (lanes((l >= kPC) & (S.plab[l] <= VD_BND_BASE + 3)) & fmask) != 0;
        now = whole || touched;
      }
      if (!now) bis = 0;
      const long long at = arena_take_all(S.ar, C, arena_counts(1, C.emit ? nface : 0, C.emit ? nc : 0, __popcll(bis)));
      pidx = readlane_ll(at, AR_PIECE);
      fb = readlane_ll(at, AR_FINT);
      fo = readlane_ll(at, AR_FACE);
      vo = readlane_ll(at, AR_VERT);
      if (GRAD && !now) {
        if (l == nwait) {
          wait_a = a;
          wait_p = pidx;
        }
        nwait++;
        if (l == 0 && pidx < C.cap_piece) {
          GL(C.piece_fint_start)[pidx] = 0;
          GL(C.piece_nfint)[pidx] = 0;
        }
      }
    }
    if (GRAD && now) face_moments<DENS>(S, Q, C, X, pidx, bis, fb);
    if (late) continue;
    // a record that does not fit its arena is dropped and counted; the per-site
    // counts below only count what was written, so the CSR built from them
    // stays inside the arenas (the clip then reports VD_ERR_CAPACITY)
    const bool fits_fv = C.emit && fo + nface <= C.cap_face && vo + nc <= C.cap_vert;
    if (pidx < C.cap_piece) {
      if (l == 0) {
        GL(C.piece_site)[pidx] = orig;
        GL(C.piece_simplex)[pidx] = a;
        GL(C.piece_nface)[pidx] = nface;
        GL(C.piece_nvert)[pidx] = nc;
        GL(C.piece_mass)[pidx] = pv;
        GL(C.piece_mom)[3 * pidx + 0] = pmx + pv * X.vx;
        GL(C.piece_mom)[3 * pidx + 1] = pmy + pv * X.vy;
        GL(C.piece_mom)[3 * pidx + 2] = pmz + pv * X.vz;
        GL(C.piece_energy)[pidx] = pe;
        GL(C.piece_fstart)[pidx] = fits_fv ? fo : -1;
        GL(C.piece_vstart)[pidx] = fits_fv ? vo : -1;
      }
      npieces++;
      if (fits_fv) {
        sum_faces += nface;
        sum_verts += nc;
        if (in_mask(fmask)) GL(C.face_label)[fo + mbcnt64(fmask)] = S.clab[l];
        if (live) {
          const long long v = vo + mbcnt64(Q.M);
          GL(C.vert_xyz)[3 * v + 0] = Q.y0 + X.vx;
          GL(C.vert_xyz)[3 * v + 1] = Q.y1 + X.vy;
          GL(C.vert_xyz)[3 * v + 2] = Q.y2 + X.vz;
          GL(C.vert_label)[3 * v + 0] = S.clab[p8(Q.cp, 0)];
          GL(C.vert_label)[3 * v + 1] = S.clab[p8(Q.cp, 1)];
          GL(C.vert_label)[3 * v + 2] = S.clab[p8(Q.cp, 2)];
        }
      } else if (C.emit) {
        dropped++;
      }
    } else {
      dropped++;
    }
    // ---- propagate: neighbours (cell planes), tetrahedra (the planes of T_a) ----
    nbmask |= fmask & cellpos;
    if (whole) break;
    for (uint64_t m = fmask >> kPC << kPC; m; m &= m - 1) {
      const int lab = uni(S.plab[__ffsll((unsigned long long)m) - 1]);
      if (lab > VD_BND_BASE + 3 && !push(-lab - 1)) { err = 2; where = VD_STAGE_SIMPLICES; break; }
    }
    lds_order();
  }
  err = uni(err);
  nbmask = uni64(nbmask);
  if (err == 9) {
    // its pieces so far become unused slots (void_pieces, before the general
    // kernel takes the site)
    if (l == 0) GL(C.pcount)[orig] = -1;
    return false;
  }
  // ---- per-site results ----
  const int nnb = __popcll(nbmask);
  const long long ns0 = arena_take(S.ar, C, AR_NBR, nnb);
  const bool nfit = ns0 + nnb <= C.cap_nbr;
  if (l == 0) {
    const double Mv = S.acc[0];
    GL(C.mass)[orig] = Mv;
    GL(C.mom)[3 * (long long)orig + 0] = S.acc[1] + Mv * X.vx;
    GL(C.mom)[3 * (long long)orig + 1] = S.acc[2] + Mv * X.vy;
    GL(C.mom)[3 * (long long)orig + 2] = S.acc[3] + Mv * X.vz;
    GL(C.energy)[orig] = S.acc[4];
    GL(C.pcount)[orig] = npieces;
    GL(C.ncount)[orig] = nfit ? nnb : 0;
    GL(C.nstart)[orig] = ns0;
    S.ar.pieces += npieces;
    S.ar.faces += sum_faces;
    S.ar.verts += sum_verts;
    if (nfit) S.ar.nbrs += nnb;
    S.ar.dropped += dropped + (nfit ? 0 : 1);
    S.ar.queries += st.queries;
    S.ar.cands += st.cands;
    S.ar.clips += st.clips;
    S.ar.gridq += st.grid;
    if (err) {
      atomicAdd(&C.cnt[err == 2 ? CNT_ERR_CAP : CNT_ERR_LOC], 1ull);
      atomicMin((int *)&C.cnt[CNT_BAD_SITE], orig);
      if (where) atomicOr((unsigned long long *)&C.cnt[CNT_STAGES], 1ull << where);
    }
  }
  if (nfit) {
    // neighbours in ascending caller index (at most one per plane slot)
    const bool mine = in_mask(nbmask);
    const int me = mine ? S.clab[l] : 0;
    int rk = 0;
    for (uint64_t m = nbmask; m; m &= m - 1)
      rk += __builtin_amdgcn_readlane(me, __ffsll((unsigned long long)m) - 1) < me ? 1 : 0;
    if (mine) GL(C.nbr_arena)[ns0 + rk] = me;
  }
  lds_order();
  return true;
}

// Persistent: every workgroup (one wave) takes sites from the queues until
// all are done; sites it cannot finish go to C.redo.
// DENS: moments weighted by the density; POW: power diagrams; CORNERS: the
// interior split by the cells' corners; LOOSE: a clip with boundary seeds (M is
// not convex or a site lies outside it),
// where cells that reach far out of it are certified piece by piece; GRAD: face
// moments (the instances without them are shorter and spill less: 25.7 against
// 27.6 ms on the 1M clustered workload).
template <bool DENS, bool POW, bool CORNERS, bool LOOSE, bool GRAD>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 4))) sweep_kernel(GridView G, DomainView D, const CellsDev *__restrict__ Cp) {
  __shared__ SweepLds S;
  const CellsDev &C = *Cp;
  arena_init(S.ar);
  for (;;) {
    const int si = queue_next(S.ar, C, G.n);
    if (si < 0) break;
    const int b = G.nb > 1 ? diagram_of(G.site_off, G.nb, si) : 0;
    if (!do_cell<DENS, POW, CORNERS, LOOSE, GRAD>(S, G.views[b], D.views[b], C, si) && vd_lane() == 0)
      GL(C.redo)[__hip_atomic_fetch_add(GL(C.cnt) + CNT_REDO, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = si;
  }
  arena_close(S.ar, C);
}

// unused: the pieces of sites that were left half done
__global__ void __launch_bounds__(256) void_pieces(const CellsDev *__restrict__ Cp) {
  const CellsDev &C = *Cp;
  if (GL(C.cnt)[CNT_REDO] == 0) return;
  const long long used = (long long)GL(C.cnt)[CNT_PIECES];
  const long long n = used < C.cap_piece ? used : C.cap_piece;
  for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) {
    const int s = GL(C.piece_site)[p];
    if (s >= 0 && GL(C.pcount)[s] < 0) GL(C.piece_site)[p] = -1;
  }
}

int resident_workgroups() {
  static int cache[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  int &w = cache[dev];
  if (!w) {
    int per_cu = 0, ncu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, sweep_kernel<false, false, false, false, false>, 64, 0) != hipSuccess ||
        per_cu < 1)
      per_cu = 1;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1) ncu = 1;
    w = per_cu * ncu;
  }
  return w;
}

}  // namespace

int vd_sweep_workgroups(long long n) {
  const int w = resident_workgroups();
  return (int)(n < w ? (n > 0 ? n : 1) : w);
}

void vd_launch_sweep(const GridView &G, const DomainView &D, const CellsDev *Cdev, int workgroups, bool density,
                     bool power, bool corners, bool bseeds, bool grad, hipStream_t st) {
  const dim3 grid(workgroups), block(64);
#define VD_SWEEP(dens, pow, cor, loose, gr) \
  hipLaunchKernelGGL((sweep_kernel<dens, pow, cor, loose, gr>), grid, block, 0, st, G, D, Cdev)
#define VD_SWEEP_GRAD(dens, cor, loose)             \
  do {                                              \
    if (grad) VD_SWEEP(dens, false, cor, loose, true); \
    else VD_SWEEP(dens, false, cor, loose, false);  \
  } while (0)
  if (power) VD_SWEEP(false, true, false, false, false);
  else if (density && corners) VD_SWEEP_GRAD(true, true, false);
  else if (corners) VD_SWEEP_GRAD(false, true, false);
  else if (density && !bseeds) VD_SWEEP_GRAD(true, false, false);
  else if (density) VD_SWEEP_GRAD(true, false, true);
  else if (!bseeds) VD_SWEEP_GRAD(false, false, false);
  else VD_SWEEP_GRAD(false, false, true);
#undef VD_SWEEP_GRAD
#undef VD_SWEEP
}

void vd_launch_void_pieces(const CellsDev *Cdev, hipStream_t st) {
  hipLaunchKernelGGL(void_pieces, dim3(1024), dim3(256), 0, st, Cdev);
}
