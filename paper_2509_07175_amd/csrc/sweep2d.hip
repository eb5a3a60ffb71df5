// sweep2d.hip -- the default restricted diagram of a triangle mesh, one
// wavefront per triangle, four pieces at a time.
//
// The sites around the triangle's centroid are copied to LDS once (vd_sweep.h)
// and from there to registers, eight to a lane, the same in each of the wave's
// four rows of 16 lanes.  A row carves one piece T_a cap Omega_i: a lane owns a
// vertex of the polygon, the row tests one vertex at a time against all the
// sites in its registers (the point-in-cell test: its nearest site), and a
// vertex with a nearer site than v_i, other than those of the vertex's own two
// edges, is cut off by that site's bisector.  A vertex that survives is tested
// once.  The sites of the triangle are found by propagation over the bisector
// edges of its pieces (Alg. 4), from the sites nearest to the centroid and to
// the three corners.  Coordinates are relative to the centroid, and a new
// vertex is interpolated on the edge that it cuts.
//
// What bounds it: the carve's chain of LDS round trips and FP64 operations (60 %
// of the kernel, four waves per SIMD, of LDS and registers): 9 vertex tests and
// 5 cuts a piece.  Icosphere of 81,920 triangles, 200,000 sites (655,000
// pieces, with segment moments): 5.2 ms with surface.hip (one piece at a time: 4
// of its 64 lanes hold vertices, grid queries and Gabriel tests), 2.35 ms here;
// of that, the copies 10 %, emission 15 %.  Coverage is looked at once per
// finished piece (2.7 ms when each vertex test did).
//
// A triangle that does not fit (a vertex that the copy does not certify, more
// than 16 vertices in a piece) is left to that kernel, which then takes
// the triangles on C.redo; pieces written before that are voided.
#include "vd_sweep.h"

namespace {

constexpr int kV = 16;   // vertices of a piece
constexpr int kS = kK / 16;  // sites a lane holds

struct __align__(16) TriSweepLds {
  union {
    struct {
      double v[4][kV][3];    // polygon vertices of each row
      int lab[4][kV];        // edge from vertex t to t + 1: site slot >= 0, or a triangle edge's flag
      int tst[4][kV];        // the vertex is certified
    };
    struct {
      unsigned short row[kCand];  // (the copy's scratch)
      int base[kRows];
    } R;
    unsigned short pre[kBatch][kNB];
  };
  union alignas(16) {
    struct {
      double s[kK][4];       // sites relative to the centroid, and half their squared norm (power: minus w)
      int p[kK];             // sorted position
      unsigned char kb[kK];
    } K;
    struct {
      unsigned long long bits[kBatch][kNB];
    } B;
  };
  unsigned rec[64];
  int orig[kK];              // caller index of each site
  double tri[3][3];          // the triangle relative to its centroid
  int tlab[3];               // flags of its edges (edge e opposite corner e)
  unsigned long long seen[2];
  double step, keep, blk[6];
  WaveArena ar;
};

struct SweepStats2 {
  long long queries = 0, clips = 0;
};

// sum over a row of 16 lanes, the same value in each of them
__device__ __forceinline__ double row_sum(double v) {
  v += perm_d<VD_DPP_QUAD_XOR1>(v);
  v += perm_d<VD_DPP_QUAD_XOR2>(v);
  v += perm_d<VD_DPP_ROW_HALF_MIRROR>(v);
  v += perm_d<VD_DPP_ROW_MIRROR>(v);
  return v;
}

__device__ __forceinline__ double row_min(double v) {
  v = fmin(v, perm_d<VD_DPP_QUAD_XOR1>(v));
  v = fmin(v, perm_d<VD_DPP_QUAD_XOR2>(v));
  v = fmin(v, perm_d<VD_DPP_ROW_HALF_MIRROR>(v));
  v = fmin(v, perm_d<VD_DPP_ROW_MIRROR>(v));
  return v;
}

__device__ __forceinline__ int row_imin(int v) {
  v = min(v, perm_i<VD_DPP_QUAD_XOR1>(v));
  v = min(v, perm_i<VD_DPP_QUAD_XOR2>(v));
  v = min(v, perm_i<VD_DPP_ROW_HALF_MIRROR>(v));
  v = min(v, perm_i<VD_DPP_ROW_MIRROR>(v));
  return v;
}

// the 16 bits of this lane's row
__device__ __forceinline__ unsigned row_of(uint64_t m) { return (unsigned)(m >> (vd_lane() & 48)) & 0xffffu; }

// One triangle; false: it has to go to the general kernel (`written` tells
// whether pieces of it are in the arenas).
template <bool DENS, bool POW, bool GRAD>
__device__ __forceinline__ bool do_tri(TriSweepLds &S, const GridView &G, const DomainView &D, const CellsDev &C, int a,
                                       bool &written) {
  const int l = vd_lane(), gl = l & 15, grp = l >> 4;
  written = false;
  double cx, cy, cz, N0, N1, N2, inrm, rho;
  {
    const auto tv = &GL(D.simp)[(long long)a * 3];
    const auto p0 = &GL(D.verts)[3 * (long long)tv[0]], p1 = &GL(D.verts)[3 * (long long)tv[1]],
               p2 = &GL(D.verts)[3 * (long long)tv[2]];
    cx = readlane_d((p0[0] + p1[0] + p2[0]) / 3.0, 0);
    cy = readlane_d((p0[1] + p1[1] + p2[1]) / 3.0, 0);
    cz = readlane_d((p0[2] + p1[2] + p2[2]) / 3.0, 0);
    const double e1[3] = {p1[0] - p0[0], p1[1] - p0[1], p1[2] - p0[2]};
    const double e2[3] = {p2[0] - p0[0], p2[1] - p0[1], p2[2] - p0[2]};
    N0 = e1[1] * e2[2] - e1[2] * e2[1];
    N1 = e1[2] * e2[0] - e1[0] * e2[2];
    N2 = e1[0] * e2[1] - e1[1] * e2[0];
    inrm = 1.0 / sqrt(N0 * N0 + N1 * N1 + N2 * N2);
    N0 = readlane_d(N0 * inrm, 0); N1 = readlane_d(N1 * inrm, 0); N2 = readlane_d(N2 * inrm, 0);
    double r2 = 0.0;
    if (l < 3) {
      const auto p = &GL(D.verts)[3 * (long long)tv[l]];
      const double x0 = p[0] - cx, x1 = p[1] - cy, x2 = p[2] - cz;
      S.tri[l][0] = x0; S.tri[l][1] = x1; S.tri[l][2] = x2;
      r2 = x0 * x0 + x1 * x1 + x2 * x2;
      const int b = GL(D.adj)[(long long)a * 3 + l];
      S.tlab[l] = b >= 0 ? -(b + 1) : VD_BND_BASE + l;
    }
    rho = sqrt_bound(fmax(readlane_d(r2, 0), fmax(readlane_d(r2, 1), readlane_d(r2, 2))));
  }
  // the copy reaches past the farthest corner by a grid cell: about two
  // distances between sites at the default density of 3.5 sites per cell
  const auto geom = GL(G.geom);
  const double hc = fmax(G.g[0] > 1 ? geom[3] : 0.0, fmax(G.g[1] > 1 ? geom[4] : 0.0, G.g[2] > 1 ? geom[5] : 0.0));
  int held = uni(fill_sites<POW>(S, G, cx, cy, cz, 0.0, rho + hc + 1e-300));
  if (held <= 0) return false;
  double eta = 0.0;  // power diagrams: the largest weight
  if (POW) {
    const int p = uni(S.K.p[0]);
    const double h = GL(G.sh)[p];
    eta = GL(G.sw)[p] + h * h;
  }
  for (int k = l; k < held; k += 64) S.orig[k] = GL(G.perm)[S.K.p[k]];
  double sx[kS], sy[kS], sz[kS], sh[kS];
#pragma unroll
  for (int b = 0; b < kS; b++) {
    const int k = 16 * b + gl;
    const bool in = k < held;
    const double *e = S.K.s[in ? k : 0];
    sx[b] = e[0]; sy[b] = e[1]; sz[b] = e[2];
    sh[b] = in ? e[3] : 1e300;
  }
  SweepStats2 st;
  // the site nearest to x (x uniform in the row): f = s.x - |s|^2 / 2 is largest.
  // Of equal ones the lowest slot: sites at the same point are neighbours in the
  // copy, by index, so that the first of them has the cell in every triangle (the
  // others none), as in surface.hip
  auto nearest = [&](double x0, double x1, double x2, double &fb, int &kb) {
    double nf = 1e300;
    int nk = 0;
#pragma unroll
    for (int b = 0; b < kS; b++) {
      if (16 * b < held) {
        const double f = sh[b] - (sx[b] * x0 + sy[b] * x1 + sz[b] * x2);
        const bool t = f < nf;
        nf = t ? f : nf;
        nk = t ? 16 * b + gl : nk;
      }
    }
    fb = row_min(nf);
    kb = row_imin(nf == fb ? nk : kK);
  };
  // does the copy hold every site that could be nearer to x than f says?
  auto covered = [&](double x0, double x1, double x2, double f) {
    const double xx = x0 * x0 + x1 * x1 + x2 * x2;
    const double s = sqrt_bound(xx) * (1.0 + 1e-9);
    const double d = sqrt_bound(fmax(xx + 2.0 * f + eta, 0.0) + 1e-12 * xx) * (1.0 + 1e-9);
    return (s + d < S.keep) & (d - x0 < S.blk[0]) & (d + x0 < S.blk[1]) & (d - x1 < S.blk[2]) & (d + x1 < S.blk[3]) &
           (d - x2 < S.blk[4]) & (d + x2 < S.blk[5]);
  };
  lds_order();
  uint64_t pend0, pend1, done0 = 0, done1 = 0;
  {
    // the cells that hold the centroid and the corners
    const double *q = S.tri[grp > 0 ? grp - 1 : 0];
    const double x0 = grp ? q[0] : 0.0, x1 = grp ? q[1] : 0.0, x2 = grp ? q[2] : 0.0;
    double f;
    int k;
    nearest(x0, x1, x2, f, k);
    if (lanes(!covered(x0, x1, x2, f))) return false;
    if (!POW) {
      // a site nearest to a point of T_a is within 2 rho of the centroid's
      // nearest distance: the others need not be looked at
      const double r = (2.0 * rho + sqrt_bound(2.0 * readlane_d(f, 0))) * (1.0 + 1e-6);
      const double lim = r * r;
      const uint64_t a0 = lanes(l < held && (double)S.K.kb[l] * S.step <= lim);
      const uint64_t a1 = lanes(l + 64 < held && (double)S.K.kb[l + 64] * S.step <= lim);
      held = __popcll(a0) + __popcll(a1);
    }
    if (l < 2) S.seen[l] = 0ull;
    lds_order();
    if (gl == 0) __hip_atomic_fetch_or(&S.seen[k >> 6], 1ull << (k & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    lds_order();
    pend0 = uni64(S.seen[0]);
    pend1 = uni64(S.seen[1]);
    st.queries += 4;
  }
  unsigned npieces = 0, nfaces = 0, dropped = 0;
#pragma unroll 1
  while (pend0 | pend1) {
    // four sites, one to a row
    int me = -1;
#pragma unroll
    for (int g = 0; g < 4; g++) {
      int b = -1;
      if (pend0) {
        b = __ffsll((unsigned long long)pend0) - 1;
        pend0 &= pend0 - 1;
        done0 |= 1ull << b;
      } else if (pend1) {
        b = 64 + __ffsll((unsigned long long)pend1) - 1;
        pend1 &= pend1 - 1;
        done1 |= 1ull << (b - 64);
      }
      me = grp == g ? b : me;
    }
    const double *e = S.K.s[me < 0 ? 0 : me];
    const double v0 = e[0], v1 = e[1], v2 = e[2], vh = e[3];
    int nv = me >= 0 ? 3 : 0;
    if (gl < 3) {
      S.v[grp][gl][0] = S.tri[gl][0]; S.v[grp][gl][1] = S.tri[gl][1]; S.v[grp][gl][2] = S.tri[gl][2];
      S.lab[grp][gl] = S.tlab[gl == 0 ? 2 : gl - 1];  // the edge from corner t to t + 1 is opposite corner t + 2
      S.tst[grp][gl] = 0;
    }
    lds_order();
    bool fail = false;
#pragma unroll 1
    for (int it = 0;; it++) {
      const unsigned open = row_of(lanes(gl < nv && !S.tst[grp][gl]));
      if (!lanes(open != 0)) break;
      if (it >= 512) { fail = true; break; }
      const int t = open ? __ffs(open) - 1 : 0;
      const double x0 = S.v[grp][t][0], x1 = S.v[grp][t][1], x2 = S.v[grp][t][2];
      const int ln = S.lab[grp][t], lp = S.lab[grp][t == 0 ? (nv > 0 ? nv - 1 : 0) : t - 1];
      double f;
      int k;
      nearest(x0, x1, x2, f, k);
      const double mine = vh - (v0 * x0 + v1 * x1 + v2 * x2);
      const bool in = (k == me) | (k == ln) | (k == lp) | !(f < mine);
      st.queries += __popcll(lanes(open != 0 && gl == 0));
      // cut off by the bisector with site k: n.x <= c
      const bool cutting = (open != 0) & !in;
      const double n0 = S.K.s[k][0] - v0, n1 = S.K.s[k][1] - v1, n2 = S.K.s[k][2] - v2, c = S.K.s[k][3] - vh;
      const bool mv = cutting & (gl < nv);
      const double a0 = S.v[grp][gl][0], a1 = S.v[grp][gl][1], a2 = S.v[grp][gl][2];
      const double da = n0 * a0 + n1 * a1 + n2 * a2 - c;
      const unsigned O = row_of(lanes(mv & (da > 0.0)));
      // certified, or outside by rounding only: it stays
      if (gl == t && open && !((O >> t) & 1u)) S.tst[grp][t] = 1;
      if (!lanes(mv & (O != 0))) { lds_order(); continue; }
      const bool go = mv & (O != 0);
      const int nx = gl + 1 < nv ? gl + 1 : 0;
      const double b0 = S.v[grp][nx][0], b1 = S.v[grp][nx][1], b2 = S.v[grp][nx][2];
      const double db = n0 * b0 + n1 * b1 + n2 * b2 - c;
      const bool ia = !((O >> gl) & 1u), ib = !((O >> nx) & 1u);
      const bool cross = go & (ia != ib);
      const unsigned I = row_of(lanes(go & ia)), X = row_of(lanes(cross));
      const int nn = __popc(I) + __popc(X);
      const int pos = __popc(I & ((1u << gl) - 1u)) + __popc(X & ((1u << gl) - 1u));
      const double tt = da / (da - db);
      const double y0 = a0 + tt * (b0 - a0), y1 = a1 + tt * (b1 - a1), y2 = a2 + tt * (b2 - a2);
      const int la = S.lab[grp][gl], ta = S.tst[grp][gl];
      if (lanes(go & (I != 0) & ((nn > kV) | (__popc(X) != 2)))) { fail = true; break; }
      lds_order();
      if (go & ia) {
        S.v[grp][pos][0] = a0; S.v[grp][pos][1] = a1; S.v[grp][pos][2] = a2;
        S.lab[grp][pos] = la;
        S.tst[grp][pos] = ta;
      }
      if (cross) {
        const int q = pos + (ia ? 1 : 0);
        S.v[grp][q][0] = y0; S.v[grp][q][1] = y1; S.v[grp][q][2] = y2;
        S.lab[grp][q] = ia ? k : la;
        S.tst[grp][q] = 0;
      }
      nv = row_of(lanes(go)) ? (I ? nn : 0) : nv;
      st.clips += __popcll(lanes(go && gl == 0));
      lds_order();
    }
    if (fail) return false;
    // ---- moments relative to v_i: fan of triangles from vertex 0, so that the
    // area's rounding error scales with the piece ----
    const bool live = gl < nv;
    const double o0 = S.v[grp][0][0], o1 = S.v[grp][0][1], o2 = S.v[grp][0][2];
    const int nx = gl + 1 < nv ? gl + 1 : 0;
    const double X0 = S.v[grp][gl][0], X1 = S.v[grp][gl][1], X2 = S.v[grp][gl][2];
    // v_i is the nearest site of every vertex: no nearer one may be missing
    if (lanes(live & !covered(X0, X1, X2, vh - (v0 * X0 + v1 * X1 + v2 * X2)))) return false;
    const double Z0 = S.v[grp][nx][0], Z1 = S.v[grp][nx][1], Z2 = S.v[grp][nx][2];
    double pa = 0, pmx = 0, pmy = 0, pmz = 0, pe = 0;
    const double vx = cx + v0, vy = cy + v1, vz = cz + v2;
    if (live) {
      const double a0 = X0 - o0, a1 = X1 - o1, a2 = X2 - o2, b0 = Z0 - o0, b1 = Z1 - o1, b2 = Z2 - o2;
      const double ar = 0.5 * ((a1 * b2 - a2 * b1) * N0 + (a2 * b0 - a0 * b2) * N1 + (a0 * b1 - a1 * b0) * N2);
      const double P0[3] = {o0 - v0, o1 - v1, o2 - v2}, P1[3] = {X0 - v0, X1 - v1, X2 - v2}, P2[3] = {Z0 - v0, Z1 - v1, Z2 - v2};
      const double s0 = P0[0] + P1[0] + P2[0], s1 = P0[1] + P1[1] + P2[1], s2 = P0[2] + P1[2] + P2[2];
      pa = ar;
      if (!DENS) {
        const double t = ar * (1.0 / 3.0);
        pmx = t * s0; pmy = t * s1; pmz = t * s2;
        pe = ar * (1.0 / 12.0) *
             (P0[0] * P0[0] + P0[1] * P0[1] + P0[2] * P0[2] + P1[0] * P1[0] + P1[1] * P1[1] + P1[2] * P1[2] +
              P2[0] * P2[0] + P2[1] * P2[1] + P2[2] * P2[2] + s0 * s0 + s1 * s1 + s2 * s2);
      }
    }
    pa = row_sum(pa);
    // a piece exists when its area is positive; with a density its moments are
    // the weighted ones
    const bool ok = nv >= 3 && pa > 0.0;
    if (DENS) {
      double dm = 0;
      if (live) {
        const double P0[3] = {o0 - v0, o1 - v1, o2 - v2}, P1[3] = {X0 - v0, X1 - v1, X2 - v2}, P2[3] = {Z0 - v0, Z1 - v1, Z2 - v2};
        const double a0 = X0 - o0, a1 = X1 - o1, a2 = X2 - o2, b0 = Z0 - o0, b1 = Z1 - o1, b2 = Z2 - o2;
        const double ar = 0.5 * ((a1 * b2 - a2 * b1) * N0 + (a2 * b0 - a0 * b2) * N1 + (a0 * b1 - a1 * b0) * N2);
        tri_density_moments(C.dens, vx, vy, vz, P0, P1, P2, ar, dm, pmx, pmy, pmz, pe);
      }
      pa = row_sum(dm);
    }
    pmx = row_sum(pmx); pmy = row_sum(pmy); pmz = row_sum(pmz); pe = row_sum(pe);
    const uint64_t lead = lanes(ok && gl == 0);
    if (!lead) continue;
    // ---- emit the pieces of the four rows ----
    const int np = __popcll(lead);
    int before = 0, tot = 0;  // vertices of the rows before this one, and of all
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int k = __builtin_amdgcn_readlane(ok ? nv : 0, 16 * g);
      before += g < grp ? k : 0;
      tot += k;
    }
    const int lab = ok && live ? S.lab[grp][gl] : -1;
    const uint64_t seg = GRAD ? lanes(lab >= 0) : 0ull;  // bisector edges
    arena_skip_pieces(S.ar, C, np);
    const long long at = arena_take_all(S.ar, C, arena_counts(np, tot, tot, __popcll(seg)));
    const long long pidx = readlane_ll(at, AR_PIECE) + __popcll(lead & low_mask(l & 48));
    const long long fo = readlane_ll(at, AR_FACE) + before;
    const long long vo = readlane_ll(at, AR_VERT) + before;
    written = true;
    // only records that fit are counted: the per-site CSR built from the
    // counts then stays inside the arenas (the clip reports the overflow)
    const bool fits_fv = fo + nv <= C.cap_face && vo + nv <= C.cap_vert;
    const bool fits_p = pidx < C.cap_piece;
    const int orig = S.orig[me < 0 ? 0 : me];
    if (GRAD) {
      // segment moments of the bisector edges: a point of the edge moves in
      // the plane of T_a with speed (x - v_i).dv / (d s), s = |n - (n.N)N|
      // (n, N unit normals of the bisector and of T_a); 2-point Gauss-Legendre
      // is exact for the cubic integrand, 3 points with a density
      const unsigned pos = row_of(seg);
      const long long base = readlane_ll(at, AR_FINT) + __popcll(seg & low_mask(l & 48));
      const int npos = __popc(pos);
      const bool ffits = base + npos <= C.cap_fint;
      if (ok && gl == 0 && fits_p) {
        GL(C.piece_fint_start)[pidx] = base;
        GL(C.piece_nfint)[pidx] = ffits ? npos : 0;
      }
      dropped += __popcll(lanes(ok && gl == 0 && fits_p && !ffits));
      const long long r = base + __popc(pos & ((1u << gl) - 1u));
      if (lab >= 0 && r < C.cap_fint) {
        const double n0 = S.K.s[lab][0] - v0, n1 = S.K.s[lab][1] - v1, n2 = S.K.s[lab][2] - v2;
        const double d = sqrt(n0 * n0 + n1 * n1 + n2 * n2);
        const double h0 = n0 / d, h1 = n1 / d, h2 = n2 / d;
        const double hn = h0 * N0 + h1 * N1 + h2 * N2;
        const double e0 = h0 - hn * N0, e1 = h1 - hn * N1, e2 = h2 - hn * N2;
        const double sfac = sqrt(e0 * e0 + e1 * e1 + e2 * e2);
        const double a0 = X0 - v0, a1 = X1 - v1, a2 = X2 - v2;
        const double b0 = Z0 - v0, b1 = Z1 - v1, b2 = Z2 - v2;
        const double len = sqrt((b0 - a0) * (b0 - a0) + (b1 - a1) * (b1 - a1) + (b2 - a2) * (b2 - a2));
        double I[12];
#pragma unroll
        for (int k = 0; k < 12; k++) I[k] = 0.0;
        const double g2 = 0.28867513459481287, g3 = 0.38729833462074170;  // 1 / (2 sqrt 3), sqrt(0.6) / 2
        constexpr int ng = DENS ? 3 : 2;
#pragma unroll
        for (int g = 0; g < ng; g++) {
          const double xi = ng == 2 ? (g == 0 ? 0.5 - g2 : 0.5 + g2) : (g == 0 ? 0.5 - g3 : (g == 1 ? 0.5 : 0.5 + g3));
          const double y0 = a0 + xi * (b0 - a0), y1 = a1 + xi * (b1 - a1), y2 = a2 + xi * (b2 - a2);
          const double w = (ng == 2 ? 0.5 : (g == 1 ? 8.0 / 18.0 : 5.0 / 18.0)) * len *
                           (DENS ? density_at(C.dens, vx + y0, vy + y1, vz + y2) : 1.0);
          const double yy = y0 * y0 + y1 * y1 + y2 * y2;
          I[0] += w * y0; I[1] += w * y1; I[2] += w * y2;
          I[3] += w * y0 * y0; I[4] += w * y0 * y1; I[5] += w * y0 * y2;
          I[6] += w * y1 * y1; I[7] += w * y1 * y2; I[8] += w * y2 * y2;
          I[9] += w * yy * y0; I[10] += w * yy * y1; I[11] += w * yy * y2;
        }
        const double sc = 1.0 / (d * sfac);
#pragma unroll
        for (int k = 0; k < 12; k++) GL(C.fint)[12 * r + k] = I[k] * sc;
        GL(C.fint_lab)[r] = S.orig[lab];
      }
    }
    if (ok && gl == 0) {
      if (fits_p && fits_fv)
        __hip_atomic_fetch_add(GL(C.pcount) + orig, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (fits_p) {
        // a piece whose edges did not fit is written as an unused slot
        GL(C.piece_site)[pidx] = fits_fv ? orig : -1;
        GL(C.piece_simplex)[pidx] = a;
        GL(C.piece_nface)[pidx] = nv;
        GL(C.piece_nvert)[pidx] = nv;
        GL(C.piece_mass)[pidx] = pa;
        GL(C.piece_mom)[3 * pidx + 0] = pmx + pa * vx;
        GL(C.piece_mom)[3 * pidx + 1] = pmy + pa * vy;
        GL(C.piece_mom)[3 * pidx + 2] = pmz + pa * vz;
        GL(C.piece_energy)[pidx] = pe;
        GL(C.piece_fstart)[pidx] = fo;
        GL(C.piece_vstart)[pidx] = vo;
      }
    }
    {
      const uint64_t fit = lanes(ok && gl == 0 && fits_p && fits_fv);
      npieces += __popcll(fit);
      dropped += np - __popcll(fit);
#pragma unroll
      for (int g = 0; g < 4; g++)
        if ((fit >> (16 * g)) & 1ull) nfaces += __builtin_amdgcn_readlane(nv, 16 * g);
    }
    if (ok && live && fits_p && fits_fv) {
      const int lp = S.lab[grp][gl == 0 ? nv - 1 : gl - 1];
      const int fl = lab >= 0 ? S.orig[lab] : lab;
      GL(C.face_label)[fo + gl] = fl;
      GL(C.vert_xyz)[3 * (vo + gl) + 0] = X0 + cx;
      GL(C.vert_xyz)[3 * (vo + gl) + 1] = X1 + cy;
      GL(C.vert_xyz)[3 * (vo + gl) + 2] = X2 + cz;
      GL(C.vert_label)[3 * (vo + gl) + 0] = lp >= 0 ? S.orig[lp] : lp;
      GL(C.vert_label)[3 * (vo + gl) + 1] = fl;
      GL(C.vert_label)[3 * (vo + gl) + 2] = 2147483647;
    }
    // ---- propagate over the bisector edges (Alg. 4) ----
    if (lab >= 0) __hip_atomic_fetch_or(&S.seen[lab >> 6], 1ull << (lab & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    lds_order();
    pend0 = uni64(S.seen[0]) & ~done0;
    pend1 = uni64(S.seen[1]) & ~done1;
  }
  if (l == 0) {
    S.ar.pieces += npieces;
    S.ar.faces += nfaces;
    S.ar.verts += nfaces;
    S.ar.dropped += dropped;
    S.ar.queries += st.queries;
    S.ar.cands += st.queries * held;
    S.ar.clips += st.clips;
  }
  return true;
}

// Persistent: every workgroup (one wave) takes triangles from the queues until
// all are done; triangles it cannot finish go to C.redo.
template <bool DENS, bool POW, bool GRAD>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 4))) tri_kernel(GridView G, DomainView D, const CellsDev *__restrict__ Cp) {
  __shared__ TriSweepLds S;
  const CellsDev &C = *Cp;
  arena_init(S.ar);
  for (;;) {
    const int a = queue_next(S.ar, C, D.m);
    if (a < 0) break;
    // the triangle's own diagram (a batch) or the only one
    const int b = D.nb > 1 ? diagram_of(D.simp_off, D.nb, a) : 0;
    bool written;
    const bool ok = do_tri<DENS, POW, GRAD>(S, G.views[b], D.views[b], C, a, written);
    if (vd_lane() == 0) {
      GL(C.voided)[a] = !ok && written ? 1 : 0;
      if (!ok)
        GL(C.redo)[__hip_atomic_fetch_add(GL(C.cnt) + CNT_REDO, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = a;
    }
    lds_order();
  }
  arena_close(S.ar, C);
}

// unused: the pieces of triangles that were left half done
__global__ void __launch_bounds__(256) void_triangles(const CellsDev *__restrict__ Cp) {
  const CellsDev &C = *Cp;
  if (GL(C.cnt)[CNT_REDO] == 0) return;
  const long long used = (long long)GL(C.cnt)[CNT_PIECES];
  const long long n = used < C.cap_piece ? used : C.cap_piece;
  for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) {
    const int s = GL(C.piece_site)[p];
    if (s >= 0 && GL(C.voided)[GL(C.piece_simplex)[p]]) {
      GL(C.piece_site)[p] = -1;
      __hip_atomic_fetch_add(GL(C.pcount) + s, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

int resident_workgroups() {
  static int cache[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  int &w = cache[dev];
  if (!w) {
    int per_cu = 0, ncu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, tri_kernel<false, false, false>, 64, 0) != hipSuccess || per_cu < 1)
      per_cu = 1;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1) ncu = 1;
    w = per_cu * ncu;
  }
  return w;
}

}  // namespace

int vd_tri_workgroups(long long m) {
  const int w = resident_workgroups();
  return (int)(m < w ? (m > 0 ? m : 1) : w);
}

void vd_launch_tri(const GridView &G, const DomainView &D, const CellsDev *Cdev, int workgroups, bool density,
                   bool power, bool grad, hipStream_t st) {
  const dim3 grid((unsigned)workgroups), block(64);
  if (power) hipLaunchKernelGGL((tri_kernel<false, true, false>), grid, block, 0, st, G, D, Cdev);
  else if (density && grad) hipLaunchKernelGGL((tri_kernel<true, false, true>), grid, block, 0, st, G, D, Cdev);
  else if (density) hipLaunchKernelGGL((tri_kernel<true, false, false>), grid, block, 0, st, G, D, Cdev);
  else if (grad) hipLaunchKernelGGL((tri_kernel<false, false, true>), grid, block, 0, st, G, D, Cdev);
  else hipLaunchKernelGGL((tri_kernel<false, false, false>), grid, block, 0, st, G, D, Cdev);
}

void vd_launch_void_triangles(const CellsDev *Cdev, hipStream_t st) {
  hipLaunchKernelGGL(void_triangles, dim3(1024), dim3(256), 0, st, Cdev);
}
