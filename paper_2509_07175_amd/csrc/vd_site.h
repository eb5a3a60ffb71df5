// vd_site.h -- what the two per-site kernels of a tetrahedral domain share: the
// site being cut, packed corner topology, the planes of a tetrahedron, and
// point location in the domain.
#pragma once
#include "vd_arena.h"

__device__ __forceinline__ int p8(int packed, int e) { return (packed >> (8 * e)) & 0xff; }
__device__ __forceinline__ int pack3(int a, int b, int c) { return a | (b << 8) | (c << 16); }
__device__ __forceinline__ uint64_t low_mask(int k) { return k >= 64 ? ~0ull : ((1ull << k) - 1ull); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The upper half of a double is its logarithm in steps of 2^-20 (up to a bias, and
// linear between powers of two); of the largest of three components here.
__device__ __forceinline__ unsigned log_size(const double *n) {
  unsigned r;
  asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(__double2hiint(n[0])), "v"(__double2hiint(n[1])), "v"(__double2hiint(n[2])));
  return r;
}

// Is the determinant of the normals of three planes more than about 2^-digits of
// their sizes?  Cramer's rule leaves the corner's coordinates 2^(digits - 53) of their
// size, and below that two planes are almost parallel, or one almost holds the edge of
// the others.
__device__ __forceinline__ bool fixed_to(unsigned digits, double det, const double *n0, const double *n1, const double *n2) {
  const unsigned one = 0x3ff00000u;
  return (int)((unsigned)__double2hiint(fabs(det)) - one + (digits << 20)) >
         (int)(log_size(n0) + log_size(n1) + log_size(n2) - 3u * one);
}

constexpr unsigned kSure = 20;  // digits that a corner may lose where nothing else is done

struct SiteCtx {
  double vx, vy, vz, delta;
  double h, w;  // power diagram: lifted coordinate and weight of the site (else 0)
  int si;
};

// Plane of face f of T_a (opposite vertex f), outward, relative to v_i, and
// its flag.  Face loops {1,2,3},{0,3,2},{0,1,3},{0,2,1} are packed 2 bits per
// vertex, 6 bits per face (no indexed local arrays).
__device__ __forceinline__ void tet_plane(const DomainView &D, const SiteCtx &X, int a, int f, double *pl,
                                          int &lab) {
  const auto tv = &GL(D.simp)[(long long)a * 4];
  const unsigned loops = (1u | 2u << 2 | 3u << 4) | (0u | 3u << 2 | 2u << 4) << 6 |
                         (0u | 1u << 2 | 3u << 4) << 12 | (0u | 2u << 2 | 1u << 4) << 18;
  const unsigned lf = loops >> (6 * f);
  const auto pA = &GL(D.verts)[3 * (long long)tv[lf & 3]];
  const auto pB = &GL(D.verts)[3 * (long long)tv[(lf >> 2) & 3]];
  const auto pC = &GL(D.verts)[3 * (long long)tv[(lf >> 4) & 3]];
  const double A0 = pA[0] - X.vx, A1 = pA[1] - X.vy, A2 = pA[2] - X.vz;
  const double ab0 = pB[0] - pA[0], ab1 = pB[1] - pA[1], ab2 = pB[2] - pA[2];
  const double ac0 = pC[0] - pA[0], ac1 = pC[1] - pA[1], ac2 = pC[2] - pA[2];
  const double n0 = ab1 * ac2 - ab2 * ac1, n1 = ab2 * ac0 - ab0 * ac2, n2 = ab0 * ac1 - ab1 * ac0;
  pl[0] = n0; pl[1] = n1; pl[2] = n2;
  pl[3] = n0 * A0 + n1 * A1 + n2 * A2;
  const int b = GL(D.adj)[(long long)a * 4 + f];
  lab = b >= 0 ? -(b + 1) : VD_BND_BASE + f;
}

// The lowest-index tetrahedron containing q (the whole wave scans the point's
// location cell), or -1.
__device__ __forceinline__ int locate_wave(const DomainView &D, double qx, double qy, double qz) {
  if (!D.lstart) return -1;
  const double q[3] = {qx, qy, qz};
  int cc[3];
  for (int k = 0; k < 3; k++) cc[k] = cell_coord(q[k], GL(D.lgeom)[k], GL(D.lgeom)[6 + k], D.lg[k]);
  const int c = cc[0] + D.lg[0] * (cc[1] + D.lg[1] * cc[2]);
  int best = 0x7fffffff;
  for (int t = GL(D.lstart)[c] + vd_lane(); t < GL(D.lstart)[c + 1]; t += 64) {
    const int a = GL(D.litems)[t];
    if (a < best && tet_contains(D, a, q)) best = a;
  }
  const int b = (int)wave_min((double)best);
  return b == 0x7fffffff ? -1 : b;
}

// Is q in M?  One lane scans q's location cell (the tolerance of tet_contains
// counts a point on the boundary as inside).
__device__ __forceinline__ bool in_domain(const DomainView &D, double qx, double qy, double qz) {
  const double q[3] = {qx, qy, qz};
  int cc[3];
  for (int k = 0; k < 3; k++) cc[k] = cell_coord(q[k], GL(D.lgeom)[k], GL(D.lgeom)[6 + k], D.lg[k]);
  const int c = cc[0] + D.lg[0] * (cc[1] + D.lg[1] * cc[2]);
  for (int t = GL(D.lstart)[c]; t < GL(D.lstart)[c + 1]; t++)
    if (tet_contains(D, GL(D.litems)[t], q)) return true;
  return false;
}

__device__ __forceinline__ int convert_label(const GridView &G, int lab) { return lab >= 0 ? GL(G.perm)[lab] : lab; }
