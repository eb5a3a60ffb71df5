// vd_sweep.h -- what the sweep kernels (sweep3d.hip, sweep2d.hip) share: the LDS
// copy of the sites around a point, and wave helpers on scalar masks.
#pragma once
#include "vd_site.h"

namespace {

constexpr int kK = 128;      // sites in the LDS copy
constexpr int kNB = 64;      // distance buckets
constexpr int kBatch = 8;    // 64-site batches of candidates
constexpr int kCand = 64 * kBatch;
constexpr int kRows = 17 * 17;  // x-rows of the largest block (half-width 8 cells)

// orders LDS accesses of the wave (they complete in issue order: no wait)
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// the lanes that hold a true value
__device__ __forceinline__ uint64_t lanes(bool b) { return __builtin_amdgcn_ballot_w64(b); }
// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ uint64_t uni64(uint64_t v) { return (uint64_t)readlane_ll((long long)v, 0); }
__device__ __forceinline__ int mbcnt64(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// maximum over the wave
__device__ __forceinline__ int wave_imax(int v) {
  v = max(v, perm_i<VD_DPP_QUAD_XOR1>(v));
  v = max(v, perm_i<VD_DPP_QUAD_XOR2>(v));
  v = max(v, perm_i<VD_DPP_ROW_HALF_MIRROR>(v));
  v = max(v, perm_i<VD_DPP_ROW_MIRROR>(v));
  return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
// a bound of doubles over the wave, none negative, at most 1e-6 above the largest:
// their upper halves compare as integers, over the whole range of sizes
__device__ __forceinline__ double wave_bound(double v) {
  return __hiloint2double(wave_imax(__double2hiint(v)) + 1, 0);
}

// inclusive prefix maximum of a non-negative int over the wave
__device__ __forceinline__ int wave_incl_max(int v) {
  v = max(v, dpp_i<VD_DPP_ROW_SHR(1)>(0, v));
  v = max(v, dpp_i<VD_DPP_ROW_SHR(2)>(0, v));
  v = max(v, dpp_i<VD_DPP_ROW_SHR(4)>(0, v));
  v = max(v, dpp_i<VD_DPP_ROW_SHR(8)>(0, v));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, VD_DPP_ROW_BCAST15, 0xa, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, VD_DPP_ROW_BCAST31, 0xc, 0xf, false));
  return v;
}

// ---------------------------------------------------------------------------
// The LDS copy: the sites of a block of grid cells around v (half-width at
// most 8 cells, sized from the density of the 3x3x3 block to hold about 2.5 kK
// sites) by bucket of squared distance, in block order within a bucket (the
// same on every run).  When more than kK are in the block, a prefix of buckets
// that fits is kept.  The row of a candidate is the last row start at or before
// it, a prefix maximum over LDS marks; then all candidates (64 a batch) are read
// together, for one wait, and stay in registers until they have their places
// (read batch by batch, and again for their places: 5M uniform sites 53.5
// against 52.1 ms).
// Returns the number of sites held, or -1 (too dense: no copy).
// ---------------------------------------------------------------------------
template <bool POW, class L>
__device__ __forceinline__ int fill_sites(L &S, const GridView &G, double vx, double vy, double vz, double w, double need) {
  const int l = vd_lane();
  const int gx = G.g[0], gy = G.g[1], gz = G.g[2];
  const auto geom = GL(G.geom);
  const int cx = cell_coord(vx, geom[0], geom[6], gx);
  const int cy = cell_coord(vy, geom[1], geom[7], gy);
  const int cz = cell_coord(vz, geom[2], geom[8], gz);
  auto cells = [&](int r) {
    return uni((min(cx + r, gx - 1) - max(cx - r, 0) + 1) * (min(cy + r, gy - 1) - max(cy - r, 0) + 1) *
               (min(cz + r, gz - 1) - max(cz - r, 0) + 1));
  };
  int r = 1;
  if (need > 0.0) {
    // a ball of radius `need` must lie in the block
    // (an axis of one cell is open on both sides)
    const double h = fmin(gx > 1 ? geom[3] : 1e300, fmin(gy > 1 ? geom[4] : 1e300, gz > 1 ? geom[5] : 1e300));
    r = uni((int)fmin(8.0, ceil(need / h)));
    r = r < 1 ? 1 : r;
  } else {
    const int c1 = block_count(G, max(cx - 1, 0), min(cx + 1, gx - 1), max(cy - 1, 0), min(cy + 1, gy - 1),
                               max(cz - 1, 0), min(cz + 1, gz - 1));
    const float dens = (float)c1 / (float)cells(1);
    while (r < 8 && uni(c1 == 0 || dens * (float)cells(r + 1) <= 2.5f * kK)) r++;
  }
  // the rows of the block: candidate t is site base[row] + t of the row that holds it
  int x0, x1, y0, y1, z0, z1, total;
  for (;;) {
    x0 = max(cx - r, 0); x1 = min(cx + r, gx - 1);
    y0 = max(cy - r, 0); y1 = min(cy + r, gy - 1);
    z0 = max(cz - r, 0); z1 = min(cz + r, gz - 1);
    const int nx = x1 - x0 + 1, ny = y1 - y0 + 1, R = ny * (z1 - z0 + 1);
    const unsigned iny = 65536u / (unsigned)ny + 1u;  // q = x / ny for x < 65536 / ny
    {
      uint4 *z4 = reinterpret_cast<uint4 *>(S.R.row);
      z4[l] = make_uint4(0u, 0u, 0u, 0u);
    }
    lds_order();
    total = 0;
    for (int r0 = 0; r0 < R; r0 += 64) {
      const int rr = r0 + l;
      int st = 0, cnt = 0;
      if (rr < R) {
        const int q = (int)(((unsigned)rr * iny) >> 16);
        const int c0 = x0 + gx * ((y0 + rr - q * ny) + gy * (z0 + q));
        st = GL(G.cstart)[c0];
        cnt = GL(G.cstart)[c0 + nx] - st;
      }
      const int inc = wave_incl_scan(cnt);
      const int ex = total + inc - cnt;
      if (rr < R) {
        S.R.base[rr] = st - ex;
        if (cnt > 0 && ex < kCand) S.R.row[ex] = (unsigned short)rr;
      }
      total += __builtin_amdgcn_readlane(inc, 63);
    }
    if (total <= kCand) break;
    if (r == 0) return -1;
    r--;
  }
  lds_order();
  const int nbat = (total + 63) >> 6;
  // distance from v to the block's sides, less a margin for the rounding of
  // cell assignment (a side at the grid's edge is open)
  double rcb = 1e300;
  {
    const double h0 = geom[3], h1 = geom[4], h2 = geom[5];
    const double mg = 1e-9 * fmin(h0, fmin(h1, h2));
    double b[6];
    b[0] = x0 > 0 ? vx - (geom[0] + x0 * h0) - mg : 1e300;
    b[1] = x1 < gx - 1 ? geom[0] + (x1 + 1) * h0 - vx - mg : 1e300;
    b[2] = y0 > 0 ? vy - (geom[1] + y0 * h1) - mg : 1e300;
    b[3] = y1 < gy - 1 ? geom[1] + (y1 + 1) * h1 - vy - mg : 1e300;
    b[4] = z0 > 0 ? vz - (geom[2] + z0 * h2) - mg : 1e300;
    b[5] = z1 < gz - 1 ? geom[2] + (z1 + 1) * h2 - vz - mg : 1e300;
#pragma unroll
    for (int k = 0; k < 6; k++) {
      rcb = fmin(rcb, b[k]);
      if (l == 0) S.blk[k] = b[k];
    }
    if (rcb < 0.0) rcb = 0.0;
  }
  // buckets of squared distance: kNB - 1 of width step over [0, rc2), the last
  // one beyond
  const bool select = total > kK;
  const double hm = fmax(geom[3], fmax(geom[4], geom[5]));
  const double rcw2 = 3.0 * ((r + 1) * hm) * ((r + 1) * hm);
  const double rc2 = select ? fmin(rcb * rcb, rcw2) : rcw2;
  const double step = rc2 / (kNB - 1);
  const double istep = rc2 > 0.0 ? (kNB - 1) / rc2 : 0.0;
  auto bucket = [&](double d2) {
    // (istep is 0 for an empty range, whose sites all belong to the last bucket)
    int k = rc2 > 0.0 ? (int)fmin((double)(kNB - 1), d2 * istep) : kNB - 1;
    k += ((k < kNB - 1) & (d2 >= (k + 1) * step)) ? 1 : 0;
    k -= ((k > 0) & (d2 < k * step)) ? 1 : 0;
    return k;
  };
#pragma unroll
  for (int w = 0; w < kBatch / 2; w++)
    reinterpret_cast<uint4 *>(&S.B.bits[0][0])[64 * w + l] = make_uint4(0u, 0u, 0u, 0u);
  lds_order();
  int pos[kBatch], kb[kBatch];
  int carry = 0;
#pragma unroll
  for (int h = 0; h < kBatch; h++) {
    pos[h] = -1;
    if (h < nbat) {
      const int t = 64 * h + l;
      const int row = max(wave_incl_max(S.R.row[t]), carry);
      carry = __builtin_amdgcn_readlane(row, 63);
      if (t < total) pos[h] = S.R.base[row] + t;
    }
  }
  // all reads of a group of batches in flight together
  double ax[kBatch], ay[kBatch], az[kBatch];
  auto read = [&](int h) {
    const int p = pos[h] >= 0 ? pos[h] : 0;
    ax[h] = GL(G.sx)[p]; ay[h] = GL(G.sy)[p]; az[h] = GL(G.sz)[p];
  };
  read(0); read(1); read(2); read(3);
  if (nbat > 4) { read(4); read(5); }
  if (nbat > 6) { read(6); read(7); }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int h = 0; h < kBatch; h++) {
    kb[h] = kNB;
    if (h < nbat) {
      ax[h] -= vx; ay[h] -= vy; az[h] -= vz;
      const int k = bucket(ax[h] * ax[h] + ay[h] * ay[h] + az[h] * az[h]);
      if (pos[h] >= 0) {
        kb[h] = k;
        __hip_atomic_fetch_or(&S.B.bits[h][k], 1ull << l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }
  lds_order();
  // lane b: the entries of bucket b before each batch, and its start
  int cnt = 0;
  {
#pragma unroll
    for (int h = 0; h < kBatch; h++)
      if (h < nbat) {
        S.pre[h][l] = (unsigned short)cnt;
        cnt += __popcll(S.B.bits[h][l]);
      }
  }
  const int cum = wave_incl_scan(cnt);
  // buckets 0 .. B-1 are kept (cum is non-decreasing, so the fitting lanes are a prefix)
  const int B = select ? __popcll(lanes(l < kNB - 1 && cum <= kK)) : kNB;
  const int held = B > 0 ? __builtin_amdgcn_readlane(cum, B - 1) : 0;
  S.rec[l] = (unsigned)(cum - cnt);
  lds_order();
  int rk[kBatch];
#pragma unroll
  for (int h = 0; h < kBatch; h++) {
    rk[h] = 0;
    if (h < nbat && kb[h] < B)
      rk[h] = (int)S.rec[kb[h]] + S.pre[h][kb[h]] + __popcll(S.B.bits[h][kb[h]] & low_mask_lt(l));
  }
  lds_order();
#pragma unroll
  for (int h = 0; h < kBatch; h++) {
    if (h < nbat && kb[h] < B) {
      const int p = pos[h];
      const double n0 = ax[h], n1 = ay[h], n2 = az[h];
      double *e = S.K.s[rk[h]];
      e[0] = n0; e[1] = n1; e[2] = n2;
      e[3] = POW ? 0.5 * (n0 * n0 + n1 * n1 + n2 * n2 + w - GL(G.sw)[p]) : 0.5 * (n0 * n0 + n1 * n1 + n2 * n2);
      S.K.p[rk[h]] = p;
      S.K.kb[rk[h]] = (unsigned char)kb[h];
    }
  }
  if (l == 0) {
    S.step = step;
    S.keep = select ? sqrt(B * step) * (1.0 - 1e-12) : 1e300;
  }
  lds_order();
  return held;
}

}  // namespace
