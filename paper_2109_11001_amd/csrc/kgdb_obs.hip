// Initial states, deterministic per-melt reductions and the R^2(n)/n observable (gfx950).
#include "kgdb_dev.h"
#include "kgdb_kernels.h"

namespace kgdb {

// Seeded freely jointed random walks: bond 0.97 sigma along isotropic unit vectors
// u = (sqrt(1-z^2) cos phi, sqrt(1-z^2) sin phi, z), z uniform in [-1,1), phi in [0, 2 pi),
// uniform start points; accumulated unwrapped in chain order, then wrapped.  One thread
// per chain (blockIdx.y = melt).  Monomer ids start as chain * N + position.
__global__ void k_random_walks(const MeltDesc* __restrict__ md, int NP, double* __restrict__ x,
                               int* __restrict__ chain, int* __restrict__ loc) {
  const MeltDesc& d = md[blockIdx.y];
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= d.M) return;
  const int N = d.N;
  U64x4 w = rng_draw(d, (uint64_t)c * N, 0, ST_WALK);
  double px = u01(w.w[0]) * d.L, py = u01(w.w[1]) * d.L, pz = u01(w.w[2]) * d.L;
  for (int p = 0; p < N; ++p) {
    if (p > 0) {
      w = rng_draw(d, (uint64_t)c * N + p, 0, ST_WALK);
      const double z = 2.0 * u01(w.w[0]) - 1.0;
      const double ph = 6.283185307179586 * u01(w.w[1]);
      const double st = sqrt(1.0 - z * z);
      px = px + 0.97 * (st * cos(ph));
      py = py + 0.97 * (st * sin(ph));
      pz = pz + 0.97 * z;
    }
    const int li = c * N + p, g = d.off + li;
    x[g] = wrap_box(px, d.L);
    x[NP + g] = wrap_box(py, d.L);
    x[2 * NP + g] = wrap_box(pz, d.L);
    chain[g] = g;
    loc[g] = li;
  }
}

// Freely rotating chains (Sec. II.B): the first bond isotropic, each later bond at angle
// theta* to the one before it (cos theta* = d.fr_cos) about a uniform azimuth phi measured in
// the frame e1 = (a x u)/|a x u|, e2 = u x e1, a the coordinate axis least aligned with the
// previous bond u (the first of them on ties); bond length l0 = 0.960897.  State t of melt k
// (tries[k] = t; < 0 skips the melt) draws from Philox counter word 1 = t.  The chain table
// of k_random_walks is kept.
__global__ void k_fr_chains(const MeltDesc* __restrict__ md, int NP, double* __restrict__ x,
                            const int* __restrict__ tries) {
  const int k = blockIdx.y;
  const MeltDesc& d = md[k];
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (tries[k] < 0 || c >= d.M) return;
  const int N = d.N;
  const uint64_t t = (uint64_t)tries[k];
  const double l0 = 0.960897, ct = d.fr_cos, st = sqrt(1.0 - ct * ct);
  U64x4 w = rng_draw(d, (uint64_t)c * N, t, ST_WALK);
  double px = u01(w.w[0]) * d.L, py = u01(w.w[1]) * d.L, pz = u01(w.w[2]) * d.L;
  double ux = 0.0, uy = 0.0, uz = 1.0;
  for (int p = 0; p < N; ++p) {
    if (p == 1) {
      w = rng_draw(d, (uint64_t)c * N + p, t, ST_WALK);
      const double z = 2.0 * u01(w.w[0]) - 1.0;
      const double ph = 6.283185307179586 * u01(w.w[1]);
      const double s = sqrt(1.0 - z * z);
      ux = s * cos(ph); uy = s * sin(ph); uz = z;
    } else if (p > 1) {
      w = rng_draw(d, (uint64_t)c * N + p, t, ST_WALK);
      const double ph = 6.283185307179586 * u01(w.w[0]);
      const double ax = fabs(ux), ay = fabs(uy), az = fabs(uz);
      double vx, vy, vz;  // a x u
      if (ax <= ay && ax <= az) { vx = 0.0; vy = -uz; vz = uy; }
      else if (ay <= az) { vx = uz; vy = 0.0; vz = -ux; }
      else { vx = -uy; vy = ux; vz = 0.0; }
      const double vn = sqrt(vx * vx + vy * vy + vz * vz);
      const double e1x = vx / vn, e1y = vy / vn, e1z = vz / vn;
      const double e2x = uy * e1z - uz * e1y, e2y = uz * e1x - ux * e1z, e2z = ux * e1y - uy * e1x;
      const double cp = cos(ph), sp = sin(ph);
      const double nx = ct * ux + st * (cp * e1x + sp * e2x);
      const double ny = ct * uy + st * (cp * e1y + sp * e2y);
      const double nz = ct * uz + st * (cp * e1z + sp * e2z);
      const double nn = sqrt(nx * nx + ny * ny + nz * nz);
      ux = nx / nn; uy = ny / nn; uz = nz / nn;
    }
    if (p > 0) { px = px + l0 * ux; py = py + l0 * uy; pz = pz + l0 * uz; }
    const int g = d.off + c * N + p;
    x[g] = wrap_box(px, d.L);
    x[NP + g] = wrap_box(py, d.L);
    x[2 * NP + g] = wrap_box(pz, d.L);
  }
}

// Maxwell-Boltzmann velocities at T (mean removed by k_remove_mean)
__global__ __launch_bounds__(256) void k_velocities(const MeltDesc* __restrict__ md, const int* __restrict__ blk_melt,
                                                    const int* __restrict__ blk_base, int NP, double* __restrict__ v) {
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int k = __builtin_amdgcn_readfirstlane(blk_melt[lb]);
  const MeltDesc& d = md[k];
  const int li = blk_base[lb] + (int)threadIdx.x;
  if (li >= d.Nm) return;
  const int g = d.off + li;
  const U64x4 w = rng_draw(d, (uint64_t)li, 0, ST_VEL);
  double z0, z1, z2, z3;
  gauss2(w.w[0], w.w[1], z0, z1);
  gauss2(w.w[2], w.w[3], z2, z3);
  const double s = sqrt(d.T);
  v[g] = s * z0; v[NP + g] = s * z1; v[2 * NP + g] = s * z2;
}

// fixed-order block sum (strided partial sums, then a tree): deterministic
template <int NT>
__device__ double block_sum(double v, double* s) {
  s[threadIdx.x] = v;
  __syncthreads();
  for (int o = NT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  const double r = s[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(256) void k_remove_mean(const MeltDesc* __restrict__ md, int NP, double* __restrict__ v) {
  __shared__ double s[256];
  const MeltDesc& d = md[blockIdx.x];
  for (int c = 0; c < 3; ++c) {
    double acc = 0.0;
    for (int i = threadIdx.x; i < d.Nm; i += 256) acc += v[c * NP + d.off + i];
    const double mean = block_sum<256>(acc, s) / d.Nm;
    for (int i = threadIdx.x; i < d.Nm; i += 256) v[c * NP + d.off + i] -= mean;
  }
}

// {U_pair, U_bond, U_ang, K} of 256 monomers, then of each melt from its blocks' sums (both in a
// fixed order).  One workgroup per melt summing everything waited on memory at every turn: 1650 us
// at 400,000 monomers against 13 us for the two launches.  (A melt's first block stands in its descriptor:
// counted up from the first melt by every workgroup, the energies of 2,048 melts of 200 monomers took 692 us
// against 293.)
__global__ __launch_bounds__(256) void k_reduce_blocks(const MeltDesc* __restrict__ md, const int* __restrict__ blk_melt,
                                                       const int* __restrict__ blk_base, int NP,
                                                       const double* __restrict__ outE, const double* __restrict__ v,
                                                       double4* __restrict__ part) {
  __shared__ double s[4][4];
  const MeltDesc& d = md[blk_melt[blockIdx.x]];
  const int li = blk_base[blockIdx.x] + (int)threadIdx.x;
  double e[4] = {0.0, 0.0, 0.0, 0.0};
  if (li < d.Nm) {
    const int g = d.off + li;
#pragma unroll
    for (int c = 0; c < 3; ++c) e[c] = outE[(size_t)c * NP + g];
    const double vx = v[g], vy = v[NP + g], vz = v[2 * NP + g];
    e[3] = 0.5 * (vx * vx + vy * vy + vz * vz);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) e[c] += __shfl_down(e[c], o, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6][c] = e[c];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double r[4];
    for (int c = 0; c < 4; ++c) r[c] = ((s[0][c] + s[1][c]) + s[2][c]) + s[3][c];
    part[blockIdx.x] = make_double4(r[0], r[1], r[2], r[3]);
  }
}
__global__ __launch_bounds__(256) void k_reduce_melt(const MeltDesc* __restrict__ md, const double4* __restrict__ part,
                                                     double* __restrict__ out4) {
  __shared__ double s[256];
  const int b0 = md[blockIdx.x].eblk_off, b1 = b0 + (md[blockIdx.x].Nm + 255) / 256;
  double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
  for (int i = b0 + (int)threadIdx.x; i < b1; i += 256) {
    const double4 p = part[i];
    acc.x += p.x; acc.y += p.y; acc.z += p.z; acc.w += p.w;
  }
  const double e[4] = {acc.x, acc.y, acc.z, acc.w};
  for (int c = 0; c < 4; ++c) {
    const double r = block_sum<256>(e[c], s);
    if (threadIdx.x == 0) out4[4 * blockIdx.x + c] = r;
  }
}

// Per chain of melt k: prefix sums s_p of minimum-image bond vectors (FP64) and the sum of
// its bond lengths.  spre is [M*N][3] local to the melt.  One workgroup per chain: 256 bonds at a
// time are gathered by as many threads, and four of them add one column each along the chain (the
// sums keep the chain's order).  A thread per chain paid the gathers' latency once per bond
// (252 us for 1000 chains of 400 beads against 16 us).
constexpr int PRE_BLOCK = 256;
__global__ __launch_bounds__(PRE_BLOCK) void k_prefix(const MeltDesc* __restrict__ md, int k, int NP,
                                                      const double* __restrict__ x, const int* __restrict__ chain,
                                                      double* __restrict__ spre, double* __restrict__ blen) {
  __shared__ double s[4][PRE_BLOCK];  // bond vectors, then their running sums; bond lengths
  const MeltDesc& d = md[k];
  const int c = blockIdx.x, N = d.N, t = threadIdx.x;
  const int* __restrict__ row = chain + d.off + c * N;
  double* __restrict__ out = spre + 3 * (size_t)c * N;
  if (t < 3) out[t] = 0.0;
  double run = 0.0;  // threads 0-3: the sum so far of column t
  for (int p0 = 1; p0 < N; p0 += PRE_BLOCK) {
    const int p = p0 + t, n = min(PRE_BLOCK, N - p0);
    if (t < n) {
      const int a = row[p - 1], b = row[p];
      const double dx = min_image(x[b] - x[a], d.L), dy = min_image(x[NP + b] - x[NP + a], d.L),
                   dz = min_image(x[2 * NP + b] - x[2 * NP + a], d.L);
      s[0][t] = dx;
      s[1][t] = dy;
      s[2][t] = dz;
      s[3][t] = sqrt(dx * dx + dy * dy + dz * dz);
    }
    __syncthreads();
    if (t < 4) {
#pragma unroll 8
      for (int q = 0; q < n; ++q) {
        run += s[t][q];
        s[t][q] = run;
      }
    }
    __syncthreads();
    for (int e = t; e < 3 * n; e += PRE_BLOCK) out[3 * p0 + e] = s[e % 3][e / 3];
    __syncthreads();
  }
  if (t == 3) blen[c] = run;
}

// block per chemical distance n (1..N-1): sum over chains and i of |s_{i+n} - s_i|^2.  Bound by
// the reads of s from L2 (48 bytes a term); R2_U terms of a thread are requested together and added in
// their order.
constexpr int R2_U = 4;
__global__ __launch_bounds__(256) void k_r2(int M, int N, const double* __restrict__ spre, double* __restrict__ r2sum) {
  __shared__ double s[256];
  const int n = blockIdx.x + 1;
  double acc = 0.0;
  const int per = N - n;
  const long total = (long)M * per;
  // (chain c, bead i) of term t, kept up by steps of 256 terms
  int c = (int)threadIdx.x / per, i = (int)threadIdx.x - c * per;
  const int dc = 256 / per, di = 256 - dc * per;
  for (long t = threadIdx.x; t < total; t += 256 * R2_U) {
    double v[R2_U];
#pragma unroll
    for (int q = 0; q < R2_U; ++q) {
      const bool on = t + 256 * q < total;
      const double* a = spre + 3 * (on ? (long)c * N + i : 0l);
      const double* b = a + 3 * n;
      const double dx = b[0] - a[0], dy = b[1] - a[1], dz = b[2] - a[2];
      v[q] = on ? dx * dx + dy * dy + dz * dz : 0.0;
      c += dc;
      i += di;
      if (i >= per) { i -= per; ++c; }
    }
#pragma unroll
    for (int q = 0; q < R2_U; ++q) acc += v[q];
  }
  const double r = block_sum<256>(acc, s);
  if (threadIdx.x == 0) r2sum[n - 1] = r;
}

// ---------------------------------------------------------------------------------------
// Structure observables of the appendices: g(r) (App. A) from a histogram of pair distances,
// S(q) (App. A) on the box's reciprocal lattice, and the monomer mean squared displacement
// (App. B) from displacements accumulated between runs of steps.
// ---------------------------------------------------------------------------------------

// Ordered pairs i != j of melt k with minimum-image distance r < r_max, counted into bins of
// width r_max / nbins.  Counts are integers, so the histogram is exact.
//
// A workgroup takes the monomers of PH_B^3 MD cells against those of the cells within R of them
// (2 R + 1 <= nc), staged in LDS up to 1,536 at a time (the cells of a batch are cut where that is
// reached): every thread holds two of these and runs over the home monomers.  Testing all pairs of a tile costs three times the distances that a
// search cell by cell would need, but no gather, cell arithmetic or division per pair.  Bound by
// latency at two wavefronts a SIMD (62 KB of LDS a workgroup): half of their time they wait for LDS, the
// coordinates and the bins' atomics (some lane of a wavefront nearly always has a hit), VALU issue takes
// 46%.  400,000 monomers to 3 sigma: 5.8 ms (a thread per monomer, gathers from L2) against 0.9 ms; 4,000 at
// density 1.2 0.78 against 0.24 (1.37 when a batch past the LDS was cut into pieces of 32 cells).
constexpr int PH_B = 4;
constexpr int PH_CELLS = 1024;  // cells per staged batch
constexpr int PH_CAP = 1536;    // staged monomers
constexpr int PH_HOMES = 256;   // home monomers per round
static_assert(CELL_CAP <= PH_CAP, "a cell always fits");

__global__ __launch_bounds__(256) void k_pair_hist(const MeltDesc* __restrict__ md, int k, int NP,
                                                   const double* __restrict__ x, const int* __restrict__ cnt,
                                                   const int* __restrict__ bucket, double r_max, int nbins, int R,
                                                   unsigned long long* __restrict__ hist) {
  extern __shared__ unsigned int s_hist[];
  __shared__ double s_p[3][PH_CAP], s_h[3][PH_HOMES];
  __shared__ int s_id[PH_CAP];              // place of a staged monomer in the buckets, then its slot
  __shared__ int s_hid[PH_B * PH_B * PH_B * CELL_CAP];
  __shared__ int s_pre[PH_CELLS + 1];       // first staged monomer of each cell of the batch
  __shared__ int s_w[4], s_nh;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  for (int b = t; b < nbins; b += 256) s_hist[b] = 0;
  const MeltDesc& d = md[k];
  const int nc = d.nc, nb = (nc + PH_B - 1) / PH_B;
  const int x0 = (int)(blockIdx.x % nb) * PH_B, y0 = (int)(blockIdx.x / nb % nb) * PH_B,
            z0 = (int)(blockIdx.x / (nb * nb)) * PH_B;
  const int bx = min(PH_B, nc - x0), by = min(PH_B, nc - y0), bz = min(PH_B, nc - z0);
  // staged cells per side: every cell once when the halo reaches round the box
  const int wx = min(bx + 2 * R, nc), wy = min(by + 2 * R, nc), wz = min(bz + 2 * R, nc);
  const int ncell = wx * wy * wz;
  const bool interior = x0 >= R && y0 >= R && z0 >= R && x0 + bx + R <= nc && y0 + by + R <= nc && z0 + bz + R <= nc;
  const double L = d.L, hL = 0.5 * d.L;
  const double dr = r_max / nbins, r2cut = r_max * r_max * (1.0 + 1e-9);
  const float scale = (float)(nbins / r_max);
  // home monomers
  if (wv == 0) {
    const int hx = lane % PH_B, hy = lane / PH_B % PH_B, hz = lane / (PH_B * PH_B);
    const bool on = hx < bx && hy < by && hz < bz;
    const int c = d.cell_off + ((z0 + hz) * nc + y0 + hy) * nc + x0 + hx;
    const int n = on ? min(cnt[c], CELL_CAP) : 0;
    int incl = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    for (int j = 0; j < n; ++j) s_hid[incl - n + j] = bucket[(size_t)c * CELL_CAP + j];
    if (lane == 63) s_nh = incl;
  }
  __syncthreads();
  const int nh_all = s_nh;
  for (int h0 = 0; h0 < nh_all; h0 += PH_HOMES) {
    const int nh = min(PH_HOMES, nh_all - h0);
    if (t < nh) {
      const int g = s_hid[h0 + t];
#pragma unroll
      for (int q = 0; q < 3; ++q) s_h[q][t] = x[(size_t)q * NP + g];
    }
    for (int c0 = 0; c0 < ncell; c0 += PH_CELLS) {
      const int nb_cells = min(PH_CELLS, ncell - c0);
      // counts of the batch's cells, four neighbouring ones a thread, and their prefix
      int cell[PH_CELLS / 256], n[PH_CELLS / 256], sum = 0;
#pragma unroll
      for (int q = 0; q < PH_CELLS / 256; ++q) {
        const int e = c0 + t * (PH_CELLS / 256) + q;
        int ax = x0 - (wx < nc ? R : 0) + e % wx, ay = y0 - (wy < nc ? R : 0) + e / wx % wy,
            az = z0 - (wz < nc ? R : 0) + e / (wx * wy);
        ax = ax < 0 ? ax + nc : (ax >= nc ? ax - nc : ax);
        ay = ay < 0 ? ay + nc : (ay >= nc ? ay - nc : ay);
        az = az < 0 ? az + nc : (az >= nc ? az - nc : az);
        const bool on = e < ncell;
        cell[q] = on ? d.cell_off + (az * nc + ay) * nc + ax : d.cell_off;
        n[q] = on ? min(cnt[cell[q]], CELL_CAP) : 0;
      }
#pragma unroll
      for (int q = 0; q < PH_CELLS / 256; ++q) sum += n[q];
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      __syncthreads();  // (the last batch's prefix and wavefront sums have been read)
      if (lane == 63) s_w[wv] = incl;
      __syncthreads();
      int at = incl - sum;
      for (int w = 0; w < wv; ++w) at += s_w[w];
      const int at0 = at;
#pragma unroll
      for (int q = 0; q < PH_CELLS / 256; ++q) {
        s_pre[t * (PH_CELLS / 256) + q] = at;
        at += n[q];
      }
      if (t == 255) s_pre[PH_CELLS] = at;
      __syncthreads();
      const int all = s_pre[PH_CELLS];
      for (int p0 = 0, p1; p0 < nb_cells; p0 = p1) {
        // cells [p0, p1): as many as fit
        const int first = s_pre[p0];
        p1 = PH_CELLS;
        if (all - first > PH_CAP) {
          int lo = p0 + 1;
          while (p1 - lo > 1) {
            const int mid = (lo + p1) >> 1;
            if (s_pre[mid] - first <= PH_CAP) lo = mid;
            else p1 = mid;
          }
          p1 = lo;
        }
        const int m = s_pre[p1] - first;
        // where each staged monomer sits in the buckets, then its position
        int a = at0 - first;
#pragma unroll
        for (int q = 0; q < PH_CELLS / 256; ++q) {
          const int c = t * (PH_CELLS / 256) + q;
          if (c >= p0 && c < p1)
            for (int j = 0; j < n[q]; ++j) s_id[a + j] = cell[q] * CELL_CAP + j;
          a += n[q];
        }
        __syncthreads();
        for (int j = t; j < m; j += 256) {
          const int g = bucket[s_id[j]];
          s_id[j] = g;
#pragma unroll
          for (int q = 0; q < 3; ++q) s_p[q][j] = x[(size_t)q * NP + g];
        }
        __syncthreads();
        for (int j0 = t; j0 < m; j0 += 512) {
          double px[2], py[2], pz[2];
          int id[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int j = j0 + 256 * q;
            const bool on = j < m;
            px[q] = on ? s_p[0][j] : 1e30;  // (no image of it comes near)
            py[q] = on ? s_p[1][j] : 1e30;
            pz[q] = on ? s_p[2][j] : 1e30;
            id[q] = on ? s_id[j] : -1;
          }
          for (int h = 0; h < nh; ++h) {
            const double xi = s_h[0][h], yi = s_h[1][h], zi = s_h[2][h];
            const int g = s_hid[h0 + h];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              double dx = px[q] - xi, dy = py[q] - yi, dz = pz[q] - zi;
              // nearest image: of a pair within r_max the same one that rounding d / L would pick
              // (r_max stays half a cell below L / 2), without the division
              if (!interior) {
                dx = dx > hL ? dx - L : (dx < -hL ? dx + L : dx);
                dy = dy > hL ? dy - L : (dy < -hL ? dy + L : dy);
                dz = dz > hL ? dz - L : (dz < -hL ? dz + L : dz);
              }
              const double r2 = dx * dx + dy * dy + dz * dz;
              if (r2 < r2cut && id[q] != g) {
                // the bin from an FP32 distance, unless that lies too near a bin's edge to tell
                const float rf = __builtin_amdgcn_sqrtf((float)r2) * scale;
                int b = (int)rf;
                const float lo = rf - (float)b, eps = rf * 1e-6f + 1e-6f;
                if (lo < eps || 1.0f - lo < eps) {
                  const double r = sqrt(r2);
                  b = r < r_max ? (int)(r / dr) : nbins;
                }
                if (b < nbins) atomicAdd(&s_hist[b], 1u);
              }
            }
          }
        }
        __syncthreads();
      }
    }
  }
  __syncthreads();
  for (int b = t; b < nbins; b += 256)
    if (s_hist[b]) atomicAdd(&hist[b], (unsigned long long)s_hist[b]);
}

// S(q) = |sum_j exp(i q . x_j)|^2 / N_m for q = (2 pi / L) nvec[3 q ..].
//
// A lane per q and a run of monomers per workgroup (one wavefront): the coordinates are the same for
// all lanes and come through scalar loads, so that a phasor costs arithmetic alone.  The phase is
// taken in turns, w in [-1/2, 1/2] after rounding, and a quarter of it through the Taylor series of
// sine and cosine (|pi w / 2| <= pi / 4: terms to the 16th power, the next below 5e-17), doubled
// twice: 29 FP64 instructions.  Bound by their issue (the VALU is busy 75% of the time).  400,000 monomers x
// 5,600 vectors: 9.6 ms (a workgroup per q with full-range sin and cos, 54 GB of coordinates read) against
// 2.2 ms.
struct TurnSeries {
  double s[8], c[9];
};
constexpr TurnSeries turn_series() {
  TurnSeries t{};
  const double h = 1.5707963267948966;
  double p = 1.0, f = 1.0;  // h^m, m!
  for (int m = 0; m <= 16; ++m) {
    if (m > 0) { p *= h; f *= m; }
    const double v = ((m / 2) % 2 ? -1.0 : 1.0) * p / f;
    if (m % 2) t.s[m / 2] = v;
    else t.c[m / 2] = v;
  }
  return t;
}

__global__ __launch_bounds__(64) void k_structure_part(const MeltDesc* __restrict__ md, int k, int NP,
                                                       const double* __restrict__ x, const int* __restrict__ nvec,
                                                       int64_t nq, int run, double2* __restrict__ part) {
  constexpr TurnSeries T = turn_series();
  const MeltDesc& d = md[k];
  const int64_t q = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int64_t qc = q < nq ? q : nq - 1;
  const double f = 1.0 / d.L;
  const double kx = f * nvec[3 * qc], ky = f * nvec[3 * qc + 1], kz = f * nvec[3 * qc + 2];
  const int i0 = (int)blockIdx.y * run, i1 = min(d.Nm, i0 + run);
  const double* __restrict__ xs = x + d.off;
  double cs = 0.0, sn = 0.0;
#pragma unroll 2
  for (int i = i0; i < i1; ++i) {
    const double t = __builtin_fma(kz, xs[2 * (size_t)NP + i], __builtin_fma(ky, xs[(size_t)NP + i], kx * xs[i]));
    const double w = t - rint(t), w2 = w * w;
    double a = T.s[7], b = T.c[8];
#pragma unroll
    for (int m = 6; m >= 0; --m) a = __builtin_fma(a, w2, T.s[m]);
#pragma unroll
    for (int m = 7; m >= 0; --m) b = __builtin_fma(b, w2, T.c[m]);
    a *= w;  // sine and cosine of a quarter of the angle
    const double a2 = a + a, s1 = a2 * b, c1 = __builtin_fma(-a2, a, 1.0), s2 = s1 + s1;
    sn = __builtin_fma(s2, c1, sn);
    cs += __builtin_fma(-s2, s1, 1.0);
  }
  if (q < nq) part[(size_t)blockIdx.y * nq + q] = make_double2(cs, sn);
}
// one wavefront per q adds the runs' sums (fixed order)
__global__ __launch_bounds__(64) void k_structure_sum(const MeltDesc* __restrict__ md, int k, int64_t nq, int nrun,
                                                      const double2* __restrict__ part, double* __restrict__ S) {
  const int64_t q = blockIdx.x;
  double cs = 0.0, sn = 0.0;
  for (int r = threadIdx.x; r < nrun; r += 64) {
    const double2 p = part[(size_t)r * nq + q];
    cs += p.x;
    sn += p.y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    cs += __shfl_down(cs, o, 64);
    sn += __shfl_down(sn, o, 64);
  }
  if (threadIdx.x == 0) S[q] = (cs * cs + sn * sn) / md[k].Nm;
}

// displacement tracking by monomer id: reset (last = x, acc = 0) or update (acc += the
// minimum-image step since last, last = x) for melt `only` (< 0: every melt)
__global__ __launch_bounds__(256) void k_msd_track(const MeltDesc* __restrict__ md, const int* __restrict__ blk_melt,
                                                   const int* __restrict__ blk_base, int NP,
                                                   const double* __restrict__ x, const int* __restrict__ mono,
                                                   double* __restrict__ last, double* __restrict__ acc, int reset,
                                                   int only) {
  const int k = blk_melt[blockIdx.x];
  if (only >= 0 && k != only) return;
  const MeltDesc& d = md[k];
  const int li = blk_base[blockIdx.x] + (int)threadIdx.x;
  if (li >= d.Nm) return;
  const int g = d.off + li, id = d.off + mono[g];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double xn = x[(size_t)c * NP + g];
    if (reset) acc[(size_t)c * NP + id] = 0.0;
    else acc[(size_t)c * NP + id] += min_image(xn - last[(size_t)c * NP + id], d.L);
    last[(size_t)c * NP + id] = xn;
  }
}

// mean over melt k's monomers of |acc|^2 (fixed-order block sum)
__global__ __launch_bounds__(256) void k_msd_reduce(const MeltDesc* __restrict__ md, int k, int NP,
                                                    const double* __restrict__ acc, double* __restrict__ out) {
  __shared__ double s[256];
  const MeltDesc& d = md[k];
  double v = 0.0;
  for (int li = threadIdx.x; li < d.Nm; li += blockDim.x) {
    const int id = d.off + li;
    for (int c = 0; c < 3; ++c) v += acc[(size_t)c * NP + id] * acc[(size_t)c * NP + id];
  }
  v = block_sum<256>(v, s);
  if (threadIdx.x == 0) out[0] = v / d.Nm;
}

void launch_pair_hist(const MeltDesc* md, int k, int nc, int NP, const double* x, const int* cnt, const int* bucket,
                      double r_max, int nbins, int R, unsigned long long* hist, hipStream_t s) {
  const int nb = (nc + PH_B - 1) / PH_B;
  hipLaunchKernelGGL(k_pair_hist, dim3(nb * nb * nb), dim3(256), sizeof(unsigned int) * nbins, s, md, k, NP, x, cnt,
                     bucket, r_max, nbins, R, hist);
}
// runs of monomers, so that the wavefronts (64 vectors each) number about 8192; the vectors' partial
// sums need runs x nq pairs of doubles
int structure_runs(int Nm, int64_t nq) {
  const int64_t qb = (nq + 63) / 64, want = 8192 / qb, most = ((int64_t)Nm + 63) / 64;
  return (int)(want < 1 ? 1 : want > most ? most : want);
}
void launch_structure_factor(const MeltDesc* md, int k, int Nm, int NP, const double* x, const int* nvec, int64_t nq,
                             double2* part, double* S, hipStream_t s) {
  if (nq <= 0) return;
  const int runs = structure_runs(Nm, nq), run = (Nm + runs - 1) / runs;
  hipLaunchKernelGGL(k_structure_part, dim3((unsigned)((nq + 63) / 64), runs), dim3(64), 0, s, md, k, NP, x, nvec, nq,
                     run, part);
  hipLaunchKernelGGL(k_structure_sum, dim3((unsigned)nq), dim3(64), 0, s, md, k, nq, runs, part, S);
}
void launch_msd_track(const MeltDesc* md, const BlockMap& pm, int NP, const double* x, const int* mono, double* last,
                      double* acc, int reset, int only, hipStream_t s) {
  hipLaunchKernelGGL(k_msd_track, dim3(pm.nblk), dim3(256), 0, s, md, pm.melt, pm.base, NP, x, mono, last, acc,
                     reset, only);
}
void launch_msd_reduce(const MeltDesc* md, int k, int NP, const double* acc, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_msd_reduce, dim3(1), dim3(256), 0, s, md, k, NP, acc, out);
}

void launch_random_walks(const MeltDesc* md, int nm, int max_M, int NP, double* x, int* chain, int* loc,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_random_walks, dim3((max_M + 63) / 64, nm), dim3(64), 0, s, md, NP, x, chain, loc);
}
void launch_fr_chains(const MeltDesc* md, int nm, int max_M, int NP, double* x, const int* tries, hipStream_t s) {
  hipLaunchKernelGGL(k_fr_chains, dim3((max_M + 63) / 64, nm), dim3(64), 0, s, md, NP, x, tries);
}
void launch_velocities(const MeltDesc* md, const BlockMap& pm, int NP, double* v, hipStream_t s) {
  hipLaunchKernelGGL(k_velocities, dim3(pm.nblk), dim3(256), 0, s, md, pm.melt, pm.base, NP, v);
}
void launch_remove_mean(const MeltDesc* md, int nm, int NP, double* v, hipStream_t s) {
  hipLaunchKernelGGL(k_remove_mean, dim3(nm), dim3(256), 0, s, md, NP, v);
}
void launch_reduce_melt(const MeltDesc* md, int nm, const BlockMap& pm, int NP, const double* outE, const double* v,
                        double4* part, double* out4, hipStream_t s) {
  if (pm.nblk == nm) part = (double4*)out4;  // melts of one block: its sums are the melt's
  hipLaunchKernelGGL(k_reduce_blocks, dim3(pm.nblk), dim3(256), 0, s, md, pm.melt, pm.base, NP, outE, v, part);
  if (pm.nblk != nm) hipLaunchKernelGGL(k_reduce_melt, dim3(nm), dim3(256), 0, s, md, part, out4);
}
void launch_prefix(const MeltDesc* md, int k, int M, int NP, const double* x, const int* chain, double* spre,
                   double* blen, hipStream_t s) {
  hipLaunchKernelGGL(k_prefix, dim3(M), dim3(PRE_BLOCK), 0, s, md, k, NP, x, chain, spre, blen);
}
void launch_r2(int M, int N, const double* spre, double* r2sum, hipStream_t s) {
  if (N > 1) hipLaunchKernelGGL(k_r2, dim3(N - 1), dim3(256), 0, s, M, N, spre, r2sum);
}

}  // namespace kgdb
