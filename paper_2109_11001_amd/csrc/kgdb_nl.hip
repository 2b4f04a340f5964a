// Production MD step on gfx950: Verlet neighbour lists over a tile-sorted storage order,
// with every workgroup's neighbourhood staged in LDS.
//
// Geometry.  The list grid has cells of edge >= r_list = r_c + skin.  Its cells are grouped
// into tiles of nl_S x nl_Sy cells of one z-plane; a tile's cells are numbered row by row, and
// the tiles of a plane, then the planes, follow one another ("sorted cell index").
//
// Rebuild (every K steps).  (1) Binning: each monomer's list cell, counted per cell and per
// tile (wave-aggregated atomics) with its storage slot, id and place in the cell (16-bit units)
// appended to the cell's bucket; the step before a rebuild bins the positions it has just
// written.  (2) A scan of the tile counts gives each tile's first storage slot.  (3) One
// workgroup per tile stages the members of the 3 (nl_S + 2)(nl_Sy + 2) cells around the tile
// in LDS, ordered by cell and by monomer id within
// a cell, at their places relative to the tile (so that periodic images need no
// offsets); it moves its own members to their new storage slots (cell order, monomer id
// within a cell: a canonical order that does not depend on the history of the run), records
// each one's position relative to its cell (its reference cell until the next rebuild), and
// lists for each one the staged members within r_list as 16-bit indices into the stage.
// (4) The chain table, chain positions and bonded-neighbour slots are carried over to the new
// slots.
//
// Step.  One workgroup per tile stages the current positions of the same neighbourhood (the
// storage of a cell is contiguous, so the stage is a set of contiguous runs), then each thread
// takes one home monomer: the truncated MLJ^n pair force over its list (LDS reads), the FENE
// and angle forces from its four chain neighbours' relative positions and cells, the Langevin
// noise, and the velocity-Verlet update.  List validity: each step records the largest
// displacement of its monomers (per melt); a list is valid while the sum of those maxima since
// its rebuild is at most skin/2, which bounds every monomer's displacement.  A run that exceeds
// it is redone by the host with more frequent rebuilds.
#include <hip/hip_ext.h>

#include <type_traits>

#include "kgdb_dev.h"
#include "kgdb_kernels.h"
#include "kgdb_list_run.h"

namespace kgdb {

__device__ __forceinline__ int pack_cell(int cx, int cy, int cz) { return cx | (cy << 10) | (cz << 20); }

// Position of a monomer relative to its reference cell (the list-grid cell it was sorted into
// at the last rebuild), and relative to a tile's frame once staged.  With FP32 forces it is
// kept in fixed point, 2^24 units per cell edge (about 1e-7 sigma per unit): displacements
// between two monomers are then exact integer differences, however far the frame extends
// (a tile and its halo span up to ~66 cells), and only the displacement itself is rounded to
// FP32.  With FP64 forces it is kept in FP64.  The fourth word holds the packed reference cell.
template <typename R> struct Rel;
template <> struct Rel<float> {
  using T = int4;
  static constexpr double UNITS = 16777216.0;  // per cell edge
  __device__ static T make(double dx, double dy, double dz, int pc, double hl) {
    const double s = UNITS / hl;
    return make_int4((int)rint(dx * s), (int)rint(dy * s), (int)rint(dz * s), pc);
  }
  __device__ static T shift(T p, int ox, int oy, int oz) {
    p.x += ox << 24;
    p.y += oy << 24;
    p.z += oz << 24;
    return p;
  }
  // a - b in units of the fixed point (the caller scales by the unit length)
  __device__ static void diff(const T& a, const T& b, float& dx, float& dy, float& dz) {
    dx = (float)(a.x - b.x);
    dy = (float)(a.y - b.y);
    dz = (float)(a.z - b.z);
  }
  __device__ static int cell(const T& p) { return p.w; }
  __host__ __device__ static double unit(double hl) { return hl / UNITS; }
  // a - b for a monomer a whose reference cell lies (ox, oy, oz) cells from b's (each in
  // (-nc/2, nc/2]), as the nearest periodic image, in units
  __device__ static void image_diff(const T& a, const T& b, int ox, int oy, int oz, int nc, double, float& dx,
                                    float& dy, float& dz) {
    int d[3] = {a.x - b.x + (ox << 24), a.y - b.y + (oy << 24), a.z - b.z + (oz << 24)};
    if (nc < 128) {  // boxes of fewer than 128 cells: the displacement may be nearer through the other image
      const int Lu = nc << 24, hLu = Lu >> 1;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        d[q] -= d[q] > hLu ? Lu : 0;
        d[q] += d[q] < -hLu ? Lu : 0;
      }
    }
    dx = (float)d[0];
    dy = (float)d[1];
    dz = (float)d[2];
  }
};
template <> struct Rel<double> {
  struct alignas(32) T { double x, y, z, w; };
  __device__ static T make(double dx, double dy, double dz, int pc, double) { return T{dx, dy, dz, (double)pc}; }
  __device__ static T shift(T p, int ox, int oy, int oz, double hl) {
    p.x += ox * hl;
    p.y += oy * hl;
    p.z += oz * hl;
    return p;
  }
  __device__ static void diff(const T& a, const T& b, double& dx, double& dy, double& dz) {
    dx = a.x - b.x;
    dy = a.y - b.y;
    dz = a.z - b.z;
  }
  __device__ static int cell(const T& p) { return (int)p.w; }
  __host__ __device__ static double unit(double) { return 1.0; }
  __device__ static void image_diff(const T& a, const T& b, int ox, int oy, int oz, int nc, double hl, double& dx,
                                    double& dy, double& dz) {
    const double L = nc * hl, iL = 1.0 / L;
    dx = a.x - b.x + ox * hl;
    dy = a.y - b.y + oy * hl;
    dz = a.z - b.z + oz * hl;
    dx -= L * rint(dx * iL);
    dy -= L * rint(dy * iL);
    dz -= L * rint(dz * iL);
  }
};
// a staged position no home monomer's cutoff reaches: 2^30 units (64 cell edges) above the
// frame's z planes in the mixed path, 10^6 sigma in FP64 (every home lies within a cell of z = 0)
template <typename R>
__device__ __forceinline__ typename Rel<R>::T stage_sentinel() {
  if constexpr (sizeof(R) == 4) return make_int4(0, 0, 1 << 30, 0);
  else return typename Rel<double>::T{0.0, 0.0, 1.0e6, 0.0};
}
template <typename R>
__device__ __forceinline__ typename Rel<R>::T rel_shift(const typename Rel<R>::T& p, int ox, int oy, int oz, double hl) {
  if constexpr (sizeof(R) == 4) {
    (void)hl;
    return Rel<float>::shift(p, ox, oy, oz);
  } else {
    return Rel<double>::shift(p, ox, oy, oz, hl);
  }
}

// ---------------------------------------------------------------------------------------
// tile geometry
// ---------------------------------------------------------------------------------------
struct TileGeo {
  int x0, y0, cz, nh, nhy;
};
__device__ __forceinline__ TileGeo tile_geo(const MeltDesc& d, int t) {
  const int seg = t % d.nl_nseg;
  t /= d.nl_nseg;
  const int yb = t % d.nl_nyb;
  TileGeo g;
  g.cz = t / d.nl_nyb;
  g.x0 = seg * d.nl_S;
  g.y0 = yb * d.nl_Sy;
  g.nh = min(d.nl_S, d.ncl - g.x0);
  g.nhy = min(d.nl_Sy, d.ncl - g.y0);
  return g;
}
// sorted index of list-grid cell (cx, cy, cz) of melt d (global over the batch) and its tile
__device__ __forceinline__ int sorted_cell(const MeltDesc& d, int cx, int cy, int cz, int* tile) {
  const int nc = d.ncl;
  const int xb = cx / d.nl_S, yb = cy / d.nl_Sy;
  const int x0 = xb * d.nl_S, y0 = yb * d.nl_Sy;
  const int nh = min(d.nl_S, nc - x0), nhy = min(d.nl_Sy, nc - y0);
  if (tile) *tile = d.tile_off + (cz * d.nl_nyb + yb) * d.nl_nseg + xb;
  return d.celll_off + cz * nc * nc + y0 * nc + x0 * nhy + (cy - y0) * nh + (cx - x0);
}
__device__ __forceinline__ int wrapc(int c, int nc) { return c < 0 ? c + nc : (c >= nc ? c - nc : c); }

// staged cell t of a tile: (x index i, y index yy, z index zz) in a frame of W x WY x 3 cells
// whose cell (1, 1, 1) is the tile's first home cell; its grid cell and sorted index
struct StagedCell {
  int i, yy, zz, ax, ay, az;
};
__device__ __forceinline__ StagedCell staged_cell(const MeltDesc& d, const TileGeo& tg, int W, int WY, int t) {
  StagedCell s;
  const int row = t / W;
  s.i = t - row * W;
  s.zz = row / WY;
  s.yy = row - s.zz * WY;
  const int nc = d.ncl;
  s.ax = wrapc(tg.x0 - 1 + s.i, nc);
  s.ay = wrapc(tg.y0 - 1 + s.yy, nc);
  s.az = wrapc(tg.cz - 1 + s.zz, nc);
  return s;
}

// ---------------------------------------------------------------------------------------
// binning: runs of lanes with the same cell (resp. tile) take their slots with one atomic
// ---------------------------------------------------------------------------------------
// first lane of the run of equal keys that this lane belongs to, its length, and the base
// returned by one atomicAdd per run; inactive lanes (and key < 0) end runs
__device__ __forceinline__ int run_add(int* ctr, int key) {
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(key, 1, 64);
  const uint64_t active = __ballot(1);
  const bool prev_on = lane > 0 && ((active >> (lane - 1)) & 1ull);
  const uint64_t heads = __ballot(!prev_on || prev != key);
  const uint64_t upto = (2ull << lane) - 1ull;  // lanes 0 .. lane
  const int hl = 63 - __builtin_clzll(heads & upto);
  int base = 0;
  if (hl == lane && key >= 0) {
    const uint64_t after = (heads | ~active) & ~upto;
    const int next = after ? __builtin_ctzll(after) : 64;
    base = atomicAdd(&ctr[key], next - lane);
  }
  base = __shfl(base, hl, 64);
  return base + (lane - hl);
}

// A bucket entry holds all that a rebuild stages of a member: its slot, its monomer id and its place in
// the cell in units of 1 / nl_u of the cell's edge (x in the low, y in the high half of the third word).
__device__ __forceinline__ void nl_bin_one(const NlArgs& a, int k, const MeltDesc& d, int g, int mono, double x,
                                           double y, double z, bool valid) {
  int sc = -1, tile = -1;
  uint32_t oxy = 0, oz = 0;
  if (valid) {
    const int nc = d.ncl, U = d.nl_u;
    const int cx = cell_coord(x, d.cinvl, nc), cy = cell_coord(y, d.cinvl, nc), cz = cell_coord(z, d.cinvl, nc);
    sc = sorted_cell(d, cx, cy, cz, &tile);
    auto place = [&](double w, int c) {
      return (uint32_t)min(max((int)__builtin_fma(__builtin_fma(w, d.cinvl, -(double)c), (double)U, 0.5), 0), U);
    };
    oxy = place(x, cx) | (place(y, cy) << 16);
    oz = place(z, cz);
  }
  const int s = run_add(a.cnt, sc);
  (void)run_add(a.tcnt, tile);
  if (!valid) return;
  if (s < NL_CELL_CAP) a.bucket[(size_t)sc * NL_CELL_CAP + s] = make_int4(g, mono, (int)oxy, (int)oz);
  else atomicOr(&a.err[k], ERR_CELL_OVERFLOW);
}

__global__ __launch_bounds__(256) void k_nl_bin(NlArgs a) {
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int k = __builtin_amdgcn_readfirstlane(a.pblk_melt[lb]);
  const MeltDesc& d = a.md[k];
  const int li = a.pblk_base[lb] + (int)threadIdx.x;
  const bool valid = li < d.Nm;
  const int g = d.off + (valid ? li : 0);
  double x = 0, y = 0, z = 0;
  if (valid) { x = a.x[g]; y = a.x[a.NP + g]; z = a.x[2 * a.NP + g]; }
  nl_bin_one(a, k, d, g, valid ? a.mono[g] : 0, x, y, z, valid);
}

// exclusive scan of the tile counts (one workgroup, runs of 1024 with a carry)
__global__ __launch_bounds__(1024) void k_tile_scan(const int* __restrict__ tcnt, int nt, int* __restrict__ tstart) {
  __shared__ int s_w[16];
  __shared__ int s_carry;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (int b0 = 0; b0 < nt; b0 += 1024) {
    const int i = b0 + (int)threadIdx.x;
    const int v = i < nt ? tcnt[i] : 0;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    if (lane == 63) s_w[wv] = incl;
    __syncthreads();
    int off = s_carry, tot = 0;
    for (int q = 0; q < 16; ++q) { off += q < wv ? s_w[q] : 0; tot += s_w[q]; }
    if (i < nt) tstart[i] = off + incl - v;
    __syncthreads();
    if (threadIdx.x == 0) s_carry += tot;
    __syncthreads();
  }
}

// inclusive prefix of s[1..n] in place (s[0] = 0), one wavefront
__device__ __forceinline__ void wave_prefix(int* s, int n) {
  const int lane = threadIdx.x & 63;
  const int per = (n + 63) >> 6;
  int sum = 0;
  for (int q = 0; q < per; ++q) {
    const int t = lane * per + q;
    if (t < n) sum += s[t + 1];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  int acc = incl - sum;
  for (int q = 0; q < per; ++q) {
    const int t = lane * per + q;
    if (t < n) { acc += s[t + 1]; s[t + 1] = acc; }
  }
  if (lane == 0) s[0] = 0;
}

// first index t in [lo, hi) with s[t + 1] > v (s ascending; s[lo] <= v)
__device__ __forceinline__ int find_cell(const int* s, int lo, int hi, int v) {
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (s[mid] <= v) lo = mid;
    else hi = mid;
  }
  return lo;
}

constexpr int NLB_CELLS = 594;  // staged cells: 3 (nl_S + 2)(nl_Sy + 2) <= 594
constexpr int NLB_HOMES = 198;  // home cells: nl_S nl_Sy < (nl_S + 2)(nl_Sy + 2) <= 198
// batches of at most this many list tiles find a tile's first slot inside the rebuild kernel
constexpr int TILE_SUM_MAX = 4096;
// A staged cell's members are read and ranked by a group of 8 lanes, an entry a lane, in melts of many
// members a cell (nl_wide: the smallest boxes, eight a cell) by 16; a cell with more goes to a
// wavefront.  (A cell a thread touched 64 cache lines with each of its loads.)
constexpr int RB_ROW = 20;  // candidates of a row tested at once (a row holds about fifteen)
// home members of a stage of `cap`: their mean is below a third of the stage's
constexpr int RB_HOME_PAD = 64;
__host__ __device__ constexpr int rb_home_cap(int cap) { return cap / 3 + RB_HOME_PAD; }
constexpr int RB_PAD = 32;  // staged entries past the capacity (a row is read up to its 32nd candidate)

// 16-byte word q (eight 16-bit entries) of the list of the monomer in slot i
__device__ __forceinline__ size_t nl_word(int i, int q) {
  return ((size_t)(i >> 6) * (NL_CAP / 8) + (size_t)q) * 64 + (size_t)(i & 63);
}

// ---------------------------------------------------------------------------------------
// rebuild 3: per tile, stage, move the home members to their new slots, list
// ---------------------------------------------------------------------------------------
// The members of staged cell t sorted by monomer id: bucket entry of the member of rank r.
__device__ __forceinline__ int4 member_entry(const NlArgs& a, int sc, int n, int r) {
  const int4* b = a.bucket + (size_t)sc * NL_CELL_CAP;
  for (int j = 0; j < n; ++j) {
    const int4 e = b[j];
    int rank = 0;
    for (int m = 0; m < n; ++m) rank += b[m].y < e.y;
    if (rank == r) return e;
  }
  return b[0];
}

// Staged positions of a rebuild decide list membership only.  They are kept in 16 bits an axis (x in
// the low, y in the high half of the first word, z in the second), U units a cell edge, U <= 10922, so
// that members up to two cells apart differ by less than 2^15 and their squared distance fits an int:
// five integer instructions test a candidate.  Each is rounded to half a unit, so two members' distance
// is off by at most sqrt(3) units; the cutoff is taken two units further out, and the few entries that
// this adds lie outside every cutoff of the step and contribute nothing.
typedef short i16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int quant_test(uint2 p, uint2 me, int minus_r2) {  // < 0: within the cutoff
  const i16x2 xy = __builtin_bit_cast(i16x2, p.x) - __builtin_bit_cast(i16x2, me.x);
  const i16x2 z = __builtin_bit_cast(i16x2, p.y) - __builtin_bit_cast(i16x2, me.y);
  return __builtin_amdgcn_sdot2(xy, xy, __builtin_amdgcn_sdot2(z, z, minus_r2, false), false);
}

// frame position of a bucket entry of staged cell (i, yy, zz)
__device__ __forceinline__ uint2 quant_pos(int4 e, int i, int yy, int zz, int U) {
  return make_uint2((uint32_t)e.z + (uint32_t)(i * U) + ((uint32_t)(yy * U) << 16), (uint32_t)(e.w + zz * U));
}

// The list of one home monomer (staged position me, staged index tme, home cell (ih, yy) of
// the frame): staged members within r_list in the 3 x 3 rows of three cells around it.  A
// row, or a side cell of it, whose nearest point is beyond r_list plus a margin holds no member
// within r_list and is skipped.
//
// A row's candidates are tested into a bit mask, so that the tests are free of the bookkeeping of an
// entry (a list takes a seventh of its candidates), and all rows' bounds, then a row's candidates, are
// requested before any is used.  The set bits then go to the thread's run in LDS, a row's first and last
// ones at a time (its count of bits says where its entries end), and the list leaves as whole 16-byte
// words.  Where a list of the wavefront has more than LB_CAP entries (it holds 19 on average at the usual
// density, temperature and step) or a row more than 32 candidates, entries go in one at a time: those past
// the run straight to the list, those of candidates past the mask after a test each.  (Such lists were built
// a second time from the start: 50,000 mixed monomers took 26.3 us a step at density 1.3 and at T = 2, now
// 19.7 and 20.8; at 0.85 and T = 1 16.7.)
// Entry j of slot g lies in word nl_word(g, j / 8) at place j % 8; the last word is filled up with
// `pad`, the index one past the stage, where the step keeps a position outside every cutoff: the step
// reads whole words without testing the list's end.
struct ListArgs {
  int W, WY, U, minus_r2;
  float rskip2;
  const int* s_off;
  int pad;
};
constexpr int LB_CAP = 32;
constexpr int LB_STRIDE = 2 * LB_CAP + 4;  // bytes of a thread's run: lanes fall on different banks
// candidates [b, b + n) of row r = 3 zz + dy + 1
__device__ __forceinline__ void list_row(const ListArgs& l, uint2 me, int ih, int yy, int r, int& bi, int& ei) {
  const float U = (float)l.U;
  const float dxl = (float)(me.x & 0xffffu) - (float)ih * U, dxr = U - dxl;
  const float dyl = (float)(me.x >> 16) - (float)yy * U, dyr = U - dyl;
  const float dzl = (float)me.y - U, dzr = U - dzl;
  const int zz = r / 3, dy = r % 3 - 1;
  const float ez = zz == 0 ? dzl : (zz == 2 ? dzr : 0.0f), ey = dy < 0 ? dyl : (dy > 0 ? dyr : 0.0f);
  const float e2 = ey * ey + ez * ez;
  const int c0 = (zz * l.WY + yy + dy) * l.W + ih - 1;  // cells c0 .. c0 + 2: x offsets -1, 0, +1
  bi = c0 + (dxl * dxl + e2 > l.rskip2 ? 1 : 0);
  ei = e2 > l.rskip2 ? bi : c0 + (dxr * dxr + e2 > l.rskip2 ? 2 : 3);
}
// the list entry by entry, members through at(t) (a stage read from global memory)
template <typename At>
__device__ __forceinline__ int nl_list_any(const NlArgs& a, const ListArgs& l, int g, uint2 me, int tme, int ih, int yy, At at) {
  uint16_t* __restrict__ out = (uint16_t*)a.nlist + nl_word(g, 0) * 8;
  int cnt = 0;
  for (int r = 0; r < 9; ++r) {
    int bi, ei;
    list_row(l, me, ih, yy, r, bi, ei);
    const int e = l.s_off[ei];
    for (int t = l.s_off[bi]; t < e; ++t)
      if (t != tme && quant_test(at(t), me, l.minus_r2) < 0) {
        if (cnt < NL_CAP) out[(cnt >> 3) * 512 + (cnt & 7)] = (uint16_t)t;
        ++cnt;
      }
  }
  for (int c = cnt; c < NL_CAP && (c & 7); ++c) out[(c >> 3) * 512 + (c & 7)] = (uint16_t)l.pad;
  return cnt;
}
__device__ __forceinline__ int nl_list_one(const NlArgs& a, const ListArgs& l, int g, uint2 me, int tme, int ih, int yy,
                                           unsigned char* s_list, const uint2* s_pos) {
  int b[9], n[9], nmax = 0;
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    int bi, ei;
    list_row(l, me, ih, yy, r, bi, ei);
    b[r] = l.s_off[bi];
    n[r] = l.s_off[ei];
  }
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    n[r] -= b[r];
    nmax = max(nmax, n[r]);
  }
  uint32_t m[9];
  int cnt = 0;
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    uint2 p[RB_ROW];
#pragma unroll
    for (int u = 0; u < RB_ROW; ++u) p[u] = s_pos[b[r] + u];
    uint32_t mask = 0;
#pragma unroll
    for (int u = 0; u < RB_ROW; ++u)  // shift the test's sign bit in
      mask = __builtin_amdgcn_alignbit(mask, (uint32_t)quant_test(p[u], me, l.minus_r2), 31);
    mask <<= 32 - RB_ROW;
    if (__ballot(n[r] > RB_ROW)) {
      uint32_t more = 0;
#pragma unroll
      for (int u = RB_ROW; u < 32; ++u)
        more = __builtin_amdgcn_alignbit(more, (uint32_t)quant_test(s_pos[b[r] + u], me, l.minus_r2), 31);
      mask |= more;
    }
    // none past the row, nor the monomer itself
    mask = row_first(mask, n[r]);
    if (r == 4) mask = row_without(mask, tme - b[r]);
    m[r] = mask;
    cnt += __popc(mask);
  }
  unsigned char* const buf = s_list + threadIdx.x * LB_STRIDE;
  if (__ballot(cnt > LB_CAP || nmax > 32)) {
    // some lane's list is longer than its run, or a row longer than a mask: what lies past them goes to the
    // list entry by entry
    uint16_t* __restrict__ o16 = (uint16_t*)a.nlist + nl_word(g, 0) * 8;
    auto put = [&](int j, int v) {
      if (j < LB_CAP) run_put(buf + 2 * j, v);
      else if (j < NL_CAP) o16[(j >> 3) * 512 + (j & 7)] = (uint16_t)v;
    };
    int j = 0;
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      for (uint32_t mask = m[r]; mask; ++j) {
        const int u = __builtin_clz(mask);
        put(j, b[r] + u);
        mask &= ~(0x80000000u >> u);
      }
      if (nmax > 32) {
        int bi, ei;
        list_row(l, me, ih, yy, r, bi, ei);
        const int e = l.s_off[ei];
        for (int t = b[r] + 32; t < e; ++t)
          if (t != tme && quant_test(s_pos[t], me, l.minus_r2) < 0) put(j++, t);
      }
    }
    cnt = j;
    for (int c = cnt; c & 7; ++c) put(c, l.pad);
  } else {
    unsigned char* front = buf;
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      uint32_t mask = m[r];
      unsigned char *f = front, *e = front + 2 * __popc(mask);
      front = e;
      while (mask) {
        const int u = __builtin_clz(mask), v = 31 - __builtin_ctz(mask);
        e -= 2;
        run_put(f, b[r] + u);
        run_put(e, b[r] + v);
        f += 2;
        mask &= ~((0x80000000u >> u) | (0x80000000u >> v));
      }
    }
    for (int c = cnt; c & 7; ++c) run_put(buf + 2 * c, l.pad);
  }
  const int words = (cnt + 7) >> 3;
  uint4* __restrict__ out = (uint4*)a.nlist + nl_word(g, 0);
#pragma unroll
  for (int w = 0; w < LB_CAP / 8; ++w)
    if (w < words) {
      const unsigned char* p = buf + 16 * w;
      out[w * 64] = make_uint4(run_word(p), run_word(p + 4), run_word(p + 8), run_word(p + 12));
    }
  return cnt;
}

template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
// number of the other lanes of a group of G (8 or 16) whose v is smaller.  Within four lanes, lane ^ 1, 2
// and 3 are quad permutations; a half row and a row reversed give lane ^ 7 and ^ 15.
template <int G>
__device__ __forceinline__ int group_rank(int v) {
  int r = 0;
  auto quad = [&](int w) {  // w and its three quad neighbours
    r += (w < v) + (dpp<0xB1>(w) < v) + (dpp<0x4E>(w) < v) + (dpp<0x1B>(w) < v);
  };
  quad(v);  // (v < v counts nothing)
  quad(dpp<0x141>(v));
  if constexpr (G == 16) {
    const int m = dpp<0x140>(v);
    quad(m);
    quad(dpp<0x141>(m));
  }
  return r;
}

// One workgroup per tile, all resident at once at 200,000 monomers (952 tiles, 3.7 a CU: at most 128
// registers, none in scratch, and a quarter of a CU's LDS each), so the launch lasts as long as its slowest
// tile.  Bound by latency (wavefronts wait 55% of their time, the VALU is busy 36%): the counts and members of
// the staged cells arrive in 5 + 6 us there (2.5 + 3 us on an idle chip), the lists take 6-8 us.  1,000 monomers 18 us, 50,000 20 us, 200,000 38 us, 1M 124 us; with a
// thread per cell, per-entry stores and FP32 positions gathered by slot 38, 41, 58 and 222 us.
template <typename R>
__global__ __launch_bounds__(NLB_THREADS, 4) void k_nl_rebuild(NlArgs a) {
  extern __shared__ __align__(16) unsigned char s_dyn[];
  uint2* const s_pos = (uint2*)s_dyn;                     // staged members, by cell and monomer id
  const int hcap = rb_home_cap(a.stage_cap);
  int* const s_old = (int*)(s_pos + a.stage_cap + RB_PAD);  // old slots of the home members
  uint16_t* const s_hmap = (uint16_t*)(s_old + hcap);       // and their home cell: y << 8 | x of the frame
  // the threads' lists; before they are begun, the cells' sorted indices and the cells left to a wavefront
  // (a workgroup's LDS then stays below a quarter of a CU's at the usual stages)
  __shared__ __align__(4) unsigned char s_list[NLB_THREADS * LB_STRIDE];
  int* const s_sc = (int*)s_list;
  int* const s_geo = s_sc + NLB_CELLS;  // x | y << 8 | z << 16 of a frame cell
  uint16_t* const s_big = (uint16_t*)(s_geo + NLB_CELLS);
  static_assert(NLB_CELLS * 10 <= NLB_THREADS * LB_STRIDE, "fits");
  __shared__ int s_off[NLB_CELLS + 1];
  __shared__ int s_home[NLB_HOMES + 1];  // prefix of the home cells' counts, sorted order
  __shared__ int s_nbig;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int k = __builtin_amdgcn_readfirstlane(a.rblk_melt[lb]);
  const int lt = a.rblk_base[lb];
  const MeltDesc& d = a.md[k];
  const TileGeo tg = tile_geo(d, lt);
  const int W = tg.nh + 2, WY = tg.nhy + 2, ncell = 3 * WY * W;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double hl = d.hl;
  const int nc = d.ncl, U = d.nl_u;

  // the first slot of this tile: with few tiles in the batch, the sum of the counts of the tiles
  // before it, read here with the cells' counts (no scan kernel); else the scan's result
  const int tile = d.tile_off + lt;
  __shared__ int s_tsum[NLB_THREADS / 64];
  const bool tile_sum = a.ntile_total <= TILE_SUM_MAX;
  const int nhc = tg.nh * tg.nhy;
  if (threadIdx.x == 0) s_nbig = 0;
  for (int t = threadIdx.x; t < ncell; t += NLB_THREADS) {
    const StagedCell s = staged_cell(d, tg, W, WY, t);
    const int sc = sorted_cell(d, s.ax, s.ay, s.az, nullptr);
    const int n = min(a.cnt[sc], NL_CELL_CAP);
    s_sc[t] = sc;
    s_geo[t] = s.i | s.yy << 8 | s.zz << 16;
    s_off[t + 1] = n;
    if (s.zz == 1 && s.yy >= 1 && s.yy <= tg.nhy && s.i >= 1 && s.i <= tg.nh)
      s_home[(s.yy - 1) * tg.nh + s.i] = n;
  }
  if (tile_sum) {
    int part = 0;
    for (int t = threadIdx.x; t < tile; t += NLB_THREADS) part += a.tcnt[t];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if (lane == 0) s_tsum[wv] = part;
  }
  __syncthreads();
  // (the members arrive while the counts' prefixes are formed)
  constexpr int BATCH = 8;  // cells a group takes at once
  int4 ent[BATCH];
  const bool wide = d.nl_wide;
  auto fetch = [&](int g, int c0) {  // lanes of a group, first cell of its batch
    const int per = NLB_THREADS / g;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int c = min(c0 + i * per + (int)threadIdx.x / g, ncell - 1);
      ent[i] = a.bucket[(size_t)s_sc[c] * NL_CELL_CAP + (threadIdx.x & (g - 1))];
    }
  };
  if (wide) fetch(16, 0);
  else fetch(8, 0);
  if (wv == 0) wave_prefix(s_off, ncell);
  if (wv == 1) wave_prefix(s_home, nhc);
  __syncthreads();
  const int total = s_off[ncell], nhome = s_home[nhc];
  const bool staged = total <= a.stage_cap && nhome <= hcap && !(d.test_flags & TF_NL_GLOBAL);
  if (threadIdx.x == 0 && !(d.test_flags & TF_NL_GLOBAL) && a.nlstat) {
    // (a capacity of the reported size holds the stage and, as a third of it, the homes)
    atomicMax(&a.nlstat[1], (uint32_t)max(total, 3 * (nhome - RB_HOME_PAD)));
    if (!staged) atomicAdd(&a.nlstat[0], 1u);
  }
  const int NP = a.NP;
  if (staged) {
    // each member's rank by id within its cell gives its place in the stage
    auto put = [&](int c, int b0, int r, const int4& e) {
      const int geo = s_geo[c], i = geo & 255, yy = (geo >> 8) & 255, zz = geo >> 16;
      s_pos[b0 + r] = quant_pos(e, i, yy, zz, U);
      if (zz == 1 && yy >= 1 && yy <= tg.nhy && i >= 1 && i <= tg.nh) {
        const int h = s_home[(yy - 1) * tg.nh + i - 1] + r;
        s_old[h] = e.x;
        s_hmap[h] = (uint16_t)(yy << 8 | i);
      }
    };
    auto stage = [&](auto gw) {
      constexpr int g = decltype(gw)::value, per = NLB_THREADS / g;
      const int j = threadIdx.x & (g - 1);
      for (int c0 = 0; c0 < ncell; c0 += BATCH * per) {
        if (c0) fetch(g, c0);
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
          const int c = c0 + i * per + (int)threadIdx.x / g;
          if (c0 + i * per >= ncell) break;  // (uniform)
          const int cc = min(c, ncell - 1), b0 = s_off[cc], n = c < ncell ? s_off[cc + 1] - b0 : 0;
          const int r = group_rank<g>(j < n ? ent[i].y : 0x7fffffff);
          if (n > g) {
            if (j == 0) s_big[atomicAdd(&s_nbig, 1)] = (uint16_t)c;
          } else if (j < n) {
            put(c, b0, r, ent[i]);
          }
        }
      }
    };
    if (wide) stage(std::integral_constant<int, 16>{});
    else stage(std::integral_constant<int, 8>{});
    __syncthreads();
    const int nbig = s_nbig;
    for (int q = wv; q < nbig; q += NLB_THREADS / 64) {  // a member a lane
      const int t = s_big[q], b0 = s_off[t], n = s_off[t + 1] - b0;
      const int4 e = a.bucket[(size_t)s_sc[t] * NL_CELL_CAP + min(lane, n - 1)];
      int r = 0;
      for (int m = 0; m < n; ++m) r += __shfl(e.y, m, 64) < e.y;
      if (lane < n) put(t, b0, r, e);
    }
    if (nbig) __syncthreads();
  }
  int first = 0;
  if (tile_sum) {
#pragma unroll
    for (int w = 0; w < NLB_THREADS / 64; ++w) first += s_tsum[w];
  } else {
    first = a.tstart[tile];
  }
  for (int c = threadIdx.x; c < nhc; c += NLB_THREADS) {
    const int ly = c / tg.nh, lx = c - ly * tg.nh;
    const int t = (WY + ly + 1) * W + lx + 1;
    a.cellsc[s_sc[t]] = make_int2(first + s_home[c], s_home[c + 1] - s_home[c]);
  }
  __syncthreads();  // (the staged list builder overwrites the cells' indices; the other one reads them)
  const float rl = (float)(sqrt(d.rlist2 * 1.0002) * d.cinvl) * (float)U + 2.0f, rsk = rl + 4.0f;
  const ListArgs la = {W, WY, U, -(int)(rl * rl) - 1, rsk * rsk, s_off, total};
  for (int h = threadIdx.x; h < nhome; h += NLB_THREADS) {
    int lx, ly, t, r;
    if (staged) {
      const int m = s_hmap[h];
      lx = (m & 255) - 1;
      ly = (m >> 8) - 1;
      t = (WY + ly + 1) * W + lx + 1;
      r = h - s_home[ly * tg.nh + lx];
    } else {
      const int c = find_cell(s_home, 0, nhc, h);
      ly = c / tg.nh;
      lx = c - ly * tg.nh;
      t = (WY + ly + 1) * W + lx + 1;
      r = h - s_home[c];
    }
    const int si = s_off[t] + r;
    const int g = first + h;
    int old;
    uint2 me;
    if (staged) {
      old = s_old[h];
      me = s_pos[si];
    } else {
      const int4 e = member_entry(a, s_sc[t], s_off[t + 1] - s_off[t], r);
      old = e.x;
      me = quant_pos(e, lx + 1, ly + 1, 1, U);
    }
    const int cx = wrapc(tg.x0 + lx, nc), cy = wrapc(tg.y0 + ly, nc), cz = tg.cz;
    const int mo = a.mono[old];
    int n;
    if (staged)
      n = nl_list_one(a, la, g, me, si, lx + 1, ly + 1, s_list, s_pos);
    else
      n = nl_list_any(a, la, g, me, si, lx + 1, ly + 1, [&](int u) {
        const int q = find_cell(s_off, 0, ncell, u);
        const int row = q / W, i = q - row * W, zz = row / WY, yy = row - zz * WY;
        return quant_pos(member_entry(a, s_sc[q], s_off[q + 1] - s_off[q], u - s_off[q]), i, yy, zz, U);
      });
    // the new slot takes the monomer's state (requested before the list was built, it arrived meanwhile, but
    // its registers sent eight others to scratch: the same times up to 200,000 monomers, 2% more at 1M)
    double xo[3], vo[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      xo[q] = a.x[(size_t)q * NP + old];
      vo[q] = a.v[(size_t)q * NP + old];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      a.xn[(size_t)q * NP + g] = xo[q];
      a.vn[(size_t)q * NP + g] = vo[q];
    }
    if (a.perm_f) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        a.fcn[(size_t)q * NP + g] = a.fc[(size_t)q * NP + old];
        a.fln[(size_t)q * NP + g] = a.fl[(size_t)q * NP + old];
      }
    }
    a.mono_n[g] = mo;
    a.inv[old] = g;
    ((typename Rel<R>::T*)a.rel_next)[g] =
        Rel<R>::make(xo[0] - cx * hl, xo[1] - cy * hl, xo[2] - cz * hl, pack_cell(cx, cy, cz), hl);
    if (n > NL_CAP) { atomicOr(&a.err[k], ERR_NLIST_OVERFLOW); n = NL_CAP; }
    if (a.side && (d.test_flags & TF_SIDE_FAULT)) {  // test hook: a failed rebuild beside a sweep
      atomicOr(&a.err[k], ERR_NLIST_OVERFLOW);
      n = 0;
    }
    a.nlen[g] = n;
  }
}

// ---------------------------------------------------------------------------------------
// rebuild 4: per old slot, carry the chain position over to the new slot, rewrite the chain
// table entry it owns, and record the new slots of its chain neighbours p-2, p-1, p+1, p+2
// (-1 past a chain end); clear the counts for the next binning and the displacement bounds
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_nl_remap(NlArgs a) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < a.ncl_total; t += gridDim.x * blockDim.x) a.cnt[t] = 0;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < a.ntile_total; t += gridDim.x * blockDim.x) a.tcnt[t] = 0;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < a.nm * 2 * DISP_SLOTS; t += gridDim.x * blockDim.x)
    a.disp[(size_t)t * DISP_STRIDE] = 0u;
  if (blockIdx.x == 0)
    for (int m = threadIdx.x; m < a.nm; m += blockDim.x) a.dacc[m] = 0.0f;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int k = __builtin_amdgcn_readfirstlane(a.pblk_melt[lb]);
  const MeltDesc& d = a.md[k];
  const int li = a.pblk_base[lb] + (int)threadIdx.x;
  if (li >= d.Nm) return;
  const int o = d.off + li;
  // (after a rebuild that overflowed a cell, entries may be stale until the run is rolled
  // back: indices are kept inside the melt)
  const int g = min(max(a.inv[o], d.off), d.off + d.Nm - 1);
  const int lc = min(max(a.loc[o], 0), d.Nm - 1);
  const int N = d.N;
  const int c = lc / N, p = lc - c * N;
  const int* row = a.chain + d.off + c * N;
  int nb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int pp = p + (q < 2 ? q - 2 : q - 1);
    nb[q] = (pp >= 0 && pp < N) ? a.inv[min(max(row[pp], d.off), d.off + d.Nm - 1)] : -1;
  }
  a.loc_n[g] = lc;
  a.chain_n[d.off + lc] = g;
  a.nb4_n[g] = make_int4(nb[0], nb[1], nb[2], nb[3]);
}

template <typename R> struct W3 { R x, y, z; };

// The step kernel's LDS stage: a fixed-point int4 per member in the mixed path; in the FP64
// path three arrays of coordinates (24 bytes per member where the relative-position record takes
// 32: three workgroups of the workload's tiles then fit a CU's LDS instead of two)
template <typename R> struct StageLds;
template <> struct StageLds<float> {
  int4* p;
  __device__ StageLds(unsigned char* base, int) : p((int4*)base) {}
  __device__ void put(int u, const int4& v) { p[u] = v; }
  __device__ int4 get(int u) const { return p[u]; }
  __host__ __device__ static size_t bytes(int cap) { return (size_t)(cap + 4) * sizeof(int4); }
};
template <> struct StageLds<double> {
  double *x, *y, *z;
  __device__ StageLds(unsigned char* base, int cap) : x((double*)base), y(x + cap + 4), z(y + cap + 4) {}
  __device__ void put(int u, const Rel<double>::T& v) { x[u] = v.x; y[u] = v.y; z[u] = v.z; }
  __device__ Rel<double>::T get(int u) const { return Rel<double>::T{x[u], y[u], z[u], 0.0}; }
  __host__ __device__ static size_t bytes(int cap) { return (size_t)(cap + 4) * 3 * sizeof(double); }
};

// fast FP32 reciprocal and square root (about 1 ulp); exact IEEE forms in FP64
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double frcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fsqrt(double x) { return sqrt(x); }

// ---------------------------------------------------------------------------------------
// the step: forces from the lists + chain, Langevin velocity Verlet
// ---------------------------------------------------------------------------------------
// NH > 0: the exponent n = 2 NH is fixed at compile time (the soft and the standard
// potential); NH = 0 reads it from the melt.
template <typename R, int MODE, int NH>
__global__ __launch_bounds__(NLB_THREADS) void k_nl_step(NlArgs a) {
  using P = typename Rel<R>::T;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  StageLds<R> s_pos(s_dyn, a.stage_cap);
  __shared__ int s_off[NLB_CELLS + 1];
  __shared__ int s_start[NLB_CELLS];
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int k = __builtin_amdgcn_readfirstlane(a.rblk_melt[lb]);
  const int lt = a.rblk_base[lb];
  const MeltDesc& d = a.md[k];
  const TileGeo tg = tile_geo(d, lt);
  const int W = tg.nh + 2, WY = tg.nhy + 2, ncell = 3 * WY * W;
  const int NP = a.NP;
  const double L = d.L, invL = d.invL, hl = d.hl;
  const P* __restrict__ rel = (const P*)a.rel_cur;
  // length of one unit of the relative coordinates (fixed point: cell edge / 2^24)
  const R u = (R)Rel<R>::unit(hl);

  // list validity: the first tile of each melt adds the previous step's largest displacement
  // to the bound accumulated since the rebuild
  const int sp = (int)(a.sp & 1u);
  uint32_t* const disp_now = a.disp + ((size_t)k * 2 + sp) * DISP_SLOTS * DISP_STRIDE;
  if (lt == 0 && threadIdx.x < 64) {  // one wavefront: the previous step's slots (then cleared)
    uint32_t* const prev = a.disp + ((size_t)k * 2 + (1 - sp)) * DISP_SLOTS * DISP_STRIDE;
    float m = threadIdx.x < DISP_SLOTS ? __uint_as_float(prev[threadIdx.x * DISP_STRIDE]) : 0.0f;
    if (threadIdx.x < DISP_SLOTS) prev[threadIdx.x * DISP_STRIDE] = 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (threadIdx.x == 0) {
      const float acc = a.dacc[k] + m;
      a.dacc[k] = acc;
      if (acc > (float)d.half_skin) atomicOr(&a.err[k], ERR_NLIST_STALE);
    }
  }

  // The stage (the members of the 3 x (nh + 2) x (nhy + 2) cells around the tile) keeps its
  // slots from one rebuild to the next.  The first step after a rebuild finds them from the cell
  // table and records them with the tile's home range; later steps read that record.  (A slot has 24
  // bits.  When the frame wraps onto itself in a small box, a slot does not fix its frame cell: bits 24
  // and 25 say whether the cell lies past one box in x and y.  A frame is at most two cells wider than
  // the box, and no deeper.  The table at every step took 22.7 us a step for 1,000 monomers in FP64 and
  // 5 x 3 tiles, 34.8 for 64 melts of 2,000, mixed; the record 18.4 and 24.7.  The loop of a frame that
  // does not wrap keeps to itself: with the bits' test in one loop for both, 200k took 3% longer.)
  const int tile = d.tile_off + lt;
  const int nc = d.ncl;
  const bool frame_ok = !(d.test_flags & TF_NL_GLOBAL);
  const bool frame_wraps = W > nc || WY > nc;
  int* const slist = a.stage_list + (size_t)tile * a.stage_stride;
  int4 meta = make_int4(0, 0, 0, 0);
  bool fast = false;
  if (!a.stage_write && frame_ok) {
    meta = a.stage_meta[tile];
    fast = meta.z <= a.stage_cap;
  }
  // the tile's home monomers occupy slots h0 .. h0 + nhome - 1
  int h0, nhome;
  if (fast) {
    h0 = meta.x;
    nhome = meta.y;
  } else {
    h0 = a.cellsc[sorted_cell(d, tg.x0, tg.y0, tg.cz, nullptr)].x;
    const int2 lastc = a.cellsc[sorted_cell(d, tg.x0 + tg.nh - 1, tg.y0 + tg.nhy - 1, tg.cz, nullptr)];
    nhome = lastc.x + lastc.y - h0;
  }
  const bool pairs_on = !(d.test_flags & (TF_NOFORCE | TF_PHANTOM));
  // a home monomer's own data (independent loads; the first one's are issued before the stage
  // is built, so that they arrive meanwhile)
  struct Home {
    P ri;
    int4 nb;
    int n;
    double x, y, z, vx, vy, vz;
    R z0, z1, z2;  // Langevin noise of this closing kick (drawn at the force precision)
    uint4 w0;
  };
  // the noise depends only on the monomer id and the step
  const uint64_t noise_idx = (MODE & F_CLOSE) ? a.step_base[k] + (uint64_t)a.s_off : 0ull;
  auto noise = [&](Home& o, int mono) {
    o.z0 = o.z1 = o.z2 = (R)0;
    if (MODE & F_CLOSE) {
      const U32x4 w = md_noise_draw(d, (uint64_t)mono, noise_idx, ST_LANGEVIN);
      double n0, n1, n2, n3;
      gauss2_md_r<R>(w.w[0], w.w[1], n0, n1);
      gauss2_md_r<R>(w.w[2], w.w[3], n2, n3);
      o.z0 = (R)n0; o.z1 = (R)n1; o.z2 = (R)n2;  // (exact: the normals are of precision R)
    }
  };
  const uint4* __restrict__ words = (const uint4*)a.nlist;
  // FP64 with an integer n / 2: position, velocity and the first chain partner wait until the pair loop
  // is over.  125 registers instead of 145 let four workgroups share a CU: the 1,020 tiles of 200,000
  // monomers run at once instead of 768 and 252 (41.3 -> 35.9 us a step with rebuilds; 400,000 74.5 ->
  // 68.1; up to 100,000, and from 700,000 on, where memory is the bound, within 1% of before).  With all
  // four partners late 1M took 5% longer; a bound on the registers spills, and changes the sums' rounding.
  constexpr bool late = sizeof(R) == 8 && NH > 0;
  auto load_home = [&](int g) {
    Home o;
    o.ri = rel[g];
    o.n = pairs_on ? a.nlen[g] : 0;
    o.nb = a.nb4[g];
    if (!late) {
      o.x = a.x[g]; o.y = a.x[NP + g]; o.z = a.x[2 * NP + g];
      o.vx = a.v[g]; o.vy = a.v[NP + g]; o.vz = a.v[2 * NP + g];
    }
    o.w0 = words[nl_word(g, 0)];
    noise(o, (MODE & F_CLOSE) ? a.mono[g] : 0);
    return o;
  };
  // (the first home's noise is drawn while its stage loads arrive)
  Home pre;
  if ((int)threadIdx.x < nhome) pre = load_home(h0 + (int)threadIdx.x);

  int total;
  bool staged;
  // staged member t: current position relative to its reference cell, moved into the frame
  auto member = [&](int t) -> P {
    const int q = find_cell(s_off, 0, ncell, t);
    const int row = q / W, i = q - row * W;
    const int zz = row / WY, yy = row - zz * WY;
    return rel_shift<R>(rel[s_start[q] + (t - s_off[q])], i - 1, yy - 1, zz - 1, hl);
  };
  if (fast) {
    total = meta.z;
    staged = true;
    // the frame cell of a member follows from its reference cell (the periodic difference) and, in a
    // frame wider than the box, the two bits of its record
    const int fx = tg.x0 - 1, fy = tg.y0 - 1, fz = tg.cz - 1;
    auto place = [&](const P& p, int wx, int wy) {
      const int c = Rel<R>::cell(p);
      int i = (c & 1023) - fx, yy = ((c >> 10) & 1023) - fy, zz = (c >> 20) - fz;
      i += i < 0 ? nc : 0;
      i -= i >= nc ? nc : 0;
      yy += yy < 0 ? nc : 0;
      yy -= yy >= nc ? nc : 0;
      zz += zz < 0 ? nc : 0;
      zz -= zz >= nc ? nc : 0;
      return rel_shift<R>(p, i + wx - 1, yy + wy - 1, zz - 1, hl);
    };
    // (slots are kept inside the storage whatever the record holds)
    if (!frame_wraps) {
#pragma unroll 4
      for (int u = threadIdx.x; u < total; u += NLB_THREADS) {
        const P p = rel[min(max(slist[u], 0), NP - 1)];
        s_pos.put(u, place(p, 0, 0));
      }
    } else {
#pragma unroll 2
      for (int u = threadIdx.x; u < total; u += NLB_THREADS) {
        const int e = slist[u];
        const P p = rel[min(e & 0xffffff, NP - 1)];
        s_pos.put(u, place(p, (e >> 24) & 1 ? nc : 0, (e >> 25) & 1 ? nc : 0));
      }
    }
  } else {
    for (int t = threadIdx.x; t < ncell; t += NLB_THREADS) {
      const StagedCell s = staged_cell(d, tg, W, WY, t);
      const int2 cs = a.cellsc[sorted_cell(d, s.ax, s.ay, s.az, nullptr)];
      s_start[t] = cs.x;
      s_off[t + 1] = cs.y;
    }
    __syncthreads();
    if (threadIdx.x < 64) wave_prefix(s_off, ncell);
    __syncthreads();
    total = s_off[ncell];
    staged = total <= a.stage_cap && !(d.test_flags & TF_NL_GLOBAL);
    const bool record = a.stage_write && staged && frame_ok;
    if (staged) {
#pragma unroll 4
      for (int u = threadIdx.x; u < total; u += NLB_THREADS) {
        const int q = find_cell(s_off, 0, ncell, u);
        const int row = q / W, i = q - row * W;
        const int zz = row / WY, yy = row - zz * WY;
        const int slot = s_start[q] + (u - s_off[q]);
        if (record) slist[u] = slot | (i >= nc ? 1 << 24 : 0) | (yy >= nc ? 1 << 25 : 0);
        s_pos.put(u, rel_shift<R>(rel[slot], i - 1, yy - 1, zz - 1, hl));
      }
    }
    if (a.stage_write && threadIdx.x == 0) a.stage_meta[tile] = make_int4(h0, nhome, total, 0);
  }
  // one place past the stage: the position that the padding of a list's last word reads
  if (staged && threadIdx.x == 0) s_pos.put(total, stage_sentinel<R>());
  __syncthreads();

  const bool forces_on = !(d.test_flags & TF_NOFORCE);
  uint32_t errbits = 0;
  float dmax = 0.0f;
  int nfloor = 0;
  const R pa = (R)d.pa, pb = (R)d.pb, n_half = (R)(0.5 * d.n_exp);
  // the cutoff in units of the relative coordinates, and 1 / unit^2
  const R rc2u = sizeof(R) == 4 ? (R)d.rc2_fx : (R)d.rc2, iu2 = sizeof(R) == 4 ? (R)d.iu2_fx : (R)1;
  const int nh = NH > 0 ? NH : d.n_half_int;

  for (int h = threadIdx.x; h < nhome; h += NLB_THREADS) {
    const int g = h0 + h;
    // (a lane's next home, in a tile of more than 256, is loaded at the end of this one: one
    // home's data live at a time)
    const Home hm = pre;
    const P ri = hm.ri;
    const int n = hm.n;
    const int4 nb = hm.nb;
    double xg = hm.x, yg = hm.y, zg = hm.z;
    double vx = hm.vx, vy = hm.vy, vz = hm.vz;
    uint4 wd = hm.w0;
    const int pc = Rel<R>::cell(ri);
    const int ix = pc & 1023, iy = (pc >> 10) & 1023, iz = pc >> 20;
    // chain neighbours p-2, p-1, p+1, p+2 (slots, or -1)
    const int nbq[4] = {nb.x, nb.y, nb.z, nb.w};
    // (the FP64 record's packed cell is taken as an int where the partner is loaded)
    P rb[4];
    int rbc[4];
    uint32_t nbmask = 0;  // bit q: partner q exists (and forces are on)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // (a slot past the storage can only come from a rebuild that overflowed, whose run is redone)
      const bool on = forces_on && nbq[q] >= 0 && nbq[q] < NP;
      nbmask |= on ? 1u << q : 0u;
      if (late && q == 0) continue;
      rb[q] = rel[on ? nbq[q] : g];
      rbc[q] = Rel<R>::cell(rb[q]);
    }

    const double z0 = hm.z0, z1 = hm.z1, z2 = hm.z2;

    W3<R> F = {(R)0, (R)0, (R)0};
    // pair force from a displacement in units (x_j - x_i); F accumulates in units too and is
    // scaled by the unit at the end
    auto pair_add = [&](R dx, R dy, R dz) {
      const R r2 = dx * dx + dy * dy + dz * dz;
      if (r2 < rc2u) {
        const R s2 = frcp(r2) * iu2;
        const R s6 = s2 * s2 * s2;
        const R sn = pow_half<R>(s2, nh, n_half);
        const R coef = (pa * sn - pb * s6) * s2;
        F.x -= coef * dx; F.y -= coef * dy; F.z -= coef * dz;
      }
    };
    // list entries: the same force without a branch; r2 is clamped away from 0 for entries
    // outside the cutoff, whose force is masked
    auto pair_add_nb = [&](R dx, R dy, R dz) {
      const R r2 = dx * dx + dy * dy + dz * dz;
      const bool in = r2 < rc2u;
      const R s2 = frcp(in ? r2 : rc2u) * iu2;
      const R s6 = s2 * s2 * s2;
      const R sn = pow_half<R>(s2, nh, n_half);
      const R coef = in ? (pa * sn - pb * s6) * s2 : (R)0;
      F.x -= coef * dx; F.y -= coef * dy; F.z -= coef * dz;
    };
    // own position in the tile frame (the reference cell is a home cell of this tile)
    const P me = rel_shift<R>(ri, ix - tg.x0, iy - tg.y0, 0, hl);
    // (mixed path, integer n / 2: the FP64 and general-exponent variants would need more
    // registers than fit four wavefronts per SIMD, and keep the guarded loop)
    constexpr bool whole_words = sizeof(R) == 4 && NH > 0;
    if (whole_words && staged) {
      // whole words without a branch: the rebuild fills a list's last word up with the
      // sentinel's index, so that the LDS reads of a word can be issued together
      for (int t = 0; t < n; t += 8) {
        const uint4 cw = wd;
        if (t + 8 < n) wd = words[nl_word(g, (t >> 3) + 1)];
        const uint32_t e2[4] = {cw.x, cw.y, cw.z, cw.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          // (an index past the stage can only come from a list left by a failed rebuild, whose
          // run is redone: it reads the sentinel)
          const P p = s_pos.get(min((int)((e2[q >> 1] >> ((q & 1) * 16)) & 0xffffu), total));
          R dx, dy, dz;
          Rel<R>::diff(p, me, dx, dy, dz);
          pair_add_nb(dx, dy, dz);
        }
      }
    } else {
      for (int t = 0; t < n; t += 8) {
        const uint4 cw = wd;
        if (t + 8 < n) wd = words[nl_word(g, (t >> 3) + 1)];
        const uint32_t e2[4] = {cw.x, cw.y, cw.z, cw.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          if (t + q < n) {
            // (an index past the stage can only come from a list left by a failed rebuild,
            // whose run is redone: it is kept inside the stage)
            const int e = min((int)((e2[q >> 1] >> ((q & 1) * 16)) & 0xffffu), total - 1);
            const P p = staged ? s_pos.get(e) : member(e);
            R dx, dy, dz;
            Rel<R>::diff(p, me, dx, dy, dz);
            pair_add_nb(dx, dy, dz);
          }
        }
      }
    }
    F.x *= u; F.y *= u; F.z *= u;  // coef * (x_j - x_i): units -> sigma

    if (late) {
      rb[0] = rel[nbmask & 1u ? nbq[0] : g];
      rbc[0] = Rel<R>::cell(rb[0]);
    }
    // bonded partners: displacement from the relative positions and the reference cells
    W3<R> Pd[5];
    bool has[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      Pd[q].x = Pd[q].y = Pd[q].z = (R)0;
      has[q] = q == 2;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int sl = q < 2 ? q : q + 1;
      if (!((nbmask >> q) & 1u)) continue;
      has[sl] = true;
      const int pj = rbc[q];
      int dx = (pj & 1023) - ix, dy = ((pj >> 10) & 1023) - iy, dz = (pj >> 20) - iz;
      // nearest periodic image of the cell difference
      dx -= nc * (dx > nc / 2) - nc * (dx < -(nc - 1) / 2);
      dy -= nc * (dy > nc / 2) - nc * (dy < -(nc - 1) / 2);
      dz -= nc * (dz > nc / 2) - nc * (dz < -(nc - 1) / 2);
      R bx, by, bz;
      Rel<R>::image_diff(rb[q], ri, dx, dy, dz, nc, hl, bx, by, bz);
      Pd[sl].x = bx * u;
      Pd[sl].y = by * u;
      Pd[sl].z = bz * u;
    }

    if (forces_on) {
      const R kf = (R)d.kfene, R0sq = (R)d.R0sq, amin = (R)d.amin, iR0sq = (R)d.iR0sq;
#pragma unroll
      for (int q = 1; q <= 3; q += 2) {
        if (!has[q]) continue;
        const W3<R> b = Pd[q];
        const R r2 = b.x * b.x + b.y * b.y + b.z * b.z;
        const bool broken = (amin > (R)0) ? !(r2 < (R)4 * R0sq) : !(r2 < R0sq);
        if (broken) errbits |= ERR_FENE;
        const R am = (R)1 - r2 * iR0sq;
        const bool floored = amin > (R)0 && am < amin;
        if ((MODE & F_CLOSE) && q == 3 && floored) ++nfloor;  // each bond once per step, by its first bead
        const R cb = kf * frcp(floored ? amin : am);  // F_i = k (x_j - x_i) / a
        F.x += cb * b.x; F.y += cb * b.y; F.z += cb * b.z;
        if (d.test_flags & TF_PHANTOM) {  // the bonded pair's MLJ^n, from the displacement in units
          const R ui = (R)1 / u;
          const W3<R> Fs = F;
          F.x = F.y = F.z = (R)0;
          pair_add(b.x * ui, b.y * ui, b.z * ui);
          F.x = Fs.x + F.x * u; F.y = Fs.y + F.y * u; F.z = Fs.z + F.z * u;
        }
      }
      const R kap = (R)d.kappa;
      if (d.kappa != 0.0) {
#pragma unroll
        for (int dv = -1; dv <= 1; ++dv) {
          const int iv = 2 + dv;
          if (!(has[iv - 1] && has[iv] && has[iv + 1])) continue;
          const W3<R> b1 = {Pd[iv].x - Pd[iv - 1].x, Pd[iv].y - Pd[iv - 1].y, Pd[iv].z - Pd[iv - 1].z};
          const W3<R> b2 = {Pd[iv + 1].x - Pd[iv].x, Pd[iv + 1].y - Pd[iv].y, Pd[iv + 1].z - Pd[iv].z};
          const R l1s = b1.x * b1.x + b1.y * b1.y + b1.z * b1.z;
          const R l2s = b2.x * b2.x + b2.y * b2.y + b2.z * b2.z;
          const R i1 = frcp(l1s), i2 = frcp(l2s);
          const R inv12 = fsqrt(i1 * i2);
          const R cs = (b1.x * b2.x + b1.y * b2.y + b1.z * b2.z) * inv12;
          const R c1 = cs * i1, c2 = cs * i2;
          const W3<R> g1 = {b2.x * inv12 - c1 * b1.x, b2.y * inv12 - c1 * b1.y, b2.z * inv12 - c1 * b1.z};
          const W3<R> g2 = {b1.x * inv12 - c2 * b2.x, b1.y * inv12 - c2 * b2.y, b1.z * inv12 - c2 * b2.z};
          if (dv == 1) { F.x -= kap * g1.x; F.y -= kap * g1.y; F.z -= kap * g1.z; }  // first bead
          else if (dv == 0) { F.x += kap * (g1.x - g2.x); F.y += kap * (g1.y - g2.y); F.z += kap * (g1.z - g2.z); }
          else { F.x += kap * g2.x; F.y += kap * g2.y; F.z += kap * g2.z; }  // last bead
        }
      }
    }

    if (late) { vx = a.v[g]; vy = a.v[NP + g]; vz = a.v[2 * NP + g]; }
    const double Fx = (double)F.x, Fy = (double)F.y, Fz = (double)F.z;
    if (!(isfinite(Fx) && isfinite(Fy) && isfinite(Fz))) errbits |= ERR_NONFINITE;
    double fx, fy, fz;
    const double dt = d.dt;
    if (MODE & F_CLOSE) {
      const double amp = d.lang_amp;  // sqrt(2 gamma T / dt)
      fx = -d.gamma * vx + amp * z0;
      fy = -d.gamma * vy + amp * z1;
      fz = -d.gamma * vz + amp * z2;
      vx = vx + 0.5 * dt * (Fx + fx);
      vy = vy + 0.5 * dt * (Fy + fy);
      vz = vz + 0.5 * dt * (Fz + fz);
    } else {
      fx = a.fl[g]; fy = a.fl[NP + g]; fz = a.fl[2 * NP + g];
    }
    if (MODE & F_STORE) {
      a.fc[g] = Fx; a.fc[NP + g] = Fy; a.fc[2 * NP + g] = Fz;
      a.fl[g] = fx; a.fl[NP + g] = fy; a.fl[2 * NP + g] = fz;
      a.v[g] = vx; a.v[NP + g] = vy; a.v[2 * NP + g] = vz;
      if (!(isfinite(vx) && isfinite(vy) && isfinite(vz))) errbits |= ERR_NONFINITE;
    }
    if (MODE & F_OPEN) {
      if (late) { xg = a.x[g]; yg = a.x[NP + g]; zg = a.x[2 * NP + g]; }
      const double hx = vx + 0.5 * dt * (Fx + fx);
      const double hy = vy + 0.5 * dt * (Fy + fy);
      const double hz = vz + 0.5 * dt * (Fz + fz);
      const double nxp = wrap_near(xg + dt * hx, L);
      const double nyp = wrap_near(yg + dt * hy, L);
      const double nzp = wrap_near(zg + dt * hz, L);
      if (!(isfinite(nxp) && isfinite(nyp) && isfinite(nzp) && isfinite(hx) && isfinite(hy) && isfinite(hz)))
        errbits |= ERR_NONFINITE;
      a.v[g] = hx; a.v[NP + g] = hy; a.v[2 * NP + g] = hz;
      a.xn[g] = nxp; a.xn[NP + g] = nyp; a.xn[2 * NP + g] = nzp;
      // (FP32, rounded up by a relative 1e-6: a bound, not a value)
      dmax = fmaxf(dmax, (float)dt * __builtin_amdgcn_sqrtf((float)(hx * hx + hy * hy + hz * hz)) * 1.000001f);
      // position relative to the reference cell (periodic image nearest to it)
      double rx = nxp - ix * hl, ry = nyp - iy * hl, rz = nzp - iz * hl;
      rx -= L * rint(rx * invL); ry -= L * rint(ry * invL); rz -= L * rint(rz * invL);
      ((P*)a.rel_next)[g] = Rel<R>::make(rx, ry, rz, pc, hl);
    }
    if (h + NLB_THREADS < nhome) pre = load_home(g + NLB_THREADS);
  }
  // the step before a rebuild bins the new positions into the list grid, in a loop of its own that
  // reads back what the lane has just written (outside the force loop, whose registers it would
  // otherwise raise past four wavefronts per SIMD)
  if (MODE & F_BIN) {
    for (int h = threadIdx.x; h < nhome; h += NLB_THREADS) {
      const int g = h0 + h;
      nl_bin_one(a, k, d, g, a.mono[g], a.xn[g], a.xn[NP + g], a.xn[2 * NP + g], true);
    }
  }
  if (MODE & F_OPEN) {
    // the step's largest displacement: per workgroup, then one atomic into one of the melt's
    // slots (non-negative floats order as their bit patterns)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dmax = fmaxf(dmax, __shfl_xor(dmax, o, 64));
    __shared__ float s_dmax[NLB_THREADS / 64];
    if ((threadIdx.x & 63) == 0) s_dmax[threadIdx.x >> 6] = dmax;
    __syncthreads();
    if (threadIdx.x == 0) {
      float m = s_dmax[0];
      for (int w = 1; w < NLB_THREADS / 64; ++w) m = fmaxf(m, s_dmax[w]);
      if (m > 0.0f) atomicMax(&disp_now[(lt % DISP_SLOTS) * DISP_STRIDE], __float_as_uint(m));
    }
  }
  if (__ballot(nfloor > 0)) {
    int c = nfloor;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(&a.fene_floored[k], (unsigned long long)c);
  }
  if (errbits) atomicOr(&a.err[k], errbits);
}

// ---------------------------------------------------------------------------------------
size_t nl_stage_bytes(int, int cap) {
  return (size_t)(cap + RB_PAD) * sizeof(uint2) + (size_t)rb_home_cap(cap) * (sizeof(int) + sizeof(uint16_t));
}
size_t rel_bytes(int prec) { return prec ? sizeof(Rel<float>::T) : sizeof(Rel<double>::T); }

void launch_nl_rebuild(int prec, const NlArgs& a, int pblk, int ntile, bool bin, hipStream_t s) {
  if (bin) hipLaunchKernelGGL(k_nl_bin, dim3(pblk), dim3(256), 0, s, a);
  if (a.ntile_total > TILE_SUM_MAX)  // (fewer tiles: each tile sums its predecessors' counts)
    hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(1024), 0, s, a.tcnt, a.ntile_total, a.tstart);
  if (prec)
    hipLaunchKernelGGL(k_nl_rebuild<float>, dim3(ntile), dim3(NLB_THREADS), nl_stage_bytes(1, a.stage_cap), s, a);
  else
    hipLaunchKernelGGL(k_nl_rebuild<double>, dim3(ntile), dim3(NLB_THREADS), nl_stage_bytes(0, a.stage_cap), s, a);
}

void launch_nl_remap(const NlArgs& a, int pblk, hipStream_t s) {
  hipLaunchKernelGGL(k_nl_remap, dim3(pblk), dim3(256), 0, s, a);
}

template <typename R, int M>
static void launch_step_nh(const NlArgs& a, int ntile, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const size_t lds = StageLds<R>::bytes(a.stage_cap);
  // with events: hipExtLaunchKernelGGL stamps them at the dispatch's own start and end
  auto go = [&](auto kern) {
    if (ev0) hipExtLaunchKernelGGL(kern, dim3(ntile), dim3(NLB_THREADS), lds, s, ev0, ev1, 0, a);
    else hipLaunchKernelGGL(kern, dim3(ntile), dim3(NLB_THREADS), lds, s, a);
  };
  if (a.nh_uniform == 1) go(k_nl_step<R, M, 1>);
  else if (a.nh_uniform == 6) go(k_nl_step<R, M, 6>);
  else go(k_nl_step<R, M, 0>);
}

void launch_nl_step(int prec, int mode, const NlArgs& a, int ntile, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
#define KG_CASE(R, M) \
  case M: launch_step_nh<R, M>(a, ntile, s, ev0, ev1); break;
  if (prec) {
    switch (mode) {
      KG_CASE(float, F_OPEN)
      KG_CASE(float, F_OPEN | F_BIN)
      KG_CASE(float, F_CLOSE | F_OPEN)
      KG_CASE(float, F_CLOSE | F_OPEN | F_BIN)
      KG_CASE(float, F_CLOSE | F_STORE)
      default: break;
    }
  } else {
    switch (mode) {
      KG_CASE(double, F_OPEN)
      KG_CASE(double, F_OPEN | F_BIN)
      KG_CASE(double, F_CLOSE | F_OPEN)
      KG_CASE(double, F_CLOSE | F_OPEN | F_BIN)
      KG_CASE(double, F_CLOSE | F_STORE)
      default: break;
    }
  }
#undef KG_CASE
}

}  // namespace kgdb
