// Anisotropic three-point function (Sec. 2.3, eq. estimator_three):
//   xi3_A = sum_A w_i d_i w_j d_j w_k d_k / sum_A w_i w_j w_k
// over triplets of pixels from three distinct forests of one realisation.  A
// triangle is binned from a main vertex i by its sides r1 = x_j - x_i and
// r2 = x_k - x_i (x = D n): lengths r1, r2 in [r_0, r_max), angles theta1,
// theta2 to the line of sight of the vertex's quasar, and the cosine of the
// inner angle, flattened as A = (((k_r1 n_r + k_r2) n_c + k_c) n_t + k_t1) n_t
// + k_t2.  Every vertex and both side orders are entered, so an unordered
// triplet contributes six entries.  theta and cos alpha bins are half-open
// with the last one closed; a side of zero length is left out.
//
// Two ways of summing.  Both need, for a vertex pixel i, its partners: the
// pixels of the other forests whose side from i lies in the r and theta grids
// (a symmetric neighbour list with the box cut r_par, r_perp < r_max, which
// every side shorter than r_max passes).
//
// Pair kernel.  An entry is symmetric under the exchange of its two sides:
// cos alpha and the products are the same, only (r1, theta1) and (r2, theta2)
// swap.  So the kernel sums each unordered partner pair once, into half
// histograms indexed by the (r, theta) cells c1 <= c2 of the two sides, and the
// expansion writes both orders.  Partner lists of a batch of vertex pixels are
// first written to device memory ordered by cell (count, scan, fill).  The half
// histogram is cut into passes, runs of consecutive bins (whole rows c1, or a
// part of one) that fit an LDS slice; a work item is one pass of a group of
// vertex pixels, so a small patch still fills the chip and the slice goes to
// the global sums once per group.
//
// Direct kernel (grids beyond the pair kernel's tables).  A work item is one
// vertex forest; the workgroup takes its pixels one at a time, lists the
// partners in LDS and adds every ordered pair to the global sums.
//
// Everything is FP64; the geometry is written with explicit operation order so
// it rounds like its definition.
#include "lya_common.h"

namespace lya {

namespace {

constexpr int kBlock3 = 1024;
constexpr int kCap3 = 3072;    // partner pixels of one vertex held in LDS (direct kernel)
constexpr int kCapC = 2048;    // partner limit of variant 0
constexpr int kSliceT = 2048;  // n_cos n_theta limit of the pair kernel's grids
constexpr int kCellC = 1024;   // (r, theta) cells of a side, pair kernel
constexpr int kCosC = 256;     // cos alpha bins held in LDS (all kernels)
// Bins of the pair kernel's LDS slice: 20 B each, two workgroups of 16 waves a
// CU (160 KB), which is every wave slot.
constexpr int kSlice3 = 3840;

// Partners of one vertex pixel: unit vector of the side, w d, w, the side's
// bins k_r | k_t << 16 and the partner's forest.
template <int CAP>
struct Partners {
  double ux[CAP], uy[CAP], uz[CAP];
  double wd[CAP], w[CAP];
  int32_t key[CAP];
  int32_t fid[CAP];
};

struct Xi3Smem {
  Partners<kCap3> p;
  double ce[kCosC + 1];  // cos alpha edges
  int32_t m;  // partners appended
  int64_t item;
};

struct Xi3SmemP {
  double hn[kSlice3], hw[kSlice3];  // the pass's slice of the half sums
  uint32_t hc[kSlice3];
  double ce[kCosC + 1];  // cos alpha edges
  uint32_t unit;
};

// The XCD (accelerator complex die) the wave runs on, from the XCC_ID hardware
// register (any value is correct: it only picks a copy of the sums).
__device__ __forceinline__ unsigned xcd_id() {
  unsigned x;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(x));
  return x;
}

// Bin of x on a uniform axis [e0, e0 + n / inv), with the guess corrected by
// comparisons against the edge array; closed_last puts x == e_n in bin n - 1.
__device__ __forceinline__ int uniform_bin(double x, const double* e, int n, double e0, double inv,
                                           bool closed_last) {
  if (x < e[0]) return -1;
  if (x >= e[n]) return (closed_last && x == e[n]) ? n - 1 : -1;
  int k = (int)__dmul_rn(__dsub_rn(x, e0), inv);
  k = k < 0 ? 0 : (k > n - 1 ? n - 1 : k);
  while (k > 0 && x < e[k]) --k;
  while (k < n - 1 && x >= e[k + 1]) ++k;
  return k;
}

// The side from the vertex (xi, yi, zi) to the pixel q: false unless its length
// is in the r grid and its angle to the line of sight n of the vertex forest
// in the theta grid; else its unit vector and bins.
__device__ __forceinline__ bool side_of(const Xi3Args& a, const ForestInfo& fi, double xi, double yi, double zi,
                                        const Point3& q, double& ux, double& uy, double& uz, int& kr, int& kt) {
  const double dx = __dsub_rn(q.x, xi), dy = __dsub_rn(q.y, yi), dz = __dsub_rn(q.z, zi);
  const double r2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
  const double rm = a.r_edges[a.n_r];
  if (!(r2 <= rm * rm * (1.0 + 1e-12))) return false;  // sqrt(r2) >= r_max for certain
  const double r = sqrt(r2);
  kr = r > 0.0 ? uniform_bin(r, a.r_edges, a.n_r, a.r_e0, a.r_inv, false) : -1;
  if (kr < 0) return false;
  ux = __ddiv_rn(dx, r);
  uy = __ddiv_rn(dy, r);
  uz = __ddiv_rn(dz, r);
  double ct = __dadd_rn(__dadd_rn(__dmul_rn(ux, fi.nx), __dmul_rn(uy, fi.ny)), __dmul_rn(uz, fi.nz));
  ct = fmin(1.0, fmax(-1.0, ct));
  // theta >= t_k  <=>  cos theta <= cos t_k (theta in [0, pi])
  kt = 0;
  for (int k = 1; k < a.n_t; ++k) kt += ct <= a.cos_theta_edges[k] ? 1 : 0;
  return ct <= a.cos_theta_edges[0] && ct >= a.cos_theta_edges[a.n_t];
}

// Stores the partners of the vertex (xi, yi, zi) of forest fi as
// store(slot, ux, uy, uz, w d, w, k_r | k_t << 16, forest).  A wave per
// neighbour forest, lanes over its pixels; one LDS atomic per wave reserves
// the slots.  *m counts every partner, also those beyond cap (not stored).
template <typename Store>
__device__ __forceinline__ void gather_partners(const Xi3Args& a, const Item& item, const ForestInfo& fi,
                                                double xi, double yi, double zi, int cap, int32_t* m,
                                                Store&& store) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int NW = kBlock3 / 64;
  for (int t = wave; t < item.nb_count; t += NW) {
    const int g = a.sorted[a.nbr[item.nb_begin + t]];
    const ForestInfo gi = a.finfo[g];
    for (int e0 = 0; e0 < gi.npix; e0 += 64) {
      const int e = e0 + lane;
      bool keep = false;
      double ux = 0.0, uy = 0.0, uz = 0.0;
      int kr = -1, kt = 0;
      const int64_t pj = gi.pix0 + e;
      if (e < gi.npix) keep = side_of(a, fi, xi, yi, zi, a.pts[pj], ux, uy, uz, kr, kt);
      const uint64_t bal = __ballot(keep);
      if (bal == 0ull) continue;
      int base = 0;
      if (lane == 0) base = atomicAdd(m, __popcll(bal));
      base = __shfl(base, 0, 64);
      if (keep) {
        const int slot = base + __popcll(bal & ((1ull << lane) - 1ull));
        if (slot < cap) store(slot, ux, uy, uz, a.pts[pj].wd, a.pts[pj].w, kr | (kt << 16), g);
      }
    }
  }
}

// The cos alpha axis with its edges in LDS and the end edges in registers (a
// load from the edge array in global memory would be a vector load waited for
// on every entry: the sums the kernels write could alias it).
struct CosAxis {
  const double* e;  // LDS copy, [n + 1]
  double lo, hi, inv;
  int n;
};

// Bin of x on the cos alpha axis, the last bin closed (-1 outside).  The host
// accepts only edges within 1e-9 bins of lo + k d, and t = (x - lo) / d is
// computed to ~1e-13 bins, so a fractional part of t farther than 1e-8 from
// 0 and 1 puts x strictly inside bin floor(t); only closer values are settled
// by comparison with the edges.
__device__ __forceinline__ int cos_axis_bin(const CosAxis& c, double x) {
  if (x < c.lo) return -1;
  if (x >= c.hi) return x == c.hi ? c.n - 1 : -1;
  const double t = __dmul_rn(__dsub_rn(x, c.lo), c.inv);
  int k = (int)t;
  k = k < 0 ? 0 : (k > c.n - 1 ? c.n - 1 : k);
  const double fr = __dsub_rn(t, (double)k);
  if (fr > 1e-8 && fr < 1.0 - 1e-8) return k;
  while (k > 0 && x < c.e[k]) --k;
  while (k < c.n - 1 && x >= c.e[k + 1]) ++k;
  return k;
}

// Copies the cos alpha edges to LDS (the caller synchronises before use).
__device__ __forceinline__ CosAxis load_cos_axis(const Xi3Args& a, double* lds) {
  for (int k = threadIdx.x; k <= a.n_c; k += kBlock3) lds[k] = a.cos_edges[k];
  return CosAxis{lds, a.cos_edges[0], a.cos_edges[a.n_c], a.c_inv, a.n_c};
}

template <int CAP>
struct LdsStore {
  Partners<CAP>& P;
  __device__ __forceinline__ void operator()(int s, double ux, double uy, double uz, double wd, double w, int key,
                                             int fid) const {
    P.ux[s] = ux;
    P.uy[s] = uy;
    P.uz[s] = uz;
    P.wd[s] = wd;
    P.w[s] = w;
    P.key[s] = key;
    P.fid[s] = fid;
  }
};

// cos alpha bin of the partners j, k (-1 outside the grid).
template <int CAP>
__device__ __forceinline__ int cos_bin(const CosAxis& cx, const Partners<CAP>& P, int j, int k) {
  double ca = __dadd_rn(__dadd_rn(__dmul_rn(P.ux[j], P.ux[k]), __dmul_rn(P.uy[j], P.uy[k])),
                        __dmul_rn(P.uz[j], P.uz[k]));
  ca = fmin(1.0, fmax(-1.0, ca));
  return cos_axis_bin(cx, ca);
}

// The sums this workgroup adds to for vertex forest f (input index): the slab
// of f's realisation (and subsample), in the copy of the workgroup's XCD when
// there is one copy per XCD (the copies spread the device-wide atomics over
// more addresses; a second kernel adds them up).
__device__ __forceinline__ int64_t sums_base(const Xi3Args& a, const ForestInfo& fi, int f) {
  const int copy = a.n_copies > 1 ? (int)(xcd_id() % (unsigned)a.n_copies) : 0;
  const int64_t slab = a.sub ? (int64_t)fi.real * a.n_sub + a.sub[f] : (int64_t)fi.real;
  return (int64_t)copy * a.copy_stride + slab * a.n_bins;
}

// Direct kernel: every entry goes to the global sums with three atomics.
__global__ __launch_bounds__(kBlock3) void xi3_kernel(Xi3Args a) {
  __shared__ Xi3Smem sm;
  const int tid = threadIdx.x;
  const int nr = a.n_r, nt = a.n_t, nc = a.n_c;
  const CosAxis cx = load_cos_axis(a, sm.ce);

  for (;;) {
    __syncthreads();  // every thread has read the previous item
    if (tid == 0) sm.item = (int64_t)atomicAdd(a.counter, 1u);
    __syncthreads();
    const int64_t it = sm.item;
    if (it >= a.n_items) break;
    const Item item = a.items[it];
    const int f = a.sorted[item.p];
    const ForestInfo fi = a.finfo[f];
    const int64_t obase = sums_base(a, fi, f);

    for (int i = 0; i < fi.npix; ++i) {
      const int64_t pi = fi.pix0 + i;
      const double wdi = a.pts[pi].wd, wi = a.pts[pi].w;
      __syncthreads();  // the previous vertex's pairs have been read
      if (tid == 0) sm.m = 0;
      __syncthreads();
      gather_partners(a, item, fi, a.pts[pi].x, a.pts[pi].y, a.pts[pi].z, kCap3, &sm.m, LdsStore<kCap3>{sm.p});
      __syncthreads();
      const int m = sm.m;
      if (m > kCap3) {
        // the call reports the overflow and its sums are not used
        if (tid == 0) atomicOr(&a.glob->flag, kBadCap3);
        continue;
      }
      if (m < 2) continue;

      // ---- ordered partner pairs (j, k) of different forests, t = j m + k
      const int64_t total = (int64_t)m * m;
      int j = tid / m, k = tid - (tid / m) * m;
      const int dj = kBlock3 / m, dk = kBlock3 - dj * m;
      for (int64_t t = tid; t < total; t += kBlock3) {
        if (sm.p.fid[j] != sm.p.fid[k]) {
          const int kc = cos_bin(cx, sm.p, j, k);
          if (kc >= 0) {
            const int kj = sm.p.key[j], kk = sm.p.key[k];
            const int64_t A = ((((int64_t)(kj & 0xffff) * nr + (kk & 0xffff)) * nc + kc) * nt + (kj >> 16)) * nt +
                              (kk >> 16);
            const double pn = __dmul_rn(__dmul_rn(wdi, sm.p.wd[j]), sm.p.wd[k]);
            const double pw = __dmul_rn(__dmul_rn(wi, sm.p.w[j]), sm.p.w[k]);
            atomicAdd(&a.num[obase + A], pn);
            atomicAdd(&a.wsum[obase + A], pw);
            atomicAdd(&a.ntrip[obase + A], 1ull);
          }
        }
        k += dk;
        j += dj;
        if (k >= m) {
          k -= m;
          ++j;
        }
      }
    }
  }
}

// ---- pair kernel: partner lists

constexpr int kListWaves = 4;    // vertex pixels per workgroup of the list kernels
constexpr int kListSplit = 8;    // workgroups per forest

// f(pixel, forest) for every pixel of the neighbours nbr[nb0, nb0 + n), lanes
// over a forest's pixels; the lanes first fetch 64 neighbours' places at once,
// so that the chain of dependent loads is paid once for them all.
template <typename F>
__device__ __forceinline__ void each_candidate(const Xi3Args& a, int64_t nb0, int64_t n, F&& f) {
  const int lane = threadIdx.x & 63;
  for (int64_t t0 = 0; t0 < n; t0 += 64) {
    const int nt = (int)min((int64_t)64, n - t0);
    int g = 0, npix = 0;
    int64_t pix0 = 0;
    if (lane < nt) {
      g = a.sorted[a.nbr[nb0 + t0 + lane]];
      pix0 = a.finfo[g].pix0;
      npix = a.finfo[g].npix;
    }
    for (int t = 0; t < nt; ++t) {
      const int gt = __builtin_amdgcn_readlane(g, t), nj = __builtin_amdgcn_readlane(npix, t);
      const int64_t p0 = ((int64_t)__builtin_amdgcn_readlane((int)(pix0 >> 32), t) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)pix0, t);
      for (int e = lane; e < nj; e += 64) f(p0 + e, gt);
    }
  }
}

// Partners of every vertex pixel (cnt[pixel]) and the largest count.  A wave
// per vertex pixel, lanes over the neighbours' pixels.
__global__ __launch_bounds__(64 * kListWaves) void xi3_count_kernel(Xi3Args a, int p0) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t p = p0 + blockIdx.x / kListSplit;
  const int f = a.sorted[p];
  const ForestInfo fi = a.finfo[f];
  const int64_t nb0 = a.nb_off[p], nbc = a.nb_cnt[p];
  int most = 0;
  for (int i = (int)(blockIdx.x % kListSplit) * kListWaves + wave; i < fi.npix; i += kListSplit * kListWaves) {
    const Point3 v = a.pts[fi.pix0 + i];
    int m = 0;
    each_candidate(a, nb0, nbc, [&](int64_t pj, int) {
      double ux, uy, uz;
      int kr, kt;
      m += side_of(a, fi, v.x, v.y, v.z, a.pts[pj], ux, uy, uz, kr, kt) ? 1 : 0;
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m += __shfl_xor(m, o, 64);
    if (lane == 0) a.p_cnt[fi.pix0 + i] = m;
    most = max(most, m);
  }
  if (lane == 0 && most > 0) atomicMax(a.p_most, most);
}

// The partner lists of vertex pixels [v0, v0 + n_v), ordered by cell k_r n_t +
// k_t: counts per cell in LDS, a scan (written as the cells' first positions),
// then the partners go to their places.  A wave per vertex pixel.
__global__ __launch_bounds__(64 * kListWaves) void xi3_fill_kernel(Xi3Args a, int p0) {
  __shared__ int32_t cell_pos[kListWaves][kCellC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t* pos = cell_pos[wave];
  const int64_t p = p0 + blockIdx.x / kListSplit;
  const int f = a.sorted[p];
  const ForestInfo fi = a.finfo[f];
  const int64_t nb0 = a.nb_off[p], nbc = a.nb_cnt[p];
  const int ncell = a.n_r * a.n_t, per = (ncell + 63) / 64;
  const int64_t off0 = a.p_off[a.v0];
  for (int i = (int)(blockIdx.x % kListSplit) * kListWaves + wave; i < fi.npix; i += kListSplit * kListWaves) {
    const int64_t v = fi.pix0 + i - a.v0;
    if (v < 0 || v >= a.n_v) continue;
    const Point3 q = a.pts[fi.pix0 + i];
    for (int c = lane; c < ncell; c += 64) pos[c] = 0;
    Partner3* list = a.plist + (a.p_off[fi.pix0 + i] - off0);
    // the wave's own LDS area and program order: no barrier between the steps
    for (int step = 0; step < 2; ++step) {
      each_candidate(a, nb0, nbc, [&](int64_t ipix, int g) {
        double ux, uy, uz;
        int kr, kt;
        const Point3 pj = a.pts[ipix];
        if (!side_of(a, fi, q.x, q.y, q.z, pj, ux, uy, uz, kr, kt)) return;
        const int cell = kr * a.n_t + kt;
        const int at = atomicAdd(&pos[cell], 1);
        if (step)
          list[at] = Partner3{ux, uy, uz, pj.wd, pj.w, g, (cell * ncell - cell * (cell - 1) / 2 - cell) * a.n_c,
                              cell * a.n_c, {0, 0, 0}};
      });
      if (step) break;
      __threadfence_block();
      const int c0 = lane * per, c1 = min(ncell, c0 + per);
      int own = 0;
      for (int c = c0; c < c1; ++c) own += pos[c];
      int incl = own;
      for (int d = 1; d < 64; d <<= 1) {
        const int x = __shfl_up(incl, d, 64);
        if (lane >= d) incl += x;
      }
      int run = incl - own;
      int32_t* cs = a.cstart + v * (ncell + 1);
      for (int c = c0; c < c1; ++c) {
        const int n = pos[c];
        cs[c] = run;
        pos[c] = run;
        run += n;
      }
      if (lane == 63) cs[ncell] = incl;
      __threadfence_block();
    }
    if (lane == 0) {
      const int slab = a.sub ? fi.real * a.n_sub + a.sub[f] : fi.real;
      a.vinfo[v] = Vertex3{a.p_off[fi.pix0 + i] - off0, slab, 0, q.wd, q.w};
    }
  }
}

// ---- pair kernel: the pass of a group of vertex pixels

// Loads through the constant address space: with a wave-uniform address the
// compiler emits scalar loads.  Only data that earlier kernels wrote.
typedef int x3_i16 __attribute__((ext_vector_type(16)));
#define X3_CONST(T, p) (*(const __attribute__((address_space(4))) T*)(p))

__device__ __forceinline__ Partner3 uniform_partner(const Partner3* p) {
  const x3_i16 v = X3_CONST(x3_i16, p);
  auto dbl = [&](int k) { return __hiloint2double(v[2 * k + 1], v[2 * k]); };
  return Partner3{dbl(0), dbl(1), dbl(2), dbl(3), dbl(4), v[10], v[11], v[12], {0, 0, 0}};
}

// What a lane keeps of its side-2 partner and of the runs it is summing.
struct Lane3 {
  double kx, ky, kz;  // side's unit vector over the cos alpha bin width
  double kwd, kw;     // w d, w times the vertex's
  int32_t kfid, kofs;
};

// Sums the pairs (j, k) of one vertex: k of the 64 lanes (each one partner of
// side 2), j over [j0, j1) of the list; with DIAG only j before k.
//
// 2^20 + x, x the coordinate of cos alpha in bins, has the bin in its upper
// word and the fraction in its lower one: three FMAs give both.  The bin is
// settled by the definition where the fraction is within 1e-8 of an edge; on axes
// with bins so narrow that the coordinate's rounding reaches that (Xi3Args::near),
// for every pair.
//
// Runs of consecutive j in one bin are summed in registers.  A finished run
// waits in the lane (one slot) and goes to LDS only when some lane needs its
// slot again: an LDS atomic costs the CU 8 (f64) or 4 (u32) clocks whatever
// number of lanes is on, and most runs end at different j in different lanes.
// Live, waiting and ending lanes are kept as 64-bit masks in scalar registers.
template <bool DIAG>
__device__ __forceinline__ void sum_pairs(const Xi3Args& a, Xi3SmemP& sm, const CosAxis& cx, const Partner3* list,
                                          int j0, int j1, const Lane3& L, uint64_t on, int kpos, double c0) {
  constexpr uint32_t kMagicHi = 0x41300000u;  // upper word of 2^20
  const int nc = a.n_c;
  uint32_t key = 0, pkey = 0;  // bin minus (first j << 16); bin plus (count << 16)
  double rn = 0.0, rw = 0.0, pn = 0.0, pw = 0.0;
  uint64_t live = 0ull, pend = 0ull;
  auto flush = [&]() __attribute__((always_inline)) {
    if (lane_in(pend)) {
      const uint32_t s = pkey & 0xffffu;
      atomicAdd(&sm.hn[s], __dmul_rn(pn, L.kwd));
      atomicAdd(&sm.hw[s], __dmul_rn(pw, L.kw));
      atomicAdd(&sm.hc[s], pkey >> 16);
    }
    pend = 0ull;
  };
  auto finish = [&](uint64_t m, uint32_t jr) __attribute__((always_inline)) {
    if (m & pend) flush();
    if (lane_in(m)) {
      keep_branch();
      pkey = key + (jr << 16);
      pn = rn;
      pw = rw;
    }
    pend |= m;
  };
  auto one = [&](const Partner3& J, int j) __attribute__((always_inline)) {
    const uint32_t jr = (uint32_t)(j - j0);
    uint64_t ok = on & __ballot(J.fid != L.kfid);
    if constexpr (DIAG) ok &= __ballot(j < kpos);
    const double u = fma(J.ux, L.kx, fma(J.uy, L.ky, fma(J.uz, L.kz, c0)));
    uint32_t kc = (uint32_t)__double2hiint(u) - kMagicHi;
    const uint64_t near = ok & __ballot((uint32_t)__double2loint(u) <= a.near);
    if (near) {
      if (lane_in(near)) {
        const Partner3 k = list[kpos];
        double ca = __dadd_rn(__dadd_rn(__dmul_rn(J.ux, k.ux), __dmul_rn(J.uy, k.uy)), __dmul_rn(J.uz, k.uz));
        ca = fmin(1.0, fmax(-1.0, ca));
        kc = (uint32_t)cos_axis_bin(cx, ca);
      }
    }
    const uint64_t in = ok & __ballot(kc < (uint32_t)nc);
    const uint32_t bin = kc + (uint32_t)(J.row + L.kofs);
    const uint64_t ne = __ballot((uint16_t)bin != (uint16_t)key);
    const uint64_t ends = live & (ne | ~in), starts = in & (ne | ~live);
    if (ends) finish(ends, jr);
    if (lane_in(starts)) {
      keep_branch();
      key = bin - (jr << 16);
      rn = 0.0;
      rw = 0.0;
    }
    live = in;
    rn += J.wd;
    rw += J.w;
  };
  int j = j0;
  for (; j + 2 <= j1; j += 2) {
    const Partner3 A = uniform_partner(list + j), B = uniform_partner(list + j + 1);
    one(A, j);
    one(B, j + 1);
  }
  if (j < j1) one(uniform_partner(list + j), j);
  if (live) finish(live, (uint32_t)(j1 - j0));
  if (pend) flush();
}

// One work item: pass `unit % n_pass` of vertex group `unit / n_pass`.  The
// waves take the (vertex, 64 side-2 partners) tasks of the group in turn, with
// no barrier but the flush's.  The lanes of a task take partners spread over
// the list, so that few lanes add to one LDS bin at once.
//
// Bound by issue, vector (~75 clocks per 64 partner pairs) and scalar (the lane
// masks) alike, at about half of each unit's rate.  120 forests at 75 / deg^2, r
// to 80 Mpc/h in 20 x 10 x 20 bins (1.3e10 partner pairs): 22 ms, and 24 ms for
// the call; one vertex pixel per workgroup with both orders of every pair, a
// pass per side-1 cell and the three sums added at the end of every run took
// 425 ms (120 workgroups, two barriers per pass).  200 forests to 40 Mpc/h: 65
// ms before, 5.5 (call 8.2).
__global__ __launch_bounds__(kBlock3, 8) void xi3_pair_kernel(Xi3Args a) {
  __shared__ Xi3SmemP sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NW = kBlock3 / 64;
  const int ncell = a.n_r * a.n_t;
  const CosAxis cx = load_cos_axis(a, sm.ce);
  const double c0 = 1048576.0 - cx.lo * cx.inv + 1e-8;  // 2^20, the axis origin and half the edge guard
  const int64_t copy = a.n_copies > 1 ? (int64_t)(xcd_id() % (unsigned)a.n_copies) * a.copy_stride : 0;

  for (int s = tid; s < kSlice3; s += kBlock3) {
    sm.hn[s] = 0.0;
    sm.hw[s] = 0.0;
    sm.hc[s] = 0u;
  }

  for (;;) {
    __syncthreads();  // the previous unit's slice has been flushed and its number read
    if (tid == 0) sm.unit = atomicAdd(a.counter, 1u);
    __syncthreads();
    const uint32_t unit = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.unit);
    if (unit >= (uint32_t)a.n_units) break;
    const int64_t va = (int64_t)(unit / (uint32_t)a.n_pass) * a.group;
    const int64_t vb = min(va + a.group, a.n_v);
    const Pass3 P = a.passes[unit % (uint32_t)a.n_pass];
    int cur = -1, task = 0;
    // adds the slice's non-zero bins to the slab's half sums and clears it
    auto flush_slice = [&]() {
      __syncthreads();
      const int64_t at = copy + (int64_t)cur * a.n_half + P.base;
      for (int s = tid; s < P.nslice; s += kBlock3) {
        const uint32_t vc = sm.hc[s];
        if (vc == 0u) continue;
        atomicAdd(&a.num[at + s], sm.hn[s]);
        atomicAdd(&a.wsum[at + s], sm.hw[s]);
        atomicAdd(&a.ntrip[at + s], (unsigned long long)vc);
        sm.hn[s] = 0.0;
        sm.hw[s] = 0.0;
        sm.hc[s] = 0u;
      }
      __syncthreads();
    };
    for (int64_t v = va; v < vb; ++v) {
      const Vertex3* vp = a.vinfo + v;
      const int32_t* cs = a.cstart + v * (ncell + 1);
      const int j0 = X3_CONST(int, cs + P.ca), j1 = X3_CONST(int, cs + P.cb);
      if (j0 == j1) continue;
      const int slab = X3_CONST(int, &vp->slab);
      if (slab != cur) {
        if (cur >= 0) flush_slice();
        cur = slab;
      }
      const Partner3* list = a.plist + X3_CONST(int64_t, &vp->off);
      const double vwd = X3_CONST(double, &vp->wd), vw = X3_CONST(double, &vp->w);
      // side-2 partners in later cells, then those in the pass's own cells
      // (there only the pairs in list order)
#pragma unroll 1
      for (int part = 0; part < 2; ++part) {
        const int ka = part ? j0 : X3_CONST(int, cs + P.k0), kb = part ? (P.diag ? j1 : j0) : X3_CONST(int, cs + P.k1);
        const int mk = kb - ka;
        if (mk <= 0) continue;
        const int nkc = (mk + 63) >> 6;
        int c = (wv - task) & (NW - 1);
        task = (task + nkc) & (NW - 1);
        for (; c < nkc; c += NW) {
          const int kk = lane * nkc + c;
          const uint64_t on = __ballot(kk < mk);
          const int kpos = ka + (kk < mk ? kk : 0);
          const Partner3 k = list[kpos];
          const Lane3 L{k.ux * cx.inv, k.uy * cx.inv, k.uz * cx.inv, __dmul_rn(vwd, k.wd), __dmul_rn(vw, k.w),
                        k.fid, k.col - (int)P.base};
          if (part) sum_pairs<true>(a, sm, cx, list, j0, j1, L, on, kpos, c0);
          else sum_pairs<false>(a, sm, cx, list, j0, j1, L, on, kpos, c0);
        }
      }
    }
    if (cur >= 0) flush_slice();
  }
}

// The full sums from the half sums' copies (copy c at c * stride): entry
// (c1, c2, k_c) is half bin (min, max, k_c), and both orders of a pair inside
// one cell meet in the same bin.
__global__ void xi3_expand_kernel(Xi3Args a, int64_t n, double* num, double* wsum, int64_t* ntrip) {
  const int nr = a.n_r, nt = a.n_t, nc = a.n_c, ncell = nr * nt;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t slab = i / a.n_bins;
    int64_t q = i - slab * a.n_bins;
    const int t2 = (int)(q % nt);
    q /= nt;
    const int t1 = (int)(q % nt);
    q /= nt;
    const int kc = (int)(q % nc);
    q /= nc;
    const int r2 = (int)(q % nr), r1 = (int)(q / nr);
    const int ca = r1 * nt + t1, cb = r2 * nt + t2;
    const int64_t lo = min(ca, cb), hi = max(ca, cb);
    const int64_t h = slab * a.n_half + (lo * ncell - lo * (lo - 1) / 2 + hi - lo) * nc + kc;
    double sn = 0.0, sw = 0.0;
    unsigned long long sc = 0;
    for (int c = 0; c < a.n_copies; ++c) {
      sn += a.num[c * a.copy_stride + h];
      sw += a.wsum[c * a.copy_stride + h];
      sc += a.ntrip[c * a.copy_stride + h];
    }
    if (ca == cb) {
      sn += sn;
      sw += sw;
      sc += sc;
    }
    num[i] = sn;
    wsum[i] = sw;
    ntrip[i] = (int64_t)sc;
  }
}

// out = sum over the copies (copy c at c * stride).
__global__ void xi3_reduce_kernel(const double* num_c, const double* wsum_c, const unsigned long long* cnt_c,
                                  int n_copies, int64_t stride, int64_t n, double* num, double* wsum,
                                  int64_t* ntrip) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double sn = 0.0, sw = 0.0;
    unsigned long long sc = 0;
    for (int c = 0; c < n_copies; ++c) {
      sn += num_c[c * stride + i];
      sw += wsum_c[c * stride + i];
      sc += cnt_c[c * stride + i];
    }
    num[i] = sn;
    wsum[i] = sw;
    ntrip[i] = (int64_t)sc;
  }
}

// Pixel positions x = D n and the products w d, w (FP64), one wave per forest.
__global__ __launch_bounds__(256) void xi3_points_kernel(lya_forests F, const ForestInfo* finfo,
                                                       const double* delta, Point3* pts) {
  const int lane = threadIdx.x & 63;
  const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (f >= F.n_forests) return;
  const ForestInfo fi = finfo[f];
  for (int k = lane; k < fi.npix; k += 64) {
    const int64_t i = fi.pix0 + k;
    const double D = F.dist[i], w = F.weight[i];
    Point3 p;
    p.x = __dmul_rn(D, fi.nx);
    p.y = __dmul_rn(D, fi.ny);
    p.z = __dmul_rn(D, fi.nz);
    p.wd = __dmul_rn(w, delta[i]);
    p.w = w;
    p.pad = 0.0;
    pts[i] = p;
  }
}

}  // namespace

hipError_t launch_xi3_points(const lya_forests* F, const ForestInfo* finfo, const double* delta, Point3* pts,
                             hipStream_t st) {
  if (F->n_forests == 0) return hipSuccess;
  hipLaunchKernelGGL(xi3_points_kernel, dim3((unsigned)((F->n_forests + 3) / 4)), dim3(256), 0, st, *F, finfo,
                     delta, pts);
  return hipGetLastError();
}

hipError_t launch_xi3_reduce(const double* num_c, const double* wsum_c, const unsigned long long* cnt_c,
                             int n_copies, int64_t stride, int64_t n, double* num, double* wsum, int64_t* ntrip,
                             hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int64_t want = (n + 255) / 256;
  const unsigned blocks = (unsigned)(want < 8192 ? want : 8192);
  hipLaunchKernelGGL(xi3_reduce_kernel, dim3(blocks), dim3(256), 0, st, num_c, wsum_c, cnt_c, n_copies, stride, n,
                     num, wsum, ntrip);
  return hipGetLastError();
}

hipError_t launch_xi3_direct(const Xi3Args& a, int blocks, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  hipLaunchKernelGGL(xi3_kernel, dim3(blocks), dim3(kBlock3), 0, st, a);
  return hipGetLastError();
}

// The list kernels over sorted positions, 2^20 of them a launch (2^31 threads; a launch
// takes less than 2^32).
template <typename Kernel>
static hipError_t launch_lists(Kernel kernel, const Xi3Args& a, int64_t n_forests, hipStream_t st) {
  constexpr int64_t kMost = 1 << 20;
  for (int64_t p0 = 0; p0 < n_forests; p0 += kMost) {
    const int64_t n = n_forests - p0 < kMost ? n_forests - p0 : kMost;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n * kListSplit)), dim3(64 * kListWaves), 0, st, a, (int)p0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_xi3_count(const Xi3Args& a, int64_t n_forests, hipStream_t st) {
  return launch_lists(xi3_count_kernel, a, n_forests, st);
}

hipError_t launch_xi3_pairs(const Xi3Args& a, int64_t n_forests, int blocks, hipStream_t st) {
  const hipError_t e = launch_lists(xi3_fill_kernel, a, n_forests, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(xi3_pair_kernel, dim3(blocks), dim3(kBlock3), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_xi3_expand(const Xi3Args& a, int64_t n, double* num, double* wsum, int64_t* ntrip, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int64_t want = (n + 255) / 256;
  hipLaunchKernelGGL(xi3_expand_kernel, dim3((unsigned)(want < 8192 ? want : 8192)), dim3(256), 0, st, a, n, num,
                     wsum, ntrip);
  return hipGetLastError();
}

int xi3_blocks_per_cu(bool pairs) {
  int n = 0;
  const hipError_t e = pairs ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, xi3_pair_kernel, kBlock3, 0)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, xi3_kernel, kBlock3, 0);
  if (e != hipSuccess) return 1;
  return n > 0 ? n : 1;
}

// Passes over the half histogram: whole rows c1 (with every c2 >= c1) while
// they fit the slice, or parts of a row that does not.
int xi3_passes(int n_r, int n_t, int n_c, Pass3* out) {
  const int ncell = n_r * n_t;
  auto at = [&](int64_t c1, int64_t c2) { return (c1 * ncell - c1 * (c1 - 1) / 2 + c2 - c1) * n_c; };
  int n = 0;
  for (int ca = 0; ca < ncell;) {
    int cb = ca;
    int64_t bins = 0;
    while (cb < ncell && bins + (int64_t)(ncell - cb) * n_c <= kSlice3) bins += (int64_t)(ncell - cb++) * n_c;
    if (cb > ca) {
      if (out) out[n] = Pass3{ca, cb, cb, ncell, 1, (int32_t)bins, at(ca, ca)};
      ++n;
      ca = cb;
      continue;
    }
    const int step = kSlice3 / n_c;  // >= 15
    for (int k = ca; k < ncell; k += step) {
      const int ke = k + step < ncell ? k + step : ncell;
      if (out) out[n] = Pass3{ca, ca + 1, k > ca ? k : ca + 1, ke, k == ca ? 1 : 0, (ke - k) * n_c, at(ca, k)};
      ++n;
    }
    ++ca;
  }
  return n;
}

// The coordinate's rounding: three sides scaled by 1 / d (half an ulp each, at most
// 1 / d in size), three FMAs and the axis origin, in all below 10 x 2^-53 / d bins,
// and 2^-33 of the sum's last bit.
uint32_t xi3_near(double c_inv) {
  constexpr uint32_t kNear = 86u;  // 2e-8 bins in units of 2^-32: 1e-8 to either side
  return c_inv <= 1e6 ? kNear : 0xffffffffu;
}

int xi3_partner_capacity() { return kCap3; }

int xi3_combine_capacity() { return kCapC; }

bool xi3_can_combine(int n_r, int n_t, int n_c) {
  return (int64_t)n_r * n_t <= kCellC && (int64_t)n_c * n_t <= kSliceT;
}

int xi3_max_cos_bins() { return kCosC; }

}  // namespace lya
