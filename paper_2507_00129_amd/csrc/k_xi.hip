// The xi pair kernel: weighted pixel-pair histograms of Sec. 2.1,
// eq. estimator_two (numerator sum w_i d_i w_j d_j, denominator sum w_i w_j,
// pair count), over every work item of the forest-pair list.
//
// Layout of the work.  A work item is one forest f (at sorted position p)
// against a few neighbour forests g; each wave takes items by itself.  The
// neighbours' pixels form one concatenated stream; the wave takes 64
// consecutive stream pixels, one per lane, and loops over the pixels of f,
// which are identical for all lanes and come through scalar loads.  Each lane
// thus evaluates one pixel pair per iteration: r_par = |D_i - D_j| c, r_perp =
// (D_i + D_j) s with the lane's own (s, c), then the bin and the two products.
//
// Geometry.  Both forms compute the bin coordinates x = (r - e0) / dr in FP64
// (on gfx950 an FP64 add, multiply or FMA issues in the 4 clocks of an FP32
// FMA, compare or conversion) as 2^20 + x + g: the upper word then holds the
// bin and the lower one the fraction, so a bin costs no conversion and the edge
// guard is one unsigned compare per axis.  A pair whose fraction is within g =
// 1e-8 of an edge (the coordinates are good to ~3e-10) is binned by comparing
// its r with the edge array.  The FP32 form's products are FP32.
//
// On other than uniform edges (kAnyEdges) a lane carries its pixel's interval on each
// axis from one pixel of f to the next: four FP64 compares a pair while both hold, else
// a step to the next interval or a search.  148 forests of 227 to 666 pixels, 15 x 15
// graded bins: 4.0 ms, against 7.3 with FP32 coordinates and a search per pair, and 9.7
// with FP64 coordinates before the search, which is as long as the rest together.
//
// Runs.  Consecutive pixels of f that fall in one bin are summed in registers
// in the form's arithmetic (a run also ends at every 32nd pixel of f); the run
// sums are added in FP64.  An LDS atomic costs its CU 8 (f64) or 4 (u32)
// clocks whatever number of lanes is on, and the lanes' runs end at different
// iterations, so a finished run waits in its lane (one slot) and the waiting
// runs go to LDS together when some lane needs its slot again.  On the
// eBOSS-like workload that is every second iteration instead of four of five
// (22 lanes each), with 0.5 Mpc/h pixels one in nine instead of one in two.
// Pairs outside the grid form runs in a bin of their own that is never read.
//
// Histograms live in LDS, one copy per workgroup (FP64 sums, u32 counts, each
// an array of its own: consecutive bins then fall on consecutive banks), and
// are added to the global FP64 outputs at the end, when the realisation changes
// and before a count could overflow.  The waves of a workgroup meet only
// there: items are ordered by output slab, and a wave whose next item needs
// another slab (or would overflow the counts) waits at a barrier that the
// others reach in turn; they then flush and go on with the smallest slab any of
// them holds.  With several slabs a workgroup takes its tickets in runs, so
// that it meets a few of the slabs only: with all workgroups going through all
// slabs together, 26 subsamples of 1961 forests spent 9 of 11 ms in flushes.
//
// Deterministic form (DET).  The run sums (at most 32 products of one lane,
// summed in a fixed order in the form's arithmetic) are scaled by 2^s (s per
// realisation, from its largest |w d| and w, so that |run sum| 2^s <= 2^55),
// rounded to integers and summed exactly in integers, in LDS and then in
// global memory; integer addition does not depend on the order, so the sums are
// bitwise reproducible and identical for a realisation alone or batched (a run
// depends only on the forest pair and the pixel, not on how the work is split).
//
// Bin means.  The MEANS form also sums w_i w_j x_par, w_i w_j x_perp (bin
// coordinates in the form's arithmetic) and w_i w_j (z_i + z_j), with the
// pixel redshift z packed with the records; a finalisation turns them into the
// weighted mean r_par, r_perp and z of each bin, the coordinate columns of the
// correlation output.
//
// Measured (MI355X, 8000 forests at 75 / deg^2, 50 x 50 bins to 200 Mpc/h,
// 4.35e10 candidate and 2.4e10 in-grid pairs, whole call): 19.5 ms, against
// 26.8 of workgroup-wide items with 16-byte bins, FP32 geometry and an atomic at
// each iteration with the end of a run; FP64, 5000 forests: 10.0 against 13.9; bin
// means (5000 forests at 100 / deg^2) 26.0 against 33.6, the deterministic form 16.0
// against 24.7, 0.5 Mpc/h pixels (4.3e11 candidate pairs) 122 against 214.  Bound by
// the vector units (about 19 instructions an iteration, three quarters of the time)
// and by the LDS atomics next.
#include <type_traits>

#include "lya_bin.h"
#include "lya_common.h"
#include "lya_pairs.h"

namespace lya {

namespace {

// Fixed-point terms of the deterministic form: q = rint(x), |q| <= 2^55.  A
// workgroup sums them in LDS in a 64-bit low and a 32-bit high word; its sum S
// goes to the global sums split as S = hi 2^28 + lo, 0 <= lo < 2^28, the two
// words in separate 64-bit integers (two's complement for hi), exact for fewer
// than 2^36 terms.  The finalisation carries lo into hi, so the result depends
// only on the total.
// A term is a run sum of at most kRunMax = 2^5 products below m^2, so the
// scale is 2^(kDetBits - 2 e) = 2^(50 - 2 e) for m < 2^e.
constexpr int kDetShift = 28;
constexpr int kDetBits = 50;

// Adds q to the 96-bit integer (hi, lo): the upper word changes only on a carry
// or borrow, once in some hundred additions.
__device__ __forceinline__ void det_add(unsigned long long* lo, int* hi, double x) {
  const long long q = __double2ll_rn(x);
  const unsigned long long old = atomicAdd(lo, (unsigned long long)q);
  const int c = (int)(old + (unsigned long long)q < old) + (q < 0 ? -1 : 0);
  if (c != 0) atomicAdd(hi, c);
}

// s for products below m^2, m given by the bits of a non-negative double:
// s = kDetBits - 2 e with m < 2^e (clamped to the double's range).  A run sum
// then stays below 2^5 m^2 2^s <= 2^55, and rounding it to an integer adds at
// most 0.5 2^-s = 2^(2 e - 51) <= 2^-49 m^2 (m >= 2^(e - 1)).
__device__ __forceinline__ int det_shift(unsigned long long mbits) {
  if (mbits == 0ull) return 0;
  const int E = (int)(mbits >> 52);
  const int e = (E == 0 ? 1 : E) - 1022;
  const int sh = kDetBits - 2 * e;
  return sh > 1000 ? 1000 : (sh < -1000 ? -1000 : sh);
}

// LDS sums: arrays of nd = n_bins + spare entries, the last ones for the pairs
// outside the grid: one per lane (one for all would be a conflict of all), or one
// where the bin means' arrays fill the LDS.  FP64 sums first: N, W and, with MEANS,
// w w x_par, w w x_perp, w w (z_i + z_j); DET: the 64-bit low words of N and W, then their 32-bit high
// words; the u32 counts last.
template <bool MEANS, bool DET>
constexpr int n_f64() { return MEANS ? 5 : 2; }
template <bool MEANS, bool DET>
constexpr size_t smem_per_bin() {
  return n_f64<MEANS, DET>() * sizeof(double) + (DET ? 2 * sizeof(int) : 0) + sizeof(unsigned);
}

// The kernel's arguments, read where they are used: what only the fetch of an
// item or a flush needs does not stay in scalar registers through the pair loop
// (8 waves per SIMD leave 80).
typedef const __attribute__((address_space(4))) XiArgs* KArgs;
__device__ __forceinline__ KArgs kargs() {
  KArgs p = (KArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// Adds the LDS sums to the output slab and clears them (the whole workgroup).  Lanes
// take consecutive output bins, so that a wave's atomics fall into few cache lines,
// and each workgroup starts at another bin: they end together, and at one address
// atomics take 12 ns each.
template <int BLOCK, bool MEANS, bool DET>
__device__ __forceinline__ void flush_hist(double* h, int slab) {
  const KArgs a = kargs();
  const int NP = a->g.n_par, NT = a->g.n_perp, nb = NP * NT, nd = nb + a->spare;
  const int64_t base = (int64_t)slab * nb;
  int* hc = (int*)(h + n_f64<MEANS, DET>() * nd);  // DET high words
  unsigned* hn = (unsigned*)(hc + (DET ? 2 * nd : 0));
  const int first = (int)((blockIdx.x * 64u) % (unsigned)nb);
  for (int n = threadIdx.x; n < nb; n += BLOCK) {
    const int o = n + first < nb ? n + first : n + first - nb, kp = o / NT, L = (o - kp * NT) * NP + kp;
    const unsigned c = hn[L];
    if (c == 0u) continue;
    hn[L] = 0u;
    const int64_t A = base + o;
    atomicAdd(&a->npairs[A], (unsigned long long)c);
    if constexpr (DET) {
      unsigned long long* hq = (unsigned long long*)h;
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const unsigned long long lo = hq[w * nd + L];
        const long long hi = hc[w * nd + L];
        atomicAdd(&a->det_acc[4 * A + 2 * w], lo & ((1ull << kDetShift) - 1));
        atomicAdd(&a->det_acc[4 * A + 2 * w + 1],
                  ((unsigned long long)hi << (64 - kDetShift)) | (lo >> kDetShift));
        hq[w * nd + L] = 0ull;
        hc[w * nd + L] = 0;
      }
    } else {
      atomicAdd(&a->num[A], h[L]);
      atomicAdd(&a->wsum[A], h[nd + L]);
      h[L] = 0.0;
      h[nd + L] = 0.0;
      if constexpr (MEANS) {
#pragma unroll
        for (int w = 0; w < 3; ++w) {
          atomicAdd(&a->msum[w * a->n_out + A], h[(2 + w) * nd + L]);
          h[(2 + w) * nd + L] = 0.0;
        }
      }
    }
  }
}

// A wave's item: first pixel, stream position, s and c of its neighbours.
template <int CH>
struct WaveTab {
  int64_t pix[CH];
  double s[CH], c[CH];
  int32_t pos[CH];
};

// Lanes whose bin is not that of the run they sum (their low 16 bits differ).
__device__ __forceinline__ uint64_t other_bin(uint32_t L, uint32_t rkey) {
  uint64_t m;
  asm("v_cmp_ne_u16_e64 %0, %1, %2" : "=s"(m) : "v"(L), "v"(rkey));
  return m;
}

// In the lanes of mask m: the run (rkey, aN, aW) becomes the waiting run
// (pkey, pN, pW), ended before pixel i (i16 = i << 16), and a new run starts in
// bin L.  Written out, under the mask and without a branch, so that the updates
// happen in place: from a branch the compiler makes a copy of every value on
// each side of it, as many instructions again.
__device__ __forceinline__ void change_run(uint64_t m, uint32_t L, uint32_t i16, uint32_t& pkey, uint32_t& rkey,
                                           float& pN, float& pW, float& aN, float& aW) {
  uint64_t t;
  asm volatile("s_and_saveexec_b64 %[t], %[m]\n\t"
               "v_add_u32_e32 %[pk], %[i], %[rk]\n\t"
               "v_mov_b32_e32 %[pn], %[an]\n\t"
               "v_mov_b32_e32 %[pw], %[aw]\n\t"
               "v_subrev_u32_e32 %[rk], %[i], %[L]\n\t"
               "v_mov_b32_e32 %[an], 0\n\t"
               "v_mov_b32_e32 %[aw], 0\n\t"
               "s_mov_b64 exec, %[t]"
               : [t] "=&s"(t), [pk] "+v"(pkey), [rk] "+v"(rkey), [pn] "+v"(pN), [pw] "+v"(pW),
                 [an] "+v"(aN), [aw] "+v"(aW)
               : [m] "s"(m), [L] "v"(L), [i] "s"(i16)
               : "scc");
}
__device__ __forceinline__ void change_run(uint64_t m, uint32_t L, uint32_t i16, uint32_t& pkey, uint32_t& rkey,
                                           double& pN, double& pW, double& aN, double& aW) {
  uint64_t t;
  asm volatile("s_and_saveexec_b64 %[t], %[m]\n\t"
               "v_add_u32_e32 %[pk], %[i], %[rk]\n\t"
               "v_mov_b64_e32 %[pn], %[an]\n\t"
               "v_mov_b64_e32 %[pw], %[aw]\n\t"
               "v_subrev_u32_e32 %[rk], %[i], %[L]\n\t"
               "v_mov_b64_e32 %[an], 0\n\t"
               "v_mov_b64_e32 %[aw], 0\n\t"
               "s_mov_b64 exec, %[t]"
               : [t] "=&s"(t), [pk] "+v"(pkey), [rk] "+v"(rkey), [pn] "+v"(pN), [pw] "+v"(pW),
                 [an] "+v"(aN), [aw] "+v"(aW)
               : [m] "s"(m), [L] "v"(L), [i] "s"(i16)
               : "scc");
}
// In the lanes of mask m: p = a, a = 0 (the bin means' further sums).
__device__ __forceinline__ void change_sum(uint64_t m, float& p, float& a) {
  uint64_t t;
  asm volatile("s_and_saveexec_b64 %[t], %[m]\n\tv_mov_b32_e32 %[p], %[a]\n\tv_mov_b32_e32 %[a], 0\n\ts_mov_b64 exec, %[t]"
               : [t] "=&s"(t), [p] "+v"(p), [a] "+v"(a) : [m] "s"(m) : "scc");
}
__device__ __forceinline__ void change_sum(uint64_t m, double& p, double& a) {
  uint64_t t;
  asm volatile("s_and_saveexec_b64 %[t], %[m]\n\tv_mov_b64_e32 %[p], %[a]\n\tv_mov_b64_e32 %[a], 0\n\ts_mov_b64 exec, %[t]"
               : [t] "=&s"(t), [p] "+v"(p), [a] "+v"(a) : [m] "s"(m) : "scc");
}

// Two workgroups of 16 waves fill a CU's wave slots at 2500 bins (50 KB of LDS
// for the sums, 14 KB for the waves' items); MEANS needs 110 KB, one workgroup.
template <typename T, int BLOCK, int AX, bool RUNS, bool MEANS, bool DET, int CH>
__global__ __launch_bounds__(BLOCK, MEANS ? 4 : 8) void xi_kernel(XiArgs) {
  static_assert(!(DET && MEANS), "the deterministic form has no bin means");
  static_assert(RUNS || !(DET || MEANS), "these forms sum runs");
  constexpr bool ZLO = AX == kZeroEdges, EDGES = AX == kAnyEdges;
  static_assert((CH & (CH - 1)) == 0, "the search for a stream pixel's neighbour halves it");
  using Rec = typename RecOf<T>::type;
  extern __shared__ double smem[];
  __shared__ WaveTab<CH> tabs[BLOCK / 64];
  __shared__ int s_next;
  __shared__ unsigned long long s_pairs;  // candidate pairs added since the last flush
  __shared__ unsigned s_lo, s_hi;         // several slabs: the workgroup's run of tickets,
  __shared__ int s_done;                  // and that there is no further one
  __shared__ int s_gone;                  // one slab: counters found to have no ticket left

  const int lane = threadIdx.x & 63;
  WaveTab<CH>& tab = tabs[uniform((int)threadIdx.x >> 6)];
  const int NP = kargs()->g.n_par, nb = NP * kargs()->g.n_perp, nd = nb + kargs()->spare;
  for (int e = threadIdx.x; e < nd * (int)(smem_per_bin<MEANS, DET>() / 4); e += BLOCK) ((unsigned*)smem)[e] = 0u;
  if (threadIdx.x == 0) {
    s_next = kWaitAll;
    s_pairs = 0ull;
    s_lo = s_hi = 0u;
    s_gone = 0;
  }
  double* const hN = smem;
  int* const hc = (int*)(smem + n_f64<MEANS, DET>() * nd);
  unsigned* const hn = (unsigned*)(hc + (DET ? 2 * nd : 0));

  const double mp = uniform(kMagic + kGuard - kargs()->g.e0_par * kargs()->g.inv_par);
  const double uphi = uniform(kMagic + NP + 2.0 * kGuard), uthi = uniform(kMagic + kargs()->g.n_perp + 2.0 * kGuard);
  // bins are carried as L = k_perp NP + k_par + G, G what the two upper words add
  const uint32_t G = (kMagicHi & 0xffffffu) * (uint32_t)NP + kMagicHi, Lout = G + (uint32_t)(nb + (lane & (kargs()->spare - 1)));
  int shN = 0, shW = 0;  // DET: s of the current realisation

  int cur = -1;        // output slab of the LDS sums
  bool have = false;   // an item is held
  unsigned turns_taken = blockIdx.x;  // thread 0: the next run of tickets
  unsigned ticket = (unsigned)uniform((int)threadIdx.x >> 6) * gridDim.x + blockIdx.x, ticket_end = 0;
  int key = 0, nbc = 0, nf = 0, total = 0, log_step = 0, part0 = 0;
  int64_t fpix0 = 0, fext = 0;
  __syncthreads();

  for (;;) {
    if (!have) {
      const KArgs a = kargs();
      have = true;
      // Tickets.  One slab: every n-th from the wave's number on (n waves), for its
      // share, then `grab` at a time from kXiCounters counters, the workgroup's own
      // first: one counter hands out a ticket in 12 ns at best, and to tell 8192
      // waves that it has none left took 0.1 ms.  Several slabs: from the
      // workgroup's run.
      const unsigned waves = (BLOCK / 64) * gridDim.x;
      unsigned t = ticket;
      if (a->chunk > 0) {
        if (lane == 0) {
          t = atomicAdd(&s_lo, 1u);
          t = t < s_hi ? t : ~0u;
        }
        t = (unsigned)uniform((int)t);
      } else if (ticket < (unsigned)a->share * waves) {
        ticket += waves;
        if (ticket >= (unsigned)a->share * waves) ticket = ticket_end = (unsigned)a->share * waves;
      } else {
        if (ticket == ticket_end) {
          ticket = t = grab_ticket(a->counter, (unsigned)a->share * waves, (unsigned)a->grab,
                                            (unsigned)(a->n_items * a->n_parts), &s_gone);
          ticket_end = ticket + (unsigned)a->grab;
        }
        if (t != ~0u) ++ticket;
      }
      key = kWaitAll;
      if ((int64_t)t < a->n_items * a->n_parts) {
        part0 = t % (unsigned)a->n_parts * kRunMax;
        t /= (unsigned)a->n_parts;
        const Item item = a->items[t];
        const int f = a->sorted[item.p];
        const ForestInfo fi = a->finfo[f];
        key = uniform(a->sub ? fi.real * a->n_sub + a->sub[f] : fi.real);
        nbc = uniform(item.nb_count);
        nf = uniform(fi.npix);
        fpix0 = ((int64_t)uniform((int)(fi.pix0 >> 32)) << 32) | (uint32_t)uniform((int)fi.pix0);
        // the neighbours in order of distance: a wave's lanes then leave the grid
        // together, and the iterations without a pair in it are skipped
        int n = 0;
        float dmin = 0.f;
        double s = 0.0, c = 1.0;
        int64_t pix = 0;
        if (lane < nbc) {
          const ForestInfo gi = a->finfo[a->sorted[a->nbr[item.nb_begin + lane]]];
          pair_sc(fi, gi, s, c);
          pix = gi.pix0;
          n = gi.npix;
          dmin = (float)gi.dmin;
        }
        int rank = 0;
        for (int t2 = 0; t2 < nbc; ++t2) {
          const float o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dmin), t2));
          rank += (o < dmin || (o == dmin && t2 < lane)) ? 1 : 0;
        }
        if (lane < nbc) {
          tab.s[rank] = s;
          tab.c[rank] = c;
          tab.pix[rank] = pix;
          tab.pos[rank] = n;
        }
        __builtin_amdgcn_wave_barrier();
        n = lane < nbc ? tab.pos[lane] : 0;
        int incl = n;
#pragma unroll
        for (int o = 1; o < CH; o <<= 1) {
          const int v = __shfl_up(incl, o, 64);
          if (lane >= o) incl += v;
        }
        if (lane < nbc) tab.pos[lane] = incl - n;
        total = __builtin_amdgcn_readlane(incl, CH - 1);
        fext = (fpix0 >> 5) + uniform(f);
        // pixels of f per r_par bin, as the power of two below 1.4 times it
        const float per = 1.4f * (float)(nf - 1) / fmaxf((float)((fi.dmax - fi.dmin) * a->g.inv_par), 1e-6f);
        log_step = uniform(per < 2.f ? 0 : (per < 4.f ? 1 : (per < 8.f ? 2 : (per < 16.f ? 3 : 4))));
      }
    }
    bool go = key == cur;
    if (go) {
      // reserve the item's pairs: no bin's count passes 2^32 between flushes
      const unsigned long long pairs = (unsigned long long)total * (unsigned long long)nf;
      int over = 0;
      if (lane == 0) {
        const unsigned long long old = atomicAdd(&s_pairs, pairs);
        if (old != 0ull && (double)(old + pairs) > kargs()->flush_pairs) {
          atomicAdd(&s_pairs, 0ull - pairs);
          over = 1;
        }
      }
      go = uniform(over) == 0;
    }
    if (!go) {
      // every wave of the workgroup comes here before any goes on; the items
      // are ordered by slab, so each of them finds an end of the work in `cur`
      if (lane == 0) atomicMin(&s_next, key);
      __syncthreads();
      const int next = uniform(s_next);
      const bool refill = next == kWaitAll && kargs()->chunk > 0;
      if (cur >= 0 && !refill) flush_hist<BLOCK, MEANS, DET>(smem, cur);
      __syncthreads();
      if (threadIdx.x == 0) {
        s_next = kWaitAll;
        if (refill) {
          const KArgs a = kargs();
          const unsigned n = (unsigned)(a->n_items * a->n_parts), c = (unsigned)a->chunk;
          const uint64_t lo = (uint64_t)turns_taken * c;
          s_lo = lo < n ? (unsigned)lo : n;
          s_hi = lo + c < n ? (unsigned)(lo + c) : n;
          s_done = lo >= n;  // not read off s_lo below: a faster wave may have taken every ticket by then
          turns_taken = gridDim.x + atomicAdd(a->counter, 1u);
        } else {
          s_pairs = 0ull;
        }
      }
      __syncthreads();
      if (refill) {
        if (uniform(s_done) == 0) {
          have = false;
          continue;
        }
        if (cur >= 0) flush_hist<BLOCK, MEANS, DET>(smem, cur);
        break;
      }
      cur = next;
      if (cur == kWaitAll) break;
      if constexpr (DET) {
        const KArgs a = kargs();
        shN = uniform(det_shift(a->det_max[2 * cur]));
        shW = uniform(det_shift(a->det_max[2 * cur + 1]));
      }
      continue;
    }
    have = false;

    const Rec* rf;
    if constexpr (sizeof(T) == 4) rf = kargs()->xrec32 + fpix0; else rf = kargs()->rec64 + fpix0;
    // Stream pixel of the lane.  Each 16 lanes (an LDS atomic takes 16 at a time)
    // take every step-th pixel, about one r_par bin apart, so that they rarely
    // meet on an address or a bank: 16 lanes on 8 addresses cost it 5 clocks
    // instead of 2.  The wave covers 64 neighbouring pixels (16 step of them in
    // step / 4 turns where step > 4).
    const int turns = log_step > 2 ? 1 << (log_step - 2) : 1;
    int lane_pix;
    {
      const int g = lane >> 4, t = lane & 15, ls = min(log_step, 2), step = 1 << log_step;
      lane_pix = ((g >> ls) << (4 + ls)) + t * step + (g & ((1 << ls) - 1));
    }
    for (int block = 0, turn = 0; block < total;) {
      const int q = block + 4 * turn + lane_pix;
      if (++turn == turns) {
        turn = 0;
        block += 64 * turns;
      }
      const bool valid = q < total;
      // the neighbour of stream pixel q: the last that starts at or before it
      int k = 0;
#pragma unroll
      for (int step = CH / 2; step > 0; step >>= 1)
        if (k + step < nbc && tab.pos[k + step] <= q) k += step;
      // (past the stream's end: no pixel)
      double Dj = 0.0, cp = 0.0, st = 0.0, bt = 0.0;  // (EDGES: cp, st are c, s)
      if constexpr (!EDGES) past_end(cp, bt);
      // EDGES: the lane's intervals (past the stream's end: in no bin), their bin, and
      // the lanes with one
      EdgeBin ep{0.0, INFINITY, -1}, et = ep;
      uint32_t Lcur = Lout;
      uint64_t incur = 0ull;
      auto set_bin = [&](int NT) __attribute__((always_inline)) {
        const bool is = ((unsigned)ep.k < (unsigned)NP) & ((unsigned)et.k < (unsigned)NT);
        Lcur = is ? G + (uint32_t)(et.k * NP + ep.k) : Lout;
        incur = ballot(is);
      };
      T wdj = 0, wj = 0, dj = 0, zj = 0, mcp = 0, mst = 0, mbt = 0, mep = 0;
      {
        const KArgs a = kargs();
        const double s64 = tab.s[k], invt = a->g.inv_perp;
        if (valid) {
          const int64_t j = tab.pix[k] + (q - tab.pos[k]);
          const Rec* recs;
          if constexpr (sizeof(T) == 4) recs = a->xrec32; else recs = a->rec64;
          const Rec r = recs[j];
          Dj = r.d;
          wdj = r.wd;
          wj = r.w;
          if constexpr (EDGES) {
            cp = tab.c[k];
            st = s64;
            double rp, rt;
            separations64(rf[0].d, Dj, cp, st, rp, rt);
            ep.search(rp, a->edges_par, NP, (int)fmin(fmax((rp - a->g.e0_par) * a->g.inv_par, 0.0), NP - 1.0));
            et.search(rt, a->edges_perp, a->g.n_perp, (int)fmin(fmax((rt - a->g.e0_perp) * invt, 0.0), a->g.n_perp - 1.0));
          } else {
            cp = tab.c[k] * a->g.inv_par;
            st = s64 * invt;
            bt = (Dj * s64 - a->g.e0_perp) * invt + (kMagic + kGuard);
          }
          if constexpr (MEANS) {
            if constexpr (sizeof(T) == 4) {
              dj = a->xaux32[j].d;
              zj = a->xaux32[j].z;
            } else {
              dj = Dj;
              zj = r.del;
            }
          }
        }
        if constexpr (EDGES) set_bin(a->g.n_perp);
        if constexpr (MEANS) {
          // coordinates in the form's arithmetic, x_par = |d_i - d_j| mcp + mep,
          // x_perp = d_i mst + mbt (FP32 distances are re-centred on dc)
          const double dcx = sizeof(T) == 4 ? a->glob->dc : 0.0;
          mcp = (T)(EDGES ? cp * a->g.inv_par : cp);
          mst = (T)(EDGES ? st * invt : st);
          mbt = (T)(((Dj + dcx) * s64 - a->g.e0_perp) * invt);
          mep = (T)(-a->g.e0_par * a->g.inv_par);
        }
      }

      T aN = 0, aW = 0, pN = 0, pW = 0;           // sums of the lane's run, and of its waiting run
      T aP = 0, aT = 0, aZ = 0, pP = 0, pT = 0, pZ = 0;
      uint32_t rkey = Lout, pkey = 0;              // bin - (first pixel << 16); bin + (pixels << 16)
      uint64_t pend = 0ull;                        // lanes with a waiting run
      uint64_t last = 0ull;                        // lanes that were inside the grid
      // chunks of kRunMax pixels of f; the item's parts take them in turn, and
      // runs count pixels in the order taken (lag behind the pixel's own index)
      int lag = part0, taken = 0;

      auto flush = [&]() __attribute__((always_inline)) {
        if (lane_in(pend)) {
          const uint32_t v = pkey - G, L = v & 0x7fffu;
          if constexpr (DET) {
            det_add((unsigned long long*)hN + L, hc + L, ldexp((double)pN, shN));
            det_add((unsigned long long*)hN + nd + L, hc + nd + L, ldexp((double)pW, shW));
          } else {
            atomicAdd(&hN[L], (double)pN);
            atomicAdd(&hN[nd + L], (double)pW);
            if constexpr (MEANS) {
              atomicAdd(&hN[2 * nd + L], (double)pP);
              atomicAdd(&hN[3 * nd + L], (double)pT);
              atomicAdd(&hN[4 * nd + L], (double)pZ);
            }
          }
          atomicAdd(&hn[L], v >> 16);
        }
        pend = 0ull;
      };
      // lanes m end their run before pixel i and start one in bin L
      auto change = [&](uint64_t m, uint32_t L, uint32_t i16) __attribute__((always_inline)) {
        if (m & pend) flush();
        pend |= m;
        change_run(m, L, i16, pkey, rkey, pN, pW, aN, aW);
        if constexpr (MEANS) {
          change_sum(m, pP, aP);
          change_sum(m, pT, aT);
          change_sum(m, pZ, aZ);
        }
      };
      // N pixels of f, from pixel i on
      auto pairs = [&](auto n_c, const UPix<T>* r, int i) __attribute__((always_inline)) {
        constexpr int N = decltype(n_c)::value;
        uint64_t in[N], some = last;
        uint32_t L[N], low = 0xffffffffu;
        if constexpr (EDGES) {
#pragma unroll
          for (int u = 0; u < N; ++u) {
            double rp, rt;
            separations64(r[u].d, Dj, cp, st, rp, rt);
            const uint64_t m = ~(ballot(ep.holds(rp)) & ballot(et.holds(rt)));
            if (m) {
              const KArgs a = kargs();
              const int NT = a->g.n_perp;
              if (lane_in(m)) {
                if (!ep.holds(rp)) ep.step(rp, a->edges_par, NP);
                if (!et.holds(rt)) et.step(rt, a->edges_perp, NT);
                if (!ep.holds(rp)) ep.search(rp, a->edges_par, NP, ep.k);
                if (!et.holds(rt)) et.search(rt, a->edges_perp, NT, et.k);
              }
              set_bin(NT);
            }
            L[u] = Lcur;
            in[u] = incur;
            some |= incur;
          }
        } else {
#pragma unroll
          for (int u = 0; u < N; ++u) {
            const double up = fma(fabs(r[u].d - Dj), cp, mp), ut = fma(r[u].d, st, bt);
            in[u] = ballot(up < uphi) & ballot(ut < uthi);
            if constexpr (!ZLO) in[u] &= ballot(up >= kMagic) & ballot(ut >= kMagic);
            some |= in[u];
            const uint32_t B = __umul24((uint32_t)__double2hiint(ut), (unsigned)NP) + (uint32_t)__double2hiint(up);
            L[u] = lane_in(in[u]) ? B : Lout;
            low = min(low, min((uint32_t)__double2loint(up), (uint32_t)__double2loint(ut)));
          }
        }
        if (some == 0ull) return;
        if constexpr (RUNS) last = in[N - 1];
        if (!EDGES && ballot(low <= kGuard2)) {
          // some pair of some lane may be within the guard of an edge: its
          // coordinates once more (kept, they would take the registers of two waves)
          const KArgs a = kargs();
          double Dj2 = Dj;
          asm volatile("" : "+v"(Dj2));
#pragma unroll
          for (int u = 0; u < N; ++u) {
            double st2 = st;
            asm volatile("" : "+v"(st2));
            const double up = fma(fabs(r[u].d - Dj2), cp, mp), ut = fma(r[u].d, st2, bt);
            const uint32_t hp = (uint32_t)__double2hiint(up), ht = (uint32_t)__double2hiint(ut);
            // r_par = 0 (aligned pixel grids) needs no guard at a zero lower edge
            uint64_t m = ballot((uint32_t)__double2loint(up) <= kGuard2);
            if (a->g.zero_lo_par) m &= ballot(hp != kMagicHi);
            m = in[u] & (m | ballot((uint32_t)__double2loint(ut) <= kGuard2));
            if (m) {
              if (lane_in(m)) {
                double rp64, rt64;
                separations64(r[u].d, Dj2, tab.c[k], tab.s[k], rp64, rt64);
                const int kp = bin_exact(rp64, a->edges_par, NP, (int)(hp - kMagicHi));
                const int kt = bin_exact(rt64, a->edges_perp, a->g.n_perp, (int)(ht - kMagicHi));
                L[u] = (kp >= 0 && kt >= 0) ? G + (uint32_t)(kt * NP + kp) : Lout;
              }
            }
          }
        }
        if constexpr (!RUNS) {
#pragma unroll
          for (int u = 0; u < N; ++u) {
            if (lane_in(in[u])) {
              const uint32_t B = L[u] & 0x7fffu;
              atomicAdd(&hN[B], (double)(r[u].wd * wdj));
              atomicAdd(&hN[nd + B], (double)(r[u].w * wj));
              atomicAdd(&hn[B], 1u);
            }
          }
          return;
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
          change(other_bin(L[u], rkey), L[u], (uint32_t)(i - lag + u) << 16);
          aN = fma(r[u].wd, wdj, aN);
          if constexpr (MEANS) {
            T di, zi;
            if constexpr (sizeof(T) == 4) {
              const lya_i2 x = LYA_CONST(lya_i2, kargs()->xaux32 + fpix0 + i + u);
              di = __int_as_float(x[0]);
              zi = __int_as_float(x[1]);
            } else {
              di = r[u].d;
              zi = LYA_CONST(double, &rf[i + u].del);
            }
            const T ad = fabs(di - dj);
            T xp;
            if constexpr (ZLO) xp = ad * mcp; else xp = fma(ad, mcp, mep);
            const T xt = fma(di, mst, mbt);
            const T ww = r[u].w * wj;
            aW += ww;
            aP = fma(ww, xp, aP);
            aT = fma(ww, xt, aT);
            aZ = fma(ww, zi + zj, aZ);
          } else {
            aW = fma(r[u].w, wj, aW);
          }
        }
      };
      constexpr int NB = Batch<T>::N;
      for (int c0 = part0; c0 < nf;) {
        const int c1 = min(nf, c0 + (int)kRunMax);
        rkey ^= 0x8000u;  // no bin: every lane starts a run
        last = RUNS ? ~0ull : 0ull;
        int i = c0;
        {
          // no pixel of this chunk within reach of any lane?  (the same rounded
          // operations from the chunk's extent, so never wrong)
          const lya_i4 e = LYA_CONST(lya_i4, kargs()->ext + fext + (c0 >> 5));
          const double lo = __hiloint2double(e[1], e[0]), hi = __hiloint2double(e[3], e[2]);
          const double gap = fmax(lo - Dj, Dj - hi);
          uint64_t near;
          if constexpr (EDGES) near = ballot(valid) & ballot(gap * cp < kargs()->g.emax_par) & ballot((lo + Dj) * st < kargs()->g.emax_perp);
          else near = ballot(fma(gap, cp, mp) < uphi) & ballot(fma(lo, st, bt) < uthi);
          if (near == 0ull) {
            if constexpr (RUNS) change(~0ull, Lout, (uint32_t)(c0 - lag) << 16);
            i = c1;
          }
        }
#pragma unroll 1
        for (; i + NB <= c1; i += NB) {
          Batch<T> b;
          b.load(rf + i);
          pairs(std::integral_constant<int, NB>{}, b.r, i);
        }
#pragma unroll 1
        for (; i < c1; ++i) {
          const UPix<T> r = load_pix(rf + i);
          pairs(std::integral_constant<int, 1>{}, &r, i);
        }
        taken = c1 - lag;
        const int skip = (int)kRunMax * (kargs()->n_parts - 1);
        lag += skip;
        c0 += (int)kRunMax + skip;
      }
      if constexpr (RUNS) {
        // the last runs, but not those outside the grid
        change(ballot((rkey & 0x7fffu) < (uint32_t)nb), Lout, (uint32_t)taken << 16);
        if (pend) flush();
      }
    }
  }
}

// Two forms, each with two workgroup sizes.  The larger size is the default:
// most waves per CU, fewest copies of the histograms; the smaller one is there for
// options.variant.  Runs where an r_par bin holds at least 1.05 pixels of a forest;
// below, where a run would rarely hold two pixels, every pair's products are added by
// themselves (xi_default_variant).
struct Variant {
  const char* name;
  int block;
  bool runs;
};
constexpr Variant kVariants[] = {
    {"b512", 512, false}, {"b1024", 1024, false}, {"b512-runs", 512, true}, {"b1024-runs", 1024, true}};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

template <typename T, int BLOCK, int AX, bool RUNS, bool MEANS = false, bool DET = false, int CH = kChunkMax>
hipError_t launch_one(const XiArgs& a, int blocks, hipStream_t st) {
  const size_t smem = ((size_t)a.g.n_par * a.g.n_perp + a.spare) * smem_per_bin<MEANS, DET>();
  auto kern = xi_kernel<T, BLOCK, AX, RUNS, MEANS, DET, CH>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(BLOCK), smem, st, a);
  return hipGetLastError();
}

// launch(std::integral_constant<int, AX>) for the axes' form.
template <typename Launch>
hipError_t with_axes(const GridDev& g, Launch&& launch) {
  switch (axis_form(g)) {
    case kZeroEdges: return launch(std::integral_constant<int, kZeroEdges>{});
    case kUniformEdges: return launch(std::integral_constant<int, kUniformEdges>{});
    default: return launch(std::integral_constant<int, kAnyEdges>{});
  }
}

template <typename T>
hipError_t launch_t(int v, const XiArgs& a, int blocks, hipStream_t st) {
  return with_axes(a.g, [&](auto ax) {
    constexpr int AX = decltype(ax)::value;
    switch (v) {
      case 0: return launch_one<T, 512, AX, false>(a, blocks, st);
      case 1: return launch_one<T, 1024, AX, false>(a, blocks, st);
      case 2: return launch_one<T, 512, AX, true>(a, blocks, st);
      case 3: return launch_one<T, 1024, AX, true>(a, blocks, st);
    }
    return hipErrorInvalidValue;
  });
}

template <typename T, int BLOCK, bool RUNS, bool MEANS = false, bool DET = false>
int occupancy(int n_bins) {
  const size_t smem = ((size_t)n_bins + 64) * smem_per_bin<MEANS, DET>();
  auto kern = xi_kernel<T, BLOCK, kZeroEdges, RUNS, MEANS, DET, kChunkMax>;
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess) return 1;
  int nblk = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nblk, kern, BLOCK, smem) != hipSuccess) return 1;
  return nblk > 0 ? nblk : 1;
}

template <typename T>
int occ_t(int v, int n_bins) {
  switch (v) {
    case 0: return occupancy<T, 512, false>(n_bins);
    case 1: return occupancy<T, 1024, false>(n_bins);
    case 2: return occupancy<T, 512, true>(n_bins);
    case 3: return occupancy<T, 1024, true>(n_bins);
  }
  return 1;
}

__global__ void zero_kernel(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

__global__ void zero3_kernel(uint32_t* a, uint32_t* b, uint32_t* c, size_t n) {
  uint32_t* const p = blockIdx.y == 0 ? a : (blockIdx.y == 1 ? b : c);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// Bin means from the sums of w_i w_j x (x in bin units) and w_i w_j (z_i + z_j):
// r = e0 + dr * sum(ww x) / W, z = sum(ww (z_i + z_j)) / (2 W); 0 where W = 0.
__global__ void finalize_means_kernel(const double* wsum, const double* msum, int64_t n, GridDev g,
                                      double* rpar, double* rperp, double* z) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double w = wsum[i];
  const bool e = w == 0.0;
  rpar[i] = e ? 0.0 : g.e0_par + (msum[i] / w) / g.inv_par;
  rperp[i] = e ? 0.0 : g.e0_perp + (msum[n + i] / w) / g.inv_perp;
  z[i] = e ? 0.0 : 0.5 * (msum[2 * n + i] / w);
}

// Largest |w delta| and w of each realisation, as bits of non-negative doubles
// (their order is the doubles' order), one wave per forest.
__global__ __launch_bounds__(256) void det_max_kernel(lya_forests F, const ForestInfo* finfo, const double* delta,
                                                    unsigned long long* det_max) {
  const int lane = threadIdx.x & 63;
  const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (f >= F.n_forests) return;
  const ForestInfo fi = finfo[f];
  double mwd = 0.0, mw = 0.0;
  for (int k = lane; k < fi.npix; k += 64) {
    const int64_t i = fi.pix0 + k;
    const double w = F.weight[i];
    mwd = fmax(mwd, fabs(__dmul_rn(w, delta[i])));
    mw = fmax(mw, w);
  }
  for (int o = 32; o > 0; o >>= 1) {
    mwd = fmax(mwd, __shfl_xor(mwd, o, 64));
    mw = fmax(mw, __shfl_xor(mw, o, 64));
  }
  if (lane == 0) {
    atomicMax(&det_max[2 * fi.real], (unsigned long long)__double_as_longlong(mwd));
    atomicMax(&det_max[2 * fi.real + 1], (unsigned long long)__double_as_longlong(mw));
  }
}

// N, W from the integer sums: (hi 2^28 + lo) 2^-s.
__global__ void finalize_det_kernel(const unsigned long long* acc, const unsigned long long* det_max,
                                    const unsigned long long* npairs, int64_t n, int n_bins, double* num,
                                    double* wsum, Globals* glob) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t r = i / n_bins;
  const int sN = det_shift(det_max[2 * r]), sW = det_shift(det_max[2 * r + 1]);
  // the low word carried into the high one: both then depend on the total only
  auto value = [](unsigned long long lo, unsigned long long hi) {
    hi += lo >> kDetShift;
    return __dadd_rn(ldexp((double)(long long)hi, kDetShift), (double)(lo & ((1ull << kDetShift) - 1)));
  };
  const double vn = value(acc[4 * i], acc[4 * i + 1]);
  const double vw = value(acc[4 * i + 2], acc[4 * i + 3]);
  num[i] = ldexp(vn, -sN);
  wsum[i] = ldexp(vw, -sW);
  if (npairs[i] >= (1ull << 36)) atomicOr(&glob->flag, kBadDet);
}

__global__ void finalize_xi_kernel(const double* num, const double* wsum, double* xi, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double w = wsum[i];
  xi[i] = w != 0.0 ? num[i] / w : 0.0;
}

}  // namespace

int xi_num_variants() { return kNumVariants; }
// Direct and runs in ms at 1.25 / 1.1 / 1.0 / 0.8 pixels per bin, 2500 log forests to 200
// Mpc/h in 10 r_perp bins: FP32 9.5, 5.8 / 8.9, 5.9 / 6.3, 6.0 / 6.9, 7.1; FP64 9.6, 6.3 /
// 8.9, 6.3 / 6.3, 6.4 / 7.0, 7.2.  500 linear forests to 60: FP32 1.82, 1.56 / 1.67, 1.54 /
// 1.63, 1.63 / 1.52, 1.68.  40 r_perp bins, FP32, at 1.1 and 1.0: 8.7, 6.1 and 6.4, 7.8.
// (While bins and pixels are nearly as wide, lanes a bin apart meet on an address.)
int xi_default_variant(double bin_par, double spacing) { return bin_par < 1.05 * spacing ? 1 : 3; }
int xi_variant_block(int v) { return kVariants[v].block; }
const char* xi_variant_name(int v) { return (v >= 0 && v < kNumVariants) ? kVariants[v].name : "?"; }

hipError_t launch_xi(int variant, int precision, const XiArgs& a, int blocks, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  return precision == LYA_FP64 ? launch_t<double>(variant, a, blocks, st)
                               : launch_t<float>(variant, a, blocks, st);
}

int xi_blocks_per_cu(int variant, int precision, int n_bins) {
  return precision == LYA_FP64 ? occ_t<double>(variant, n_bins) : occ_t<float>(variant, n_bins);
}

// The deterministic form: 28 B of LDS per bin, two workgroups per CU at 2500 bins.
constexpr int kDetBlock = 1024;

hipError_t launch_xi_det(int precision, const XiArgs& a, int blocks, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  return with_axes(a.g, [&](auto ax) {
    constexpr int AX = decltype(ax)::value;
    return precision == LYA_FP64 ? launch_one<double, kDetBlock, AX, true, false, true>(a, blocks, st)
                                 : launch_one<float, kDetBlock, AX, true, false, true>(a, blocks, st);
  });
}

int xi_det_blocks_per_cu(int precision, int n_bins) {
  return precision == LYA_FP64 ? occupancy<double, kDetBlock, true, false, true>(n_bins)
                               : occupancy<float, kDetBlock, true, false, true>(n_bins);
}

hipError_t launch_det_max(const lya_forests* F, const ForestInfo* finfo, const double* delta,
                          unsigned long long* det_max, hipStream_t st) {
  if (F->n_forests == 0) return hipSuccess;
  hipLaunchKernelGGL(det_max_kernel, dim3((unsigned)((F->n_forests + 3) / 4)), dim3(256), 0, st, *F, finfo, delta,
                     det_max);
  return hipGetLastError();
}

hipError_t launch_finalize_det(const unsigned long long* det_acc, const unsigned long long* det_max,
                               const unsigned long long* npairs, int64_t n_out, int n_bins, double* num,
                               double* wsum, Globals* glob, hipStream_t st) {
  if (n_out == 0) return hipSuccess;
  hipLaunchKernelGGL(finalize_det_kernel, dim3((unsigned)((n_out + 255) / 256)), dim3(256), 0, st, det_acc, det_max,
                     npairs, n_out, n_bins, num, wsum, glob);
  return hipGetLastError();
}

// The bin-means form: 44 B of LDS per bin, one workgroup of 16 waves per CU at
// 2500 bins.
constexpr int kMeansBlock = 1024;

// Bin means over 3490 bins fill the LDS: one entry for the pairs outside the grid and
// items of two neighbours then leave room up to 3698 bins.
bool xi_means_tight(int n_bins) {
  return ((size_t)n_bins + 64) * smem_per_bin<true, false>() + sizeof(WaveTab<kChunkMax>) * (kMeansBlock / 64) + 64 > kLdsBytes;
}

hipError_t launch_xi_means(int precision, const XiArgs& a, int blocks, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  return with_axes(a.g, [&](auto ax) {
    constexpr int AX = decltype(ax)::value;
    if (a.spare == 1)
      return precision == LYA_FP64 ? launch_one<double, kMeansBlock, AX, true, true, false, kChunkTight>(a, blocks, st)
                                   : launch_one<float, kMeansBlock, AX, true, true, false, kChunkTight>(a, blocks, st);
    return precision == LYA_FP64 ? launch_one<double, kMeansBlock, AX, true, true>(a, blocks, st)
                                 : launch_one<float, kMeansBlock, AX, true, true>(a, blocks, st);
  });
}

int xi_means_blocks_per_cu(int precision, int n_bins) {
  if (xi_means_tight(n_bins)) return 1;
  return precision == LYA_FP64 ? occupancy<double, kMeansBlock, true, true>(n_bins)
                               : occupancy<float, kMeansBlock, true, true>(n_bins);
}

hipError_t launch_finalize_means(const double* wsum, const double* msum, int64_t n, const GridDev& g,
                                 double* rpar, double* rperp, double* z, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(finalize_means_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, wsum, msum,
                     n, g, rpar, rperp, z);
  return hipGetLastError();
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  const size_t n = bytes / 4;
  const unsigned blocks = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(zero_kernel, dim3(blocks), dim3(256), 0, st, (uint32_t*)p, n);
  return hipGetLastError();
}

hipError_t launch_zero3(void* a, void* b, void* c, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  const size_t n = bytes / 4;
  const unsigned blocks = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(zero3_kernel, dim3(blocks, c ? 3 : 2), dim3(256), 0, st, (uint32_t*)a, (uint32_t*)b, (uint32_t*)c, n);
  return hipGetLastError();
}

hipError_t launch_finalize_xi(const double* num, const double* wsum, double* xi, int64_t n,
                              hipStream_t st) {
  if (n == 0 || xi == nullptr) return hipSuccess;
  hipLaunchKernelGGL(finalize_xi_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, num, wsum, xi, n);
  return hipGetLastError();
}

}  // namespace lya
