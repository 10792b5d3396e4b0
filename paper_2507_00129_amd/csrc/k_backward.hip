// Backward pass of the xi estimator (Sec. 2.1, eq. estimator_two):
// with gamma_A = (dL/dxi_A) / W_A,
//   dL/d delta_i = w_i sum_j gamma_{A(i,j)} w_j delta_j
//   dL/d w_i     = sum_j gamma_{A(i,j)} w_j (delta_i delta_j - xi_{A(i,j)})
//                = delta_i S1_i - S2_i,  S1_i = sum_j gamma w_j delta_j,
//                                        S2_i = sum_j gamma xi w_j
// over every pixel j of every other forest of the same realisation.
//
// Work item = one forest f with some of its neighbours (a symmetric neighbour
// list); each wave takes items by itself.  Lanes own 64 pixels i of f at a time;
// the neighbour's pixels j are wave-uniform (scalar loads, several records at a
// time).  Bins come from FP64 coordinates 2^20 + x (upper word: the bin, lower:
// the fraction), as in the forward kernel.  Over a run of consecutive pixels j
// in one bin the lane sums w_j delta_j and w_j in the form's arithmetic; gamma
// and gamma xi come from an LDS table once per run.  A finished run waits in its
// lane (one slot), so that the lanes' runs, which end at different pixels, meet
// the table together.  A neighbour's sums are added to FP64 registers in the
// form's precision, an item's to S1 and S2 in global memory; a last kernel makes
// the gradients of them.
//
// The table holds one realisation; items are ordered by realisation, and a wave
// whose item belongs to the next one waits until the others get there too.
//
// Measured (MI355X, FP32, 3.3e10 candidate pairs counted once, 50 x 50 bins to 200
// Mpc/h): 15.6 ms, against 44 of one workgroup of 8 waves per forest with FP32
// geometry, which kept 4 waves on a SIMD, gathered from the table at each
// iteration with the end of a run (36 vector instructions an iteration) and had 6
// forests per workgroup to balance.  Bound by the vector units; a quarter of the
// lanes have no pixel (forests of 100).
#include "lya_bin.h"
#include "lya_common.h"
#include "lya_pairs.h"

namespace lya {

namespace {

typedef const __attribute__((address_space(4))) BwdArgs* BArgs;
// The kernel's arguments, read again where they are used: what only an item or
// the exact path needs does not stay in scalar registers through the pair loop.
__device__ __forceinline__ BArgs bargs() {
  BArgs p = (BArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// A wave's item: its neighbours.
struct BwdTab {
  int64_t pix[kChunkMax];
  double s[kChunkMax], c[kChunkMax];
  int32_t n[kChunkMax], f[kChunkMax];
};

template <typename T> struct Pair2;
template <> struct Pair2<float> { using type = float2; };
template <> struct Pair2<double> { using type = double2; };

// In the lanes of mask m: the run (rkey, aN, aW) becomes the waiting run and a
// run in bin L starts (under the mask and in place, see k_xi.hip's change_run).
__device__ __forceinline__ void next_run(uint64_t m, uint32_t L, uint32_t& pkey, uint32_t& rkey, float& pN, float& pW,
                                         float& aN, float& aW) {
  uint64_t t;
  asm volatile("s_and_saveexec_b64 %[t], %[m]\n\t"
               "v_mov_b32_e32 %[pk], %[rk]\n\t"
               "v_mov_b32_e32 %[pn], %[an]\n\t"
               "v_mov_b32_e32 %[pw], %[aw]\n\t"
               "v_mov_b32_e32 %[rk], %[L]\n\t"
               "v_mov_b32_e32 %[an], 0\n\t"
               "v_mov_b32_e32 %[aw], 0\n\t"
               "s_mov_b64 exec, %[t]"
               : [t] "=&s"(t), [pk] "+v"(pkey), [rk] "+v"(rkey), [pn] "+v"(pN), [pw] "+v"(pW),
                 [an] "+v"(aN), [aw] "+v"(aW)
               : [m] "s"(m), [L] "v"(L)
               : "scc");
}
__device__ __forceinline__ void next_run(uint64_t m, uint32_t L, uint32_t& pkey, uint32_t& rkey, double& pN, double& pW,
                                         double& aN, double& aW) {
  uint64_t t;
  asm volatile("s_and_saveexec_b64 %[t], %[m]\n\t"
               "v_mov_b32_e32 %[pk], %[rk]\n\t"
               "v_mov_b64_e32 %[pn], %[an]\n\t"
               "v_mov_b64_e32 %[pw], %[aw]\n\t"
               "v_mov_b32_e32 %[rk], %[L]\n\t"
               "v_mov_b64_e32 %[an], 0\n\t"
               "v_mov_b64_e32 %[aw], 0\n\t"
               "s_mov_b64 exec, %[t]"
               : [t] "=&s"(t), [pk] "+v"(pkey), [rk] "+v"(rkey), [pn] "+v"(pN), [pw] "+v"(pW),
                 [an] "+v"(aN), [aw] "+v"(aW)
               : [m] "s"(m), [L] "v"(L)
               : "scc");
}

// Two workgroups of 16 waves fill a CU's wave slots (2500 bins: 20 KB of table in
// FP32, 40 KB in FP64, and 10 KB for the waves' items).
template <typename T, int BLOCK, bool ZLO>
__global__ __launch_bounds__(BLOCK, 8) void xi_bwd_kernel(BwdArgs) {
  using Rec = typename RecOf<T>::type;
  using T2 = typename Pair2<T>::type;
  extern __shared__ __align__(16) double smem[];
  T2* const gam = (T2*)smem;  // [nb]: gamma, gamma xi  (local layout)
  __shared__ BwdTab tabs[BLOCK / 64];
  __shared__ int s_next, s_done, s_gone;
  __shared__ unsigned s_lo, s_hi;  // several realisations: the workgroup's run of tickets

  const int lane = threadIdx.x & 63;
  BwdTab& tab = tabs[uniform((int)threadIdx.x >> 6)];
  const int NP = bargs()->g.n_par;
  const double guard = bargs()->g.exact_all ? kWideGuard : kGuard;
  const double mp = uniform(kMagic + guard - bargs()->g.e0_par * bargs()->g.inv_par);
  const double uphi = uniform(kMagic + NP + 2.0 * guard), uthi = uniform(kMagic + bargs()->g.n_perp + 2.0 * guard);
  const uint32_t thr = bargs()->g.exact_all ? 0xffffffffu : kGuard2;
  // bins are carried as L = k_perp NP + k_par + G, G what the two upper words add
  const uint32_t G = (kMagicHi & 0xffffffu) * (uint32_t)NP + kMagicHi;
  const uint32_t Lout = G + (uint32_t)(NP * bargs()->g.n_perp);
  if (threadIdx.x == 0) {
    s_next = kWaitAll;
    s_lo = s_hi = 0u;
    s_gone = 0;
  }

  int cur = -1;        // realisation of the table
  bool have = false;   // an item is held
  unsigned turns_taken = blockIdx.x;  // thread 0: the next run of tickets
  unsigned ticket = (unsigned)uniform((int)threadIdx.x >> 6) * gridDim.x + blockIdx.x, ticket_end = 0;
  int key = 0, nbc = 0, nf = 0, part = 0;
  int64_t fpix0 = 0;
  __syncthreads();

  for (;;) {
    if (!have) {
      // tickets as in the forward kernel
      const BArgs a = bargs();
      have = true;
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
        part = t % (unsigned)a->n_parts;
        t /= (unsigned)a->n_parts;
        const Item item = a->items[t];
        const ForestInfo fi = a->finfo[a->sorted[item.p]];
        key = uniform(fi.real);
        nbc = uniform(item.nb_count);
        nf = uniform(fi.npix);
        fpix0 = ((int64_t)uniform((int)(fi.pix0 >> 32)) << 32) | (uint32_t)uniform((int)fi.pix0);
        if (lane < nbc) {
          const int g = a->sorted[a->nbr[item.nb_begin + lane]];
          const ForestInfo gi = a->finfo[g];
          double s, c;
          pair_sc(fi, gi, s, c);
          tab.pix[lane] = gi.pix0;
          tab.s[lane] = s;
          tab.c[lane] = c;
          tab.n[lane] = gi.npix;
          tab.f[lane] = g;
        }
      }
    }
    if (key != cur) {
      // every wave of the workgroup comes here before any goes on
      if (lane == 0) atomicMin(&s_next, key);
      __syncthreads();
      const BArgs a = bargs();
      const int next = uniform(s_next);
      const bool refill = next == kWaitAll && a->chunk > 0;
      if (next != kWaitAll) {
        const int nb = NP * a->g.n_perp;
        const double2* src = a->gtab + (int64_t)next * nb;
        for (int L = threadIdx.x; L < nb; L += BLOCK) {
          const double2 v = src[L];
          T2 g;
          g.x = (T)v.x;
          g.y = (T)v.y;
          gam[L] = g;
        }
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        s_next = kWaitAll;
        if (refill) {
          const unsigned n = (unsigned)(a->n_items * a->n_parts), c = (unsigned)a->chunk;
          const uint64_t lo = (uint64_t)turns_taken * c;
          s_lo = lo < n ? (unsigned)lo : n;
          s_hi = lo + c < n ? (unsigned)(lo + c) : n;
          s_done = lo >= n;
          turns_taken = gridDim.x + atomicAdd(a->counter, 1u);
        }
      }
      __syncthreads();
      if (refill) {
        if (uniform(s_done) != 0) break;
        have = false;
        continue;
      }
      cur = next;
      if (cur == kWaitAll) break;
      continue;
    }
    have = false;

    for (int i0 = 64 * part; i0 < nf; i0 += 64 * bargs()->n_parts) {
      const int i = i0 + lane;
      const bool valid = i < nf;
      double Di = 0.0, s1 = 0.0, s2 = 0.0;
      {
        const BArgs a = bargs();
        const Rec* recs;
        if constexpr (sizeof(T) == 4) recs = a->xrec32; else recs = a->rec64;
        if (valid) Di = recs[fpix0 + i].d;
      }
#pragma unroll 1
      for (int k = 0; k < nbc; ++k) {
        // lanes past the forest's end: outside the grid and off the edge guard
        double cp, st = 0.0, bt;
        past_end(cp, bt);
        const int ng = uniform(tab.n[k]);
        const int64_t gp = tab.pix[k];
        const int64_t gpix0 = ((int64_t)uniform((int)(gp >> 32)) << 32) | (uint32_t)uniform((int)gp);
        const Rec* rg;
        const double2* ext;
        {
          const BArgs a = bargs();
          if (valid) {
            const double s64 = tab.s[k], invt = a->g.inv_perp;
            cp = tab.c[k] * a->g.inv_par;
            st = s64 * invt;
            bt = (Di * s64 - a->g.e0_perp) * invt + (kMagic + (a->g.exact_all ? kWideGuard : kGuard));
          }
          if constexpr (sizeof(T) == 4) rg = a->xrec32 + gpix0; else rg = a->rec64 + gpix0;
          ext = a->ext + (gpix0 >> 5) + uniform(tab.f[k]);
        }
        T p1 = 0, p2 = 0, aN = 0, aW = 0, pN = 0, pW = 0;
        uint32_t rkey = Lout, pkey = Lout;
        uint64_t pend = 0ull, last = 0ull;  // lanes with a waiting run; that were inside the grid
        auto flush = [&]() __attribute__((always_inline)) {
          if (lane_in(pend) && pkey != Lout) {
            const T2 g = gam[pkey - G];
            p1 += g.x * pN;
            p2 += g.y * pW;
          }
          pend = 0ull;
        };
        auto change = [&](uint64_t m, uint32_t L) __attribute__((always_inline)) {
          if (m == 0ull) return;
          if (m & pend) flush();
          pend |= m;
          next_run(m, L, pkey, rkey, pN, pW, aN, aW);
        };
        auto pairs = [&](auto n_c, const UPix<T>* r) __attribute__((always_inline)) {
          constexpr int N = decltype(n_c)::value;
          uint64_t in[N], some = last;
          uint32_t L[N], low = 0xffffffffu;
#pragma unroll
          for (int u = 0; u < N; ++u) {
            const double up = fma(fabs(r[u].d - Di), cp, mp), ut = fma(r[u].d, st, bt);
            in[u] = ballot(up < uphi) & ballot(ut < uthi);
            if constexpr (!ZLO) in[u] &= ballot(up >= kMagic) & ballot(ut >= kMagic);
            some |= in[u];
            const uint32_t B = __umul24((uint32_t)__double2hiint(ut), (unsigned)NP) + (uint32_t)__double2hiint(up);
            L[u] = lane_in(in[u]) ? B : Lout;
            low = min(low, min((uint32_t)__double2loint(up), (uint32_t)__double2loint(ut)));
          }
          if (some == 0ull) return;
          last = in[N - 1];
          if (ballot(low <= thr)) {
            // some pair may be within the guard of an edge: by the edges then
            const BArgs a = bargs();
            double Di2 = Di;
            asm volatile("" : "+v"(Di2));
            int kt_last = -1;  // non-uniform edges: the bin of the pixel before is the better guess
#pragma unroll
            for (int u = 0; u < N; ++u) {
              double st2 = st;
              asm volatile("" : "+v"(st2));
              const double up = fma(fabs(r[u].d - Di2), cp, mp), ut = fma(r[u].d, st2, bt);
              const uint32_t hp = (uint32_t)__double2hiint(up), ht = (uint32_t)__double2hiint(ut);
              // r_par = 0 (aligned pixel grids) needs no guard at a zero lower edge
              uint64_t m = ballot((uint32_t)__double2loint(up) <= thr);
              if (a->g.zero_lo_par && !a->g.exact_all) m &= ballot(hp != kMagicHi);
              m = in[u] & (m | ballot((uint32_t)__double2loint(ut) <= thr));
              if (m) {
                if (lane_in(m)) {
                  double rp64, rt64;
                  separations64(Di2, r[u].d, tab.c[k], tab.s[k], rp64, rt64);
                  const int kp = bin_exact(rp64, a->edges_par, NP, (int)(hp - kMagicHi));
                  const int kt = bin_exact(rt64, a->edges_perp, a->g.n_perp,
                                           a->g.exact_all && kt_last >= 0 ? kt_last : (int)(ht - kMagicHi));
                  kt_last = kt;
                  L[u] = (kp >= 0 && kt >= 0) ? G + (uint32_t)(kt * NP + kp) : Lout;
                }
              }
            }
          }
#pragma unroll
          for (int u = 0; u < N; ++u) {
            change(ballot(L[u] != rkey), L[u]);
            aN += r[u].wd;
            aW += r[u].w;
          }
        };
        constexpr int NB = Batch<T>::N;
        for (int c0 = 0; c0 < ng; c0 += (int)kRunMax) {
          const int c1 = min(ng, c0 + (int)kRunMax);
          int j = c0;
          {
            // no pixel of this chunk within reach of any lane?  (the same rounded
            // operations from the chunk's extent, so never wrong)
            const lya_i4 e = LYA_CONST(lya_i4, ext + (c0 >> 5));
            const double lo = __hiloint2double(e[1], e[0]), hi = __hiloint2double(e[3], e[2]);
            const double gap = fmax(lo - Di, Di - hi);
            if ((ballot(fma(gap, cp, mp) < uphi) & ballot(fma(lo, st, bt) < uthi)) == 0ull) {
              change(ballot(rkey != Lout), Lout);
              last = 0ull;
              j = c1;
            }
          }
#pragma unroll 1
          for (; j + NB <= c1; j += NB) {
            Batch<T> b;
            b.load(rg + j);
            pairs(std::integral_constant<int, NB>{}, b.r);
          }
#pragma unroll 1
          for (; j < c1; ++j) {
            const UPix<T> r = load_pix(rg + j);
            pairs(std::integral_constant<int, 1>{}, &r);
          }
        }
        change(ballot(rkey != Lout), Lout);
        if (pend) flush();
        s1 += (double)p1;
        s2 += (double)p2;
      }
      if (valid) {
        const BArgs a = bargs();
        atomicAdd(&a->grad_delta[fpix0 + i], s1);
        atomicAdd(&a->grad_weight[fpix0 + i], s2);
      }
    }
  }
}

// The gradients from the sums S1 (in grad_delta) and S2 (in grad_weight).
__global__ __launch_bounds__(256) void bwd_finish_kernel(const double* weight, const double* delta, int64_t n,
                                                         double* grad_delta, double* grad_weight) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const double s1 = grad_delta[i], s2 = grad_weight[i];
  if (s1 == 0.0 && s2 == 0.0) return;
  grad_delta[i] = weight[i] * s1;
  grad_weight[i] = delta[i] * s1 - s2;
}

// gamma_A = dL/dxi_A / W_A (0 where W_A = 0) and gamma_A xi_A, in the local
// (LDS) bin order L = kt * NP + kp.
__global__ void gamma_kernel(const double* grad_xi, const double* xi, const double* wsum,
                             double2* out, int64_t n, int NP, int NT) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n) return;
  const int nb = NP * NT;
  const int64_t r = idx / nb;
  const int L = (int)(idx - r * nb);
  const int kt = L / NP, kp = L - kt * NP;
  const int64_t A = r * nb + (int64_t)kp * NT + kt;
  const double w = wsum[A];
  const double g = w != 0.0 ? grad_xi[A] / w : 0.0;
  out[idx] = make_double2(g, g * xi[A]);
}

// Adjoint of the per-forest projection delta' = eta delta (Sec. 2.2) applied
// to the gradient.  eta moves with w through W, the weighted mean of Lambda
// and S; differentiating delta'_i = delta_i - m - a_i t (m = sum w delta / W,
// t = sum w a delta / S, a = Lambda - Lambda_bar) and collapsing the sums
// gives, with g'_k = dL/d delta'_k and h'_k = dL/dw_k at fixed delta':
//   c_k = G0 / W + a_k G1 / S,  G0 = sum_i g'_i,  G1 = sum_i a_i g'_i,
//   dL/d delta_k = g'_k - w_k c_k,   dL/dw_k = h'_k - delta'_k c_k.
// The slope part is used only where the forward used the slope term, and
// c = 0 where eta = I (identity mode, or a forest with W = 0).  One wave per
// forest, FP64, in place.
__global__ __launch_bounds__(256) void project_adjoint_kernel(lya_forests F, const EtaInfo* einfo,
                                                              const double* delta_proj,
                                                              double* grad_delta, double* grad_weight) {
  const int lane = threadIdx.x & 63;
  const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (f >= F.n_forests) return;
  const EtaInfo e = einfo[f];
  if (!e.active) return;
  const int64_t p0 = F.offsets[f], p1 = F.offsets[f + 1];
  double g0 = 0.0, g1 = 0.0;
  for (int64_t k = p0 + lane; k < p1; k += 64) {
    const double g = grad_delta[k];
    g0 += g;
    g1 += (F.loglam[k] - e.lbar) * g;
  }
  g0 = wave_sum(g0);
  g1 = wave_sum(g1);
  const double c0 = g0 / e.W, c1 = e.slope ? g1 / e.S : 0.0;
  for (int64_t k = p0 + lane; k < p1; k += 64) {
    const double c = c0 + (F.loglam[k] - e.lbar) * c1;
    grad_delta[k] -= F.weight[k] * c;
    grad_weight[k] -= delta_proj[k] * c;
  }
}

constexpr int kBlock = 1024;

template <typename T>
hipError_t launch_one(const BwdArgs& a, int blocks, hipStream_t st) {
  const size_t smem = (size_t)a.g.n_par * a.g.n_perp * 2 * sizeof(T);
  auto kern = (a.g.zero_lo_par && a.g.zero_lo_perp) ? xi_bwd_kernel<T, kBlock, true> : xi_bwd_kernel<T, kBlock, false>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBlock), smem, st, a);
  return hipGetLastError();
}

template <typename T>
int occupancy(int n_bins) {
  const size_t smem = (size_t)n_bins * 2 * sizeof(T);
  auto kern = xi_bwd_kernel<T, kBlock, true>;
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess) return 1;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, kBlock, smem) != hipSuccess) return 1;
  return n > 0 ? n : 1;
}

}  // namespace

hipError_t launch_gamma(const double* grad_xi, const double* xi, const double* wsum, double2* out,
                        int64_t n, int NP, int NT, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(gamma_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, grad_xi, xi, wsum,
                     out, n, NP, NT);
  return hipGetLastError();
}

hipError_t launch_project_adjoint(const lya_forests* F, const EtaInfo* einfo, const double* delta_proj,
                                  double* grad_delta, double* grad_weight, hipStream_t st) {
  if (F->n_forests == 0) return hipSuccess;
  const unsigned blocks = (unsigned)((F->n_forests + 3) / 4);
  hipLaunchKernelGGL(project_adjoint_kernel, dim3(blocks), dim3(256), 0, st, *F, einfo, delta_proj,
                     grad_delta, grad_weight);
  return hipGetLastError();
}

hipError_t launch_xi_bwd(int precision, const BwdArgs& a, int blocks, hipStream_t st) {
  if (a.n_items == 0) return hipSuccess;
  const hipError_t e = precision == LYA_FP64 ? launch_one<double>(a, blocks, st) : launch_one<float>(a, blocks, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(bwd_finish_kernel, dim3((unsigned)((a.n_pix + 255) / 256)), dim3(256), 0, st, a.weight, a.delta,
                     a.n_pix, a.grad_delta, a.grad_weight);
  return hipGetLastError();
}

int xi_bwd_block() { return kBlock; }
int xi_bwd_blocks_per_cu(int precision, int n_bins) {
  return precision == LYA_FP64 ? occupancy<double>(n_bins) : occupancy<float>(n_bins);
}

}  // namespace lya
