// Phase A of a messenger sweep: m-parallel work in harmonic space (FP64 VALU path).
//
// For each m the Legendre functions lambda_lm(z) of every ring pair are generated
// on the fly, l = m..lmax, by the three-term recurrence in FP64 and contracted
// against the ring Fourier coefficients:
//
//   analysis   a_lm = sum_pairs lambda_lm(z) (S if l-m even else D),  S/D = G_N +/- G_S
//   filter     s_lm = f_l(lambda) a_lm, f_l = C_l / (C_l + lambda tau Omega)     (Eq. 4)
//   synthesis  E = sum_{l-m even} lambda_lm s_lm, O = sum_{l-m odd} lambda_lm s_lm,
//              F_N = E + O, F_S = E - O
//
// using lambda_lm(-z) = (-1)^(l+m) lambda_lm(z) for the mirror rings.
//
// The recurrence runs on rescaled values mu_l = lambda_lm / C_lm that obey
//   mu_l = (A_lm z) mu_{l-1} - mu_{l-2}
// (A and C are plan-time FP64 tables derived from
//  a_lm = sqrt((4 l^2 - 1)/(l^2 - m^2)) with C_l = C_{l-2} a_l / a_{l-1}, A_l = a_l C_{l-1} / C_l),
// i.e. one multiply and one FMA per value; C is applied once per (l, m) after the
// ring sum (analysis) or folded into s_lm (synthesis).
//
// Two values of l per step (Ishioka 2018, J. Meteorol. Soc. Japan 96, 241: a recurrence in z^2 for
// lambda_{m+2k+1} / z, from which the even functions follow as a combination of two) take half of
// these operations, and were measured and taken back: the even functions are then differences of
// values l times larger next to the equator, and elsewhere the step's coefficients cost digits.
// Relative error of the lambda_lm of one ring over all l and m, in FP64 against 80 bits, Nside 512,
// lmax 1024, pairs 0, 16, 64, 256, 512, 800 from the equator on: 5e-17, 5e-16, 6e-16, 1.6e-15, 3.7e-15,
// 9e-15 with the step in l; 1e-13, 9e-15, 2.4e-15, 5e-15, 1.5e-14, 5e-14 with the best form of the other.
//
// The sectoral seed lambda_mm = norm_m sin^m(theta) underflows FP64 near the
// poles: every value carries an integer scale s (value = v 2^(-512 s)). The scale
// is checked once per chunk of l (|v| > 2^64 with s > 0: v *= 2^-512, s -= 1);
// a ring whose scale is still positive at the start of a chunk contributes
// nothing in that chunk (its values are below 2^-448 times the growth of one
// chunk, far under FP64 resolution of the sums). The recurrence alternates
// between two registers, so a step is one multiply and one FMA and no moves.
//
// Work items are (m, block of 64 R ring pairs, range of l), one wavefront each; a lane owns R
// ring pairs. An item starts from a recurrence state made at plan time, so its seeds cost a
// load, it can start anywhere in l, and the l at which every ring of the block is still below
// 2^-128 (m well above l sin(theta)) are not generated, summed or written at all: of the steps, 10 %
// in the analysis and 12 % in the synthesis at Nside 512, lmax 1024 (blocks of 256 and 128 pairs), 14 % at
// Nside 1024, lmax 2048, none at Nside 64, lmax 191. The analysis splits a block's l into several items, since their outputs are
// independent: with one item per (m, block) at Nside 512, 3500 items for 3072 waves, the
// longest set the launch's time (1.67 of the mean). A batch, whose maps fill the chip together, takes
// longer items where one map's are short. The synthesis sums over l and takes smaller
// blocks instead where there are few items.
//
// A launch is one workgroup per CU (and map) of up to 12 (analysis) or 16 waves, for such a batch
// more of four. The items are balanced over the workgroups at plan time; inside one the waves take them
// from a shared queue.
//
// The recurrence coefficients are fetched 64 values of l ahead with one vector load and read
// from LDS; the synthesis coefficients, twice as many, are held 16 to a row of lanes and
// broadcast by the FMAs themselves (see accumulate). The analysis reduces over lanes through
// LDS once per chunk of 16 values of l and writes one partial sum per block; a small kernel sums
// the partials of each (l, m), applies the filter and forms the synthesis coefficients.
//
// Kernel times for one map, one wave per packed bin of whole blocks -> now: Nside 512, lmax 1024
// analysis 145 -> 116 us, synthesis 110 -> 91 us; Nside 1024, lmax 2048 891 -> 687 and 687 -> 512 us;
// Nside 64, lmax 191 16 -> 6.0 and 10.5 -> 6.5 us. FP64 issue bounds both: at Nside 1024 the items run
// 3.42e9 (l, m, ring pair) units of four FP64 instructions (one multiply, three FMAs), which 1024 SIMDs
// of 16 lanes could issue in 348 us at 2.4 GHz: 0.68 of the synthesis and 0.51 of the analysis, which
// also sums over the lanes. At Nside 512 an item's set-up (ring states and S/D, 256 rows of G apart)
// weighs more.
#include <type_traits>

#include "mwf_internal.hpp"

namespace mwf {
namespace {

constexpr double BIG_THRESH = 0x1p64;
constexpr double RESCALE = 0x1p-512;
constexpr double RISE_THRESH = 0x1p-128;   // values below this are left out of the FP64 sums' work

__device__ __forceinline__ int wave_any(int pred) { return __any(pred); }

// a + b over lanes l and l + 32 with the halves exchanged (v_permlane32_swap): lanes
// 0..31 return a[l] + a[l + 32], lanes 32..63 return b[l - 32] + b[l].
__device__ __forceinline__ double fold_halves(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false,
                                                   false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false,
                                                   false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// Recurrence state of a lane's ring pairs: z, the two registers (mu of the latest odd and even
// l - m), and the scales.
template <int R>
struct RingState {
  double z[R], mu1[R], mu2[R];
  unsigned sc;   // a byte per ring pair (at most four)
};

// The plan's start state of item k (zero past the active ring pairs).
template <int R>
__device__ __forceinline__ void init_rings(const PlanDev& P, const Leg64List& T, const double* __restrict__ zt, int k,
                                           int blk, int lane, int nact, RingState<R>& st) {
  st.sc = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int q = blk * (LANES * R) + r * LANES + lane;
    const size_t at = (size_t)k * (LANES * R) + r * LANES + lane;
    const double2 mu = T.state[at];
    st.z[r] = q < nact ? zt[min(q, P.npairs - 1)] : 0.0;
    st.mu1[r] = mu.x;
    st.mu2[r] = mu.y;
    st.sc |= (unsigned)T.scale[at] << (8 * r);
  }
}

// Steps to l (l - m even, into mu2) and l + 1 (into mu1) of a ring.
__device__ __forceinline__ void step_pair(double& mu1, double& mu2, double z, double A0, double A1) {
  mu2 = fma(A0 * z, mu1, -mu2);
  mu1 = fma(A1 * z, mu2, -mu1);
}

// Once per chunk: bring large scaled values back by 2^-512. Returns a bit mask of
// the rings whose scale reached zero in this call.
template <int R>
__device__ __forceinline__ int rescale_chunk(RingState<R>& st) {
  int woke = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (((st.sc >> (8 * r)) & 0xff) != 0 && fmax(fabs(st.mu1[r]), fabs(st.mu2[r])) > BIG_THRESH) {
      st.mu1[r] *= RESCALE;
      st.mu2[r] *= RESCALE;
      st.sc -= 1u << (8 * r);
      if (((st.sc >> (8 * r)) & 0xff) == 0) woke |= 1 << r;
    }
  }
  return woke;
}

constexpr int LTILE = 64;  // values of l per prefetched coefficient tile (one per lane)

// Orders a wave's LDS accesses around it (one wave's LDS operations execute in
// order; this keeps the compiler from moving them across).
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }
constexpr int ACH = 16;    // analysis: values of l per cross-lane reduction (and scale check)
static_assert(LTILE % ACH == 0 && (2 * ACH) <= LANES, "analysis chunking");

// LDS of one wave: the cross-lane reduction (values x 32 lanes, padded) and the coefficient tile.
constexpr int RED_STRIDE = LANES / 2 + 1;
constexpr int ANA_LDS = 2 * ACH * RED_STRIDE + LTILE;   // doubles per wave

// The items of this workgroup, taken by its waves one at a time, most costly first, through a
// counter in LDS. A SIMD issues from its oldest ready wave, so with the items dealt to the
// waves beforehand the first wave of each SIMD finished at 0.59 of the launch, the second at
// 0.79, and the last ran its rest alone, with nothing to hide its latencies.
struct ItemQueue {
  int* ctr;
  int first, end, k = 0;
  __device__ __forceinline__ ItemQueue(const Leg64List& T, double* lds)
      : ctr(reinterpret_cast<int*>(lds)), first(T.wg[blockIdx.x]), end(T.wg[blockIdx.x + 1]) {
    if (threadIdx.x == 0) *ctr = first;
    __syncthreads();
  }
  __device__ __forceinline__ bool next(int lane) {
    int v = 0;
    if (lane == 0) v = atomicAdd(ctr, 1);
    k = __builtin_amdgcn_readfirstlane(v);
    return k < end;
  }
};

template <int R>
__device__ __forceinline__ void analysis_item(const PlanDev& P, const Leg64Dev& L, const int k, const Item64 it,
                                              const int map, const int lane, double* __restrict__ lds,
                                              const double* __restrict__ G, double2* __restrict__ partial) {
  double* red = lds;
  double* sA = lds + 2 * ACH * RED_STRIDE;
  const int m = it.m, blk = it.blk;
  const int nact = P.n_active[m];
  const double* __restrict__ Arow = P.A + P.row_off[m] + it.i0;
  const size_t pstride = gf_stride(P.lmax);
  const double* Gm = G + (size_t)map * P.npairs * pstride + (size_t)m * 4;

  RingState<R> st;
  init_rings<R>(P, L.ana, L.z, k, blk, lane, nact, st);
  // S and D of each ring, zero while the ring's values are still scaled
  double Sre[R], Sim[R], Dre[R], Dim[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int q = blk * (LANES * R) + r * LANES + lane;
    // (loaded whatever the scale, so that the load does not wait for the state)
    const double4 sd = *reinterpret_cast<const double4*>(Gm + (size_t)min(q, nact - 1) * pstride);
    const bool on = q < nact && ((st.sc >> (8 * r)) & 0xff) == 0;
    Sre[r] = on ? sd.x : 0.0;
    Sim[r] = on ? sd.y : 0.0;
    Dre[r] = on ? sd.z : 0.0;
    Dim[r] = on ? sd.w : 0.0;
  }

  // the item's part of the block's partial sums
  const int nl = it.i1 - it.i0;
  double* out = reinterpret_cast<double*>(partial + ((size_t)map * P.nblk_max + blk) * P.nalm +
                                          alm_index(P.lmax, m, m) + it.i0);

  // recurrence coefficients of LTILE values of l: lane i loads l = base + i one tile ahead, the
  // tile in use is read from LDS (the same address in every lane). The loads are unconditional,
  // with the index clamped to the first entry of the row's zero padding, so that no wait for
  // them lands inside the loop.
  const int na = P.lmax - m + 1 - it.i0;
  auto tile_a = [&](int i) { return Arow[min(i, na)]; };
  sA[lane] = tile_a(lane);
  // every load issued so far (ring states, S/D, tile 0) completes here, so the loop
  // body waits on nothing but its own LDS reads
  __builtin_amdgcn_s_waitcnt(0);
  wave_sync();
  double An = tile_a(LTILE + lane);

  for (int i = 0; i < nl; i += ACH) {
    const int t0 = i & (LTILE - 1);
    if (t0 == 0 && i > 0) {
      sA[lane] = An;      // the previous tile's last readers passed the barrier below
      wave_sync();
      An = tile_a(i + LTILE + lane);
    }
    double are[ACH], aim[ACH];
#pragma unroll
    for (int j = 0; j < ACH; ++j) are[j] = aim[j] = 0.0;
    const double2* Ac = reinterpret_cast<const double2*>(sA + t0);
#pragma unroll
    for (int j = 0; j < ACH; j += 4) {
      const double2 A0 = Ac[j / 2], A1 = Ac[j / 2 + 1];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int v = j + 2 * h;
        const double2 A = h ? A1 : A0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          step_pair(st.mu1[r], st.mu2[r], st.z[r], A.x, A.y);
          are[v] = fma(st.mu2[r], Sre[r], are[v]);
          aim[v] = fma(st.mu2[r], Sim[r], aim[v]);
          are[v + 1] = fma(st.mu1[r], Dre[r], are[v + 1]);
          aim[v + 1] = fma(st.mu1[r], Dim[r], aim[v + 1]);
        }
      }
      // keeps the tile reads of all the steps from moving up here, where they cost the
      // registers that let a third wave in
      if (j == ACH / 2) __builtin_amdgcn_sched_barrier(0);
    }
    // reduce the NV = 2 ACH values (v = 2 j + re/im) over the 64 lanes: first lanes
    // l and l + 32 in registers, the lower half keeping values 0..NV/2-1 and the
    // upper half the rest, then the remaining 32 lanes through LDS, LPV lanes per
    // value each adding 32 / LPV entries, and LPV - 1 shuffles
    constexpr int NV = 2 * ACH, LPV = LANES / NV;
#pragma unroll
    for (int x = 0; x < ACH; ++x) {
      const int ja = x >> 1, jb = ACH / 2 + (x >> 1);
      const double va = (x & 1) ? aim[ja] : are[ja];
      const double vb = (x & 1) ? aim[jb] : are[jb];
      red[(x + (lane >> 5) * ACH) * RED_STRIDE + (lane & 31)] = fold_halves(va, vb);
    }
    wave_sync();
    const int v = lane / LPV;
    const double* rv = red + v * RED_STRIDE + (lane % LPV) * (32 / LPV);
    double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int x = 0; x < 32 / LPV; ++x) part[x & 3] += rv[x];
    double sum = (part[0] + part[1]) + (part[2] + part[3]);
#pragma unroll
    for (int x = 1; x < LPV; x <<= 1) sum += __shfl_xor(sum, x);
    if (lane % LPV == 0 && i + (v >> 1) < nl) out[2 * (i + (v >> 1)) + (v & 1)] = sum;
    wave_sync();
    const int woke = wave_any(st.sc != 0) ? rescale_chunk<R>(st) : 0;
    if (woke) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (woke & (1 << r)) {
          const int q = blk * (LANES * R) + r * LANES + lane;
          const double4 sd = *reinterpret_cast<const double4*>(Gm + (size_t)q * pstride);
          Sre[r] = sd.x;
          Sim[r] = sd.y;
          Dre[r] = sd.z;
          Dim[r] = sd.w;
        }
      // (rare) complete these loads here rather than at their first use, where the
      // wait would also cover the tile prefetch
      __builtin_amdgcn_s_waitcnt(0);
    }
  }
  wave_sync();   // the next item's tile 0 is written after this one's last reads
}

template <int R>
__global__ void __launch_bounds__(FP64_ANA_WAVES * LANES) legendre_analysis_f64_kernel(PlanDev P, Leg64Dev L,
                                                                     const double* __restrict__ G,
                                                                     double2* __restrict__ partial) {
  // the queue's counter, then per-wave LDS: waves run unrelated items and never synchronise
  extern __shared__ __attribute__((aligned(16))) double leg64_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);
  const int lane = threadIdx.x % LANES;
  double* lds = leg64_lds + 2 + wave * ANA_LDS;
  for (ItemQueue q(L.ana, leg64_lds); q.next(lane);) {
    const int k = q.k;
    analysis_item<R>(P, L, k, L.ana.items[k], blockIdx.y, lane, lds, G, partial);
  }
}

// Filtered coefficients for the synthesis, one thread per (l, m, map):
//   SY_FROM_PARTIAL  a = C_l sum_blk partial, s = f_l(lambda) a
//   SY_ALM_ONLY      a = C_l sum_blk partial (the forward transform), s = a
//   SY_FROM_ALM      s = caller's alm (imaginary part of m = 0 dropped)
// s goes to alm_out when requested; bcoef = C_l s, in the padded row layout of
// the recurrence tables (zeros beyond lmax) so the synthesis can read whole chunks.
// A flat grid over the padded rows r of every m (m = row_m[r], l = m + r - row_off[m];
// padding rows get zeros) and the maps: with one workgroup per m instead, the long rows
// of small m went to a few waves in turn, each waiting on its loads.
__global__ void legendre_coeff_kernel(PlanDev P, Leg64Dev L, SynthArgs a) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int map = blockIdx.y;
  const bool chi = a.chi2 != nullptr && a.mode == SY_FROM_PARTIAL;
  double chi_acc = 0.0;
  if (r < P.rows_total) {
    const int lmax = P.lmax;
    const int m = P.row_m[r];
    const int i = (int)(r - P.row_off[m]);
    double2 b = make_double2(0.0, 0.0);
    if (i < lmax - m + 1) {
      const int64_t at = alm_index(lmax, m, m) + i;
      const double c = P.C[r];
      double2 alm;
      if (a.mode == SY_FROM_ALM) {
        alm = a.alm_in[(size_t)map * P.nalm + at];
        if (m == 0) alm.y = 0.0;
      } else {
        // the ring phase already applied Omega to G
        const double2 p = block_partials(P, L, a.partial + (size_t)map * P.nblk_max * P.nalm + at, m, i);
        alm = make_double2(p.x * c, p.y * c);
        if (a.mode == SY_FROM_PARTIAL) {
          const double cl = P.cl[m + i];
          const double f = cl > 0.0 ? cl / (cl + a.lambda * P.tau * P.omega) : 0.0;
          alm.x *= f;
          alm.y *= f;
          // chi^2 prior term of the new iterate: w_m |s_lm|^2 / C_l (w = 1 at m = 0, else 2)
          if (chi && cl > 0.0) chi_acc = (m == 0 ? 1.0 : 2.0) * (alm.x * alm.x + alm.y * alm.y) / cl;
        }
      }
      if (a.alm_out) a.alm_out[(size_t)map * P.nalm + at] = alm;
      b = make_double2(alm.x * c, alm.y * c);
    }
    if (a.mode != SY_ALM_ONLY) a.bcoef[(size_t)map * P.rows_total + r] = b;
  }
  if (chi) block_sum_add(chi_acc, a.chi2 + map * a.chi2_stride);
}

constexpr int SCH = 16;   // synthesis: values of l per coefficient tile and scale check
static_assert(LTILE % SCH == 0 && SCH == CHUNK, "synthesis chunking");

// e_r += u_r b_V and o_r += w_r b_{V+1} (complex b) for the R ring pairs of a lane. Lane i of
// every row of 16 holds b_i of a tile of 16; the FMAs take the lane of the row they need as an
// operand (DPP row_newbcast), so the coefficients cost neither LDS nor registers: read from LDS
// as broadcasts they took as long as the FP64 work (32 bytes per lane and FMA quartet, and one
// LDS for four SIMDs), through the scalar cache every chunk waited on it. The s_nop covers a
// write of bx or by just before (two wait states before a DPP read).
#define MWF_FMAC(ACC, B, U, LANE) "\n\tv_fmac_f64_dpp %" ACC ", %" B ", %" U " row_newbcast:%" LANE " row_mask:0xf bank_mask:0xf"
#define MWF_RING(A0, A1, A2, A3, U, W) \
  MWF_FMAC(A0, "[x]", U, "[v]") MWF_FMAC(A1, "[y]", U, "[v]") MWF_FMAC(A2, "[x]", W, "[w]") MWF_FMAC(A3, "[y]", W, "[w]")
#define MWF_OUT(r) "+v"(er[r]), "+v"(ei[r]), "+v"(orr[r]), "+v"(oi[r])
#define MWF_IN [x] "v"(bx), [y] "v"(by), [v] "n"(V), [w] "n"(V + 1)
template <int V, int R>
__device__ __forceinline__ void accumulate(double (&er)[R], double (&ei)[R], double (&orr)[R], double (&oi)[R],
                                           const double (&u)[R], const double (&w)[R], double bx, double by) {
  static_assert(R == 1 || R == 2 || R == 4, "ring pairs per lane");
  if constexpr (R == 1)
    asm volatile("s_nop 1" MWF_RING("0", "1", "2", "3", "[u0]", "[w0]") : MWF_OUT(0) : MWF_IN, [u0] "v"(u[0]), [w0] "v"(w[0]));
  else if constexpr (R == 2)
    asm volatile("s_nop 1" MWF_RING("0", "1", "2", "3", "[u0]", "[w0]") MWF_RING("4", "5", "6", "7", "[u1]", "[w1]")
                 : MWF_OUT(0), MWF_OUT(1)
                 : MWF_IN, [u0] "v"(u[0]), [w0] "v"(w[0]), [u1] "v"(u[1]), [w1] "v"(w[1]));
  else
    asm volatile("s_nop 1" MWF_RING("0", "1", "2", "3", "[u0]", "[w0]") MWF_RING("4", "5", "6", "7", "[u1]", "[w1]")
                 MWF_RING("8", "9", "10", "11", "[u2]", "[w2]") MWF_RING("12", "13", "14", "15", "[u3]", "[w3]")
                 : MWF_OUT(0), MWF_OUT(1), MWF_OUT(2), MWF_OUT(3)
                 : MWF_IN, [u0] "v"(u[0]), [w0] "v"(w[0]), [u1] "v"(u[1]), [w1] "v"(w[1]), [u2] "v"(u[2]), [w2] "v"(w[2]),
                   [u3] "v"(u[3]), [w3] "v"(w[3]));
}
#undef MWF_IN
#undef MWF_OUT
#undef MWF_RING
#undef MWF_FMAC

template <int R>
__device__ __forceinline__ void synthesis_item(const PlanDev& P, const Leg64Dev& L, const int k, const Item64 it,
                                               const int map, const int lane, double* __restrict__ sA,
                                               const double2* __restrict__ bcoef, double* __restrict__ F) {
  const int m = it.m, blk = it.blk;
  const int64_t roff = P.row_off[m] + it.i0;
  const double* __restrict__ Arow = P.A + roff;
  const double2* __restrict__ brow = bcoef + (size_t)map * P.rows_total + roff;
  const int nact = P.n_active[m];
  const int nl = it.i1 - it.i0;
  // recurrence coefficients of LTILE values of l: lane i loads l = base + i one tile ahead,
  // the tile in use is read from LDS (the same address in every lane); synthesis coefficients
  // of SCH values of l likewise, in registers. The loads are unconditional, with the index
  // clamped to the first entry of the row's zero padding.
  auto tile_a = [&](int i) { return Arow[min(i, nl)]; };
  auto tile_b = [&](int i) { return brow[min(i + (lane & (SCH - 1)), nl)]; };
  RingState<R> st;
  init_rings<R>(P, L.syn, L.z, k, blk, lane, nact, st);
  sA[lane] = tile_a(lane);
  double2 b = tile_b(0);
  // every load issued so far (ring states, tile 0) completes here
  __builtin_amdgcn_s_waitcnt(0);
  wave_sync();
  double An = tile_a(LTILE + lane);
  double Ere[R], Eim[R], Ore[R], Oim[R];
#pragma unroll
  for (int r = 0; r < R; ++r) Ere[r] = Eim[r] = Ore[r] = Oim[r] = 0.0;

  for (int i = 0; i < nl; i += SCH) {
    const int t0 = i & (LTILE - 1);
    if (t0 == 0 && i > 0) {
      wave_sync();
      sA[lane] = An;
      wave_sync();
      An = tile_a(i + LTILE + lane);
    }
    const double2 bn = tile_b(i + SCH);
    const unsigned scaled = st.sc;
    const double2* Ac = reinterpret_cast<const double2*>(sA + t0);
    auto step = [&](auto V) {
      constexpr int v = decltype(V)::value;     // l - m = i + v .. i + v + 3
      const double2 A0 = Ac[v / 2], A1 = Ac[v / 2 + 1];
#pragma unroll
      for (int r = 0; r < R; ++r) step_pair(st.mu1[r], st.mu2[r], st.z[r], A0.x, A0.y);
      accumulate<v>(Ere, Eim, Ore, Oim, st.mu2, st.mu1, b.x, b.y);
#pragma unroll
      for (int r = 0; r < R; ++r) step_pair(st.mu1[r], st.mu2[r], st.z[r], A1.x, A1.y);
      accumulate<v + 2>(Ere, Eim, Ore, Oim, st.mu2, st.mu1, b.x, b.y);
    };
    step(std::integral_constant<int, 0>());
    step(std::integral_constant<int, 4>());
    step(std::integral_constant<int, 8>());
    step(std::integral_constant<int, 12>());
    b = bn;
    // a ring still scaled at the chunk start has contributed nothing so far: clear it
    if (wave_any(scaled != 0)) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (scaled & (0xffu << (8 * r))) Ere[r] = Eim[r] = Ore[r] = Oim[r] = 0.0;
      rescale_chunk<R>(st);
    }
  }

  const size_t pstride = gf_stride(P.lmax);
  double* Fm = F + (size_t)map * P.npairs * pstride + (size_t)m * 4;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int q = blk * (LANES * R) + r * LANES + lane;
    if (q < nact)
      *reinterpret_cast<double4*>(Fm + (size_t)q * pstride) =
          make_double4(Ere[r], Eim[r], Ore[r], Oim[r]);
  }
  wave_sync();   // the next item's tile 0 is written after this one's last reads
}

template <int R>
__global__ void __launch_bounds__(FP64_SYN_WAVES * LANES) legendre_synthesis_f64_kernel(PlanDev P, Leg64Dev L,
                                                                      const double2* __restrict__ bcoef,
                                                                      double* __restrict__ F) {
  // the queue's counter, then per-wave LDS: waves run unrelated items and never synchronise
  extern __shared__ __attribute__((aligned(16))) double leg64_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);
  const int lane = threadIdx.x % LANES;
  double* sA = leg64_lds + 2 + wave * LTILE;
  for (ItemQueue q(L.syn, leg64_lds); q.next(lane);) {
    const int k = q.k;
    synthesis_item<R>(P, L, k, L.syn.items[k], blockIdx.y, lane, sA, bcoef, F);
  }
}

// Plan time, per (m, ring pair): the first l - m + 1 at which lambda_lm(z_q) has
// risen above the scaled range (its scale reached 0; 0 if it starts there), or
// WAKE_NEVER if that does not happen for l <= lmax (the pair is skipped for m); and
// likewise in `rise`, unless that is null, the first l - m at which it exceeds 2^-128.
__global__ void reach_kernel(PlanDev P, uint16_t* __restrict__ wake, uint16_t* __restrict__ rise) {
  const int m = blockIdx.y;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= P.npairs) return;
  const RingPair rp = P.pairs[q];
  double v;
  int s;
  sectoral_seed(m, rp.sin_t, P.norm_m[m], &v, &s);
  uint16_t w = s == 0 ? 0 : WAKE_NEVER, e = s == 0 && fabs(v) > RISE_THRESH ? 0 : WAKE_NEVER;
  if (rise ? e != 0 : w != 0) {
    const double* Arow = P.A + P.row_off[m];
    double mu1 = 0.0, mu2 = -v;
    for (int l = m; l <= P.lmax; ++l) {
      const double mu = fma(Arow[l - m] * rp.z, mu1, -mu2);
      mu2 = mu1;
      mu1 = mu;
      if (s > 0 && fabs(mu1) > BIG_THRESH) {
        mu1 *= RESCALE;
        mu2 *= RESCALE;
        if (--s == 0) {
          w = (uint16_t)(l - m + 1);
          if (!rise) break;
        }
      }
      if (s == 0 && fabs(mu1) > RISE_THRESH) {
        e = (uint16_t)(l - m);
        break;
      }
    }
  }
  wake[(size_t)m * P.npairs + q] = w;
  if (rise) rise[(size_t)m * P.npairs + q] = e;
}

// Plan time: the recurrence state of every ring pair of every item at its first l (workgroup k:
// item k, thread t: pair t of the block), run with the kernels' own steps and scale checks (ch
// values of l per check; items start at multiples of it).
__global__ void start_state_kernel(PlanDev P, const Item64* __restrict__ items, int ch,
                                   double2* __restrict__ state, uint8_t* __restrict__ scale) {
  const Item64 it = items[blockIdx.x];
  const int m = it.m, rb = blockDim.x, q = it.blk * rb + threadIdx.x;
  const size_t at = (size_t)blockIdx.x * rb + threadIdx.x;
  double mu1 = 0.0, mu2 = 0.0;   // mu_{m-1}; with A_mm = 0 the first step yields mu_m = -mu2
  int s = 0;
  if (q < P.n_active[m]) {
    const RingPair rp = P.pairs[q];
    double v;
    sectoral_seed_full(m, rp.z, P.norm_m[m], &v, &s);
    mu2 = -v;
    const double* Arow = P.A + P.row_off[m];
    for (int i = 0; i < it.i0; i += ch) {
      for (int j = i; j < i + ch; j += 2) step_pair(mu1, mu2, rp.z, Arow[j], Arow[j + 1]);
      if (s > 0 && fmax(fabs(mu1), fabs(mu2)) > BIG_THRESH) {
        mu1 *= RESCALE;
        mu2 *= RESCALE;
        s -= 1;
      }
    }
  }
  state[at] = make_double2(mu1, mu2);
  scale[at] = (uint8_t)s;
}

template <int R>
hipError_t launch_ana_r(const PlanDev& P, const Leg64Dev& L, int nmaps, const double* G, double2* partial,
                        hipStream_t s) {
  const size_t lds = ((size_t)L.ana.waves * ANA_LDS + 2) * sizeof(double);
  if (hipError_t e = ensure_dynamic_lds((const void*)legendre_analysis_f64_kernel<R>, lds)) return e;
  hipLaunchKernelGGL(legendre_analysis_f64_kernel<R>, dim3(L.ana.nwg, nmaps),
                     dim3(L.ana.waves * LANES), lds, s, P, L, G, partial);
  return hipGetLastError();
}

template <int R>
hipError_t launch_syn_r(const PlanDev& P, const Leg64Dev& L, const SynthArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(legendre_synthesis_f64_kernel<R>, dim3(L.syn.nwg, a.nmaps),
                     dim3(L.syn.waves * LANES), ((size_t)L.syn.waves * LTILE + 2) * sizeof(double), s, P, L, a.bcoef, a.F);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_legendre_analysis_f64(const PlanDev& P, const Leg64Dev& lists, int nmaps, const double* G,
                                        double2* partial, hipStream_t s) {
  Leg64Dev L = lists;
  if (nmaps >= L.batch_from) L.ana = L.ana_batch;
  switch (L.ana.rb / LANES) {
    case 1: return launch_ana_r<1>(P, L, nmaps, G, partial, s);
    case 2: return launch_ana_r<2>(P, L, nmaps, G, partial, s);
    case 4: return launch_ana_r<4>(P, L, nmaps, G, partial, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_legendre_coeff(const PlanDev& P, const Leg64Dev& L, const SynthArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(legendre_coeff_kernel, dim3((unsigned)((P.rows_total + 255) / 256), a.nmaps), dim3(256), 0, s, P, L,
                     a);
  return hipGetLastError();
}

hipError_t launch_legendre_synthesis_f64(const PlanDev& P, const Leg64Dev& L, const SynthArgs& a, hipStream_t s) {
  switch (L.syn.rb / LANES) {
    case 1: return launch_syn_r<1>(P, L, a, s);
    case 2: return launch_syn_r<2>(P, L, a, s);
    case 4: return launch_syn_r<4>(P, L, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_reach(const PlanDev& P, uint16_t* wake, uint16_t* rise, hipStream_t s) {
  dim3 grid((P.npairs + 127) / 128, P.lmax + 1);
  hipLaunchKernelGGL(reach_kernel, grid, dim3(128), 0, s, P, wake, rise);
  return hipGetLastError();
}

hipError_t launch_start_state(const PlanDev& P, const Leg64List& T, int nitems, int ch,
                              double2* state, uint8_t* scale, hipStream_t s) {
  hipLaunchKernelGGL(start_state_kernel, dim3(nitems), dim3(T.rb), 0, s, P, T.items, ch, state, scale);
  return hipGetLastError();
}

}  // namespace mwf
