// Plan-time tables shared by every plan of a given (device, nside, lmax):
// HEALPix ring geometry (Gorski et al. 2005), the rescaled Legendre recurrence
// coefficients, FFT twiddles, mixed-radix and Bluestein tables, and the polar-skip work
// lists.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <complex>
#include <map>
#include <queue>
#include <tuple>

#include "runtime.hpp"

namespace mwf {

namespace {

constexpr long double PI_L = 3.141592653589793238462643383279502884L;
// Ring pairs whose class length (n; twice n for mixed radix; the Bluestein length M) is at
// most this many points run one wave per pair when batched; longer ones a larger workgroup
// (512 threads for rings that are not a power of two, 256 for power-of-two rings).
constexpr int SMALL_FFT = 1024;

bool is_pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }

int ilog2_ceil(int64_t x) {
  int l = 0;
  while ((int64_t(1) << l) < x) ++l;
  return l;
}

// In-place iterative radix-2 FFT in long double (plan time only).
void host_fft(std::vector<std::complex<long double>>& a, int sign) {
  const size_t n = a.size();
  for (size_t i = 1, j = 0; i < n; ++i) {
    size_t bit = n >> 1;
    for (; j & bit; bit >>= 1) j ^= bit;
    j ^= bit;
    if (i < j) std::swap(a[i], a[j]);
  }
  for (size_t len = 2; len <= n; len <<= 1) {
    for (size_t k = 0; k < len / 2; ++k) {
      const long double ang = sign * 2.0L * PI_L * (long double)k / (long double)len;
      const std::complex<long double> w(cosl(ang), sinl(ang));
      for (size_t i = k; i < n; i += len) {
        const auto u = a[i], v = a[i + len / 2] * w;
        a[i] = u + v;
        a[i + len / 2] = u - v;
      }
    }
  }
}

std::mutex g_geo_mu;
// Weak entries: the tables of a shape live while a plan or serving lane holds them.
std::map<std::tuple<int, int, int>, std::weak_ptr<Geometry>> g_geo;

// Per (m, ring pair), what launch_reach gives; rise is empty where it was not asked for.
struct Reach {
  std::vector<uint16_t> wake, rise;
};

// Runs the reach kernel of a geometry whose recurrence tables are on the device.
int run_reach(const Geometry& g, bool rise, Reach* out) {
  PlanDev D{};
  D.nside = g.nside;
  D.lmax = g.lmax;
  D.npairs = g.npairs;
  D.pairs = g.pairs;
  D.A = g.A;
  D.row_off = g.row_off;
  D.norm_m = g.norm;
  const size_t n = (size_t)(g.lmax + 1) * g.npairs;
  uint16_t *dw = nullptr, *dr = nullptr;
  DevMem tmp;
  int rc;
  if ((rc = tmp.alloc(&dw, n)) || (rise && (rc = tmp.alloc(&dr, n)))) return rc;
  MWF_HIP(launch_reach(D, dw, dr, nullptr));
  out->wake.resize(n);
  MWF_HIP(hipMemcpy(out->wake.data(), dw, n * sizeof(uint16_t), hipMemcpyDeviceToHost));
  if (rise) {
    out->rise.resize(n);
    MWF_HIP(hipMemcpy(out->rise.data(), dr, n * sizeof(uint16_t), hipMemcpyDeviceToHost));
  }
  return WF_OK;
}

// Work items (m, block of rb ring pairs) over the active pairs of every m, largest first.
std::vector<WorkItem> items_by_size(const Geometry& g, int rb) {
  const int lmax = g.lmax;
  std::vector<WorkItem> items;
  for (int m = 0; m <= lmax; ++m) {
    const int nb = (g.n_active[m] + rb - 1) / rb;
    for (int b = 0; b < nb; ++b) items.push_back({m, b});
  }
  std::stable_sort(items.begin(), items.end(), [&](const WorkItem& a, const WorkItem& b) {
    auto c = [&](const WorkItem& w) {
      const int rings = std::min(rb, g.n_active[w.m] - w.blk * rb);
      return (double)(lmax - w.m + 1) * (double)std::max(rings, 1);
    };
    return c(a) > c(b);
  });
  if (items.empty()) items.push_back({0, 0});
  return items;
}

// reach receives the polar reach of every (m, ring pair), with the rises for an FP64 plan.
int build_geometry(Geometry& g, bool fp64, Reach* reach) {
  const int nside = g.nside, lmax = g.lmax;
  g.npix = 12LL * nside * nside;
  g.nalm = (int64_t)(lmax + 1) * (lmax + 2) / 2;
  g.nrings = 4 * nside - 1;
  g.npairs = 2 * nside;
  g.omega = 4.0 * 3.141592653589793238462643383279502884 / (double)g.npix;
  int rc;

  // ---- ring pairs, equator first
  std::vector<RingPair> pairs(g.npairs);
  std::vector<int> blue_len;
  for (int q = 0; q < g.npairs; ++q) {
    const int i = 2 * nside - q;
    const RingGeo gn = ring_geometry(nside, i);
    RingPair rp{};
    rp.z = gn.z;
    rp.sin_t = std::sqrt((1.0 - gn.z) * (1.0 + gn.z));
    rp.start_n = gn.start;
    rp.start_s = (q == 0) ? -1 : ring_geometry(nside, 4 * nside - i).start;
    rp.nphi = gn.nphi;
    rp.ph_num = gn.ph_num;
    rp.ph_den = gn.ph_den;
    if (is_pow2(gn.nphi)) {
      rp.log2n = ilog2_ceil(gn.nphi);
      rp.bl_M = 0;
      g.tw_len = std::max(g.tw_len, gn.nphi);
    } else if ((rp.mix = mixed_radix_passes(gn.nphi)) != 0) {
      // 2^a 3^b 5^c 7^d points: radix-2/4/8 passes (their twiddles from the power-of-two
      // table, as for a 2^a-point transform), then the odd passes
      rp.log2n = -1;
      rp.bl_M = 0;
      g.tw_len = std::max(g.tw_len, gn.nphi & -gn.nphi);
    } else {
      rp.log2n = -1;
      rp.bl_M = 1 << ilog2_ceil(2 * gn.nphi - 1);
      g.tw_len = std::max(g.tw_len, rp.bl_M);
      blue_len.push_back(gn.nphi);
    }
    pairs[q] = rp;
  }

  // ---- Bluestein chirps exp(-i pi j^2 / n) and filter spectra H = FFT_M(h),
  //      h_j = exp(+i pi j^2 / n) for |j| < n
  std::vector<double2> blue, chirp;
  {
    std::vector<int64_t> off_of(4 * nside + 1, -1), coff_of(4 * nside + 1, -1);
    for (int n : blue_len) {
      if (off_of[n] >= 0) continue;
      coff_of[n] = (int64_t)chirp.size();
      for (int j = 0; j < n; ++j) {
        const long double ang = -PI_L * (long double)(((int64_t)j * j) % (2LL * n)) / (long double)n;
        chirp.push_back(make_double2((double)cosl(ang), (double)sinl(ang)));
      }
      const int M = 1 << ilog2_ceil(2 * n - 1);
      std::vector<std::complex<long double>> h(M, 0.0L);
      for (int j = 0; j < n; ++j) {
        const long double ang = PI_L * (long double)(((int64_t)j * j) % (2LL * n)) / (long double)n;
        const std::complex<long double> w(cosl(ang), sinl(ang));
        h[j] = w;
        if (j) h[M - j] = w;
      }
      host_fft(h, -1);
      off_of[n] = (int64_t)blue.size();
      for (int k = 0; k < M; ++k) blue.push_back(make_double2((double)h[k].real(), (double)h[k].imag()));
    }
    for (auto& rp : pairs)
      if (rp.bl_M > 0) {
        rp.bl_off = off_of[rp.nphi];
        rp.chirp_off = coff_of[rp.nphi];
      }
    if (blue.empty()) blue.push_back(make_double2(0.0, 0.0));
    if (chirp.empty()) chirp.push_back(make_double2(0.0, 0.0));
  }
  // ---- mixed-radix rings: exp(-2 pi i t / n), t < n, per distinct length
  std::vector<double2> mixtw;
  {
    std::vector<int64_t> off_of(4 * nside + 1, -1);
    for (auto& rp : pairs) {
      if (!rp.mix) continue;
      const int n = rp.nphi;
      if (off_of[n] < 0) {
        off_of[n] = (int64_t)mixtw.size();
        for (int t = 0; t < n; ++t) {
          const long double ang = -2.0L * PI_L * (long double)t / (long double)n;
          mixtw.push_back(make_double2((double)cosl(ang), (double)sinl(ang)));
        }
      }
      rp.bl_off = off_of[n];
    }
    if (mixtw.empty()) mixtw.push_back(make_double2(0.0, 0.0));
  }
  std::vector<double2> tw(g.tw_len / 2);
  for (int k = 0; k < g.tw_len / 2; ++k) {
    const long double ang = -2.0L * PI_L * (long double)k / (long double)g.tw_len;
    tw[k] = make_double2((double)cosl(ang), (double)sinl(ang));
  }
  auto to32 = [](const std::vector<double2>& v) {
    std::vector<float2> o(v.size());
    for (size_t i = 0; i < v.size(); ++i) o[i] = make_float2((float)v[i].x, (float)v[i].y);
    return o;
  };

  // ---- recurrence tables mu_l = (A z) mu_{l-1} - mu_{l-2}, lambda = C mu; padded rows
  std::vector<int64_t> row_off(lmax + 1);
  std::vector<int32_t> row_m;             // m of every padded row
  std::vector<double> A, C, norm(lmax + 1);
  {
    int64_t off = 0;
    for (int m = 0; m <= lmax; ++m) {
      row_off[m] = off;
      off += (lmax - m + 1) + ROW_PAD;
    }
    g.rows_total = off;
    row_m.resize(off);
    for (int m = 0; m <= lmax; ++m)
      for (int64_t r = row_off[m]; r < (m < lmax ? row_off[m + 1] : off); ++r) row_m[r] = m;
    A.assign(off, 0.0);
    C.assign(off, 0.0);
    long double nm = 1.0L / sqrtl(4.0L * PI_L);
    for (int m = 0; m <= lmax; ++m) {
      if (m > 0) nm *= -sqrtl((2.0L * m + 1.0L) / (2.0L * m));
      norm[m] = (double)nm;
      auto alpha = [&](int l) {
        return sqrtl((4.0L * l * l - 1.0L) / ((long double)(l - m) * (long double)(l + m)));
      };
      const int64_t r = row_off[m];
      long double c_lm2 = 1.0L, c_lm1 = 1.0L, alm1 = 0.0L;
      A[r] = 0.0;
      C[r] = 1.0;
      if (m + 1 <= lmax) {
        alm1 = alpha(m + 1);
        A[r + 1] = (double)alm1;
        C[r + 1] = 1.0;
      }
      for (int l = m + 2; l <= lmax; ++l) {
        const long double al = alpha(l);
        const long double cl_ = c_lm2 * al / alm1;
        A[r + (l - m)] = (double)(al * c_lm1 / cl_);
        C[r + (l - m)] = (double)cl_;
        c_lm2 = c_lm1;
        c_lm1 = cl_;
        alm1 = al;
      }
    }
  }

  DevMem& M = g.mem;
  if ((rc = M.upload(&g.pairs, pairs))) return rc;
  if ((rc = M.upload(&g.A, A))) return rc;
  if ((rc = M.upload(&g.C, C))) return rc;
  if ((rc = M.upload(&g.row_off, row_off))) return rc;
  if ((rc = M.upload(&g.row_m, row_m))) return rc;
  if ((rc = M.upload(&g.norm, norm))) return rc;
  if ((rc = M.upload(&g.tw, tw))) return rc;
  if ((rc = M.upload(&g.chirp, chirp))) return rc;
  if ((rc = M.upload(&g.blue, blue))) return rc;
  if ((rc = M.upload(&g.tw32, to32(tw)))) return rc;
  if ((rc = M.upload(&g.chirp32, to32(chirp)))) return rc;
  if ((rc = M.upload(&g.blue32, to32(blue)))) return rc;
  if ((rc = M.upload(&g.mixtw, mixtw))) return rc;
  if ((rc = M.upload(&g.mixtw32, to32(mixtw)))) return rc;

  // ---- ring launch classes by transform kind and length
  {
    std::vector<int32_t> lists[2][NRING_CLASSES];
    int lens[2][NRING_CLASSES];
    for (auto& row : lens)
      for (int& l : row) l = 4;
    // a ring that is not a power of two (mixed radix or Bluestein) goes with the Bluestein
    // rings, its class length at least twice its own (the kernels of that kind assume it)
    auto class_len = [&](const RingPair& rp) {
      return rp.bl_M > 0 ? rp.bl_M : (rp.mix ? 2 * rp.nphi : rp.nphi);
    };
    for (int q = 0; q < g.npairs; ++q) {
      const bool npot = pairs[q].log2n < 0;
      const int L = class_len(pairs[q]);
      const int c0 = npot ? 0 : 1;                    // few maps: by kind only
      const int c1 = L <= SMALL_FFT ? 2 : c0;          // batched: short ones apart
      lists[0][c0].push_back(q);
      lens[0][c0] = std::max(lens[0][c0], L);
      lists[1][c1].push_back(q);
      lens[1][c1] = std::max(lens[1][c1], L);
    }
    for (int k = 0; k < 2; ++k)
      for (int c = 0; c < NRING_CLASSES; ++c) {
        int32_t* d = nullptr;
        if ((rc = M.upload(&d, lists[k][c]))) return rc;
        g.ring_cls[k][c] = RingClass{d, (int32_t)lists[k][c].size(), lens[k][c]};
      }
    // All ring pairs in one list, longest transforms first, up to Nside 512 (at 1024 the FP64 buffer
    // of the longest leaves one workgroup a CU, and the other rings would take its size): one or a
    // few maps take one launch. The launches by kind, the event pair that forked and joined their
    // streams and the gaps around them were half of a sweep at Nside 16 to 64.
    if (std::max(lens[0][0], lens[0][1]) <= RING_ONE_LAUNCH) {
      std::vector<int32_t> all(g.npairs);
      for (int q = 0; q < g.npairs; ++q) all[q] = q;
      auto own_len = [&](int q) { return pairs[q].mix ? pairs[q].nphi : class_len(pairs[q]); };
      std::stable_sort(all.begin(), all.end(), [&](int a, int b) {
        auto cost = [&](int q) { return (pairs[q].bl_M > 0 ? 2 : 1) * own_len(q); };
        return cost(a) > cost(b);
      });
      int len = 4;
      for (int q : all) len = std::max(len, own_len(q));
      int32_t* d = nullptr;
      if ((rc = M.upload(&d, all))) return rc;
      g.ring_all = RingClass{d, g.npairs, len};
    } else {
      // Few maps otherwise: Bluestein rings of the longest transform apart from the shorter ones: at the
      // longest length alone they can hold all of the chip's LDS. The mixed-radix rings go
      // with the shorter ones at their own length: these two launches run only the plain
      // ring kernel, whose transforms need n <= 4 MAXB NT, not the half-length bound of
      // the class lists (with the longest ones, or at twice their length, they made the
      // one-map ring phase 5 and 16 us slower).
      std::vector<int32_t> bl[2];
      int bl_len[2] = {4, 4};
      for (int q : lists[0][0]) {
        const int k = pairs[q].bl_M == lens[0][0] ? 0 : 1;
        bl[k].push_back(q);
        bl_len[k] = std::max(bl_len[k], pairs[q].mix ? pairs[q].nphi : class_len(pairs[q]));
      }
      for (int k = 0; k < 2; ++k) {
        int32_t* d = nullptr;
        if ((rc = M.upload(&d, bl[k]))) return rc;
        g.blue_split[k] = RingClass{d, (int32_t)bl[k].size(), bl_len[k]};
      }
    }
    // such a split of the batched class 0, whatever the size: at 64 maps the 2048-point Bluestein rings and
    // the long mixed-radix rings ran in the launch sized for the 4096-point ones
    std::vector<int32_t> ls[2];
    int ls_len[2] = {4, 4};
    for (int q : lists[1][0]) {
      const int k = pairs[q].bl_M == lens[1][0] ? 0 : 1;
      ls[k].push_back(q);
      ls_len[k] = std::max(ls_len[k], pairs[q].mix ? pairs[q].nphi : class_len(pairs[q]));
    }
    for (int k = 0; k < 2; ++k) {
      int32_t* d = nullptr;
      if ((rc = M.upload(&d, ls[k]))) return rc;
      g.long_split[k] = RingClass{d, (int32_t)ls[k].size(), ls_len[k]};
    }
  }

  // ---- polar skip: ring pairs whose lambda_lm never leaves the negligible range
  {
    if ((rc = run_reach(g, fp64, reach))) return rc;
    const std::vector<uint16_t>& wake = reach->wake;
    g.n_active.assign(lmax + 1, 0);
    g.units_active = 0;
    for (int m = 0; m <= lmax; ++m) {
      int na = 0;
      for (int q = 0; q < g.npairs; ++q)
        if (wake[(size_t)m * g.npairs + q] != WAKE_NEVER) na = q + 1;
      g.n_active[m] = na;
      g.units_active += (int64_t)na * (lmax - m + 1);
    }
  }
  auto make_items = [&](int rb) { return items_by_size(g, rb); };
  // Matrix-core lists, ordered for the L2 caches of the XCDs. A row of G or F holds the
  // entries of consecutive m side by side (16 bytes each in FP32), so the items of one ring
  // block and eight consecutive m read or write the same one or two 128-byte lines of every
  // row. Such a group, taken in the
  // order of its most costly item, is dealt with seven others so that group g of the eight
  // holds positions g, g + 8, ..., g + 56: a dispatch that deals workgroups to the XCDs in
  // turn runs each group on one XCD, its members one after another. Missing members are
  // empty items (m = -1, the kernels return at once).
  auto xcd_order = [&](const std::vector<WorkItem>& items) {
    std::vector<std::vector<WorkItem>> groups;
    std::map<std::pair<int, int>, int> index;
    for (const WorkItem& w : items) {
      const auto key = std::make_pair(w.blk, w.m >> 3);
      auto f = index.find(key);
      if (f == index.end()) {
        f = index.emplace(key, (int)groups.size()).first;
        groups.emplace_back();
      }
      groups[f->second].push_back(w);
    }
    for (auto& g : groups)
      std::sort(g.begin(), g.end(), [](const WorkItem& a, const WorkItem& b) { return a.m < b.m; });
    std::vector<WorkItem> out;
    for (size_t s0 = 0; s0 < groups.size(); s0 += 8)
      for (size_t k = 0; k < 8; ++k)
        for (size_t g = s0; g < s0 + 8; ++g)
          out.push_back(g < groups.size() && k < groups[g].size() ? groups[g][k] : WorkItem{-1, 0});
    return out;
  };
  g.ring_block_ana = ana_ring_block(g.npairs);
  g.nblk_max_ana = (g.npairs + g.ring_block_ana - 1) / g.ring_block_ana;
  std::vector<int32_t> nblk(lmax + 1);
  for (int m = 0; m <= lmax; ++m) nblk[m] = (g.n_active[m] + g.ring_block_ana - 1) / g.ring_block_ana;
  const auto i128 = xcd_order(make_items(128)), i256 = xcd_order(make_items(256)), i64 = xcd_order(make_items(64));
  g.n_a128 = (int)i128.size();
  g.n_a256 = (int)i256.size();
  g.n_s64 = (int)i64.size();
  if ((rc = M.upload(&g.nact, g.n_active))) return rc;
  if ((rc = M.upload(&g.nblk_ana, nblk))) return rc;
  if ((rc = M.upload(&g.items_a128, i128))) return rc;
  if ((rc = M.upload(&g.items_a256, i256))) return rc;
  if ((rc = M.upload(&g.items_s64, i64))) return rc;
  return WF_OK;
}

// Workgroups and waves of a launch of one map: one workgroup per CU, of as many waves as give every
// CU work where items are few.
void one_map_shape(size_t items, int n_cu, int max_waves, int* nwg, int* waves) {
  int W = 1;
  while (W < max_waves && (int64_t)W * n_cu < (int64_t)items) W = std::min(2 * W, max_waves);
  *waves = W;
  *nwg = std::max(1, std::min(n_cu, (int)((items + W - 1) / W)));
}

// Packs items (with their costs) into nwg workgroups: items, most costly first, each go to the
// least-loaded workgroup, which keeps that order. off: the item range of each workgroup.
// In a full launch the items of eight consecutive m go to the workgroups of one XCD (workgroup b
// runs on XCD b mod 8): their 32-byte entries of G and F share 128-byte lines, which then are
// fetched into one L2 and written back from one (Nside 512: analysis 121 -> 116 us, synthesis
// 93 -> 91 us).
std::vector<Item64> pack_items(const std::vector<Item64>& items, const std::vector<int64_t>& cost, int nwg,
                               std::vector<int32_t>* off) {
  const int nx = nwg % 8 == 0 && nwg >= 64 ? 8 : 1;
  // least-loaded dealing of ids (in the order given, with their loads) to n places
  auto deal = [](const std::vector<int>& ids, const std::vector<int64_t>& load, int n) {
    std::vector<std::vector<int>> to(n);
    using Load = std::pair<int64_t, int>;
    std::priority_queue<Load, std::vector<Load>, std::greater<Load>> least;
    for (int b = 0; b < n; ++b) least.push({0, b});
    for (int i : ids) {
      const Load l = least.top();
      least.pop();
      to[l.second].push_back(i);
      least.push({l.first + load[i], l.second});
    }
    return to;
  };
  auto by_load = [](const std::vector<int64_t>& load) {
    std::vector<int> order(load.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return load[a] > load[b]; });
    return order;
  };
  std::vector<int64_t> group;
  for (size_t i = 0; i < items.size(); ++i) {
    const size_t g = items[i].m / 8;
    if (g >= group.size()) group.resize(g + 1, 0);
    group[g] += cost[i];
  }
  std::vector<int> xcd(group.size(), 0);
  if (nx > 1) {
    const auto to = deal(by_load(group), group, nx);
    for (int x = 0; x < nx; ++x)
      for (int g : to[x]) xcd[g] = x;
  }
  std::vector<std::vector<int>> ids(nx);
  for (int i : by_load(cost)) ids[xcd[items[i].m / 8]].push_back(i);
  std::vector<std::vector<std::vector<int>>> to(nx);
  for (int x = 0; x < nx; ++x) to[x] = deal(ids[x], cost, nwg / nx);
  std::vector<Item64> packed;
  off->assign(1, 0);
  for (int b = 0; b < nwg; ++b) {
    for (int i : to[b % nx][b / nx]) packed.push_back(items[i]);
    off->push_back((int32_t)packed.size());
  }
  return packed;
}

// Work lists of the FP64 Legendre kernels (Leg64Dev), made for the first FP64 plan of the shape.
int build_leg64(Geometry& g, const Reach& reach) {
  const int lmax = g.lmax, nbm = g.nblk_max_ana;
  // (m, block of rb pairs) with the first l - m, in chunks of 16, at which a ring pair of it exceeds
  // 2^-128, and the l - m up to which a ring of it is still scaled
  const std::vector<uint16_t>&wake = reach.wake, &rise = reach.rise;
  struct Block {
    int m, blk, first, scaled;
  };
  auto blocks = [&](int rb) {
    std::vector<Block> out;
    for (int m = 0; m <= lmax; ++m)
      for (int b = 0; b * rb < g.n_active[m]; ++b) {
        const int nl = lmax - m + 1, q1 = std::min(g.n_active[m], (b + 1) * rb);
        int first = nl, scaled = 0;
        for (int q = b * rb; q < q1; ++q) {
          const size_t at = (size_t)m * g.npairs + q;
          if (rise[at] != WAKE_NEVER) first = std::min(first, (int)rise[at] / CHUNK * CHUNK);
          if (wake[at] != WAKE_NEVER) scaled = std::max(scaled, std::min((int)wake[at], nl));
        }
        out.push_back({m, b, first, scaled});
      }
    return out;
  };
  auto item_cost = [&](const Item64& w, int scaled, int scaled_cost) {
    const int64_t n = w.i1 - w.i0, sc = std::min<int64_t>(n, std::max(0, scaled - w.i0));
    return 4 * (n - sc) + scaled_cost * sc + 4 * FP64_ITEM_COST_L;
  };
  const auto whole = blocks(g.ring_block_ana);
  std::vector<int32_t> start((size_t)(lmax + 1) * nbm);
  for (int m = 0; m <= lmax; ++m)
    for (int b = 0; b < nbm; ++b) start[(size_t)m * nbm + b] = lmax - m + 1;
  int64_t total = 0;
  for (const Block& b : whole) {
    start[(size_t)b.m * nbm + b.blk] = b.first;
    total += lmax - b.m + 1 - b.first;
  }
  std::vector<Item64> items;
  std::vector<int64_t> cost;
  // analysis items: the l of a block in parts of about `part` (in chunks of 16)
  auto split = [&](int64_t part) {
    items.clear();
    cost.clear();
    for (const Block& b : whole) {
      const int nl = lmax - b.m + 1, n = nl - b.first;
      if (n == 0) continue;
      const int parts = std::max(1, (int)((n + part / 2) / part));
      const int len = ((n + parts - 1) / parts + CHUNK - 1) / CHUNK * CHUNK;
      for (int i = b.first; i < nl; i += len) {
        const Item64 w{b.m, b.blk, i, std::min(nl, i + len)};
        items.push_back(w);
        cost.push_back(item_cost(w, b.scaled, FP64_SCALED_COST_ANA));
      }
    }
  };
  std::vector<int32_t> wg_ana, wg_batch, wg_syn;
  int nwg = 1, waves_ana = 1, waves_syn = 1;
  // few maps: parts of about half a wave's share of one map, 32 at least
  const int64_t part = std::max<int64_t>(32, (total / (2 * FP64_ANA_WAVES * g.n_cu) + CHUNK - 1) / CHUNK * CHUNK);
  split(part);
  one_map_shape(items.size(), g.n_cu, FP64_ANA_WAVES, &nwg, &waves_ana);
  const auto ia = pack_items(items, cost, nwg, &wg_ana);
  // Where these are short, the set-up of an item (ring states and S/D, 256 rows of G apart) is half of
  // its time, which pays only while waves would idle otherwise: batches take longer ones, in small
  // workgroups of two items a wave. Analysis of 3, 8, 16 and 48 maps (us) with the items of one
  // map and with these: Nside 256, lmax 300 41, 94, 179, 490 and 32, 58, 101, 274; Nside 256, lmax
  // 512 64, 158, 325, 971 and 63, 131, 258, 742; Nside 128, lmax 256 18, 33, 56, 152 and 22, 31, 51, 120; Nside
  // 64, lmax 128 8, 11, 16, 33 and 11, 13, 17, 31. From that the rule: two maps, and 80 l a
  // wave of a full launch. One map of more than FP64_BATCH_PART l per item has items as long already.
  std::vector<Item64> ib;
  int batch_from = INT_MAX;
  if (part < FP64_BATCH_PART) {
    split(FP64_BATCH_PART);
    const int per_wg = 2 * FP64_BATCH_WAVES;
    nwg = std::max(1, (int)((items.size() + per_wg - 1) / per_wg));
    if (nwg > 8) nwg = (nwg + 7) / 8 * 8;
    ib = pack_items(items, cost, nwg, &wg_batch);
    const int64_t from = ((int64_t)80 * FP64_ANA_WAVES * g.n_cu + total - 1) / std::max<int64_t>(total, 1);
    batch_from = (int)std::min<int64_t>(std::max<int64_t>(from, 2), INT_MAX);
  }
  // synthesis: the largest blocks, up to 256 pairs, that still give every wave of a full launch an
  // item and a half (a wave's share is then not set by its longest item). A smaller block that
  // never rises inside one of the analysis's that does gets an item of no steps, which writes
  // zeros: the entries of F that a plan writes then grow with its band limit, and the others,
  // zero from the start, stay so when the coefficients of a truncated sweep are carried over.
  int rb_syn = g.ring_block_ana;
  for (;; rb_syn /= 2) {
    const auto bl = blocks(rb_syn);
    items.clear();
    cost.clear();
    for (const Block& b : bl) {
      const int nl = lmax - b.m + 1;
      if (start[(size_t)b.m * nbm + b.blk * rb_syn / g.ring_block_ana] >= nl) continue;
      const Item64 w{b.m, b.blk, b.first, nl};
      items.push_back(w);
      cost.push_back(item_cost(w, b.scaled, FP64_SCALED_COST_SYN));
    }
    if (rb_syn == LANES || (int64_t)items.size() * 2 >= (int64_t)FP64_SYN_WAVES * g.n_cu * 3) break;
  }
  one_map_shape(items.size(), g.n_cu, FP64_SYN_WAVES, &nwg, &waves_syn);
  const auto is = pack_items(items, cost, nwg, &wg_syn);
  std::vector<double> z(g.npairs);
  for (int q = 0; q < g.npairs; ++q) z[q] = ring_geometry(g.nside, 2 * g.nside - q).z;

  // handed to the geometry when all is made: plans of other types keep it after a failure here
  DevMem M;
  double* dz = nullptr;
  int32_t* dstart = nullptr;
  int rc;
  if ((rc = M.upload(&dz, z)) || (rc = M.upload(&dstart, start))) return rc;
  Leg64Dev L{};
  L.z = dz;
  L.start = dstart;
  PlanDev D{};
  D.nside = g.nside;
  D.lmax = lmax;
  D.npairs = g.npairs;
  D.pairs = g.pairs;
  D.A = g.A;
  D.row_off = g.row_off;
  D.norm_m = g.norm;
  D.n_active = g.nact;
  auto make_list = [&](Leg64List& T, const std::vector<Item64>& it, const std::vector<int32_t>& wg, int waves,
                       int rb) -> int {
    Item64* di = nullptr;
    int32_t* db = nullptr;
    double2* ds = nullptr;
    uint8_t* dc = nullptr;
    int rc;
    if ((rc = M.upload(&di, it)) || (rc = M.upload(&db, wg)) || (rc = M.alloc(&ds, it.size() * rb)) ||
        (rc = M.alloc(&dc, it.size() * rb)))
      return rc;
    T.items = di;
    T.wg = db;
    T.nwg = (int)wg.size() - 1;
    T.waves = waves;
    T.rb = rb;
    MWF_HIP(launch_start_state(D, T, (int)it.size(), CHUNK, ds, dc, nullptr));
    T.state = ds;
    T.scale = dc;
    return WF_OK;
  };
  if ((rc = make_list(L.ana, ia, wg_ana, waves_ana, g.ring_block_ana)) ||
      (rc = make_list(L.syn, is, wg_syn, waves_syn, rb_syn)))
    return rc;
  L.batch_from = batch_from;
  if (!ib.empty() && (rc = make_list(L.ana_batch, ib, wg_batch, FP64_BATCH_WAVES, g.ring_block_ana))) return rc;
  MWF_HIP(hipStreamSynchronize(nullptr));
  g.mem.ptrs.insert(g.mem.ptrs.end(), M.ptrs.begin(), M.ptrs.end());
  M.ptrs.clear();
  g.leg64 = L;
  g.leg64_ready = true;
  return WF_OK;
}

}  // namespace

RingGeo ring_geometry(int n, int i) {
  RingGeo g{};
  const int64_t npix = 12LL * n * n;
  if (i < n) {
    g.z = 1.0 - (double)((int64_t)i * i) / (3.0 * n * n);
    g.nphi = 4 * i;
    g.ph_num = 1;
    g.ph_den = 4 * i;
    g.start = 2LL * i * (i - 1);
  } else if (i <= 3 * n) {
    g.z = 2.0 * (2 * n - i) / (3.0 * n);
    g.nphi = 4 * n;
    g.ph_num = (i - n + 1) % 2;
    g.ph_den = 4 * n;
    g.start = 2LL * n * (n - 1) + 4LL * n * (i - n);
  } else {
    const int ip = 4 * n - i;
    g.z = -(1.0 - (double)((int64_t)ip * ip) / (3.0 * n * n));
    g.nphi = 4 * ip;
    g.ph_num = 1;
    g.ph_den = 4 * ip;
    g.start = npix - 2LL * ip * (ip + 1);
  }
  return g;
}

int get_geometry(int nside, int lmax, bool fp64, std::shared_ptr<Geometry>* out) {
  int dev = 0;
  MWF_HIP(hipGetDevice(&dev));
  const auto key = std::make_tuple(dev, nside, lmax);
  std::lock_guard<std::mutex> lock(g_geo_mu);
  auto it = g_geo.find(key);
  if (it != g_geo.end()) {
    if (auto live = it->second.lock()) {
      if (fp64 && !live->leg64_ready) {
        Reach reach;
        if (int rc = run_reach(*live, true, &reach)) return rc;
        if (int rc = build_leg64(*live, reach)) return rc;
      }
      *out = live;
      return WF_OK;
    }
  }
  auto g = std::make_shared<Geometry>();
  g->device = dev;
  MWF_HIP(hipDeviceGetAttribute(&g->n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  if (g->n_cu <= 0) g->n_cu = 1;
  g->nside = nside;
  g->lmax = lmax;
  Reach reach;
  int rc = build_geometry(*g, fp64, &reach);
  if (!rc && fp64) rc = build_leg64(*g, reach);
  if (rc) return rc;
  g_geo[key] = g;
  *out = g;
  return WF_OK;
}

}  // namespace mwf
