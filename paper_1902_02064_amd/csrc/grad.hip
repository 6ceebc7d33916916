// Gradient of sum_k w_k E_k with respect to the J-coupled two-body matrix elements
// and the single-particle energies. H is linear in its parameters, so by
// Hellmann-Feynman dE_k/dtheta = <psi_k| dH/dtheta |psi_k>; with
// H2 = sum_terms h_term O_term and h_term = sum_t c(term, t) V_t,
//   d(sum_k w_k E_k)/dV_t = sum_terms c(term, t) rho_term,
//   rho_term = sum_k w_k <psi_k| O_term |psi_k>   (two-body densities).
// The densities are regrouped by spectator cores like the products (App. B): a pn term leaves a core of
// n_prot - 1 protons and n_neut - 1 neutrons in place, a pp (nn) term n - 2 protons (neutrons) and the whole
// other species. With the pair states of one pair 2M listed once, the densities of a pair block are
//   rho[i][j] = sum over cores and vectors of w_k x_i x_j,   x_i = sign_i X[core + pair i][k],
// a product of a tall matrix with its own transpose: it runs on the matrix cores (both operands of
// v_mfma_f64_16x16x4f64 are the same registers), 16 x 16 or 32 x 32 pairs at a time with the sums in registers,
// and a work item adds its sums to the block once. The contraction with the coefficients c(term, t) of
// the J -> m conversion is done on the host.
// 20 vectors of sd 6+6 (D = 93,710): 0.66 ms a call, of which the pn densities 0.29 and the identical
// particles 0.31 ms; walking the stored operators and jump pairs with one atomic per element took 6.96 ms
// (5.4 and 1.4). The items are short (about 24 cores a group there), so what is left is mostly the chain
// of table lookups that starts each of them.
#include <algorithm>
#include <map>

#include "dense.h"
#include "tilecore.h"

namespace trbl {

namespace {

constexpr int GRAD_MAXPAIR = 1024;  // pairs of one block: at most 64 states x 16 orbits of one m

// One work item: a core and a run of the states it is combined with (pn: neutron cores of one group,
// identical particles: states of the other species in one block; core is the index of the core's list).
struct GradItem {
  int rect, core, first, count;
};
// What a run of items shares. pn: pair block and first entry of the target blocks of its pairs;
// identical particles: pair block and product block.
struct GradRect {
  int k, list, blk, pad;
};
// Identical particles: a pair outside a core (its index in the pair block) and the state that they form
// (index in its sector << 1 | sign).
struct GradPair {
  int id, state;
};

struct GradArgs {
  const double* X;  // [D][n] eigenvectors
  int n, lq, ns;    // lq: lanes (of two columns each) of a row
  const double* w;  // [n] weights (device)
  const GradItem* items;
  const GradRect* rect;
  const int* pr_off;  // pair blocks: pairs and densities
  const int* rho_off;
  double* rho;
  const int64_t* blk_off;
  const int* blk_dn;
  // pn
  const int* pr_xu;  // x | u << 8
  const int* rblk;   // target block of each pair (-1: none)
  const int* rkp;    // [core * ns + state]: position of state << 24 | local index of core + state, -1 inside
  const int* rkn;
  // identical particles: the pairs outside a core that reach one sector are list_pair[list_off[core] ..
  // list_off[core + 1])
  const int* list_off;
  const GradPair* list_pair;
  int species;
};

typedef double v2d __attribute__((ext_vector_type(2)));

// The sums of the 16 NT x 16 NT pairs from (i0, j0) on over a run of states, in `acc`. Vectors are taken
// ST * 2 lq columns at a time (with one tile all of them up to 24), so that a lane's weights stay in
// registers; a wavefront works on UO steps of the run at once: their loads are issued together.
template <bool PN, int NT>
__device__ __forceinline__ void dens_sums(const GradArgs& a, const GradItem& it, int64_t stride, int d, int i0, int j0,
                                          const int64_t* row, const int* us, const int* sg,
                                          tiles::Mfma<double>::acc (&acc)[NT][NT]) {
  using namespace tiles;
  constexpr int ST = NT == 1 ? 3 : 1, UO = 2, NR = 2 * NT;  // row tiles: NT of i, NT of j
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, c = l & 15, kq = l >> 4;
  const bool diag = i0 == j0;
  const int per = 4 / a.lq;                                // states of the run per step
  const int o_lane = kq / a.lq, c_lane = 2 * (kq % a.lq);  // this lane's state and first column
  int64_t r0[NR];
  int un[NR], sn[NR];
  bool in[NR];
#pragma unroll
  for (int t = 0; t < NR; t++) {
    const int i = (t < NT ? i0 + 16 * t : j0 + 16 * (t - NT)) + c;
    in[t] = i < d;
    r0[t] = row[min(i, d - 1)];
    un[t] = us[min(i, d - 1)];
    sn[t] = sg[min(i, d - 1)];
  }
  for (int s0 = 0; s0 < a.n; s0 += 2 * a.lq * ST) {
    double wt[ST][2];
#pragma unroll
    for (int s = 0; s < ST; s++)
#pragma unroll
      for (int t = 0; t < 2; t++) {
        const int k = s0 + c_lane + 2 * a.lq * s + t;
        wt[s][t] = k < a.n ? a.w[k] : 0.0;
      }
    for (int o0 = w * per * UO; o0 < it.count; o0 += 4 * per * UO) {
      v2d v[UO][NR][ST];
#pragma unroll
      for (int u = 0; u < UO; u++) {
        const int o = o0 + u * per + o_lane;
#pragma unroll
        for (int t = 0; t < NR; t++) {
          if (t >= NT && diag) continue;
          bool on = in[t] && o < it.count;
          unsigned flip = (unsigned)sn[t];
          const double* x = a.X;
          if constexpr (PN) {
            const int rn = on ? a.rkn[(it.first + o) * a.ns + un[t]] : -1;
            on = rn >= 0;
            if (on) x += (r0[t] + (rn & 0xFFFFFF)) * a.n;
            flip += (unsigned)(rn >> 24);
          } else {
            if (on) x += (r0[t] + (it.first + o) * stride) * a.n;
          }
#pragma unroll
          for (int s = 0; s < ST; s++) {
            const int k = s0 + c_lane + 2 * a.lq * s;
            v2d y = v2d(0.0);
            if (on && k + 1 < a.n) __builtin_memcpy(&y, x + k, 16);
            else if (on && k < a.n) y[0] = x[k];
            y[0] = flip_if((double)y[0], flip);
            y[1] = flip_if((double)y[1], flip);
            v[u][t][s] = y;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < UO; u++)
#pragma unroll
        for (int s = 0; s < ST; s++) {
          if (s0 + 2 * a.lq * s >= a.n) continue;  // uniform
#pragma unroll
          for (int p = 0; p < NT; p++)
#pragma unroll
            for (int q = 0; q < NT; q++) {
              if (diag && q < p) continue;
              const v2d y = diag ? v[u][q][s] : v[u][NT + q][s];
              acc[p][q] = Mfma<double>::run(v[u][p][s][0], wt[s][0] * y[0], acc[p][q]);
              acc[p][q] = Mfma<double>::run(v[u][p][s][1], wt[s][1] * y[1], acc[p][q]);
            }
        }
    }
  }
}

// the sums of the four wavefronts added to the block of densities
template <int NT>
__device__ __forceinline__ void dens_add(const GradArgs& a, const GradRect& rc, int D2, int d, int i0, int j0,
                                         const int* id, double* red, const tiles::Mfma<double>::acc (&acc)[NT][NT]) {
  using namespace tiles;
  constexpr int R = 16 * NT;
  const int l = threadIdx.x & 63, c = l & 15, kq = l >> 4;
  for (int e = threadIdx.x; e < R * R; e += 256) red[e] = 0.0;
  __syncthreads();
#pragma unroll
  for (int p = 0; p < NT; p++)
#pragma unroll
    for (int q = 0; q < NT; q++)
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const int i = 16 * p + Mfma<double>::row(kq, v), j = 16 * q + c;
        if (i0 + i <= j0 + j && j0 + j < d) atomicAdd(&red[i * R + j], (double)acc[p][q][v]);
      }
  __syncthreads();
  double* rho = a.rho + a.rho_off[rc.k];
  for (int e = threadIdx.x; e < R * R; e += 256) {
    const int i = i0 + e / R, j = j0 + e % R;
    if (i <= j && j < d) atomicAdd(rho + (int64_t)min(id[i], id[j]) * D2 + max(id[i], id[j]), red[e]);
  }
  __syncthreads();
}

template <bool PN>
__global__ __launch_bounds__(256, 4) void dens_kernel(GradArgs a, int maxpair) {
  using namespace tiles;
  extern __shared__ __align__(16) char lds_[];
  int64_t* row = reinterpret_cast<int64_t*>(lds_);  // first row of pair i (pn: of its proton row; else of state 0)
  int* id = reinterpret_cast<int*>(row + maxpair);  // pair, neutron state, sign (pn: position of the proton state)
  int* us = id + maxpair;
  int* sg = us + maxpair;
  double* red = reinterpret_cast<double*>(sg + maxpair);  // 32 x 32
  __shared__ int nd;
  const GradItem it = a.items[blockIdx.x];
  const GradRect rc = a.rect[it.rect];
  const int q0 = a.pr_off[rc.k], D2 = a.pr_off[rc.k + 1] - q0;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  int64_t stride = 1;  // rows between consecutive states of the run
  if (!PN && a.species == 1) stride = a.blk_dn[rc.blk];
  if constexpr (!PN) {  // the pairs outside the core are listed
    const int e0 = a.list_off[it.core], d = a.list_off[it.core + 1] - e0;
    const int64_t off = a.blk_off[rc.blk], rs = a.species == 0 ? a.blk_dn[rc.blk] : 1;
    for (int i = threadIdx.x; i < d; i += 256) {
      const GradPair p = a.list_pair[e0 + i];
      row[i] = off + (p.state >> 1) * rs;
      id[i] = p.id;
      us[i] = 0;
      sg[i] = p.state & 1;
    }
    if (threadIdx.x == 0) nd = d;
  } else if (w == 0) {  // the pairs outside the core, in order
    int d = 0;
    for (int e0 = 0; e0 < D2; e0 += 64) {
      const int e = min(e0 + l, D2 - 1);
      bool ok = e0 + l < D2;
      int64_t r0 = 0;
      const int xu = a.pr_xu[q0 + e], b = a.rblk[rc.list + e], rp = a.rkp[it.core * a.ns + (xu & 255)];
      ok = ok && b >= 0 && rp >= 0;
      if (ok) r0 = a.blk_off[b] + (int64_t)(rp & 0xFFFFFF) * a.blk_dn[b];
      const uint64_t mask = __ballot(ok);
      if (ok) {
        const int i = d + __popcll(mask & ((1ull << l) - 1));
        row[i] = r0;
        id[i] = e0 + l;
        us[i] = xu >> 8;
        sg[i] = rp >> 24;
      }
      d += __popcll(mask);
    }
    if (l == 0) nd = d;
  }
  __syncthreads();
  const int d = nd;
  if (d == 0) return;
  if (d <= 16) {
    Mfma<double>::acc acc[1][1] = {};
    dens_sums<PN, 1>(a, it, stride, d, 0, 0, row, us, sg, acc);
    dens_add<1>(a, rc, D2, d, 0, 0, id, red, acc);
    return;
  }
  for (int i0 = 0; i0 < d; i0 += 32)
    for (int j0 = i0; j0 < d; j0 += 32) {
      Mfma<double>::acc acc[2][2] = {};
      dens_sums<PN, 2>(a, it, stride, d, i0, j0, row, us, sg, acc);
      dens_add<2>(a, rc, D2, d, i0, j0, id, red, acc);
    }
}

struct OccArgs {
  const double* X;
  int n, nblocks, norb;
  const double* w;
  const int* blk_dn;
  const int64_t* blk_off;
  const int* blk_p0;
  const int* blk_n0;
  const uint64_t* pwords;
  const uint64_t* nwords;
  uint64_t orbmask[16];
  double* occ;  // [2][norb]
};

// occupation densities of every orbit, per species: sum_i (sum_k w_k X[i,k]^2) * N_a(i); a workgroup sums
// its rows in LDS and adds them to the result once
__global__ __launch_bounds__(256) void dens_occ_kernel(OccArgs a, int64_t D) {
  __shared__ double sum[32];
  if (threadIdx.x < 32) sum[threadIdx.x] = 0.0;
  __syncthreads();
  double mine[2][16] = {};
  for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < D; i += (int64_t)gridDim.x * 256) {
    int lo = 0, hi = a.nblocks - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.blk_off[mid] <= i) lo = mid;
      else hi = mid - 1;
    }
    const int64_t rel = i - a.blk_off[lo];
    const int dn = a.blk_dn[lo];
    const uint64_t pw = a.pwords[a.blk_p0[lo] + rel / dn], nw = a.nwords[a.blk_n0[lo] + rel % dn];
    const double* x = a.X + i * a.n;
    double u = 0.0;
    for (int c = 0; c < a.n; c++) u += a.w[c] * x[c] * x[c];
#pragma unroll
    for (int o = 0; o < 16; o++)
      if (o < a.norb) {
        mine[0][o] += u * __popcll(pw & a.orbmask[o]);
        mine[1][o] += u * __popcll(nw & a.orbmask[o]);
      }
  }
#pragma unroll
  for (int s = 0; s < 2; s++)
#pragma unroll
    for (int o = 0; o < 16; o++)
      if (o < a.norb) {
        double v = mine[s][o];
        for (int h = 32; h; h >>= 1) v += __shfl_down(v, h);
        if ((threadIdx.x & 63) == 0) atomicAdd(&sum[16 * s + o], v);
      }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < 32 && (t & 15) < a.norb) atomicAdd(a.occ + (t >> 4) * a.norb + (t & 15), sum[t]);
}

// Pair blocks of one channel (0 pp, 1 nn, 2 pn): they depend on the space alone.
struct Channel {
  std::vector<int> pid, pblk;             // [a * ns + b]: index in its block, block (-1: none)
  std::vector<int> pr_off, rho_off;
  std::vector<int> pr_xu;
  size_t nitems = 0;
};

// Cores and work items of one channel while they are built for the device.
struct ChannelWork {
  std::vector<int> rblk, rk[2];           // pn
  std::vector<int> list_off;              // identical particles
  std::vector<GradPair> list_pair;
  std::vector<GradRect> rect;
  std::vector<GradItem> items;
};

// all n-subsets of ns states (colex)
template <class F>
void subsets(int ns, int n, F&& f) {
  if (n == 0) {
    f((uint64_t)0);
    return;
  }
  uint64_t w = n == 64 ? ~0ull : (1ull << n) - 1;
  while (true) {
    f(w);
    const uint64_t lo = w & (~w + 1), hi = w + lo;
    if (hi == 0) break;
    const uint64_t nw = (((hi ^ w) >> 2) / lo) | hi;
    if ((ns < 64 && nw >= (1ull << ns)) || nw <= w) break;
    w = nw;
  }
}

struct CoreGroup {
  int tm, par, start, count;
};

// cores of `n` particles grouped by (2M, parity)
std::vector<CoreGroup> core_groups(const Model& m, int n, std::vector<uint64_t>& words) {
  std::map<std::pair<int, int>, std::vector<uint64_t>> by;
  subsets(m.ns, n, [&](uint64_t w) {
    int tm = 0, par = 0;
    for (uint64_t x = w; x; x &= x - 1) {
      const int s = __builtin_ctzll(x);
      tm += m.st_tm[s];
      par ^= m.orbits[m.st_orb[s]].l & 1;
    }
    by[{tm, par}].push_back(w);
  });
  std::vector<CoreGroup> g;
  words.clear();
  for (auto& kv : by) {
    g.push_back({kv.first.first, kv.first.second, (int)words.size(), (int)kv.second.size()});
    words.insert(words.end(), kv.second.begin(), kv.second.end());
  }
  return g;
}

void pair_blocks(const Model& m, bool identical, Channel& ch, std::map<std::pair<int, int>, int>& kid) {
  const int ns = m.ns;
  ch.pid.assign(ns * ns, -1);
  ch.pblk.assign(ns * ns, -1);
  std::vector<std::vector<int>> pairs;
  for (int a = 0; a < ns; a++)
    for (int b = identical ? a + 1 : 0; b < ns; b++) {
      const int odd = (m.orbits[m.st_orb[a]].l + m.orbits[m.st_orb[b]].l) & 1;
      const auto at = kid.emplace(std::make_pair(m.st_tm[a] + m.st_tm[b], odd), (int)pairs.size());
      if (at.second) pairs.emplace_back();
      ch.pblk[a * ns + b] = at.first->second;
      ch.pid[a * ns + b] = (int)pairs[at.first->second].size();
      pairs[at.first->second].push_back(a | (b << 8));
    }
  ch.pr_off.assign(1, 0);
  ch.rho_off.assign(1, 0);
  for (auto& v : pairs) {
    TRBL_REQUIRE((int)v.size() <= GRAD_MAXPAIR, TRBL_E_INVALID, "pair block too wide for the gradient");
    ch.pr_off.push_back(ch.pr_off.back() + (int)v.size());
    ch.rho_off.push_back(ch.rho_off.back() + (int)(v.size() * v.size()));
    ch.pr_xu.insert(ch.pr_xu.end(), v.begin(), v.end());
  }
}

int below_odd(uint64_t w, int s) { return __builtin_popcountll(w & ((1ull << s) - 1)) & 1; }

std::vector<int> sector_map(const Model& m, std::map<std::pair<int, int>, int> (&secid)[2]) {
  for (int s = 0; s < 2; s++)
    for (int q = 0; q < (int)m.sp[s].sectors.size(); q++)
      secid[s][{m.sp[s].sectors[q].twoM, m.sp[s].sectors[q].par < 0 ? 1 : 0}] = q;
  const int nn = (int)m.sp[1].sectors.size();
  std::vector<int> bos(m.sp[0].sectors.size() * nn, -1);
  for (size_t b = 0; b < m.blocks.size(); b++) bos[m.blocks[b].psec * nn + m.blocks[b].nsec] = (int)b;
  return bos;
}

void pn_channel(const Model& m, Channel& ch, ChannelWork& cw) {
  if (m.n_prot == 0 || m.n_neut == 0) return;
  const int ns = m.ns;
  std::map<std::pair<int, int>, int> kid, secid[2];
  pair_blocks(m, false, ch, kid);
  const std::vector<int> bos = sector_map(m, secid);
  const int nnsec = (int)m.sp[1].sectors.size();
  std::vector<CoreGroup> groups[2];
  for (int s = 0; s < 2; s++) {
    std::vector<uint64_t> words;
    groups[s] = core_groups(m, m.sp[s].npart - 1, words);
    cw.rk[s].assign(words.size() * ns, -1);
    for (size_t q = 0; q < words.size(); q++)
      for (int st = 0; st < ns; st++) {
        if ((words[q] >> st) & 1) continue;
        const auto at = m.sp[s].index.find(words[q] | (1ull << st));
        if (at == m.sp[s].index.end()) continue;  // its sector is in no block
        const int loc = at->second - m.sp[s].sectors[m.sp[s].sector_of[at->second]].start;
        TRBL_REQUIRE(loc < (1 << 24), TRBL_E_INVALID, "sector too large for the gradient tables");
        cw.rk[s][q * ns + st] = __builtin_popcountll(words[q] & ((1ull << st) - 1)) << 24 | loc;
      }
  }
  // rectangles of core groups whose pair block reaches some block of the space
  struct Rect {
    const CoreGroup *p, *n;
  };
  std::vector<Rect> of;
  for (const CoreGroup& gp : groups[0])
    for (const CoreGroup& gn : groups[1])
      for (int odd = 0; odd < 2; odd++) {
        const auto k = kid.find({m.twoM - gp.tm - gn.tm, odd});
        if (k == kid.end()) continue;
        bool any = false;
        const int list = (int)cw.rblk.size();
        for (int e = ch.pr_off[k->second]; e < ch.pr_off[k->second + 1]; e++) {
          const int x = ch.pr_xu[e] & 255, u = ch.pr_xu[e] >> 8;
          const auto ip = secid[0].find({gp.tm + m.st_tm[x], gp.par ^ (m.orbits[m.st_orb[x]].l & 1)});
          const auto in = secid[1].find({gn.tm + m.st_tm[u], gn.par ^ (m.orbits[m.st_orb[u]].l & 1)});
          const int b = ip != secid[0].end() && in != secid[1].end() ? bos[ip->second * nnsec + in->second] : -1;
          cw.rblk.push_back(b);
          any = any || b >= 0;
        }
        if (!any) {
          cw.rblk.resize(list);
          continue;
        }
        cw.rect.push_back({k->second, list, 0, 0});
        of.push_back({&gp, &gn});
      }
  // up to 256 neutron cores an item, more where that would take more than 2^24 items
  int chunk = 256;
  auto total = [&] {
    size_t t = 0;
    for (const Rect& r : of) t += (size_t)r.p->count * ((r.n->count + chunk - 1) / chunk);
    return t;
  };
  while (chunk < (1 << 20) && total() > (size_t)1 << 24) chunk *= 2;
  cw.items.reserve(total());
  for (size_t r = 0; r < of.size(); r++)
    for (int cp = of[r].p->start; cp < of[r].p->start + of[r].p->count; cp++)
      for (int n0 = 0; n0 < of[r].n->count; n0 += chunk)
        cw.items.push_back({(int)r, cp, of[r].n->start + n0, std::min(chunk, of[r].n->count - n0)});
}

// Words numbered in the order of their first appearance.
class WordIndex {
 public:
  int at(uint64_t w) {
    if (2 * (words.size() + 1) > slot_.size()) grow();
    size_t h = home(w);
    while (slot_[h] >= 0 && words[slot_[h]] != w) h = (h + 1) & (slot_.size() - 1);
    if (slot_[h] < 0) {
      slot_[h] = (int)words.size();
      words.push_back(w);
    }
    return slot_[h];
  }
  std::vector<uint64_t> words;

 private:
  size_t home(uint64_t w) const { return (size_t)((w * 0x9E3779B97F4A7C15ull) >> 20) & (slot_.size() - 1); }
  void grow() {
    slot_.assign(std::max<size_t>(256, 2 * slot_.size()), -1);
    for (size_t i = 0; i < words.size(); i++) {
      size_t h = home(words[i]);
      while (slot_[h] >= 0) h = (h + 1) & (slot_.size() - 1);
      slot_[h] = (int)i;
    }
  }
  std::vector<int> slot_;
};

// The lists come from the states that the space stores: every pair of a state's nucleons belongs to the core of
// the others, so that the tables hold C(n, 2) entries a state, whatever the number of subsets of the m-states
// (28 protons in 32 states: 0.6 million entries, against 906,192 cores x 496 pairs).
void identical_channel(const Model& m, int s, Channel& ch, ChannelWork& cw) {
  const Species& S = m.sp[s];
  if (S.npart < 2) return;
  const int ns = m.ns;
  std::map<std::pair<int, int>, int> kid;
  pair_blocks(m, true, ch, kid);
  // product blocks of every sector; sectors in none of them are left out
  std::vector<std::vector<int>> blocks(S.sectors.size());
  for (size_t b = 0; b < m.blocks.size(); b++)
    if ((s == 0 ? m.blocks[b].dn : m.blocks[b].dp) > 0)
      blocks[s == 0 ? m.blocks[b].psec : m.blocks[b].nsec].push_back((int)b);
  cw.list_off.assign(1, 0);
  for (size_t q = 0; q < S.sectors.size(); q++) {
    if (blocks[q].empty()) continue;
    const SpeciesSector& sec = S.sectors[q];
    // entries of the sector, then by core in the order of the states. A core fixes the (2M, parity) of the
    // pair that completes it to the sector, so its list belongs to one pair block.
    struct Entry {
      int core;
      GradPair p;
    };
    WordIndex cores;
    std::vector<int> kblk, count;
    std::vector<Entry> entry;
    entry.reserve((size_t)sec.size * S.npart * (S.npart - 1) / 2);
    for (int g = 0; g < sec.size; g++) {
      const uint64_t w = S.words[sec.start + g];
      for (uint64_t x = w; x; x &= x - 1) {
        const int a = __builtin_ctzll(x);
        for (uint64_t y = x & (x - 1); y; y &= y - 1) {
          const int b = __builtin_ctzll(y);
          const uint64_t core = w ^ (1ull << a) ^ (1ull << b);
          const int c = cores.at(core);
          if (c == (int)kblk.size()) {
            kblk.push_back(ch.pblk[a * ns + b]);
            count.push_back(0);
          }
          count[c]++;
          entry.push_back({c, {ch.pid[a * ns + b], g << 1 | (below_odd(core, a) ^ below_odd(core, b))}});
        }
      }
    }
    const size_t base = cw.list_pair.size(), l0 = cw.list_off.size() - 1;
    TRBL_REQUIRE(base + entry.size() < ((size_t)1 << 31), TRBL_E_NOMEM, "too many states for the gradient tables");
    for (int c : count) cw.list_off.push_back(cw.list_off.back() + c);
    cw.list_pair.resize(base + entry.size());
    std::vector<int> next(cw.list_off.begin() + l0, cw.list_off.end() - 1);
    for (const Entry& e : entry) cw.list_pair[next[e.core]++] = e.p;
    for (int b : blocks[q]) {
      const int other = s == 0 ? m.blocks[b].dn : m.blocks[b].dp;
      std::map<int, int> rect_of;  // pair block -> rectangle
      for (size_t c = 0; c < kblk.size(); c++) {
        const auto r = rect_of.emplace(kblk[c], (int)cw.rect.size());
        if (r.second) cw.rect.push_back({kblk[c], 0, b, 0});
        for (int o = 0; o < other; o += 1024)
          cw.items.push_back({r.first->second, (int)(l0 + c), o, std::min(1024, other - o)});
      }
    }
  }
}

}  // namespace

struct GradTables {
  Channel ch[3];
  DevBuf pr_off[3], rho_off[3], pr_xu, rblk, rk[2], list_off[2], list_pair[2], rect[3], items[3];
  DevBuf work;  // weights, then the densities of the three channels and the occupations
};

void GradTablesDelete::operator()(GradTables* t) const { delete t; }

// the pair, core and work tables of the space, built by the first gradient and kept with the model
static GradTables& tables_for(const Model& m) {
  if (m.grad_tables) return *m.grad_tables;
  std::unique_ptr<GradTables, GradTablesDelete> t(new GradTables());
  for (int k = 0; k < 3; k++) {
    ChannelWork cw;
    if (k == 2) pn_channel(m, t->ch[k], cw);
    else identical_channel(m, k, t->ch[k], cw);
    t->ch[k].nitems = cw.items.size();
    t->pr_off[k].upload(t->ch[k].pr_off);
    t->rho_off[k].upload(t->ch[k].rho_off);
    t->rect[k].upload(cw.rect);
    t->items[k].upload(cw.items);
    if (k == 2) {
      t->pr_xu.upload(t->ch[k].pr_xu);
      t->rblk.upload(cw.rblk);
      for (int s = 0; s < 2; s++) t->rk[s].upload(cw.rk[s]);
    } else {
      t->list_off[k].upload(cw.list_off);
      t->list_pair[k].upload(cw.list_pair);
    }
  }
  m.grad_tables = std::move(t);
  return *m.grad_tables;
}

void tbme_gradient(const Model& m, int n_eig, const double* w, const double* X, double* grad_v, double* grad_spe,
                   hipStream_t s) {
  TRBL_REQUIRE(m.has_h, TRBL_E_STATE, "no Hamiltonian set");
  TRBL_REQUIRE(!m.fly, TRBL_E_INVALID, "no gradient for wide single-species spaces (generated per element)");
  TRBL_REQUIRE((int)m.orbits.size() <= 16, TRBL_E_INVALID, "gradient supports at most 16 orbits");
  GradTables& t = tables_for(m);
  const DeviceTables& d = m.dt;
  const int norb = (int)m.orbits.size(), ns = m.ns;
  // one work block: weights, densities by channel, occupations
  size_t at[5] = {(size_t)n_eig, 0, 0, 0, 0};
  for (int k = 0; k < 3; k++) at[k + 1] = at[k] + (t.ch[k].rho_off.empty() ? 0 : (size_t)t.ch[k].rho_off.back());
  at[4] = at[3] + 2 * (size_t)norb;
  t.work.alloc(at[4] * sizeof(double));
  double* work = t.work.as<double>();
  TRBL_HIP(hipMemcpyAsync(work, w, n_eig * sizeof(double), hipMemcpyHostToDevice, s));
  TRBL_HIP(hipMemsetAsync(work + at[0], 0, (at[4] - at[0]) * sizeof(double), s));
  GradArgs a{};
  a.X = X;
  a.n = n_eig;
  a.lq = n_eig <= 2 ? 1 : n_eig <= 4 ? 2 : 4;
  a.ns = ns;
  a.w = work;
  a.blk_off = d.blk_off.as<int64_t>();
  a.blk_dn = d.blk_dn.as<int>();
  a.pr_xu = t.pr_xu.as<int>();
  a.rblk = t.rblk.as<int>();
  a.rkp = t.rk[0].as<int>();
  a.rkn = t.rk[1].as<int>();
  for (int k = 2; k >= 0; k--) {
    const size_t ni = t.ch[k].nitems;
    if (ni == 0) continue;
    a.items = t.items[k].as<GradItem>();
    a.rect = t.rect[k].as<GradRect>();
    a.pr_off = t.pr_off[k].as<int>();
    a.rho_off = t.rho_off[k].as<int>();
    a.rho = work + at[k];
    a.species = k;
    if (k < 2) {
      a.list_off = t.list_off[k].as<int>();
      a.list_pair = t.list_pair[k].as<GradPair>();
    }
    int maxpair = 0;  // widest block, in whole wavefronts
    for (size_t b = 0; b + 1 < t.ch[k].pr_off.size(); b++)
      maxpair = std::max(maxpair, (t.ch[k].pr_off[b + 1] - t.ch[k].pr_off[b] + 63) / 64 * 64);
    const size_t shm = (size_t)maxpair * (sizeof(int64_t) + 3 * sizeof(int)) + 32 * 32 * sizeof(double);
    // a launch takes at most 2^22 workgroups
    for (size_t i0 = 0; i0 < ni; i0 += (size_t)1 << 22) {
      const dim3 grid((unsigned)std::min<size_t>(ni - i0, (size_t)1 << 22));
      if (k == 2) hipLaunchKernelGGL(dens_kernel<true>, grid, dim3(256), shm, s, a, maxpair);
      else hipLaunchKernelGGL(dens_kernel<false>, grid, dim3(256), shm, s, a, maxpair);
      a.items += grid.x;
    }
  }
  OccArgs oc{};
  oc.X = X;
  oc.n = n_eig;
  oc.w = work;
  oc.nblocks = (int)m.blocks.size();
  oc.norb = norb;
  oc.blk_dn = a.blk_dn;
  oc.blk_off = a.blk_off;
  oc.blk_p0 = d.blk_p0.as<int>();
  oc.blk_n0 = d.blk_n0.as<int>();
  oc.pwords = d.pwords.as<uint64_t>();
  oc.nwords = d.nwords.as<uint64_t>();
  for (int q = 0; q < ns; q++) oc.orbmask[m.st_orb[q]] |= 1ull << q;
  oc.occ = work + at[3];
  hipLaunchKernelGGL(dens_occ_kernel, dim3((unsigned)std::min<int64_t>((m.dim + 255) / 256, 1024)), dim3(256), 0, s, oc,
                     m.dim);
  TRBL_HIP(hipGetLastError());
  std::vector<double> h(at[4] - at[0]);
  TRBL_HIP(hipMemcpyAsync(h.data(), work + at[0], h.size() * sizeof(double), hipMemcpyDeviceToHost, s));
  TRBL_HIP(hipStreamSynchronize(s));
  // contraction with the J -> m coefficients; densities are stored for index i <= j of a block
  for (size_t q = 0; q < m.tbme.size(); q++) grad_v[q] = 0.0;
  const std::vector<MTerm>* terms[3] = {&m.terms_pp, &m.terms_nn, &m.terms_pn};
  const std::vector<std::vector<std::pair<int, double>>>* coef[3] = {&m.coef_pp, &m.coef_nn, &m.coef_pn};
  for (int k = 0; k < 3; k++) {
    const Channel& ch = t.ch[k];
    if (ch.nitems == 0) continue;
    for (size_t q = 0; q < terms[k]->size(); q++) {
      const MTerm& u = (*terms[k])[q];  // c+_a c+_b c_d c_c (pn: a, c protons)
      const int blk = ch.pblk[u.a * ns + u.b], D2 = ch.pr_off[blk + 1] - ch.pr_off[blk];
      const int i = ch.pid[u.a * ns + u.b], j = ch.pid[u.c * ns + u.d];
      const double r = h[at[k] - at[0] + ch.rho_off[blk] + (size_t)std::min(i, j) * D2 + std::max(i, j)];
      for (const auto& cv : (*coef[k])[q]) grad_v[cv.first] += cv.second * r;
    }
  }
  if (grad_spe)
    for (int q = 0; q < 2 * norb; q++) grad_spe[q] = h[at[3] - at[0] + q];
}

}  // namespace trbl
