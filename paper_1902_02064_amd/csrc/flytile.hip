// Identical-particle (two-body) part of the block H.V of single-species spaces as dense pair
// blocks on the matrix cores (App. B, the terms regrouped by their spectator nucleons).
#include <algorithm>
#include <cstdlib>
#include <map>

#include "tilecore.h"

namespace trbl {

using namespace tiles;

namespace {

// 4-pair steps of the kernel instance for a block of d pairs
__host__ __device__ inline int fly_steps(int d) {
  const int k = (d + 3) / 4;
  return k <= 6 ? k : k <= 12 ? (k + 1) / 2 * 2 : 16;
}

// ------------------------------------------------------------------ one species: pairs of identical nucleons
// A two-body term c+_a c+_b c_d c_c (a < b, c < d) of one species leaves n - 2 nucleons in place,
// a core L. With the pairs (a, b) of one (2M, parity) listed once, the terms acting on the
// states L + a + b form the dense symmetric block h(ab; cd) restricted to pairs outside L. The
// sign of the term on L + c + d is sigma(L, a) sigma(L, b) sigma(L, c) sigma(L, d) (the operators
// act on L in the order c, d, then b, a, and a < b, c < d), a target and a source factor. Every
// term application belongs to exactly one core (the target minus a and b), so the two-body part
// of W is the sum over the C(n, 2) cores of a target, slot (position of a, position of b) each.
//
// A block is the same for every core, so the 16 columns of a matrix instruction are shared by several
// cores; the pairs that a core blocks read zeros and write nothing.
template <class T>
struct FlyTileArgs {
  const T* V;  // internal order, packed nb
  T* Z;
  // column tile: first column, valid columns, lanes of a row (a power of two)
  int c0, cval, lr;
  int half, D, vrow;
  unsigned vbytes;
  const uint64_t* cw;  // cores, grouped
  const int* base;     // two-level ranking (sector-major low-part offsets, high-part ranks)
  const int* rank;
  const int* sstart;   // first internal index of each sector
  const int* pr_off;
  const int* pr_ab;
  const int* hb_off;
  const T* hb;
  const int* rect;    // per rectangle: pair block, target sector
  const int4* items;  // per work item: rectangle, first core, count, -
  int nitems;
};

#if defined(__HIP_DEVICE_COMPILE__)  // buffer descriptors exist only in the device pass
// The cores of one item for a block of at most 4 KS pairs. Lane c of the 16 columns serves core c / lr of
// KN and VPL adjacent columns (one load or store of up to 16 bytes); VPL instructions take a lane's columns
// one after the other. A wavefront lists KN cores at a time, a lane per pair (V offset, halved, with the
// sign of pair and core on top, NO_ROW where the core blocks the pair; slot row), with the rank-table
// lookups of the next KN issued ahead, runs the KS steps of each 16-target tile over the block's fragments,
// and during the last tile gathers the source rows of the next KN cores into the registers it has just used.
template <class T, int VPL, int KN, int KS>
struct FlyCores {
  static constexpr int LP = KS <= 4 ? 16 : KS <= 8 ? 32 : 64, PPO = 64 / LP;  // lanes of a core's list
  static constexpr int NO = KN > PPO ? KN / PPO : 1, DT = (KS + 3) / 4;
  static constexpr int LW = NO * 64;  // words of one list
  typedef typename Cols<T, VPL>::type cols;
  typedef typename Cols<T, VPL>::stored stored;
  typedef Buf<(int)sizeof(cols)> B;
  const FlyTileArgs<T>& a;
  const T* Af;
  unsigned* L;  // this wavefront's lists: [stage][V offsets, slot rows][LW]
  const uint64_t* Lc;
  int count, l, kq, sa, sb, st;
  const int* bk;
  bool have;
  unsigned vh, cb, sbyte, rowb, at0;
  uint64_t pair, lmask;
  __amdgpu_buffer_rsrc_t vs;
  int eb[NO], er[NO];

  __device__ __forceinline__ FlyCores(const FlyTileArgs<T>& a_, const int* Ps, int D2, int sk, const T* Af_,
                                      unsigned* L_, const uint64_t* Lc_, int count_)
      : a(a_), Af(Af_), L(L_), Lc(Lc_), count(count_) {
    l = threadIdx.x & 63;
    kq = l >> 4;
    const int c = l & 15, ab = Ps[min(l % LP, D2 - 1)];
    have = l % LP < D2;
    sa = ab & 255;
    sb = ab >> 8;  // sa < sb
    pair = (1ull << sa) | (1ull << sb);
    lmask = (1ull << a.half) - 1;
    st = a.sstart[sk];
    bk = a.base + ((int64_t)sk << a.half);
    vh = (unsigned)a.vrow >> 1;
    rowb = (unsigned)(a.lr * VPL * (int)sizeof(T));
    const int q = min(c / a.lr, KN - 1);  // lanes beyond KN * lr repeat the last core
    // columns of this lane: the last one of a ragged row overlaps its neighbour (the same values at the same
    // place), and lanes beyond it repeat those columns and fill the slot row up
    const int c1 = VPL * (c % a.lr), c2 = max(min(c1, a.cval - VPL), 0);
    cb = (unsigned)c2 * (unsigned)sizeof(T);
    sbyte = (unsigned)(c1 < a.cval ? c2 : c1) * (unsigned)sizeof(T);
    at0 = (unsigned)(q * LP + kq);
    vs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.V + a.c0), (short)0, (int)a.vbytes, 0x00020000);
  }
  __device__ __forceinline__ uint64_t core(int n, int o) const {
    const int j = n + o * PPO + l / LP;
    return j < count && o * PPO + l / LP < KN ? Lc[j] : ~0ull;
  }
  __device__ __forceinline__ bool free_pair(uint64_t K) const { return have && (K & pair) == 0; }
  // rank-table lookups of the KN cores from n on
  __device__ __forceinline__ void entries(int n) {
#pragma unroll
    for (int o = 0; o < NO; o++) {
      const uint64_t K = core(n, o), x = free_pair(K) ? K | pair : 0ull;
      eb[o] = bk[x & lmask];
      er[o] = a.rank[x >> a.half];
    }
  }
  // lists the KN cores from n on, whose lookups are held, then issues those of the cores from `next` on
  __device__ __forceinline__ void list(int buf, int n, int next) {
    unsigned* const Rv = L + buf * 2 * LW;
#pragma unroll
    for (int o = 0; o < NO; o++) {
      const uint64_t K = core(n, o);
      const unsigned t = (unsigned)(st + eb[o] + er[o]);
      const int pa = __popcll(K & ((1ull << sa) - 1)), pb = __popcll(K & ((1ull << sb) - 1)) + 1;
      const unsigned sg = (unsigned)(pa + pb + 1) << 31;  // sigma(K, a) sigma(K, b)
      Rv[o * 64 + l] = free_pair(K) ? __umul24(t, vh) | sg : NO_ROW >> 1;
      Rv[LW + o * 64 + l] = __umul24((unsigned)(pb * (pb - 1) / 2 + pa), (unsigned)a.D) + t;
    }
    entries(next);
    // the lists are written and read by this wavefront only: LDS operations of one wavefront
    // complete in order, so only the compiler must keep them in place
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ cols gather(const unsigned* Rv, int j) {
    return __builtin_bit_cast(cols, B::load(vs, (Rv[at0 + 4 * j] << 1) + cb));
  }
  static __device__ __forceinline__ T value(const cols& x, int t) {
    if constexpr (VPL == 1) return x;
    else return x[t];
  }
  static __device__ __forceinline__ cols flipped(cols x, unsigned o) {
    if constexpr (VPL == 1) {
      return flip_if(x, o >> 31);
    } else {
#pragma unroll
      for (int t = 0; t < VPL; t++) x[t] = flip_if((T)x[t], o >> 31);
      return x;
    }
  }
  __device__ __forceinline__ void run() {
    int n = (int)(threadIdx.x >> 6) * KN;
    if (n >= count) return;
    cols b[KS];
    entries(n);
    list(0, n, n + 4 * KN);
#pragma unroll
    for (int j = 0; j < KS; j++) b[j] = gather(L, j);
    char* const Zb = reinterpret_cast<char*>(a.Z) + sbyte;
    int buf = 0;
    for (; n < count; n += 4 * KN) {
      const unsigned* const Rv = L + buf * 2 * LW;
      buf ^= 1;
      list(buf, n + 4 * KN, n + 8 * KN);  // beyond the last core: no rows
      const unsigned* const Nv = L + buf * 2 * LW;
#pragma unroll
      for (int mt = 0; mt < DT; mt++) {
        typename Mfma<T>::acc acc[VPL];
#pragma unroll
        for (int t = 0; t < VPL; t++) acc[t] = typename Mfma<T>::acc{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < KS; j++) {
          if (mt == 0) b[j] = flipped(b[j], Rv[at0 + 4 * j]);
          const T av = Af[(mt * KS + j) * 64 + l];
#pragma unroll
          for (int t = 0; t < VPL; t++) acc[t] = Mfma<T>::run(av, value(b[j], t), acc[t]);
          if (mt == DT - 1) b[j] = gather(Nv, j);
        }
#pragma unroll
        for (int v = 0; v < 4; v++) {
          const int i = at0 - kq + 16 * mt + Mfma<T>::row(kq, v);
          if (sizeof(T) == 8 && 4 * mt + v >= KS) continue;  // beyond the block in every lane
          const unsigned o = Rv[i], z = Rv[LW + i];
          cols x;
          if constexpr (VPL == 1) {
            x = (T)acc[0][v];
          } else {
#pragma unroll
            for (int t = 0; t < VPL; t++) x[t] = (T)acc[t][v];
          }
          if (o != NO_ROW >> 1) {
            stored* p = reinterpret_cast<stored*>(Zb + (uint64_t)z * rowb);
            if constexpr (VPL > 1 && KN <= 4) __builtin_nontemporal_store(flipped(x, o), p);
            else *p = flipped(x, o);
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
};
#endif

// One work item: up to PN_TPB cores of one (2M, parity) group and one pair block, which is laid out as the
// matrix instructions read it (one conflict-free LDS read per fragment). Blocks of up to 16, 32 and 64
// pairs are launches of their own: registers and LDS of the narrow ones allow 8, 5 and 4 workgroups a CU (64 pairs with
// eight cores a turn, FP64 up to 4 columns: 3 by their LDS, 2 beyond 48 pairs).
// 112Sn-like space (D = 6,210,638, 53.8 M cores of 7.5 allowed pairs on average; ms per product): 8 columns
// FP64 38.0 -> 21.1, 1 column 32.4 -> 8.8, 16 columns 82.0 -> 44.0, 16 columns FP32 64.4 -> 21.7. (Before,
// each core compacted its allowed pairs: 114 instructions a core and block elements gathered from LDS; in
// one launch 25.7.) At 8 columns FP64 the slots are 27 GB written and read back and 28 GB of rows come from
// beyond the L2; the matrix cores are busy 35 % and the vector units 20 % of the kernel, the rest waits for rows.
template <class T, int VPL, int KN, int LP>
__global__ __launch_bounds__(256, LP == 16 ? 8 : LP == 32 ? 5 : 4) void fly_tile_kernel(FlyTileArgs<T> a) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __align__(16) char hs_[];  // fragments of the widest block
  T* Af = reinterpret_cast<T*>(hs_);
  __shared__ int Ps[LP];
  __shared__ uint64_t Lc[PN_TPB];
  constexpr int LW = 4 * std::max(KN * LP, 64);  // words of one wavefront's lists
  __shared__ unsigned L[4 * LW];
  const int item = pn_xcd_item(blockIdx.x, a.nitems);
  if (item >= a.nitems) return;
  const int4 it = a.items[item];
  const int k = a.rect[2 * it.x], sk = a.rect[2 * it.x + 1];
  const int q0 = a.pr_off[k], D2 = a.pr_off[k + 1] - q0;
  const T* hg = a.hb + a.hb_off[k];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  for (int e = threadIdx.x; e < D2; e += 256) Ps[e] = a.pr_ab[q0 + e];
  for (int e = threadIdx.x; e < it.z; e += 256) Lc[e] = a.cw[it.y + e];
  const int KS = fly_steps(D2), nf = (KS + 3) / 4 * KS;
  for (int f = w; f < nf; f += 4) {
    const int i = f / KS * 16 + (l & 15), j = f % KS * 4 + (l >> 4);
    Af[f * 64 + l] = i < D2 && j < D2 ? hg[i * D2 + j] : T(0);
  }
  __syncthreads();
#define TRBL_CORES(K) \
  case K: FlyCores<T, VPL, KN, K>(a, Ps, D2, sk, Af, L + w * LW, Lc, it.z).run(); break
  if constexpr (LP == 16) {
    switch (KS) {
      TRBL_CORES(1);
      TRBL_CORES(2);
      TRBL_CORES(3);
      TRBL_CORES(4);
    }
  } else if constexpr (LP == 32) {
    switch (KS) {
      TRBL_CORES(5);
      TRBL_CORES(6);
      TRBL_CORES(8);
    }
  } else {
    switch (KS) {
      TRBL_CORES(10);
      TRBL_CORES(12);
      TRBL_CORES(16);
    }
  }
#undef TRBL_CORES
#endif
}

// W[t][c0 ..] = (single-particle energies of t) V[t][c0 ..] + the slots of t in slot order, 16 bytes of
// columns a thread (t and V in the internal order, V packed nb, cpr chunks to a slot row; W in Table-1 order)
template <class T>
__global__ void fly_finalize_kernel(const T* __restrict__ V, int nb, T* __restrict__ W, int64_t ldw,
                                    const T* __restrict__ Z, int S, int64_t D, int cpr, int c0, int cval,
                                    const uint64_t* words, const T* e, const int* sstart, const int64_t* soff,
                                    const int* perm, int nsec) {
  constexpr int VPC = 16 / (int)sizeof(T);
  typedef T zv __attribute__((ext_vector_type(VPC)));
  const int64_t n = D * cpr;
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = q / cpr;
    const int c = (int)(q - t * cpr) * VPC;
    if (c >= cval) continue;
    T d = T(0);
    for (uint64_t x = words[t]; x; x &= x - 1) d += e[__builtin_ctzll(x)];
    const T* vt = V + t * nb + c0 + c;
    zv s;
#pragma unroll
    for (int j = 0; j < VPC; j++) s[j] = c + j < cval ? d * vt[j] : T(0);
    const zv* z = reinterpret_cast<const zv*>(Z) + q;
    int k = 0;
    for (; k + 8 <= S; k += 8) {
      zv zq[8];
#pragma unroll
      for (int j = 0; j < 8; j++) zq[j] = __builtin_nontemporal_load(z + (k + j) * n);
#pragma unroll
      for (int j = 0; j < 8; j++) s += zq[j];
    }
    for (; k < S; k++) s += __builtin_nontemporal_load(z + k * n);
    int sec = 0;
    while (sec + 1 < nsec && t >= sstart[sec + 1]) sec++;
    T* wt = W + (soff[sec] + perm[t]) * ldw + c0 + c;
#pragma unroll
    for (int j = 0; j < VPC; j++)
      if (c + j < cval) wt[j] = s[j];
  }
}

template <class T, int VPL, int KN, int LP>
void launch_class(FlyTileArgs<T> a, const int4* items, const int* first, int max_pairs, hipStream_t s) {
  const int cl = LP == 16 ? 0 : LP == 32 ? 1 : 2, ks = fly_steps(std::min(LP, max_pairs));
  a.items = items + first[cl];
  a.nitems = first[cl + 1] - first[cl];
  if (a.nitems == 0) return;
  hipLaunchKernelGGL((fly_tile_kernel<T, VPL, KN, LP>), dim3((unsigned)((a.nitems + 7) / 8 * 8)), dim3(256),
                     (size_t)((ks + 3) / 4 * ks) * 64 * sizeof(T), s, a);
}
template <class T, int VPL, int KN>
void launch_tile(const FlyTileArgs<T>& a, const FlyTiles& F, hipStream_t s) {
  const int4* items = F.items_buf.as<int4>();
  launch_class<T, VPL, KN, 64>(a, items, F.first, F.max_pairs, s);
  launch_class<T, VPL, KN, 32>(a, items, F.first, F.max_pairs, s);
  launch_class<T, VPL, KN, 16>(a, items, F.first, F.max_pairs, s);
}

}  // namespace

// ------------------------------------------------------------------ one species: host tables and launch
void build_fly_tiles(Model& m) {
  FlyTiles& F = m.flyt;
  F.on = false;
  F.z.release();
  const char* env = std::getenv("TRBL_PN_TILES");
  if (env && env[0] == '0') return;
  const Species& SP = m.sp[m.fly_s];
  const int ns = m.ns, npart = SP.npart, tj = m.cl.tjmax;
  if (npart < 2) return;
  const std::vector<MTerm>& terms = m.fly_s == 1 ? m.terms_nn : m.terms_pp;
  auto stpar = [&](int st) { return (m.orbits[m.st_orb[st]].l & 1) ? 1 : 0; };  // 1: odd
  // pair blocks by (2M, parity) of the pair, pairs a < b
  std::map<std::pair<int, int>, int> kid;
  std::vector<std::vector<int>> pairs;
  std::vector<int> pid(ns * ns, -1), pk(ns * ns, -1);
  for (int a0 = 0; a0 < ns; a0++)
    for (int b0 = a0 + 1; b0 < ns; b0++) {
      const std::pair<int, int> key{m.st_tm[a0] + m.st_tm[b0], stpar(a0) ^ stpar(b0)};
      auto itk = kid.find(key);
      if (itk == kid.end()) {
        itk = kid.emplace(key, (int)pairs.size()).first;
        pairs.emplace_back();
      }
      pk[a0 * ns + b0] = itk->second;
      pid[a0 * ns + b0] = (int)pairs[itk->second].size();
      pairs[itk->second].push_back(a0 | (b0 << 8));
    }
  const int nk = (int)pairs.size();
  int maxp = 0;
  for (auto& v : pairs) maxp = std::max(maxp, (int)v.size());
  if (maxp > PN_MAXPAIR) return;
  std::vector<int> pr_off(nk + 1, 0), pr_ab, hb_off(nk + 1, 0);
  for (int k = 0; k < nk; k++) {
    pr_off[k + 1] = pr_off[k] + (int)pairs[k].size();
    hb_off[k + 1] = hb_off[k] + (int)(pairs[k].size() * pairs[k].size());
    pr_ab.insert(pr_ab.end(), pairs[k].begin(), pairs[k].end());
  }
  std::vector<double> hb(hb_off[nk], 0.0);
  for (const MTerm& t : terms) {  // c+_a c+_b c_d c_c, a < b, c < d
    TRBL_REQUIRE(t.a < t.b && t.c < t.d, TRBL_E_INVALID, "identical-particle term not in canonical order");
    const int k = pk[t.a * ns + t.b];
    TRBL_REQUIRE(k == pk[t.c * ns + t.d], TRBL_E_INVALID, "two-body term breaks M or parity conservation");
    const int D2 = (int)pairs[k].size();
    hb[hb_off[k] + pid[t.a * ns + t.b] * D2 + pid[t.c * ns + t.d]] += t.h;
  }
  // cores: (n - 2)-subsets grouped by (2M, parity); only groups whose pairs reach a stored sector
  const int nc = npart - 2;
  if (binom(ns, nc) > (int64_t)1 << 27) return;
  std::map<std::pair<int, int>, int> secid;
  for (int q = 0; q < (int)SP.sectors.size(); q++) secid[{SP.sectors[q].twoM, SP.sectors[q].par < 0 ? 1 : 0}] = q;
  std::map<std::pair<int, int>, std::vector<uint64_t>> by;
  auto visit = [&](uint64_t w) {
    int tm = 0, par = 0;
    for (uint64_t x = w; x; x &= x - 1) {
      const int st = __builtin_ctzll(x);
      tm += m.st_tm[st];
      par ^= stpar(st);
    }
    by[{tm, par}].push_back(w);
  };
  if (nc == 0) {
    visit(0);
  } else {
    uint64_t w = (1ull << nc) - 1;
    const uint64_t limit = ns == 64 ? 0ull : (1ull << ns);
    while (true) {
      visit(w);
      const uint64_t lo = w & (~w + 1), hi = w + lo;
      if (hi == 0) break;
      const uint64_t nw = (((hi ^ w) >> 2) / lo) | hi;
      if ((ns < 64 && nw >= limit) || nw <= w) break;
      w = nw;
    }
  }
  std::vector<uint64_t> cw;
  std::vector<int> rect, items, cls[3];  // work items by lanes of a core's list: 16, 32, 64
  for (auto& kv : by) {
    std::vector<std::pair<int, int>> rs;  // (pair block, sector)
    for (const auto& sv : secid) {
      const int tmp = sv.first.first - kv.first.first, parp = sv.first.second ^ kv.first.second;
      auto itk = kid.find({tmp, parp});
      if (itk != kid.end()) rs.push_back({itk->second, sv.second});
    }
    if (rs.empty()) continue;
    // cores in the order of the internal numbering (low part of the m-states first): consecutive
    // cores then reach targets and sources in nearby ranges of V and of the slots
    const uint64_t lm = (1ull << m.fly_half) - 1;
    std::sort(kv.second.begin(), kv.second.end(), [&](uint64_t x, uint64_t y) {
      return (x & lm) != (y & lm) ? (x & lm) < (y & lm) : (x >> m.fly_half) < (y >> m.fly_half);
    });
    const int c0 = (int)cw.size();
    cw.insert(cw.end(), kv.second.begin(), kv.second.end());
    const int n = (int)kv.second.size();
    for (const auto& r : rs) {
      const int ri = (int)(rect.size() / 2);
      rect.insert(rect.end(), {r.first, r.second});
      const int np = (int)pairs[r.first].size();
      std::vector<int>& to = cls[np <= 16 ? 0 : np <= 32 ? 1 : 2];
      for (int q = 0; q < n; q += PN_TPB) to.insert(to.end(), {ri, c0 + q, std::min(PN_TPB, n - q), 0});
    }
  }
  for (int q = 0; q < 3; q++) {
    items.insert(items.end(), cls[q].begin(), cls[q].end());
    F.first[q + 1] = (int)(items.size() / 4);
  }
  if (items.empty()) return;
  TRBL_REQUIRE(items.size() / 4 < ((size_t)1 << 31) / 256, TRBL_E_INVALID, "too many cores for one launch");
  const int S = npart * (npart - 1) / 2;
  const size_t zbytes = (size_t)S * (size_t)m.dim * 64;  // slot rows of at most 64 bytes
  size_t fr = 0, tot = 0;
  TRBL_HIP(hipMemGetInfo(&fr, &tot));
  // (V of 64 columns below NO_ROW bytes)
  if (zbytes > fr / 4 || (double)m.dim * 64 * 8 > (double)NO_ROW || (double)S * m.dim >= 4294967296.0) return;
  F.S = S;
  F.max_pairs = maxp;
  F.cw.upload(cw);
  F.pr_off.upload(pr_off);
  F.pr_ab.upload(pr_ab);
  F.hb_off.upload(hb_off);
  F.hb.upload(hb);
  F.hb32.upload(std::vector<float>(hb.begin(), hb.end()));
  F.rect.upload(rect);
  F.items_buf.upload(items);
  F.z.alloc(zbytes);
  F.on = true;
}

template <class T>
void launch_fly_tiles(const Model& m, int nb, const T* Vint, T* W, int64_t ldw, hipStream_t s) {
  constexpr int VPC = 16 / (int)sizeof(T), WIDE = 64 / (int)sizeof(T);  // values per lane, most columns at once
  const FlyTiles& F = m.flyt;
  const DeviceTables& d = m.dt;
  FlyTileArgs<T> a{};
  a.V = Vint;
  a.Z = F.z.as<T>();
  a.half = m.fly_half;
  a.D = (int)m.dim;
  a.vrow = (int)(nb * sizeof(T));
  a.cw = F.cw.as<uint64_t>();
  a.base = d.fly_base.as<int>();
  a.rank = d.fly_rank.as<int>();
  a.sstart = d.fly_sstart.as<int>();
  a.pr_off = F.pr_off.as<int>();
  a.pr_ab = F.pr_ab.as<int>();
  a.hb_off = F.hb_off.as<int>();
  a.hb = (sizeof(T) == 8 ? F.hb : F.hb32).as<T>();
  a.rect = F.rect.as<int>();
  for (int c0 = 0; c0 < nb; c0 += WIDE) {
    a.c0 = c0;
    a.cval = std::min(WIDE, nb - c0);
    a.vbytes = (unsigned)(m.dim * a.vrow - c0 * (int64_t)sizeof(T));
    const int cpr = pn_slot_stride(sizeof(T), a.cval);  // 16-byte chunks of a slot row
    if (a.cval < VPC) {
      a.lr = VPC;  // one value a lane
      launch_tile<T, 1, 16 / VPC>(a, F, s);
    } else {
      a.lr = cpr;
      if (cpr <= 2) launch_tile<T, VPC, 8>(a, F, s);
      else launch_tile<T, VPC, 4>(a, F, s);
    }
    hipLaunchKernelGGL(fly_finalize_kernel<T>, dim3(elementwise_grid(m.dim * cpr)), dim3(256), 0, s, Vint, nb, W, ldw,
                       (const T*)a.Z, F.S, m.dim, cpr, c0, a.cval, d.fly_wint.as<uint64_t>(),
                       (sizeof(T) == 8 ? d.fly_e64 : d.fly_e32).as<T>(), a.sstart, d.fly_soff.as<int64_t>(),
                       d.fly_perm.as<int>(), (int)m.sp[m.fly_s].sectors.size());
  }
  TRBL_HIP(hipGetLastError());
}
template void launch_fly_tiles<double>(const Model&, int, const double*, double*, int64_t, hipStream_t);
template void launch_fly_tiles<float>(const Model&, int, const float*, float*, int64_t, hipStream_t);

}  // namespace trbl
