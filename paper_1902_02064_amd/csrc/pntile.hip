// Proton-neutron part of the block H.V (App. B) as dense pair blocks on the matrix cores.
//
// Every pn term c+_a(p) c+_b(n) c_d(n) c_c(p) moves one proton (c -> a) and one neutron (d -> b).
// Acting on a basis state it keeps the other protons, a core K_p of n_prot - 1 particles, and the
// other neutrons, a core K_n. Take the pair states (x, u), x a proton m-state and u a neutron
// m-state, grouped by their total 2m. For a fixed core pair (K_p, K_n) the states K_p+x, K_n+u
// with x outside K_p and u outside K_n, and 2m(x) + 2m(u) = 2M - 2M(K_p) - 2M(K_n), are linked
// by the pn terms as a dense symmetric block: the m-scheme pn matrix H_M[(x,u)][(y,v)] of that
// pair 2m, restricted to the allowed pairs. The Jordan-Wigner sign of c+_x c_y on K_p+y is
// sigma(K_p, x) sigma(K_p, y), sigma(K, s) = (-1)^(occupied states of K below s), and the same on
// the neutron side, so the sign of an element factorises into a target and a source sign.
//
// Each term is counted in exactly one core pair (the core is the set of spectator nucleons;
// a = c is a proton number operator, and its core is the target minus a), so the pn part of W is
//   W[t] += sum over the n_prot * n_neut core pairs of t of  s_t (H_M (s V))[t].
// A work item fixes one core (of protons, or of neutrons where their runs are short) and runs over cores of the
// other species. The pair states that the fixed core leaves free are compacted once, by a ballot, and the block of H_M
// over them is laid out in LDS as the matrix instructions read it. Several cores of the run share the 16 columns of an
// instruction, a lane serving one core and up to 16 bytes of adjacent columns: it gathers the source rows with their
// signs and writes each target row into a slot of its own; pairs that the run's core blocks read zeros and write
// nothing.
//
// Slots. The proton cores are worked through in batches. A batch owns a slot row for every
// (core K_p, x, position of u in the target's neutron word, target neutron state), so each slot is
// written exactly once, and the target rows K_p + x then add their slots to W in a fixed order:
// no atomics, and the result does not depend on scheduling. With several batches two slot buffers
// alternate: one launch computes a batch and adds the previous one to W. With one batch the slots of
// all targets lie position pair by position pair, and the own-row kernel or pn_sum_kernel adds them.
#include <algorithm>
#include <array>
#include <cstdlib>
#include <map>

#include "tilecore.h"

namespace trbl {

using namespace tiles;

namespace {

template <class T>
struct PNTileArgs {
  const T* V;
  T* Z;
  // column tile: first column, valid columns, lanes of a row (a power of two), 16-byte chunks of a slot row
  // (written, and holding valid columns)
  int c0, cval, lr, cpr, cprv;
  int ns;
  int64_t vrow;  // bytes per row of V
  // [core * ns + state]: position << 24 | local index of core + state, -1 inside; of the species whose core an item
  // fixes and of the species whose cores it runs over
  const int* rkf;
  const int* rkr;
  int swap;           // the neutron core is fixed
  const int* blk_off;  // block offsets (the tables are used only while D < 2^31)
  const int* blk_dn;
  const int* pr_off;
  const int* pr_xu;
  const int* hb_off;
  const T* hb;
  const int* rect;    // per rectangle: pair block, first entry of its list in rblk
  const int* rblk;    // per rectangle and pair: target block << 1 | parity of its neutron sector, -1 if none
  const int* zoff;    // several batches: [(core * ns + x) * 2 + neutron parity], first slot row in the batch
  int zstep;          // one batch: slot rows between positions of u (0: the neutron states of the target's sector)
  const int4* items;  // per work item: rectangle, fixed core, first core of the run, count
  int nitems, spread;  // spread: taken in order by all XCDs, else a contiguous range for each
  unsigned vbytes, zbytes;  // of V (where it stays below 4 GiB) and of a slot buffer
  // the previous batch, added to W by the first nred workgroups
  const T* Zr;
  T* W;
  int64_t ldw;
  const PNRow* rows;
  const int* tent;
  int nred, nchunk, nrows, nneut, wvec;
};

constexpr int RED_ROWS = 64;  // target rows of one reducing workgroup

// 16 bytes of a row of W += the `per` slots of each of n entries (first slot chunk z(i), `step` chunks apart),
// entry by entry
template <class T, class F>
__device__ __forceinline__ void add_chunk(const PNTileArgs<T>& a, int64_t row, int k, int n, int per, int64_t step,
                                          F&& z) {
  constexpr int VPC = 16 / (int)sizeof(T);  // values per 16 bytes
  typedef T zv __attribute__((ext_vector_type(VPC)));
  T* w = a.W + row * a.ldw + a.c0 + VPC * k;
  const bool full = a.wvec && VPC * k + VPC <= a.cval;
  zv v;
  if (full) {
    v = *reinterpret_cast<const zv*>(w);
  } else {
#pragma unroll
    for (int j = 0; j < VPC; j++) v[j] = VPC * k + j < a.cval ? w[j] : T(0);
  }
  for (int i = 0; i < n; i++) {
    const zv* x = reinterpret_cast<const zv*>(a.Zr) + z(i) + k;
    int q = 0;
    for (; q + 4 <= per; q += 4) {  // four in flight
      zv zq[4];
#pragma unroll
      for (int j = 0; j < 4; j++) zq[j] = __builtin_nontemporal_load(x + (q + j) * step);
#pragma unroll
      for (int j = 0; j < 4; j++) v += zq[j];
    }
    for (; q < per; q++) v += __builtin_nontemporal_load(x + q * step);
  }
  if (full) {
    *reinterpret_cast<zv*>(w) = v;
  } else {
#pragma unroll
    for (int j = 0; j < VPC; j++)
      if (VPC * k + j < a.cval) w[j] = v[j];
  }
}

// the slots of the target rows of a batch, entry by entry and position by position
template <class T>
__device__ __forceinline__ void add_slots(const PNTileArgs<T>& a, int bid) {
  const int ri = bid / a.nchunk, t0 = (bid % a.nchunk) * RED_ROWS;
  if (ri >= a.nrows) return;
  const PNRow r = a.rows[ri];
  const int n = min(RED_ROWS, r.dn - t0) * a.cprv;  // not positive: a chunk beyond this row
  const int64_t step = (int64_t)r.dn * a.cpr;
  for (int e = threadIdx.x; e < n; e += 256) {
    const int t = t0 + e / a.cprv;
    add_chunk(a, r.row + t, e % a.cprv, r.ne, a.nneut, step,
              [&](int i) { return ((int64_t)a.tent[r.e0 + i] + t) * a.cpr; });
  }
}

// One batch: every target has the same number of slots, `zstep` slot rows apart, so a thread takes 16 bytes of
// any row (a workgroup a target row leaves most of its threads idle where the rows have few neutron states:
// pf 5+1, 32 columns FP64, 28.5 us against 6.7 us a tile).
template <class T>
__global__ __launch_bounds__(256) void pn_sum_kernel(PNTileArgs<T> a, int rows, int slots) {
  const int64_t step = (int64_t)rows * a.cpr;  // all slots together stay below 4 GiB
  for (int e = blockIdx.x * 256 + threadIdx.x; e < rows * a.cprv; e += gridDim.x * 256) {
    const int t = e / a.cprv;
    add_chunk(a, t, e - t * a.cprv, 1, slots, step, [&](int) { return (int64_t)t * a.cpr; });
  }
}

// Per-item tables in LDS: the pair states that the fixed core allows, in order. Below, `state` is the m-state of
// the run's species and `loc` the index of core + state in its sector: V row row + mul * loc, slot row
// z + step * (position of state) + mul * loc; pos: position of the fixed species' state; id: index in the pair block.
struct PairList {
  int state[PN_MAXPAIR], row[PN_MAXPAIR], mul[PN_MAXPAIR], z[PN_MAXPAIR], pos[PN_MAXPAIR], step[PN_MAXPAIR],
      id[PN_MAXPAIR];
};

#if defined(__HIP_DEVICE_COMPILE__)
// The core pairs of one item whose fixed core allows d <= 4 KS pair states. The block is the same for
// every core of the run, so the 16 columns of a matrix instruction are shared by KN of them: lane c
// serves core c / lr and VPL adjacent columns (one load or store of up to 16 bytes), and VPL
// instructions take a lane's columns one after the other. A wavefront lists KN cores at a
// time, a lane per pair state (V offset and slot offset, halved, with the sign on top; NO_ROW where the
// core holds the state), runs the KS k-steps of each 16-target tile over the block's fragments, and
// during the last tile gathers each k-step's source rows of the next KN cores into the registers that
// the step has just used.
template <class T, int VPL, int KN, bool BIG, int KS>
struct CorePairs {
  static constexpr int LP = KS <= 4 ? 16 : KS <= 8 ? 32 : 64, PPO = 64 / LP;
  static constexpr int NO = KN > PPO ? KN / PPO : 1, DT = (KS + 3) / 4;
  static constexpr int LW = NO * 64;  // words of one list
  typedef typename Cols<T, VPL>::type cols;
  typedef Buf<(int)sizeof(cols)> B;
  const PNTileArgs<T>& a;
  const T* Af;
  unsigned* L;  // this wavefront's lists: [stage][V offsets, slot offsets][LW]
  int first, count;
  int l, c, kq, q, pst;
  bool have;
  unsigned vrow, vmul, zmul, prow, pz, pstep, psg, cb, sb, at0;
  __amdgpu_buffer_rsrc_t vs, zs;
  int en[NO];

  __device__ __forceinline__ CorePairs(const PNTileArgs<T>& a_, const PairList& P, int d, const T* Af_, unsigned* L_,
                                       int first_, int count_)
      : a(a_), Af(Af_), L(L_), first(first_), count(count_) {
    l = threadIdx.x & 63;
    c = l & 15;
    kq = l >> 4;
    const int i = min(l % LP, d - 1);
    have = l % LP < d;
    vrow = (unsigned)a.vrow;
    const unsigned vh = vrow >> 1, rh = (unsigned)(a.lr * VPL * (int)sizeof(T)) >> 1, mul = (unsigned)P.mul[i];
    pst = P.state[i];
    prow = BIG ? (unsigned)P.row[i] : (unsigned)P.row[i] * vh;
    vmul = BIG ? mul : mul * vh;
    pz = (unsigned)P.z[i] * rh;
    zmul = mul * rh;
    pstep = (unsigned)P.step[i] * rh;
    psg = (unsigned)P.pos[i];
    q = min(c / a.lr, KN - 1);  // lanes beyond KN * lr repeat the last core
    // columns of this lane: the last one of a ragged row overlaps its neighbour (the same values at the same
    // place), and lanes beyond it repeat those columns and fill the slot row up
    const int c1 = VPL * (c % a.lr), c2 = min(c1, a.cval - VPL);
    cb = (unsigned)c2 * (unsigned)sizeof(T);
    sb = (unsigned)(c1 < a.cval ? c2 : c1) * (unsigned)sizeof(T);
    at0 = (unsigned)(q * LP + kq);
    vs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.V + a.c0), (short)0, (int)a.vbytes, 0x00020000);
    zs = __builtin_amdgcn_make_buffer_rsrc((void*)a.Z, (short)0, (int)a.zbytes, 0x00020000);
  }
  // table entries of the KN cores from n on
  __device__ __forceinline__ void entries(int n) {
#pragma unroll
    for (int o = 0; o < NO; o++) {
      const int core = n + o * PPO + l / LP;
      en[o] = core < count && o * PPO + l / LP < KN ? a.rkr[(first + core) * a.ns + pst] : -1;
    }
  }
  // lists the KN cores whose entries are held, then fetches the entries from `next` on
  __device__ __forceinline__ void list(int buf, int next) {
    unsigned* const Rv = L + buf * 2 * LW;
#pragma unroll
    for (int o = 0; o < NO; o++) {
      const int rn = en[o];
      const bool ok = have && rn >= 0;
      const unsigned loc = (unsigned)rn & 0xFFFFFFu, pos = (unsigned)rn >> 24;
      const unsigned sg = (psg + pos) << 31;
      Rv[o * 64 + l] = ok ? (prow + __umul24(loc, vmul)) | sg : BIG ? ~0u : NO_ROW >> 1;
      Rv[LW + o * 64 + l] = ok ? (pz + pos * pstep + __umul24(loc, zmul)) | sg : NO_ROW >> 1;
    }
    entries(next);
    // the lists are written and read by this wavefront only: LDS operations of one wavefront
    // complete in order, so only the compiler must keep them in place
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ cols gather(const unsigned* Rv, int j) {
    const unsigned o = Rv[at0 + 4 * j];
    if constexpr (BIG) {
      const bool no = o == ~0u;
      const char* p = reinterpret_cast<const char*>(a.V + a.c0) + ((uint64_t)(no ? 0u : o & 0x7FFFFFFFu) * vrow + cb);
      cols x;
      __builtin_memcpy(&x, p, sizeof(x));
      return no ? cols(0) : x;
    } else {
      return __builtin_bit_cast(cols, B::load(vs, (o << 1) + cb));
    }
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
    list(0, n + 4 * KN);
#pragma unroll
    for (int j = 0; j < KS; j++) b[j] = gather(L, j);
    int buf = 0;
    for (; n < count; n += 4 * KN) {
      const unsigned* const Rv = L + buf * 2 * LW;
      buf ^= 1;
      list(buf, n + 8 * KN);  // beyond the last core: no rows
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
          const unsigned z = Rv[LW + q * LP + 16 * mt + Mfma<T>::row(kq, v)];
          cols x;
          if constexpr (VPL == 1) {
            x = (T)acc[0][v];
          } else {
#pragma unroll
            for (int t = 0; t < VPL; t++) x[t] = (T)acc[t][v];
          }
          B::template store<(VPL > 1 && KN <= 4)>(__builtin_bit_cast(typename B::raw, flipped(x, z)), zs, (z << 1) + sb);
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
};
#endif

// One work item: a proton core K_p and a run of neutron cores of one (2M, parity) group, or a neutron core and
// a run of proton cores. The pair states that the fixed core leaves free are listed once, and the block of H_M
// over them is laid out as the matrix instructions read it (one conflict-free LDS read per fragment). The cores
// of the run then only mask sources and targets: their blocked pairs read zeros and write nothing. The first
// workgroups of a launch add the previous batch.
// Registers allow 4 workgroups a CU. LDS, sized for the widest block of the space, allows 3 or 4 at two and four cores
// a turn and 2 or 3 at eight (FP64 up to 4 columns, FP32 from 4 to 8): the lists of eight cores take 32 KB, the
// fragments of a block of 60 pairs 32 KB in FP64.
template <class T, int VPL, int KN, bool BIG>
__global__ __launch_bounds__(256, 4) void pn_tile_kernel(PNTileArgs<T> a) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __align__(16) char hs_[];  // fragments of the widest block
  T* Af = reinterpret_cast<T*>(hs_);
  __shared__ PairList P;
  constexpr int LW = 4 * KN * 64;  // words of one wavefront's lists
  __shared__ unsigned L[4 * LW];
  if ((int)blockIdx.x < a.nred) {
    add_slots<T>(a, blockIdx.x);
    return;
  }
  const int item = a.spread ? blockIdx.x - a.nred : pn_xcd_item(blockIdx.x - a.nred, a.nitems);
  if (item >= a.nitems) return;
  const int4 it = a.items[item];
  const int k = a.rect[2 * it.x], rb0 = a.rect[2 * it.x + 1];
  const int q0 = a.pr_off[k], D2 = a.pr_off[k + 1] - q0;
  const T* hg = a.hb + a.hb_off[k];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int xu = a.pr_xu[q0 + min(l, D2 - 1)], fst = a.swap ? xu >> 8 : xu & 255;
  const int tb = a.rblk[rb0 + min(l, D2 - 1)];
  const int rf = a.rkf[it.y * a.ns + fst];
  const bool lok = l < D2 && tb >= 0 && rf >= 0;
  const uint64_t mask = __ballot(lok);
  const int d = __popcll(mask);
  if (d == 0) return;  // the same for every wavefront
  if (w == 0 && lok) {
    const int i = __popcll(mask & ((1ull << l) - 1));
    const int dn = a.blk_dn[tb >> 1], row = a.blk_off[tb >> 1] + (rf & 0xFFFFFF) * (a.swap ? 1 : dn), pos = rf >> 24;
    P.state[i] = a.swap ? xu & 255 : xu >> 8;
    P.row[i] = row;
    P.mul[i] = a.swap ? dn : 1;
    P.pos[i] = pos;
    if (a.zstep) {  // one batch: [position of x][position of u][target]
      P.z[i] = pos * (a.swap ? a.zstep : a.nneut * a.zstep) + row;
      P.step[i] = a.swap ? a.nneut * a.zstep : a.zstep;
    } else {
      P.z[i] = a.zoff[(it.y * a.ns + fst) * 2 + (tb & 1)];
      P.step[i] = dn;
    }
    P.id[i] = l;
  }
  __syncthreads();
  const int KS = (d + 7) / 8 * 2, nf = (KS + 3) / 4 * KS;
  for (int f = w; f < nf; f += 4) {
    const int i = f / KS * 16 + (l & 15), j = f % KS * 4 + (l >> 4);
    Af[f * 64 + l] = i < d && j < d ? hg[P.id[i] * D2 + P.id[j]] : T(0);
  }
  __syncthreads();
#define TRBL_PAIRS(K) \
  case K: CorePairs<T, VPL, KN, BIG, K>(a, P, d, Af, L + w * LW, it.z, it.w).run(); break
  switch (KS) {
    TRBL_PAIRS(2);
    TRBL_PAIRS(4);
    TRBL_PAIRS(6);
    TRBL_PAIRS(8);
    TRBL_PAIRS(10);
    TRBL_PAIRS(12);
    TRBL_PAIRS(14);
    TRBL_PAIRS(16);
  }
#undef TRBL_PAIRS
#endif
}

}  // namespace

void build_pn_tiles(Model& m) {
  PNTiles& T = m.pn;
  T.on = false;
  T.z.release();
  T.batches.clear();
  const char* env = std::getenv("TRBL_PN_TILES");
  if (env && env[0] == '0') return;
  T.force = env && env[0] == '2';
  if (m.fly || m.n_prot == 0 || m.n_neut == 0) return;
  const int ns = m.ns, tj = m.cl.tjmax;
  const int nk = 2 * tj + 1;
  // pair blocks by pair 2m: (x, u) with 2m(x) + 2m(u) = 2 (k - tj)
  std::vector<std::vector<int>> pairs(nk);
  std::vector<int> pid(ns * ns, -1);
  for (int x = 0; x < ns; x++)
    for (int u = 0; u < ns; u++) {
      const int k = (m.st_tm[x] + m.st_tm[u] + 2 * tj) / 2;
      pid[x * ns + u] = (int)pairs[k].size();
      pairs[k].push_back(x | (u << 8));
    }
  int maxp = 0;
  for (auto& v : pairs) maxp = std::max(maxp, (int)v.size());
  if (maxp > PN_MAXPAIR) return;
  // Where the pair blocks are built and taken (ms per product, jump lists / pair blocks; TRBL_PN_TILES=2 takes them
  // regardless). A slot row, written and read back, carries the products of one core pair: on average about
  // L = (pair-weighted mean block size) x (share of the proton states outside a proton core) x (the same for
  // neutrons) source pairs. A product on pair blocks costs at least about 0.06 ms of launches.
  // L >= 16 (pf spaces): from 2,500 states on, FP64 at 1, 8, 16, 32 columns: pf 4+4 (L = 31) 1.85 / 0.90, 3.18 / 1.62,
  // 5.56 / 3.25, 11.4 / 7.2; pf 3+3 0.184 / 0.083, 0.259 / 0.122, 0.356 / 0.178, 0.547 / 0.388; pf 1+4 0.062 / 0.066,
  // 0.092 / 0.074, 0.127 / 0.090, 0.146 / 0.112; pf 3+1 (D = 2,550) 0.062 / 0.059, 0.069 / 0.064, 0.079 / 0.068,
  // 0.160 / 0.082; pf 2+1 (D = 472) 0.028 / 0.062, 0.031 / 0.064, 0.037 / 0.063, 0.048 / 0.078. Below 5,000 states
  // spaces of several protons keep the jump lists where these share a row as below (8, 12, 16, 32 columns: pf 2+2
  // 0.034 / 0.060, 0.047 / 0.060, 0.043 / 0.061, 0.059 / 0.077), and with one proton, where twenty rows leave the chip
  // empty, the pair blocks take rows of 65 to 128 bytes (pf 1+3 0.042 / 0.062, 0.090 / 0.065, 0.072 / 0.068, 0.072 /
  // 0.082).
  // L from 11 to 16 (sd): the same rows (8, 12, 16, 32 columns: sd 4+4 (L = 11.4) 0.051 / 0.065, 0.117 / 0.079, 0.106 /
  // 0.084, 0.110 / 0.160; sd 2+5 0.032 / 0.063, 0.093 / 0.065, 0.072 / 0.067, 0.073 / 0.079), but not where the jump
  // lists can share a row between four parts of a workgroup (sectors of up to 90 neutron states, up to 256 proton
  // rows: sd 3+4 0.037 / 0.062, 0.055 / 0.068, 0.049 / 0.069, 0.088 / 0.098), and from 33 bytes on where there are
  // more than 512 proton rows, which they share between two (sd 5+3, FP32, 9 columns: 0.080 / 0.066).
  // L < 11: never (sd 4+5 (10.1) 0.057 / 0.085, 0.169 / 0.127, 0.131 / 0.136, 0.152 / 0.238; sd 6+6 (6.9) 0.125 /
  // 0.178, 0.210 / 0.286, 0.179 / 0.288, 0.332 / 0.574).
  {
    double n1 = 0.0, n2 = 0.0;
    for (auto& v : pairs) {
      n1 += (double)v.size();
      n2 += (double)v.size() * (double)v.size();
    }
    const double L = n2 / n1 * (double)(ns - (m.n_prot - 1)) / ns * (double)(ns - (m.n_neut - 1)) / ns;
    const bool split = m.n_prot > 1 && m.max_dn <= 90 && m.np_total <= 256;
    if ((m.dim < 2500 || L < 11.0 || ((L < 16.0 || m.dim < 5000) && split)) && !T.force) return;
    T.one_tile = !T.force && (L < 16.0 || (m.dim < 5000 && m.n_prot == 1));
    T.min_row = m.np_total > 512 ? 32 : 64;
  }
  std::vector<int> pr_off(nk + 1, 0), pr_xu, hb_off(nk + 1, 0);
  for (int k = 0; k < nk; k++) {
    pr_off[k + 1] = pr_off[k] + (int)pairs[k].size();
    hb_off[k + 1] = hb_off[k] + (int)(pairs[k].size() * pairs[k].size());
    pr_xu.insert(pr_xu.end(), pairs[k].begin(), pairs[k].end());
  }
  std::vector<double> hb(hb_off[nk], 0.0);
  for (const MTerm& t : m.terms_pn) {  // c+_a(p) c+_b(n) c_d(n) c_c(p): target pair (a, b), source pair (c, d)
    const int k = (m.st_tm[t.a] + m.st_tm[t.b] + 2 * tj) / 2;
    const int kc = (m.st_tm[t.c] + m.st_tm[t.d] + 2 * tj) / 2;
    TRBL_REQUIRE(k == kc, TRBL_E_INVALID, "pn term breaks M conservation");
    const int D2 = (int)pairs[k].size();
    hb[hb_off[k] + pid[t.a * ns + t.b] * D2 + pid[t.c * ns + t.d]] += t.h;
  }
  // cores of each species: all (N - 1)-subsets, grouped by (2M, parity)
  struct Group {
    int tm, par, start, count;
  };
  std::vector<Group> groups[2];
  std::vector<uint64_t> cw[2];
  std::vector<int> rk[2];
  std::map<std::pair<int, int>, int> secid[2];
  for (int s = 0; s < 2; s++) {
    const Species& S = m.sp[s];
    for (int q = 0; q < (int)S.sectors.size(); q++) secid[s][{S.sectors[q].twoM, S.sectors[q].par}] = q;
    const int nc = S.npart - 1;
    if (binom(ns, nc) > (1 << 21)) return;
    std::map<std::pair<int, int>, std::vector<uint64_t>> by;
    auto visit = [&](uint64_t w) {
      int tm = 0, ls = 0;
      for (uint64_t x = w; x; x &= x - 1) {
        const int st = __builtin_ctzll(x);
        tm += m.st_tm[st];
        ls += m.orbits[m.st_orb[st]].l;
      }
      by[{tm, (ls & 1) ? -1 : 1}].push_back(w);
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
    for (auto& kv : by) {
      groups[s].push_back({kv.first.first, kv.first.second, (int)cw[s].size(), (int)kv.second.size()});
      for (uint64_t w : kv.second) {
        cw[s].push_back(w);
        for (int st = 0; st < ns; st++) {
          if ((w >> st) & 1) {
            rk[s].push_back(-1);
            continue;
          }
          const auto it = S.index.find(w | (1ull << st));
          if (it == S.index.end()) {  // sector not stored: no block of the space holds it
            rk[s].push_back(-1);
            continue;
          }
          const int q = S.sector_of[it->second];
          const int loc = it->second - S.sectors[q].start;
          TRBL_REQUIRE(loc < (1 << 24), TRBL_E_INVALID, "sector too large for the pair-block tables");
          rk[s].push_back((__builtin_popcountll(w & ((1ull << st) - 1)) << 24) | loc);
        }
      }
    }
  }
  // block of (proton sector, neutron sector)
  const int nnsec = (int)m.sp[1].sectors.size();
  std::vector<int> bos(m.sp[0].sectors.size() * nnsec, -1);
  for (size_t b = 0; b < m.blocks.size(); b++) bos[m.blocks[b].psec * nnsec + m.blocks[b].nsec] = (int)b;
  auto stpar = [&](int st) { return (m.orbits[m.st_orb[st]].l & 1) ? -1 : 1; };
  // rectangles of core groups whose pair block reaches some block of the space
  std::vector<int> rect, rblk;
  std::vector<int> rect_of;  // per (proton group, neutron group): rectangle or -1
  for (const Group& gp : groups[0])
    for (const Group& gn : groups[1]) {
      rect_of.push_back(-1);
      const int tmp = m.twoM - gp.tm - gn.tm;
      if (tmp < -2 * tj || tmp > 2 * tj) continue;
      const int k = (tmp + 2 * tj) / 2;
      bool any = false;
      std::vector<int> pb;
      for (int xu : pairs[k]) {
        const int x = xu & 255, u = xu >> 8;
        auto ip = secid[0].find({gp.tm + m.st_tm[x], gp.par * stpar(x)});
        auto in = secid[1].find({gn.tm + m.st_tm[u], gn.par * stpar(u)});
        const int b = (ip != secid[0].end() && in != secid[1].end()) ? bos[ip->second * nnsec + in->second] : -1;
        pb.push_back(b >= 0 ? b << 1 | (m.sp[1].sectors[in->second].par < 0 ? 1 : 0) : -1);
        any = any || b >= 0;
      }
      if (!any) continue;
      rect_of.back() = (int)(rect.size() / 2);
      rect.insert(rect.end(), {k, (int)rblk.size()});
      rblk.insert(rblk.end(), pb.begin(), pb.end());
    }
  if (rect.empty()) return;
  // V rows and slot rows are counted in 31 and 32 bits
  if ((double)m.dim >= 2147483648.0) return;
  // Slot rows of every proton core: for each x outside it and each neutron sector that completes
  // K_p + x to a block of the space, n_neut rows per neutron state.
  const int nc0 = (int)cw[0].size();
  std::vector<int64_t> crow(nc0, 0);
  std::vector<int> zoff((size_t)nc0 * ns * 2, -1);  // here: the target block
  for (const Group& gp : groups[0])
    for (int cp = gp.start; cp < gp.start + gp.count; cp++)
      for (int x = 0; x < ns; x++) {
        if (rk[0][(size_t)cp * ns + x] < 0) continue;
        const auto ip = secid[0].find({gp.tm + m.st_tm[x], gp.par * stpar(x)});
        if (ip == secid[0].end()) continue;
        for (int q = 0; q < nnsec; q++) {
          const int b = bos[ip->second * nnsec + q];
          if (b < 0) continue;
          zoff[((size_t)cp * ns + x) * 2 + (m.sp[1].sectors[q].par < 0 ? 1 : 0)] = b;
          crow[cp] += (int64_t)m.n_neut * m.blocks[b].dn;
        }
      }
  // Batches: a single one while the slots of all cores stay below 4 GiB (128-byte rows) and a quarter of
  // the free memory, else runs of proton cores of at most 4 Mi rows, two buffers of 512 MiB (pf 6+6,
  // FP32 at 32 columns: 645 ms; 1 Mi rows 756, 2 Mi 658, 8 Mi 646, 32 Mi 614 to 634 ms, at 8 GB).
  // TRBL_PN_BATCH: the most slot rows of a batch (a testing and tuning override).
  size_t fr = 0, tot = 0;
  TRBL_HIP(hipMemGetInfo(&fr, &tot));
  int64_t all = 0, cap = 1 << 22;
  for (int64_t r : crow) all += r;
  if (all * 128 <= (int64_t)std::min<size_t>(NO_ROW, fr / 4)) cap = all;
  if (const char* ev = std::getenv("TRBL_PN_BATCH")) cap = std::max(1ll, std::atoll(ev));
  for (int64_t r : crow) cap = std::max(cap, r);
  if (cap * 128 > (int64_t)NO_ROW) return;  // slot byte offsets in 32 bits
  std::vector<int> bat0(1, 0);
  int64_t run = 0, most = 0;
  for (int cp = 0; cp < nc0; cp++) {
    if (run + crow[cp] > cap) {
      bat0.push_back(cp);
      run = 0;
    }
    run += crow[cp];
    most = std::max(most, run);
  }
  bat0.push_back(nc0);
  const int nbat = (int)bat0.size() - 1;
  // one batch: the slots of all targets lie one position pair after the other, [x][u][target]
  T.zstep = nbat == 1 ? (int)m.dim : 0;
  // Work items: per fixed core, the cores of one group of the other species that make a rectangle with it, up to
  // `chunk` at a time. An item's set-up, and the lanes of a matrix instruction that the cores share, pay for
  // runs of some cores, so with one batch the items run over the protons where they would hold fewer than 4
  // neutron cores on average and the proton runs are longer (ms, over neutrons / protons, FP64 8 and 32 columns: pf
  // 4+2 0.148 / 0.099, 0.408 / 0.306; pf 5+1 0.175 / 0.139, 0.280 / 0.203; pf 3+2 0.068 / 0.064, 0.141 / 0.124; the
  // other way round pf 2+4 0.106 / 0.169, 0.288 / 0.391). TRBL_PN_RUN=p or n: a testing override.
  auto count_items = [&](bool sw, int ch) {
    int64_t n = 0;
    for (size_t ip = 0; ip < groups[0].size(); ip++)
      for (size_t in = 0; in < groups[1].size(); in++)
        if (rect_of[ip * groups[1].size() + in] >= 0) {
          const int np = groups[0][ip].count, nn = groups[1][in].count;
          n += (int64_t)(sw ? nn : np) * (((sw ? np : nn) + ch - 1) / ch);
        }
    return n;
  };
  T.swap = nbat == 1 && count_items(false, 1) < 4 * count_items(false, PN_TPB) &&
           count_items(true, PN_TPB) < count_items(false, PN_TPB);
  if (const char* ev = std::getenv("TRBL_PN_RUN")) T.swap = ev[0] == 'p' && nbat == 1;
  // One batch: as many as 256 cores an item while that makes 768 items, three for a CU, else fewer, down to 8 (two
  // cores a wavefront; FP64 8 and 32 columns, 256 / 8 cores: pf 1+4 0.107 / 0.068, 0.272 / 0.113; pf 1+5 0.254 /
  // 0.189, 0.495 / 0.233; with 32 cores pf 2+4 0.126 / 0.106, 0.358 / 0.288). The fixed cores of a group go in runs of 16
  // consecutive (colex) ones, one chunk after the other, so that the items in flight on an XCD, which
  // takes a contiguous range of them, share source rows in its L2. Several batches: 64 cores and
  // one fixed core after the other, so that a batch has enough items for the chip (pf 6+6: 645 against 696 ms).
  // TRBL_PN_CHUNK: a tuning override.
  int chunk = nbat == 1 ? PN_TPB : 64;
  while (nbat == 1 && chunk > 8 && count_items(T.swap, chunk) < 768) chunk /= 2;
  if (const char* ev = std::getenv("TRBL_PN_CHUNK")) chunk = std::max(8, std::min(PN_TPB, std::atoi(ev)));
  const int core_run = nbat == 1 ? 16 : 1;
  const std::vector<Group>&gf = groups[T.swap ? 1 : 0], &gr = groups[T.swap ? 0 : 1];
  const int nfix = (int)cw[T.swap ? 1 : 0].size();
  std::vector<int> group_of(nfix);
  for (int g = 0; g < (int)gf.size(); g++)
    for (int c = gf[g].start; c < gf[g].start + gf[g].count; c++) group_of[c] = g;
  std::vector<int64_t> blk_row0(m.blocks.size() + 1, 0);
  for (size_t b = 0; b < m.blocks.size(); b++) blk_row0[b + 1] = blk_row0[b] + m.blocks[b].dp;
  TRBL_REQUIRE(blk_row0.back() < ((int64_t)1 << 31), TRBL_E_INVALID, "too many proton rows");
  const int ngn = (int)groups[1].size();
  std::vector<int> items, tent;
  std::vector<PNRow> trow;
  for (int ib = 0; ib < nbat; ib++) {
    PNTiles::Batch B{};
    B.item0 = (int)(items.size() / 4);
    B.row0 = (int)trow.size();
    for (int t0 = bat0[ib], te = nbat == 1 ? nfix : bat0[ib + 1]; t0 < te;) {
      const int g = group_of[t0];
      const int t1 = std::min(std::min(te, gf[g].start + gf[g].count), t0 + core_run);
      for (int ir = 0; ir < (int)gr.size(); ir++) {
        const int r = T.swap ? rect_of[ir * ngn + g] : rect_of[g * ngn + ir];
        if (r < 0) continue;
        for (int c0 = 0; c0 < gr[ir].count; c0 += chunk)
          for (int cf = t0; cf < t1; cf++)
            items.insert(items.end(), {r, cf, gr[ir].start + c0, std::min(chunk, gr[ir].count - c0)});
      }
      t0 = t1;
    }
    if (nbat > 1) {  // the costliest items first: a batch is a few items per workgroup slot
      std::vector<std::pair<int64_t, std::array<int, 4>>> by_cost;
      for (size_t i = 4 * (size_t)B.item0; i < items.size(); i += 4) {
        const int k = rect[2 * items[i]], rb0 = rect[2 * items[i] + 1];
        int d = 0;
        for (size_t e = 0; e < pairs[k].size(); e++)
          d += rblk[rb0 + e] >= 0 && rk[0][(size_t)items[i + 1] * ns + (pairs[k][e] & 255)] >= 0;
        const int ks = (d + 7) / 8 * 2;
        by_cost.push_back({-(int64_t)items[i + 3] * (400 + 64 * ks * ((ks + 3) / 4)),
                           {items[i], items[i + 1], items[i + 2], items[i + 3]}});
      }
      std::stable_sort(by_cost.begin(), by_cost.end(), [](const auto& x, const auto& y) { return x.first < y.first; });
      for (size_t i = 0; i < by_cost.size(); i++)
        for (int q = 0; q < 4; q++) items[4 * ((size_t)B.item0 + i) + q] = by_cost[i].second[q];
    }
    if (nbat > 1) {  // slot rows and target rows of the batch
      std::map<int64_t, std::vector<int>> to;  // target row (block row0 + proton row) -> first slot rows
      int64_t at = 0;
      for (int cp = bat0[ib]; cp < bat0[ib + 1]; cp++)
        for (int x = 0; x < ns; x++)
          for (int q = 0; q < 2; q++) {
            int& z = zoff[((size_t)cp * ns + x) * 2 + q];
            if (z < 0) continue;
            const int b = z, pl = rk[0][(size_t)cp * ns + x] & 0xFFFFFF;
            z = (int)at;
            to[blk_row0[b] + pl].push_back(z);
            at += (int64_t)m.n_neut * m.blocks[b].dn;
          }
      size_t b = 0;
      for (auto& kv : to) {
        while (kv.first >= blk_row0[b + 1]) b++;
        const int dn = m.blocks[b].dn;
        trow.push_back({m.blocks[b].off + (kv.first - blk_row0[b]) * dn, dn, (int)tent.size(), (int)kv.second.size(), 0});
        tent.insert(tent.end(), kv.second.begin(), kv.second.end());
        B.maxdn = std::max(B.maxdn, dn);
      }
    }
    B.nitems = (int)(items.size() / 4) - B.item0;
    B.nrows = (int)trow.size() - B.row0;
    const int64_t nred = (int64_t)B.nrows * ((B.maxdn + RED_ROWS - 1) / RED_ROWS);  // reducing workgroups
    TRBL_REQUIRE(B.nitems < (1 << 22) && nred < (1 << 22), TRBL_E_INVALID, "too many core pairs for one launch");
    if (B.nitems > 0) T.batches.push_back(B);
  }
  TRBL_REQUIRE(items.size() < ((size_t)1 << 31), TRBL_E_INVALID, "too many core pairs");
  T.nbuf = T.batches.size() > 1 ? 2 : 1;
  T.buf_rows = most;
  const size_t zbytes = (size_t)T.nbuf * (size_t)most * 128;
  if (zbytes > fr / 4) return;
  T.max_pairs = maxp;
  T.rk[0].upload(rk[0]);
  T.rk[1].upload(rk[1]);
  T.pr_off.upload(pr_off);
  T.pr_xu.upload(pr_xu);
  T.hb_off.upload(hb_off);
  T.hb.upload(hb);
  std::vector<float> hb32(hb.begin(), hb.end());
  T.hb32.upload(hb32);
  T.rect.upload(rect);
  T.rblk.upload(rblk);
  T.items.upload(items);
  T.zoff.upload(zoff);
  T.trow.upload(trow);
  T.tent.upload(tent);
  std::vector<int> boff32(m.blocks.size());
  for (size_t b = 0; b < m.blocks.size(); b++) boff32[b] = (int)m.blocks[b].off;
  T.boff.upload(boff32);
  T.z.alloc(zbytes);
  if (!T.side) TRBL_HIP(hipStreamCreateWithFlags(&T.side, hipStreamNonBlocking));
  for (auto& e : T.ev)
    if (!e) TRBL_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  T.on = true;
}

template <class T, int VPL, int KN>
static void run_batches(const Model& m, PNTileArgs<T>& a, bool big, bool reduce, hipStream_t s) {
  const PNTiles& P = m.pn;
  const int ks = (P.max_pairs + 7) / 8 * 2;
  const size_t shm = (size_t)((ks + 3) / 4 * ks) * 64 * sizeof(T);
  const int4* items = P.items.as<int4>();
  const PNRow* rows = P.trow.as<PNRow>();
  const int64_t bytes = P.buf_rows * a.cpr * 16;
  a.zbytes = (unsigned)bytes;
  char* const z = P.z.as<char>();
  const int n = (int)P.batches.size();
  for (int i = 0; i < n + (reduce ? 1 : 0); i++) {
    a.nred = a.nitems = 0;
    if (n == 1 && i == 1) {
      a.Zr = reinterpret_cast<const T*>(z);
      hipLaunchKernelGGL(pn_sum_kernel<T>, dim3(elementwise_grid(m.dim * a.cprv)), dim3(256), 0, s, a, (int)m.dim,
                         m.n_prot * m.n_neut);
      break;
    }
    if (i > 0) {
      const PNTiles::Batch& R = P.batches[i - 1];
      a.nchunk = (R.maxdn + RED_ROWS - 1) / RED_ROWS;
      a.nrows = R.nrows;
      a.nred = (int)(((int64_t)R.nrows * a.nchunk + 7) / 8 * 8);
      a.rows = rows + R.row0;
      a.Zr = reinterpret_cast<const T*>(z + (size_t)((i - 1) % P.nbuf) * bytes);
    }
    if (i < n) {
      const PNTiles::Batch& B = P.batches[i];
      a.items = items + B.item0;
      a.nitems = B.nitems;
      a.Z = reinterpret_cast<T*>(z + (size_t)(i % P.nbuf) * bytes);
    }
    const dim3 grid((unsigned)(a.nred + (a.nitems + 7) / 8 * 8));
    if (big) hipLaunchKernelGGL((pn_tile_kernel<T, VPL, KN, true>), grid, dim3(256), i < n ? shm : 0, s, a);
    else hipLaunchKernelGGL((pn_tile_kernel<T, VPL, KN, false>), grid, dim3(256), i < n ? shm : 0, s, a);
  }
}

// 16-byte chunks of a slot row: those with valid columns, and as laid out (a power of two, so that whole
// lines are written)
int pn_slot_chunks(size_t elt, int cols) { return (cols * (int)elt + 15) / 16; }
int pn_slot_stride(size_t elt, int cols) {
  int p = 1;
  while (p < pn_slot_chunks(elt, cols)) p <<= 1;
  return p;
}

template <class T>
void launch_pn_tiles(const Model& m, int nb, const T* V, int64_t ldv, T* W, int64_t ldw, hipStream_t s, bool reduce) {
  constexpr int VPC = 16 / (int)sizeof(T), WIDE = 128 / (int)sizeof(T);  // values per lane, most columns at once
  const PNTiles& P = m.pn;
  PNTileArgs<T> a{};
  a.V = V;
  a.W = W;
  a.ldw = ldw;
  a.ns = m.ns;
  a.nneut = m.n_neut;
  a.vrow = ldv * (int64_t)sizeof(T);
  a.swap = P.swap;
  a.rkf = P.rk[P.swap ? 1 : 0].as<int>();
  a.rkr = P.rk[P.swap ? 0 : 1].as<int>();
  a.blk_off = P.boff.as<int>();
  a.blk_dn = m.dt.blk_dn.as<int>();
  a.pr_off = P.pr_off.as<int>();
  a.pr_xu = P.pr_xu.as<int>();
  a.hb_off = P.hb_off.as<int>();
  a.hb = (sizeof(T) == 8 ? P.hb : P.hb32).as<T>();
  a.rect = P.rect.as<int>();
  a.rblk = P.rblk.as<int>();
  a.zoff = P.zoff.as<int>();
  a.zstep = P.zstep;
  a.spread = P.batches.size() > 1;
  a.tent = P.tent.as<int>();
  // (row steps between states of the run are multiplied in 24 bits)
  const bool big = (double)m.dim * (double)a.vrow > (double)NO_ROW ||
                   (double)a.vrow * (P.swap ? m.max_dn : 1) >= (double)(1 << 25);
  for (int c0 = 0; c0 < nb; c0 += WIDE) {
    a.c0 = c0;
    a.cval = std::min(WIDE, nb - c0);
    a.vbytes = big ? 0u : (unsigned)(m.dim * a.vrow - c0 * (int64_t)sizeof(T));
    a.wvec = (uintptr_t)(W + c0) % 16 == 0 && (ldw * (int64_t)sizeof(T)) % 16 == 0;
    // neutron cores that share the 16 columns of a matrix instruction
    a.cprv = pn_slot_chunks(sizeof(T), a.cval);
    a.cpr = pn_slot_stride(sizeof(T), a.cval);
    if (a.cval < VPC) {
      a.lr = VPC;  // one value a lane
      run_batches<T, 1, 16 / VPC>(m, a, big, reduce, s);
      continue;
    }
    a.lr = a.cpr;
    if (a.lr <= 2) run_batches<T, VPC, 8>(m, a, big, reduce, s);
    else if (a.lr <= 4) run_batches<T, VPC, 4>(m, a, big, reduce, s);
    else run_batches<T, VPC, 2>(m, a, big, reduce, s);
  }
  TRBL_HIP(hipGetLastError());
}
template void launch_pn_tiles<double>(const Model&, int, const double*, int64_t, double*, int64_t, hipStream_t, bool);
template void launch_pn_tiles<float>(const Model&, int, const float*, int64_t, float*, int64_t, hipStream_t, bool);

}  // namespace trbl
