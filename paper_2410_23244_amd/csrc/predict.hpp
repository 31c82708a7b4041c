// predict.hpp -- sum-of-trees prediction f(x) = offset + sum_j g(x; T_j, M_j)
// (eq. bartdef) at many points, on gfx950.
//
// Algorithm 1 follows every point through every level of every tree, which
// costs a table read and a byte gather per level and point.  Here the trees
// are compiled first, once per call (k_pred_program): the reachable internal
// nodes of a tree in heap order, and the leaf value of every combination of
// their decisions.  A point's leaf value is then a table read at the number
// whose bits are the decisions "x >= cut", and because the nodes are the same
// for all lanes, a decision for 4 points costs one coalesced word of the
// node's predictor row, and a compare and an add-with-carry per point (the
// visited nodes' decisions are those of Algorithm 1; the others do not change
// the table's value).  Trees of more than 6 nodes use bit masks of the leaves
// that each decision leaves (the QuickScorer method of Lucchese et al., SIGIR
// 2015), the largest Algorithm 1.
#pragma once
#include "common.hpp"

namespace bart {

constexpr int kPredTrees = 16;      // trees per group of the compiled program
constexpr int kPredTabNodes = 6;    // most internal nodes of a tree with a decision table
constexpr int kPredTab = 1 << kPredTabNodes;
constexpr int kPredListNodes = 31;  // most internal nodes of a tree with a leaf bit mask
constexpr int kPredBatch = 8;       // nodes whose predictor words are in flight together
constexpr int kPredTile = 256;      // points per tile: 4 per lane
constexpr uint32_t kPredNop = 256u << 16;  // a decision no byte takes
constexpr int kPredList = kPredTrees * kPredListNodes;  // nodes of a group's trees with a mask
static_assert(kPredList % kPredBatch == 0 && kPredTrees * kPredTabNodes % kPredBatch == 0,
              "whole batches");

// One group of the program: batches of kPredBatch nodes, filled up with
// kPredNop.  A node: axis, cut << 16 (9 bits), bit 25 the tree's last node, the
// tree's place in the group << 26.
struct alignas(16) PredGroup {
  uint32_t nbatch;    // batches of trees with a decision table, at least 1
  uint32_t nlist;     // batches of trees with a leaf mask
  uint32_t nspecial;  // trees of more nodes
  uint32_t pad[13];
  // trees of up to kPredTabNodes nodes (a tree without a node gets one that
  // decides nothing)
  uint32_t node[kPredTrees * kPredTabNodes];
  // trees of up to kPredListNodes nodes, and the leaves outside a node's left
  // subtree (bit k: k-th leaf from the left)
  uint32_t list[kPredList], keep[kPredList];
  uint32_t special[kPredTrees];  // place in the group of a tree for Algorithm 1
  // leaf value by decisions (the first node's the highest bit), or by leaf
  // from the left
  float tab[kPredTrees][kPredTab];
};

// The program of one chain (blockIdx.y), a group per block and a tree per
// wave: lane l holds heap slots l and l + 64.
__global__ void __launch_bounds__(64 * kPredTrees)
    k_pred_program(const uint16_t *axis0, const uint8_t *cut0, const float *leaf0, PredGroup *prog0,
                   int m, int p, int D, int H, size_t chain_bytes) {
  __shared__ int s_nodes[kPredTrees], s_list[kPredTrees], s_special[kPredTrees];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const size_t cb = blockIdx.y * chain_bytes;
  const int j = blockIdx.x * kPredTrees + w;
  const bool live = j < m;
  const int64_t row = (int64_t)(live ? j : 0);
  const uint16_t *ax = (const uint16_t *)((const char *)axis0 + cb) + row * H;
  const uint8_t *ct = cut0 + cb + row * H;
  const float *lf = (const float *)((const char *)leaf0 + cb) + row * 2 * H;
  PredGroup &P = ((PredGroup *)((char *)prog0 + cb))[blockIdx.x];

  int c[2], a[2];
  uint64_t im[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int h = l + 64 * r;
    const bool in = live && h >= 1 && h < H;
    c[r] = in ? ct[h] : 0;
    a[r] = in ? ax[h] : 0;
    if (a[r] >= p) a[r] = 0;
  }
  // internal nodes: a cut at the node and at each of its ancestors
  {
    const uint64_t raw[2] = {__ballot(c[0] != 0), __ballot(c[1] != 0)};
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      bool ok = c[r] != 0;
#pragma unroll
      for (int s = 1; s < 7; ++s) {
        const int q = (l + 64 * r) >> s;
        ok = ok && (q == 0 || ((raw[q >> 6] >> (q & 63)) & 1ull));
      }
      im[r] = __ballot(ok);
    }
  }
  const int n = __popcll(im[0]) + __popcll(im[1]);
  auto inner = [&](int h) { return h < H && (((h < 64 ? im[0] : im[1]) >> (h & 63)) & 1ull); };
  auto below = [](const uint64_t (&b)[2], int k) {  // bits of b below bit k < 128
    return k < 64 ? __popcll(b[0] & ((1ull << k) - 1ull))
                  : __popcll(b[0]) + __popcll(b[1] & ((1ull << (k - 64)) - 1ull));
  };
  const bool table = n <= kPredTabNodes, list = !table && n <= kPredListNodes;
  if (l == 0) {
    s_nodes[w] = live && table ? (n > 0 ? n : 1) : 0;
    s_list[w] = live && list ? n : 0;
    s_special[w] = live && !table && !list;
  }
  __syncthreads();
  int first = 0, total = 0, lfirst = 0, ltotal = 0, sfirst = 0, stotal = 0;
  for (int q = 0; q < kPredTrees; ++q) {
    if (q == w) first = total, lfirst = ltotal, sfirst = stotal;
    total += s_nodes[q];
    ltotal += s_list[q];
    stotal += s_special[q];
  }
  const int nbatch = total > 0 ? (total + kPredBatch - 1) / kPredBatch : 1;
  const int nlist = (ltotal + kPredBatch - 1) / kPredBatch;
  if (threadIdx.x == 0) {
    P.nbatch = (uint32_t)nbatch;
    P.nlist = (uint32_t)nlist;
    P.nspecial = (uint32_t)stotal;
  }
  if (w == 0 && total + l < nbatch * kPredBatch) P.node[total + l] = kPredNop;
  if (w == 0 && ltotal + l < nlist * kPredBatch) {
    P.list[ltotal + l] = kPredNop;
    P.keep[ltotal + l] = ~0u;
  }
  if (!live) return;
  if (table) {
    const uint32_t tag = (uint32_t)w << 26;
    if (n == 0 && l == 0) P.node[first] = kPredNop | 1u << 25 | tag;
#pragma unroll
    for (int r = 0; r < 2; ++r)
      if ((im[r] >> l) & 1ull) {
        const int k = below(im, l + 64 * r);
        P.node[first + k] = (uint32_t)a[r] | (uint32_t)c[r] << 16 | (k == n - 1 ? 1u << 25 : 0u) | tag;
      }
    // lane l: the leaf that decisions l reach
    int h = 1;
    for (int lvl = 1; lvl < D; ++lvl)
      if (inner(h)) h = 2 * h + ((l >> (n - 1 - below(im, h))) & 1);
    if (l < 1 << n) P.tab[w][l] = lf[h];
    return;
  }
  if (!list) {
    if (l == 0) P.special[sfirst] = (uint32_t)w;
    return;
  }
  // leaves from the left: bottom position k (of H) starts a leaf if the leaf
  // above it begins there
  uint64_t start[2];
  int leaf_of[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int k = l + 64 * r;
    int h = 1, d = 0;
    for (int lvl = 1; lvl < D; ++lvl)
      if (inner(h)) {
        h = 2 * h + ((k >> (D - 2 - d)) & 1);
        ++d;
      }
    leaf_of[r] = h;
    start[r] = __ballot(k < H && (k & ((1 << (D - 1 - d)) - 1)) == 0);
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int h = l + 64 * r;
    if ((start[r] >> l) & 1ull) P.tab[w][below(start, h)] = lf[leaf_of[r]];
    if ((im[r] >> l) & 1ull) {
      const int d = 31 - __clz(h), half = 1 << (D - 2 - d);
      const int pos = (h << (D - 1 - d)) - H;  // its first bottom position; pos + half < H
      const uint32_t left = (1u << below(start, pos + half)) - (1u << below(start, pos));
      const int k = below(im, h);
      P.list[lfirst + k] = (uint32_t)a[r] | (uint32_t)c[r] << 16 | (k == n - 1 ? 1u << 25 : 0u) |
                           (uint32_t)w << 26;
      P.keep[lfirst + k] = ~left;
    }
  }
}

// One decision of 4 points: code = 2 code + (byte >= cut) each, as a byte
// compare and an add with carry (from C++ a third instruction selects 0 or 1
// first).  The compares come together: a lane mask written by a vector
// instruction may be read by one three instructions later at the earliest.
__device__ __forceinline__ void pred_decide4(uint32_t (&code)[4], uint32_t x, uint32_t cut) {
  uint64_t m0, m1, m2, m3;
  asm("v_cmp_ge_u32_sdwa %4, %8, %9 src0_sel:BYTE_0 src1_sel:DWORD\n\t"
      "v_cmp_ge_u32_sdwa %5, %8, %9 src0_sel:BYTE_1 src1_sel:DWORD\n\t"
      "v_cmp_ge_u32_sdwa %6, %8, %9 src0_sel:BYTE_2 src1_sel:DWORD\n\t"
      "v_cmp_ge_u32_sdwa %7, %8, %9 src0_sel:BYTE_3 src1_sel:DWORD\n\t"
      "v_addc_co_u32_e64 %0, %4, %0, %0, %4\n\t"
      "v_addc_co_u32_e64 %1, %5, %1, %1, %5\n\t"
      "v_addc_co_u32_e64 %2, %6, %2, %2, %6\n\t"
      "v_addc_co_u32_e64 %3, %7, %3, %3, %7"
      : "+v"(code[0]), "+v"(code[1]), "+v"(code[2]), "+v"(code[3]), "=&s"(m0), "=&s"(m1),
        "=&s"(m2), "=&s"(m3)
      : "v"(x), "s"(cut));
}

// The same for a tree with a leaf mask: code &= keep where byte >= cut.
__device__ __forceinline__ void pred_mask4(uint32_t (&code)[4], uint32_t x, uint32_t cut,
                                           uint32_t keep) {
  uint64_t m0, m1, m2, m3;
  uint32_t t;
  asm("v_cmp_ge_u32_sdwa %5, %9, %10 src0_sel:BYTE_0 src1_sel:DWORD\n\t"
      "v_cmp_ge_u32_sdwa %6, %9, %10 src0_sel:BYTE_1 src1_sel:DWORD\n\t"
      "v_cmp_ge_u32_sdwa %7, %9, %10 src0_sel:BYTE_2 src1_sel:DWORD\n\t"
      "v_cmp_ge_u32_sdwa %8, %9, %10 src0_sel:BYTE_3 src1_sel:DWORD\n\t"
      "v_cndmask_b32_e64 %4, -1, %11, %5\n\t"
      "v_and_b32_e32 %0, %4, %0\n\t"
      "v_cndmask_b32_e64 %4, -1, %11, %6\n\t"
      "v_and_b32_e32 %1, %4, %1\n\t"
      "v_cndmask_b32_e64 %4, -1, %11, %7\n\t"
      "v_and_b32_e32 %2, %4, %2\n\t"
      "v_cndmask_b32_e64 %4, -1, %11, %8\n\t"
      "v_and_b32_e32 %3, %4, %3"
      : "+v"(code[0]), "+v"(code[1]), "+v"(code[2]), "+v"(code[3]), "=&v"(t), "=&s"(m0),
        "=&s"(m1), "=&s"(m2), "=&s"(m3)
      : "v"(x), "s"(cut), "v"(keep));
}

// The compiled trees at a tile of 64 x 4 points per wave: lane l's word holds
// the 4 points at 4 (64 tile + l).  split = 1: every wave has a tile of its
// own.  Else the waves of a block share one tile and the groups of trees, in
// order, among them.  The groups are cut into `ranges` ranges, a power of two
// that the number of groups fixes (pred_ranges), `per_wave` of them for each
// of the waves; a range is summed in fp64 in
// order, and the ranges by a binary tree, of which a wave makes the part over
// its own: the split, which is chosen by the number of points and chains,
// changes no bit of a sum.  blockIdx.y = chain.  ACC: add f and f^2 (fp64) to sum and sumsq instead of
// writing fp32(f) to out.  What bounds it is the issue of the decisions, two
// instructions each per point, then the words' loads: 1e6 points, 200 trees of
// the branching prior, 402 us by Algorithm 1 for every tree, 104 us here (a
// call, with the program).  Trees of 7 to 31 nodes cost three instructions per
// node and point, larger ones a gather per level and point; both wait until the
// stream of the others is done, so that their registers are not held beside
// it (105 of them instead of 79, a wave per SIMD less).  100 trees, every node
// split with probability 0.85 / 1, against Algorithm 1 for every tree (8 trees
// of a point in flight per thread): 1e5 points, depth 6 135 / 145 us, now 72 /
// 124, depth 8 217 / 231, now 136 / 173; 1e6 points, depth 6 265 / 353, now 214
// / 371, depth 8 416 / 593, now 460 / 623 (one node's word at a time and the
// trees read from memory at every level, before: 852 for complete trees of depth 6,
// 1,801 of depth 8).
constexpr int kPredRanges = 16;  // most ranges, and most waves that share a tile
constexpr int pred_ranges(int ngroups) {
  int r = 1;
  while (r < kPredRanges && 2 * r <= ngroups) r *= 2;
  return r;
}
// LDS of a wave with 1 or 2 ranges: the tables of a group (its fp64 sums in
// their place at the end), and the sums of the first of two
constexpr int kPredSums = kPredTile * sizeof(double);
__host__ __device__ constexpr int pred_wave_lds(int per_wave) {
  return kPredTrees * kPredTab * (int)sizeof(float) + (per_wave > 1 ? kPredSums : 0);
}

typedef uint32_t u32_any __attribute__((aligned(1)));  // Xt has no alignment of its own
template <class T>
using cptr = const __attribute__((address_space(4))) T *;  // scalar loads

// (at most 80 VGPRs, 6 waves per SIMD: three blocks of 8 waves on a compute unit,
// not two; without ACC the compiler gets there by itself, and asked for it made
// code 2 % slower)
template <bool ACC>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(ACC ? 6 : 4)))
    k_pred_eval(const uint8_t *Xt, int64_t ldx, int64_t nt, int p, const PredGroup *prog0,
                const uint16_t *axis0, const uint8_t *cut0, const float *leaf0, int ngroups, int D,
                int H, double offset, size_t chain_bytes, int split, int per_wave, int lg_ranges,
                float *out0, double *sum0, double *sumsq0) {
  extern __shared__ __align__(16) char s_raw[];
  static_assert(kPredTrees * kPredTab * sizeof(float) >= kPredSums,
                "the partial sums reuse the tables");
  const int wave_lds = pred_wave_lds(per_wave);
  const int l = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nw = (int)blockDim.x >> 6;
  float *const tab = (float *)(s_raw + w * wave_lds);
  double *const held = (double *)(tab + kPredTrees * kPredTab);  // [4][64]
  const size_t cb = blockIdx.y * chain_bytes;
  const char *prog = (const char *)prog0 + cb;
  const int64_t tiles = (nt + kPredTile - 1) / kPredTile;
  const int64_t step = (int64_t)gridDim.x * (split > 1 ? 1 : nw);
  const int r0 = split > 1 ? w * per_wave : 0;  // its first range
  auto range_start = [&](int r) { return (int)((uint32_t)ngroups * (uint32_t)r >> lg_ranges); };
  const int g0 = range_start(r0), g1 = range_start(r0 + per_wave);
  const int mid = per_wave > 1 ? range_start(r0 + 1) : -1;  // start of its second range

  for (int64_t tile = split > 1 ? blockIdx.x : (int64_t)blockIdx.x * nw + w; tile < tiles;
       tile += step) {
    // byte offset of this lane's word in a predictor row (the first word
    // stands in past the last point)
    const int64_t base = kPredTile * tile;
    const int64_t at = base + 4 * l;
    uint32_t vo = at < nt ? (uint32_t)(4 * l) : 0u;
    const uint8_t *X = Xt + base;
    double acc[4];
    float pend[4];  // leaf values read but not yet added
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = 0.0, pend[b] = 0.f;

    struct Batch {
      uint32_t node[kPredBatch];
      uint32_t x[kPredBatch];
    };
    auto group = [&](int g) {
      return (cptr<PredGroup>)(prog + (size_t)g * sizeof(PredGroup));
    };
    auto fetch = [&](int g, int b, Batch &B) {
      const cptr<PredGroup> G = group(g);
#pragma unroll
      for (int e = 0; e < kPredBatch; ++e) B.node[e] = G->node[b * kPredBatch + e];
#pragma unroll
      for (int e = 0; e < kPredBatch; ++e) {
        // (a 32-bit lane offset from a uniform row, kept that way)
        asm volatile("" : "+v"(vo));
        const gptr<const uint8_t> xr = gbl(X) + (int64_t)(B.node[e] & 0xffffu) * ldx;
        B.x[e] = *(gptr<const u32_any>)(xr + vo);
      }
    };
    uint32_t code[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) code[b] = 0;
    auto process = [&](const Batch &B) {
#pragma unroll
      for (int e = 0; e < kPredBatch; ++e) {
        const uint32_t node = B.node[e];
        const uint32_t cut = (node >> 16) & 0x1ffu;
        pred_decide4(code, B.x[e], cut);
        if ((node >> 25) & 1u) {  // uniform
          const float *tt = tab + (node >> 26) * kPredTab;
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            acc[b] += (double)pend[b];
            pend[b] = tt[code[b]];
            code[b] = 0;
          }
        }
      }
    };
    // trees of more nodes, by leaf masks: every node clears the leaves of its
    // left subtree for a point that goes right; the leaf is the leftmost one
    // left.  The next batch is in flight, as above
    auto masks = [&](int g) {
      const cptr<PredGroup> G = group(g);
      const int nl = (int)G->nlist;
      const float *const values = (const float *)(prog + (size_t)g * sizeof(PredGroup) +
                                                  offsetof(PredGroup, tab));
      auto fetch_list = [&](int b, Batch &B) {
#pragma unroll
        for (int e = 0; e < kPredBatch; ++e) B.node[e] = G->list[b * kPredBatch + e];
#pragma unroll
        for (int e = 0; e < kPredBatch; ++e) {
          asm volatile("" : "+v"(vo));
          const gptr<const uint8_t> xr = gbl(X) + (int64_t)(B.node[e] & 0xffffu) * ldx;
          B.x[e] = *(gptr<const u32_any>)(xr + vo);
        }
      };
#pragma unroll
      for (int b = 0; b < 4; ++b) code[b] = ~0u;
      auto apply = [&](int k, const Batch &B) {
        uint32_t keep[kPredBatch];
#pragma unroll
        for (int e = 0; e < kPredBatch; ++e) keep[e] = G->keep[k * kPredBatch + e];
#pragma unroll
        for (int e = 0; e < kPredBatch; ++e) {
          const uint32_t node = B.node[e];
          pred_mask4(code, B.x[e], (node >> 16) & 0x1ffu, keep[e]);
          if ((node >> 25) & 1u) {  // uniform
            const gptr<const float> tt = gbl(values) + (node >> 26) * kPredTab;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              acc[b] += (double)pend[b];
              pend[b] = tt[__ffs((int)code[b]) - 1];
              code[b] = ~0u;
            }
          }
        }
      };
      if (nl > 0) {
        Batch C0, C1;
        fetch_list(0, C0);
#pragma unroll 1
        for (int k = 0; k < nl; k += 2) {
          fetch_list(min(k + 1, nl - 1), C1);
          apply(k, C0);
          if (k + 1 < nl) {
            fetch_list(min(k + 2, nl - 1), C0);
            apply(k + 1, C1);
          }
        }
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        acc[b] += (double)pend[b];
        pend[b] = 0.f;
      }
    };
    // trees of more nodes, by Algorithm 1, two at a time: their nodes (the
    // offset of the predictor row, 56 bits, and the cut above; 0 at a leaf) and
    // leaf values in LDS in place of the tables, which are done with.
    // One LDS read and one byte gather per level and point; the loads of 8
    // descents are in flight together.
    auto special = [&](int g) {
      const cptr<PredGroup> G = group(g);
      const int ns = (int)G->nspecial;
      static_assert(2 * 4 * 128 <= kPredTrees * kPredTab, "two trees of depth 8 in the tables");
#pragma unroll 1
      for (int q = 0; q < ns; q += 2) {
        const bool both = q + 1 < ns;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int64_t j = (int64_t)g * kPredTrees + (int)G->special[u && both ? q + 1 : q];
          const gptr<const uint16_t> ax = gbl((const uint16_t *)((const char *)axis0 + cb)) + j * H;
          const gptr<const uint8_t> ct = gbl(cut0 + cb) + j * H;
          const gptr<const float> lf = gbl((const float *)((const char *)leaf0 + cb)) + j * 2 * H;
          float *const t = tab + u * 4 * H;
          int ll = l;  // opaque: else the lane's addresses are kept over the whole tile loop
          asm volatile("" : "+v"(ll));
#pragma unroll 1
          for (int k = ll; k < H; k += 64) {
            const uint32_t cv = ct[k], a = ax[k];
            const uint64_t off = cv && a < (uint32_t)p ? (uint64_t)a * (uint64_t)ldx : 0u;
            t[2 * k] = __uint_as_float((uint32_t)off);
            t[2 * k + 1] = __uint_as_float((uint32_t)(off >> 32) | cv << 24);
          }
#pragma unroll 1
          for (int k = ll; k < 2 * H; k += 64) t[2 * H + k] = lf[k];
        }
        int h[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int b = 0; b < 4; ++b) h[u][b] = 1;
#pragma unroll 1
        for (int lvl = 1; lvl < D; ++lvl) {  // (an internal slot until the last level: below H)
          uint32_t cv[2][4], xv[2][4];
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              const float *t = tab + u * 4 * H + 2 * h[u][b];
              const uint32_t lo = __float_as_uint(t[0]), hi = __float_as_uint(t[1]);
              cv[u][b] = hi >> 24;
              xv[u][b] = gbl(X)[(int64_t)((uint64_t)(hi & 0xffffffu) << 32 | lo) + vo + b];
            }
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int b = 0; b < 4; ++b)
              if (cv[u][b]) h[u][b] = 2 * h[u][b] + (xv[u][b] >= cv[u][b] ? 1 : 0);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (u == 0 || both)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[b] += (double)tab[u * 4 * H + 2 * H + h[u][b]];
      }
    };

    if (g0 < g1) {
      // the stream of batches of all groups, the next one always in flight;
      // the tables of a group are read ahead likewise and stored to LDS when
      // the group begins (this wave's own copy: no barrier)
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      constexpr int kQuads = kPredTrees * kPredTab / 256;
      u32x4 tq[kQuads];
      auto fetch_tab = [&](int g) {
        const gptr<const u32x4> q =
            gbl((const u32x4 *)(prog + (size_t)g * sizeof(PredGroup) + offsetof(PredGroup, tab)));
#pragma unroll
        for (int k = 0; k < kQuads; ++k) tq[k] = q[64 * k + l];
      };
      auto store_tab = [&]() {
#pragma unroll
        for (int k = 0; k < kQuads; ++k) ((u32x4 *)tab)[64 * k + l] = tq[k];
      };
      int more = 0;  // trees without a table
      int g = g0, b = 0, nb = (int)group(g)->nbatch;
      int others = (int)(group(g)->nlist | group(g)->nspecial);
      fetch_tab(g);
      Batch B0, B1;
      fetch(g, 0, B0);
      store_tab();
      if (g + 1 < g1) fetch_tab(g + 1);
      // the batch after (g, b): in this group, or the first of the next (the
      // same one again where there is none)
      auto fetch_next = [&](Batch &B) {
        const bool here = b + 1 < nb;
        const int gn = here || g + 1 >= g1 ? g : g + 1;
        fetch(gn, here ? b + 1 : 0, B);
      };
      // past a batch; at the end of a group the tables of the next; false at
      // the end
      auto advance = [&]() -> bool {
        if (++b < nb) return true;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[q] += (double)pend[q];
          pend[q] = 0.f;
        }
        more |= others;
        if (++g == mid)  // its first range is summed: held until the second is
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            held[q * 64 + l] = acc[q];
            acc[q] = 0.0;
          }
        if (g >= g1) return false;
        store_tab();
        if (g + 1 < g1) fetch_tab(g + 1);
        b = 0;
        nb = (int)group(g)->nbatch;
        others = (int)(group(g)->nlist | group(g)->nspecial);
        return true;
      };
      for (;;) {
        fetch_next(B1);
        process(B0);
        if (!advance()) break;
        fetch_next(B0);
        process(B1);
        if (!advance()) break;
      }
      // a range's trees of more nodes, behind its others: the second range's
      // first, whose other trees' sums are at hand
      if (__builtin_expect(more, 0))
#pragma unroll 1
        for (int part = 0; part < per_wave; ++part) {
          if (part > 0)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const double t = held[q * 64 + l];
              held[q * 64 + l] = acc[q];
              acc[q] = t;
            }
          const int ga = part == 0 && per_wave > 1 ? mid : g0, gb = part > 0 ? mid : g1;
#pragma unroll 1
          for (g = ga; g < gb; ++g) {
            masks(g);
            special(g);
          }
        }
      if (per_wave > 1)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] += held[q * 64 + l];
    }

    auto emit = [&](int64_t i, double s) {
      const int64_t o = blockIdx.y * nt + i;
      const double f = offset + s;
      if (ACC) {
        sum0[o] += f;
        sumsq0[o] += f * f;
      } else {
        out0[o] = (float)f;
      }
    };
    if (split > 1) {
      double *const part = (double *)tab;  // [4][64] of this wave
#pragma unroll
      for (int b = 0; b < 4; ++b) part[b * 64 + l] = acc[b];
      __syncthreads();
      for (int q = threadIdx.x; q < kPredTile; q += blockDim.x) {
        const int k = (q & 3) * 64 + (q >> 2);  // point q of the tile: lane q / 4
        auto two = [&](int v) {
          return ((const double *)(s_raw + v * wave_lds))[k] +
                 ((const double *)(s_raw + (v + 1) * wave_lds))[k];
        };
        auto four = [&](int v) { return two(v) + two(v + 2); };
        double s = split > 2 ? four(0) : two(0);
        if (split > 4) s += four(4);
        if (split > 8) s += four(8) + four(12);
        if (base + q < nt) emit(base + q, s);
      }
      __syncthreads();
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (at + b < nt) emit(at + b, acc[b]);
    }
  }
}

}  // namespace bart
