// Batched products: many independent products of uneven sizes in one launch
// sequence, captured once per batch shape in a HIP graph.
//
// A batch plan (per host thread, device, stream and shape: format, slice
// form, and every product's m, n, k and D) owns one device workspace holding
// every product's maxima and exponents and the planes of the products that are
// formed at one time (all of them, or run by run where they would take too much:
// FormatPlan), plus
//   - the descriptors of all operands and products (rewritten before every
//     launch: they carry the caller's pointers),
//   - prefix sums of the split work per operand and the work items of the
//     persistent GEMM kernels, in one list per XCD (written once).
// The graph holds, for the products by residues: clear the maxima and work
// counters, one max-exponent launch (and the FLOAT form's samples), one residue split over all operands'
// blocks, the persistent INT8 GEMMs over (product, tile, k chunk, unit group)
// items and the combine; for those by slices: the split (fused, or clear the
// maxima, the max-exponent launch and dmax pass launches), clear the work
// counter, and one persistent GEMM over (product, tile) items.  In the FLOAT form
// the residue products' slice launches follow, and end at once unless the split
// flagged a product; the slices take the place of the operands' residue planes, so
// their split comes behind the residue GEMM.  Kernels take the caller's pointers from the descriptors, so
// a cached graph is replayed with new pointers after one small host-to-device
// copy of the descriptors.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstring>
#include <vector>

#include "../../include/mpgemm.h"
#include "host.h"
#include "internal.h"
#include "layout.h"
#include "residue.h"

namespace mp {
namespace host {
namespace {

constexpr int kMaxPlans = 6;
constexpr int kPersistentGrid = 512;  // 2 workgroups per CU on 256 CUs

// Tile configuration of one product by residues of a batch: the one set for the
// thread (2 and 4 run as 3); else the 256 x 256 tiles unless padding to them
// exceeds 1.5 times the area padded to 128 x 128.  Against one configuration for all
// products (by this rule, 128 x 128, 256 x 256): 128 QD products of 64 to 1024 in the
// FLOAT form 3347, 3471 and 3477 us; 256 DD ones, INT8, 2993, 2991 and 3069; 64 DD
// ones of 64 to 300, INT8, 322, 287 and 315; 200 QD ones of 64 to 200 917, 886, 1086.
int batch_int8_cfg(int64_t m, int64_t n, int cfg_override) {
  if (cfg_override >= 1) return int8_tile_config(m, n, cfg_override) == 1 ? 1 : 3;
  const int64_t area3 = ceil_div(m, 256) * ceil_div(n, 256) * 4, area1 = ceil_div(m, 128) * ceil_div(n, 128);
  return 2 * area3 <= 3 * area1 ? 3 : 1;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int tiles64(int64_t a, int64_t b) { return (int)(ceil_div(a, 64) * ceil_div(b, 64)); }

// The work items of a persistent launch as kXcds per-XCD lists (take_item):
// runs of items with the same key (the tiles of one product, or of one
// product's k chunk and diagonal group) stay together in one list, so that the
// workgroups of one XCD read the same operand panels through its L2.  Runs are
// dealt out in decreasing total work, each to the list with the least work so
// far, and every list is ordered by decreasing item work (longest first).
// bounds receives the kXcds + 1 running offsets of the lists in the result.
template <typename Item, typename Key>
std::vector<Item> xcd_lists(const std::vector<Item> &items, Key key, int *bounds) {
  struct Run {
    int64_t key, item_cost, total;
    std::vector<int> idx;
  };
  std::vector<Run> runs;
  {
    std::vector<std::pair<int64_t, int>> keyed(items.size());
    for (size_t i = 0; i < items.size(); ++i) keyed[i] = {key(items[i]), (int)i};
    std::stable_sort(keyed.begin(), keyed.end(),
                     [](const std::pair<int64_t, int> &a, const std::pair<int64_t, int> &b) { return a.first < b.first; });
    for (const auto &ki : keyed) {
      if (runs.empty() || runs.back().key != ki.first) runs.push_back({ki.first, items[ki.second].cost, 0, {}});
      runs.back().idx.push_back(ki.second);
      runs.back().total += items[ki.second].cost;
    }
  }
  std::stable_sort(runs.begin(), runs.end(), [](const Run &a, const Run &b) { return a.total > b.total; });
  std::vector<std::vector<const Run *>> lists(kXcds);
  int64_t load[kXcds] = {};
  for (const Run &r : runs) {
    const int q = (int)(std::min_element(load, load + kXcds) - load);
    lists[q].push_back(&r);
    load[q] += r.total;
  }
  std::vector<Item> out;
  out.reserve(items.size());
  bounds[0] = 0;
  for (int q = 0; q < kXcds; ++q) {
    std::stable_sort(lists[q].begin(), lists[q].end(),
                     [](const Run *a, const Run *b) { return a->item_cost > b->item_cost; });
    for (const Run *r : lists[q])
      for (int i : r->idx) out.push_back(items[i]);
    bounds[q + 1] = (int)out.size();
  }
  return out;
}

// The products of a batch that are formed by residues (residue.h): one split
// over all their operands, one persistent INT8 GEMM per tile configuration over
// (product, tile, k chunk, unit group) items in per-XCD lists, and one combine.
struct ResidueBatch {
  struct Slot {
    int g;  // product of the batch
    int m, n, k, D, cfg, groups = 1;
    ResiduePlan plan;
    int64_t mbp, nbp, kbp;
    size_t a, b, r;  // planes, counted from `scratch`
    size_t exp_a, exp_b, mu_a, mu_b, st_a, st_b, table;
    size_t operand_bytes() const {
      return align256((size_t)plan.nplanes * mbp * kbp * 1024) + align256((size_t)plan.nplanes * nbp * kbp * 1024);
    }
    size_t result_bytes() const { return align256((size_t)plan.nplanes * plan.nchunks * mbp * nbp * 1024); }
  };
  std::vector<Slot> slots;
  int nw = 0, tiles0 = 0, strips = 0, nitems1 = 0, nitems3 = 0;
  int blocks = 0;
  size_t scratch = 0, planes_bytes = 0;  // where the planes' part of the workspace begins; the operands' planes
  bool shared = false;                   // other runs write to it
  size_t off_ran = 0;  // FLOAT form: a word set once slices have been written to the operands' planes
  size_t off_static = 0, off_tables = 0, off_items = 0, off_bounds = 0, off_counter = 0, off_zero = 0, zero_bytes = 0;
  bool float_form = false;
  size_t off_flags = 0;            // FLOAT form: a word set if any product is flagged, then one per product
  std::vector<int> prefix;         // 2 n + 1 max tiles, 2 n + 1 split blocks, n + 1 combine blocks, 2 n + 1 sampled strips
  std::vector<uint32_t> tables;    // the distinct combine tables
  std::vector<int4> items;
  int bounds[2 * (kXcds + 1)] = {};

  int nops() const { return 2 * (int)slots.size(); }
  size_t ops_bytes(size_t elem) const { return (size_t)nops() * elem; }

  static Slot slot(int g, int m, int n, int k, int D, const ResiduePlan &plan, int cfg) {
    Slot s;
    s.g = g;
    s.m = m;
    s.n = n;
    s.k = k;
    s.D = D;
    s.cfg = cfg;
    s.plan = plan;
    const int tb = int8_tile_blocks(cfg);
    s.mbp = nblocks8_padded(m, tb);
    s.nbp = nblocks8_padded(n, tb);
    s.kbp = kblocks8_padded(k);
    return s;
  }

  // The planes, counted from `scratch`: the operands' from 0 on, the results' from
  // max(their end, after) on.  Returns the end of all.
  size_t place_planes(size_t after) {
    size_t o = 0;
    for (Slot &s : slots) {
      s.a = o;
      s.b = o + align256((size_t)s.plan.nplanes * s.mbp * s.kbp * 1024);
      o += s.operand_bytes();
    }
    planes_bytes = o;
    o = std::max(o, after);
    for (Slot &s : slots) {
      s.r = o;
      o += s.result_bytes();
    }
    return o;
  }

  // Places everything but the planes in the workspace (take: bytes -> offset);
  // elem: bytes of a maximum.
  template <typename Take>
  void layout(Take take, size_t elem, bool float_slices) {
    float_form = float_slices;
    // products of one combine size together: each size has its launch
    std::stable_sort(slots.begin(), slots.end(), [](const Slot &a, const Slot &b) { return a.plan.nwc < b.plan.nwc; });
    for (Slot &s : slots) nw = std::max(nw, s.plan.nw);
    for (Slot &s : slots) {
      s.exp_a = take((size_t)s.m * 4);
      s.exp_b = take((size_t)s.n * 4);
    }
    off_zero = take(0);
    for (Slot &s : slots) {
      s.mu_a = take((size_t)s.m * elem);
      s.mu_b = take((size_t)s.n * elem);
      s.st_a = take(float_form ? (size_t)s.m * 4 : 0);
      s.st_b = take(float_form ? (size_t)s.n * 4 : 0);
    }
    off_flags = take(float_form ? (slots.size() + 1) * 4 : 0);
    off_counter = take(2 * kXcds * 4);
    zero_bytes = take(0) - off_zero;

    const int n = (int)slots.size();
    prefix.assign((size_t)3 * (2 * n + 1) + n + 1, 0);
    int *pre0 = prefix.data(), *preb = pre0 + 2 * n + 1, *prec = preb + 2 * n + 1, *pres = prec + n + 1;
    std::vector<std::pair<std::array<int, 3>, size_t>> known;
    for (int i = 0; i < n; ++i) {
      Slot &s = slots[i];
      const int64_t kbl = ceil_div((int64_t)s.k, (int64_t)kKBlk8);
      pre0[2 * i + 1] = pre0[2 * i] + tiles64(s.m, s.k);
      pre0[2 * i + 2] = pre0[2 * i + 1] + tiles64(s.n, s.k);
      pres[2 * i + 1] = pres[2 * i] + ceil_div(s.m, 16);
      pres[2 * i + 2] = pres[2 * i + 1] + ceil_div(s.n, 16);
      // A's blocks cover the padding of k, which has to be zero in one operand (it is
      // cleared with the plan, and written where something else may lie there since:
      // ResidueOperand::padded); that of m and n takes part in no element of C
      preb[2 * i + 1] = preb[2 * i] + (int)(ceil_div((int64_t)s.m, (int64_t)kBlk8) * s.kbp);
      preb[2 * i + 2] = preb[2 * i + 1] + (int)(ceil_div((int64_t)s.n, (int64_t)kBlk8) * kbl);
      // blocks of its combine launch, counted from the launch's first product
      const bool first = i == 0 || slots[i - 1].plan.nwc != s.plan.nwc;
      prec[i] = first ? 0 : prec[i - 1] + (int)(slots[i - 1].mbp * slots[i - 1].nbp);
      const std::array<int, 3> key{s.plan.nunits, s.plan.nsq, s.plan.nwc};
      size_t at = SIZE_MAX;
      for (const auto &kn : known)
        if (kn.first == key) at = kn.second;
      if (at == SIZE_MAX) {
        at = tables.size();
        const std::vector<uint32_t> &t = residue_table(key[0], key[1], key[2]);
        tables.insert(tables.end(), t.begin(), t.end());
        tables.resize((tables.size() + 3) / 4 * 4, 0u);  // read 16 bytes at a time
        known.push_back({key, at});
      }
      s.table = at;
    }
    tiles0 = pre0[2 * n];
    strips = pres[2 * n];
    blocks = preb[2 * n];
    make_items();
    off_static = take(prefix.size() * 4);
    off_tables = take(tables.size() * 4);
    off_items = take(items.size() * sizeof(int4));
    off_bounds = take(sizeof(bounds));
    off_ran = take(4);
  }

  void make_items() {
    // unit groups: items of about 1/4 of a persistent workgroup's fair share
    int64_t work = 0;
    for (const Slot &s : slots)
      work += (s.mbp / 4) * (s.nbp / 4) * s.plan.products() * s.kbp;  // in 128 x 128 tile units
    const int64_t target = std::max<int64_t>(1, work / (4 * (int64_t)kPersistentGrid));
    struct Item {
      int slot, tile, chunk, group;
      int64_t cost;
    };
    std::vector<Item> items1, items3;
    for (int i = 0; i < (int)slots.size(); ++i) {
      Slot &s = slots[i];
      const int tb = int8_tile_blocks(s.cfg);
      const int64_t unit = (tb / 4) * (tb / 4), kbc = std::min<int64_t>(s.kbp, kChunkBlocks);
      s.groups = (int)std::min<int64_t>(s.plan.nunits,
                                        std::max<int64_t>(1, ceil_div(s.plan.products() * kbc * unit, target)));
      const int ntiles = (int)((s.mbp / tb) * (s.nbp / tb));
      std::vector<Item> &dst = s.cfg == 1 ? items1 : items3;
      for (int z = 0; z < s.groups; ++z) {
        const int nsq = s.plan.nsq, nu = s.plan.nunits;
        const int pairs = residue_pairs_below(residue_group_start(0, nu, nsq, z + 1, s.groups), nsq) -
                          residue_pairs_below(residue_group_start(0, nu, nsq, z, s.groups), nsq);
        if (pairs == 0) continue;
        for (int c = 0; c < s.plan.nchunks; ++c) {
          const int64_t kb = std::min<int64_t>(kChunkBlocks, s.kbp - (int64_t)c * kChunkBlocks);
          for (int t = 0; t < ntiles; ++t) dst.push_back({i, t, c, z, pairs * kb});
        }
      }
    }
    // one list per XCD for each configuration; a run is one (product, k chunk,
    // unit group): its tiles
    auto run_key = [](const Item &it) { return ((int64_t)it.slot << 32) | ((int64_t)it.chunk << 12) | it.group; };
    items1 = xcd_lists(items1, run_key, bounds);
    items3 = xcd_lists(items3, run_key, bounds + kXcds + 1);
    nitems1 = (int)items1.size();
    nitems3 = (int)items3.size();
    for (const auto *v : {&items1, &items3})
      for (const Item &it : *v) items.push_back(make_int4(it.slot, it.tile, it.chunk, it.group));
  }

  // Static device data of a new plan.  Planes of zeros in the padding also leave the
  // matrix cores less to do than what lay there (the clock follows their power).
  bool upload(char *ws) const {
    if (slots.empty()) return true;
    return hipMemset(ws + scratch, 0, planes_bytes) == hipSuccess && hipMemset(ws + off_ran, 0, 4) == hipSuccess &&
           hipStreamSynchronize(nullptr) == hipSuccess &&
           hipMemcpy(ws + off_static, prefix.data(), prefix.size() * 4, hipMemcpyHostToDevice) == hipSuccess &&
           hipMemcpy(ws + off_tables, tables.data(), tables.size() * 4, hipMemcpyHostToDevice) == hipSuccess &&
           hipMemcpy(ws + off_items, items.data(), items.size() * sizeof(int4), hipMemcpyHostToDevice) == hipSuccess &&
           hipMemcpy(ws + off_bounds, bounds, sizeof(bounds), hipMemcpyHostToDevice) == hipSuccess;
  }

  // Whether every block and work item can be numbered in an int.
  bool countable() const {
    int64_t split = 0, combine = 0, tiles = 0, groups = 0;
    for (const Slot &s : slots) {
      split += (s.mbp + s.nbp) * s.kbp;
      combine += s.mbp * s.nbp;
      tiles += ceil_div((int64_t)s.m + s.n + 64, (int64_t)64) * ceil_div((int64_t)s.k, (int64_t)64);
      groups += s.mbp * s.nbp / 16 * s.plan.nchunks * s.plan.nunits;
    }
    return std::max(std::max(split, combine), std::max(tiles, groups)) <= 0x7fffffffLL;
  }

  // The launch sequence in three parts (descriptors at off_ops, off_descs of the workspace).
  template <typename T, int C>
  hipError_t launch_split(char *ws, size_t off_ops, hipStream_t st) const {
    if (slots.empty()) return hipSuccess;
    const auto *ops = reinterpret_cast<const ResidueOperand<T> *>(ws + off_ops);
    const int n = (int)slots.size();
    const int *pre0 = reinterpret_cast<const int *>(ws + off_static), *preb = pre0 + 2 * n + 1;
    hipError_t e = launch_fill32(ws + off_zero, (int64_t)(zero_bytes / 4), 0u, st);
    if (e == hipSuccess) e = launch_residue_max_batched<T>(ops, pre0, 2 * n, tiles0, st);
    if (e == hipSuccess && float_form)
      e = launch_residue_sample<T, C>(ops, preb + 2 * n + 1 + n + 1, 2 * n, strips, st);
    if (e == hipSuccess) e = launch_residue_split_batched<T, C>(nw, ops, preb, 2 * n, blocks, st);
    return e;
  }
  hipError_t launch_gemm(char *ws, size_t off_descs, hipStream_t st) const {
    if (slots.empty()) return hipSuccess;
    return launch_gemm_residue_batched(reinterpret_cast<const ResidueDesc *>(ws + off_descs),
                                       reinterpret_cast<const int4 *>(ws + off_items), nitems1, nitems3,
                                       reinterpret_cast<const int *>(ws + off_bounds),
                                       reinterpret_cast<int *>(ws + off_counter), st);
  }
  template <typename T, int C>
  hipError_t launch_combine(char *ws, size_t off_descs, hipStream_t st) const {
    const auto *descs = reinterpret_cast<const ResidueDesc *>(ws + off_descs);
    const int n = (int)slots.size();
    const int *prec = reinterpret_cast<const int *>(ws + off_static) + 4 * n + 2;
    hipError_t e = hipSuccess;
    for (int i = 0; i < n && e == hipSuccess;) {
      int j = i;
      int64_t sum = 0;
      bool chunks = false;
      for (; j < n && slots[j].plan.nwc == slots[i].plan.nwc; ++j) {
        sum += slots[j].mbp * slots[j].nbp;
        chunks = chunks || slots[j].plan.nchunks > 1;
      }
      e = launch_residue_combine_batched<T, C>(slots[i].plan.nwc, chunks, descs + i, prec + i, j - i, sum, st);
      i = j;
    }
    return e;
  }

  // Descriptors carrying a call's pointers, into the pinned stage.
  template <typename T>
  void write(char *ws, ResidueOperand<T> *ops, ResidueDesc *descs, const T *const *A, const int *lda,
             const T *const *B, const int *ldb, T *const *Cm, const int *ldc) const {
    const char *tab = ws + off_tables;
    for (size_t i = 0; i < slots.size(); ++i) {
      const Slot &s = slots[i];
      const int g = s.g;
      for (int side = 0; side < 2; ++side) {
        ResidueOperand<T> o{};
        o.X = side == 0 ? A[g] : B[g];
        o.comp_stride = side == 0 ? (int64_t)lda[g] * s.k : (int64_t)ldb[g] * s.n;
        o.sv = side == 0 ? 1 : ldb[g];
        o.sp = side == 0 ? lda[g] : 1;
        o.nvec = side == 0 ? s.m : s.n;
        o.len = s.k;
        o.orient = side;
        o.bits = s.plan.bits;
        o.float_form = float_form;
        if (float_form) {
          o.slice_bits = (sizeof(T) == 8 ? 53 : 24) - rho_of(sizeof(T) == 8 ? 53 : 24, s.k);
          o.passes = s.D;
          o.state = reinterpret_cast<int *>(ws + (side == 0 ? s.st_a : s.st_b));
          o.any = reinterpret_cast<int *>(ws + off_flags);
          o.flag = o.any + i + 1;
        }
        o.planes = reinterpret_cast<int8_t *>(ws + scratch + (side == 0 ? s.a : s.b));
        o.nbp = side == 0 ? s.mbp : s.nbp;
        o.kbp = s.kbp;
        o.mu = ws + (side == 0 ? s.mu_a : s.mu_b);
        o.exps = reinterpret_cast<int *>(ws + (side == 0 ? s.exp_a : s.exp_b));
        o.nunits = s.plan.nunits;
        o.nsq = s.plan.nsq;
        o.padded = shared ? nullptr : reinterpret_cast<const int *>(ws + off_ran);
        ops[2 * i + side] = o;
      }
      ResidueDesc d{};
      d.A = reinterpret_cast<const int8_t *>(ws + scratch + s.a);
      d.B = reinterpret_cast<const int8_t *>(ws + scratch + s.b);
      d.R = reinterpret_cast<int8_t *>(ws + scratch + s.r);
      d.table = reinterpret_cast<const uint32_t *>(tab) + s.table;
      d.EA = reinterpret_cast<const int *>(ws + s.exp_a);
      d.EB = reinterpret_cast<const int *>(ws + s.exp_b);
      d.mbp = s.mbp;
      d.nbp = s.nbp;
      d.kbp = s.kbp;
      d.plane = s.mbp * s.nbp * 1024;
      d.nunits = s.plan.nunits;
      d.nsq = s.plan.nsq;
      d.nplanes = s.plan.nplanes;
      d.nchunks = s.plan.nchunks;
      d.groups = s.groups;
      d.bits = s.plan.bits;
      d.m = s.m;
      d.n = s.n;
      d.ldc = ldc[g];
      d.C = Cm[g];
      d.c_stride = (int64_t)ldc[g] * s.n;
      if (float_form) d.skip = reinterpret_cast<const int *>(ws + off_flags) + i + 1;
      descs[i] = d;
    }
  }
};

// The part of an operand that decides its split kernel.
struct OperandShape {
  int64_t kbp, nbp, nvec;
};

// The products of a batch that are formed from slices: the split of all their
// operands and one persistent slice-product kernel over (product, tile) items
// in per-XCD lists.  A FLOAT-form batch has two: the products that do not go by
// residues, and, behind them, those that do, whose kernels run only for the
// products that the residue split flagged.
template <typename T, int C>
struct PlainBatch {
  struct Slot {
    int g;  // product of the batch
    int m, n, k, D, rho;
    int64_t mbp, nbp, kbp;
    size_t resid_a, resid_b, pack_a, pack_b;  // counted from `scratch`
    size_t mu_a, mu_b, exp_a, exp_b;
    bool fused_a, fused_b;  // operand split by the fused kernel (no residual)
    size_t flag;            // offset of its condition word (SIZE_MAX: always formed)
  };
  std::vector<Slot> slots;
  size_t scratch = 0, scratch_bytes = 0;  // of the residuals and slices
  size_t off_static = 0, off_items = 0, off_bounds = 0, off_counter = 0, off_mu = 0, mu_bytes = 0;
  size_t off_any = SIZE_MAX;  // condition word of all launches
  size_t off_ran = SIZE_MAX;  // set by launches that run
  int tiles0 = 0, tilesp = 0, stripsf = 0, dpass = 0;
  int fused_nt = 512;  // threads of the fused-split workgroups
  std::vector<int> prefix;  // 2 n + 1 max tiles, 2 n + 1 pass tiles, 2 n + 1 fused strips
  std::vector<int2> items;
  int bounds[kXcds + 1] = {};

  size_t ops_bytes() const { return 2 * slots.size() * sizeof(SplitOperand<T>); }
  size_t stage_bytes() const { return ops_bytes() + slots.size() * sizeof(PlainGemmDesc); }

  static Slot slot(int g, int m, int n, int k, int D) {
    Slot s{};
    s.g = g;
    s.m = m;
    s.n = n;
    s.k = k;
    s.D = D;
    s.rho = rho_of(sizeof(T) == 8 ? 53 : 24, k);
    s.mbp = nblocks_padded(m);
    s.nbp = nblocks_padded(n);
    s.kbp = kblocks_padded(k);
    s.flag = SIZE_MAX;
    return s;
  }
  // Bytes of its slices, and of its residuals where the fused kernel does not split it.
  static size_t scratch_of(const Slot &s, int split_kernel) {
    const bool fused = split_kernel == 0 && fused_threads<T, C>(s.kbp * kKBlk) > 0;
    return (size_t)s.D * (s.mbp + s.nbp) * s.kbp * 256 * sizeof(T) +
           (fused || s.D <= 1 ? 0 : (size_t)C * (s.m + s.n) * s.k * sizeof(T));
  }

  template <typename Take>
  void layout(Take take, int split_kernel) {
    const size_t w = sizeof(T);
    auto take_scratch = [&](size_t bytes) {
      const size_t at = scratch_bytes;
      scratch_bytes += align256(bytes);
      return at;
    };
    // one fused-split launch: 512-thread workgroups when every product's vectors
    // allow them, else 1024
    for (const Slot &s : slots)
      if (fused_threads<T, C>(s.kbp * kKBlk) == 1024) fused_nt = 1024;
    for (Slot &s : slots) {
      s.fused_a = split_kernel == 0 && fused_strips<T, C>(OperandShape{s.kbp, s.mbp, s.m}, fused_nt) >= 0;
      s.fused_b = split_kernel == 0 && fused_strips<T, C>(OperandShape{s.kbp, s.nbp, s.n}, fused_nt) >= 0;
      s.resid_a = take_scratch(s.D > 1 && !s.fused_a ? (size_t)C * s.m * s.k * w : 0);
      s.resid_b = take_scratch(s.D > 1 && !s.fused_b ? (size_t)C * s.k * s.n * w : 0);
      s.pack_a = take_scratch((size_t)s.D * s.mbp * s.kbp * 256 * w);
      s.pack_b = take_scratch((size_t)s.D * s.nbp * s.kbp * 256 * w);
      s.exp_a = take((size_t)s.D * s.m * 4);
      s.exp_b = take((size_t)s.D * s.n * 4);
    }
    // one region for all maxima (cleared by a single fill)
    size_t mo = 0;
    for (Slot &s : slots) {
      s.mu_a = mo;
      mo += (size_t)s.D * s.m * w;
      s.mu_b = mo;
      mo += (size_t)s.D * s.n * w;
    }
    off_mu = take(mo);
    mu_bytes = (mo + 3) / 4 * 4;
    for (Slot &s : slots) {
      s.mu_a += off_mu;
      s.mu_b += off_mu;
    }

    // prefix sums of the split work.  An operand whose vectors fit a fused
    // workgroup is split by the fused kernel alone; the others by the max and
    // pass kernels.
    const int n = 2 * (int)slots.size();
    prefix.assign((size_t)3 * (n + 1), 0);
    int *pre0 = prefix.data(), *prep = pre0 + n + 1, *pref = prep + n + 1;
    for (int i = 0; i < n; ++i) {
      const Slot &s = slots[i / 2];
      const bool side_b = i % 2 == 1, fused = side_b ? s.fused_b : s.fused_a;
      const int64_t nvec = side_b ? s.n : s.m, nbp = side_b ? s.nbp : s.mbp;
      pref[i + 1] = pref[i] + (fused ? fused_strips<T, C>(OperandShape{s.kbp, nbp, nvec}, fused_nt) : 0);
      pre0[i + 1] = pre0[i] + (fused ? 0 : tiles64(nvec, s.k));
      prep[i + 1] = prep[i] + (fused ? 0 : tiles64(nbp * kBlk, s.kbp * kKBlk));
      if (!fused) dpass = std::max(dpass, s.D);
    }
    tiles0 = pre0[n];
    tilesp = prep[n];
    stripsf = pref[n];

    // work items: (slot, tile)
    struct Item {
      int slot, tile;
      int64_t cost;
    };
    std::vector<Item> list;
    for (int i = 0; i < (int)slots.size(); ++i) {
      const Slot &s = slots[i];
      const int ntiles = (int)((s.mbp / kTileBlocks) * (s.nbp / kTileBlocks));
      const int64_t cost = (int64_t)s.D * (s.D + 1) / 2 * s.kbp;
      for (int t = 0; t < ntiles; ++t) list.push_back({i, t, cost});
    }
    list = xcd_lists(list, [](const Item &it) { return (int64_t)it.slot; }, bounds);
    for (const Item &it : list) items.push_back(make_int2(it.slot, it.tile));
    off_static = take(prefix.size() * 4);
    off_items = take(items.size() * sizeof(int2));
    off_bounds = take(sizeof(bounds));
    off_counter = take(kXcds * 4);
  }

  bool upload(char *ws) const {
    if (slots.empty()) return true;
    return hipMemcpy(ws + off_static, prefix.data(), prefix.size() * 4, hipMemcpyHostToDevice) == hipSuccess &&
           hipMemcpy(ws + off_items, items.data(), items.size() * sizeof(int2), hipMemcpyHostToDevice) == hipSuccess &&
           hipMemcpy(ws + off_bounds, bounds, sizeof(bounds), hipMemcpyHostToDevice) == hipSuccess;
  }

  // The launch sequence in two parts, with the descriptors at `off` of the workspace.
  hipError_t launch_split(char *ws, size_t off, hipStream_t st) const {
    if (slots.empty()) return hipSuccess;
    const int n = 2 * (int)slots.size();
    const int *pre0 = reinterpret_cast<const int *>(ws + off_static), *prep = pre0 + n + 1, *pref = prep + n + 1;
    const int *any = off_any == SIZE_MAX ? nullptr : reinterpret_cast<const int *>(ws + off_any);
    return launch_split_plain_batched<T, C>(reinterpret_cast<const SplitOperand<T> *>(ws + off), pre0, prep, pref, n,
                                            tiles0, tilesp, stripsf, fused_nt, dpass, ws + off_mu,
                                            (int64_t)(mu_bytes / 4), any, st);
  }
  hipError_t launch_products(char *ws, size_t off, int gemm_layout, hipStream_t st) const {
    if (slots.empty()) return hipSuccess;
    const int *any = off_any == SIZE_MAX ? nullptr : reinterpret_cast<const int *>(ws + off_any);
    hipError_t e = launch_fill32(ws + off_counter, kXcds, 0u, st);
    if (e == hipSuccess)
      e = launch_gemm_plain_batched<T, C>(reinterpret_cast<const PlainGemmDesc *>(ws + off + ops_bytes()),
                                          reinterpret_cast<const int2 *>(ws + off_items),
                                          reinterpret_cast<const int *>(ws + off_bounds),
                                          reinterpret_cast<int *>(ws + off_counter),
                                          std::min((int)items.size(), kPersistentGrid), gemm_layout, any,
                                          off_ran == SIZE_MAX ? nullptr : reinterpret_cast<int *>(ws + off_ran), st);
    return e;
  }

  // Descriptors carrying a call's pointers, into the pinned stage.
  void write(char *ws, char *stage, int last_slice, const T *const *A, const int *lda, const T *const *B,
             const int *ldb, T *const *Cm, const int *ldc) const {
    auto *ops = reinterpret_cast<SplitOperand<T> *>(stage);
    auto *descs = reinterpret_cast<PlainGemmDesc *>(stage + ops_bytes());
    for (size_t i = 0; i < slots.size(); ++i) {
      const Slot &s = slots[i];
      const int g = s.g;
      const int *run_if = s.flag == SIZE_MAX ? nullptr : reinterpret_cast<const int *>(ws + s.flag);
      for (int side = 0; side < 2; ++side) {
        SplitOperand<T> o{};
        o.X = side == 0 ? A[g] : B[g];
        o.comp_stride = side == 0 ? (int64_t)lda[g] * s.k : (int64_t)ldb[g] * s.n;
        o.sv = side == 0 ? 1 : ldb[g];
        o.sp = side == 0 ? lda[g] : 1;
        o.nvec = side == 0 ? s.m : s.n;
        o.len = s.k;
        o.orient = side;
        o.resid = reinterpret_cast<T *>(ws + scratch + (side == 0 ? s.resid_a : s.resid_b));
        o.packed = ws + scratch + (side == 0 ? s.pack_a : s.pack_b);
        o.nbp = side == 0 ? s.mbp : s.nbp;
        o.kbp = s.kbp;
        o.mu = ws + (side == 0 ? s.mu_a : s.mu_b);
        o.exps = reinterpret_cast<int *>(ws + (side == 0 ? s.exp_a : s.exp_b));
        o.D = s.D;
        o.rho = s.rho;
        o.last_literal = last_slice;
        o.run_if = run_if;
        ops[2 * i + side] = o;
      }
      PlainGemmDesc d{};
      d.Apk = ws + scratch + s.pack_a;
      d.Bpk = ws + scratch + s.pack_b;
      d.mbp = s.mbp;
      d.nbp = s.nbp;
      d.kbp = s.kbp;
      d.m = s.m;
      d.n = s.n;
      d.D = s.D;
      d.ldc = ldc[g];
      d.C = Cm[g];
      d.c_stride = (int64_t)ldc[g] * s.n;
      d.run_if = run_if;
      descs[i] = d;
    }
  }
};

// The plan of a batch, without its format's part.
struct BatchPlan {
  int device = 0, fmt = 0, mode = 0, layout = 1, int8_tile = 0, split_kernel = 0, last_slice = 0;
  bool automatic = true;  // slice counts chosen by the library
  hipStream_t stream = nullptr;
  std::vector<int> m, n, k, D;
  bool any_order = false;   // every operand is read before the first C is written
  bool needs_apart = false; // built for C's apart from all operands (any_order = false, and it makes use of it)
  std::vector<int> alone;   // products formed by a call of their own
  bool empty = true;
  char *ws = nullptr;
  size_t off_desc = 0, desc_bytes = 0, total = 0;
  void *stage = nullptr;
  hipEvent_t stage_done = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  uint64_t last_use = 0;
  virtual ~BatchPlan() {}

  void release() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (stage_done) (void)hipEventDestroy(stage_done);
    if (stage) (void)hipHostFree(stage);
    if (ws) (void)hipFree(ws);
    exec = nullptr;
    graph = nullptr;
    stage_done = nullptr;
    stage = nullptr;
    ws = nullptr;
  }
};

struct BatchCache {
  std::vector<BatchPlan *> plans;
  hipStream_t capture[64] = {};
  uint64_t clock = 0;
};
// Owned by the thread and intentionally not destroyed at thread exit (the HIP
// runtime may already be gone then); mpgemm_batched_cache_clear frees it.
thread_local BatchCache *g_batch = nullptr;

BatchCache &cache() {
  if (!g_batch) g_batch = new BatchCache();
  return *g_batch;
}

// A plan of one format: the products by slices, and runs of products by residues
// with, in the FLOAT form, their slices where the residue split flags them.  The
// runs come one after the other and share the workspace of their planes: one run
// holds all products unless their planes exceed residue_room.  A product whose planes
// alone do so is formed by a call of its own.  Both write some C before the last
// operand is read; with any_order (C's that share memory with operands) FLOAT
// products that do not fit in one run go by slices, INT8 ones in one run all the same.
template <typename T, int C>
struct FormatPlan : BatchPlan {
  struct Run {
    ResidueBatch res;
    PlainBatch<T, C> fallback;
    size_t off_fallback = 0, off_ops = 0, off_res = 0;  // descriptors, from off_desc
  };
  PlainBatch<T, C> plain;
  std::vector<Run> runs;

  // Bytes of the digits and sums that an INT8 product took before it had residues.
  static size_t digit_bytes(int64_t m, int64_t n, int64_t k, int D, int cfg) {
    const int tb = int8_tile_blocks(cfg);
    const int64_t mbp = nblocks8_padded(m, tb), nbp = nblocks8_padded(n, tb), kbp = kblocks8_padded(k);
    return (size_t)D * 1024 * ((mbp + nbp) * kbp + 4 * ceil_div(kbp, (int64_t)int8_kblocks_per_chunk(D)) * mbp * nbp);
  }

  // Deals the products to `plain`, `runs` and `alone`.
  int deal() {
    const int count = (int)m.size();
    const bool slices = mode == MPGEMM_MODE_FLOAT;
    std::vector<ResidueBatch::Slot> res;
    size_t least = 0, operands = 0, packed = 0, results = 0;  // of the slices or digits; of the residues
    for (int g = 0; g < count; ++g) {
      if (m[g] <= 0 || n[g] <= 0 || k[g] <= 0) continue;
      const auto ps = PlainBatch<T, C>::slot(g, m[g], n[g], k[g], D[g]);
      const int cfg = batch_int8_cfg(m[g], n[g], int8_tile);
      ResiduePlan rp;
      if (!slices) {
        if (!residue_plan(7 * D[g] - 1, k[g], rp)) return MPGEMM_ERR_TOO_LARGE;  // none: D <= 40, k <= 2^20
        least += digit_bytes(m[g], n[g], k[g], D[g], cfg);
      } else {
        const size_t own = PlainBatch<T, C>::scratch_of(ps, split_kernel);
        least += own;
        if (!automatic || last_slice != 0 || !float_residue_plan(fmt, D[g], k[g], rp)) {
          plain.slots.push_back(ps);
          continue;
        }
        packed += own;
      }
      res.push_back(ResidueBatch::slot(g, m[g], n[g], k[g], D[g], rp, cfg));
      operands += res.back().operand_bytes();
      results += res.back().result_bytes();
    }
    // 7/4 of the slices hold all planes of products of like m, n and k: 512 DD products
    // of 64 to 1024 take 6.8 ms in one run (10.8 GB, 1.6 times their slices), 7.1 in two
    const size_t all = std::max(operands, packed) + results, room = residue_room(all, least, 7);
    const bool fits = all <= room;
    if (any_order && !fits && slices) {
      for (const auto &s : res) plain.slots.push_back(PlainBatch<T, C>::slot(s.g, s.m, s.n, s.k, s.D));
      return 0;
    }
    size_t ro = 0, rp = 0, rr = 0;  // of the run being filled
    for (const auto &s : res) {
      const auto ps = PlainBatch<T, C>::slot(s.g, s.m, s.n, s.k, s.D);
      const size_t o = s.operand_bytes(), r = s.result_bytes(),
                   q = slices ? PlainBatch<T, C>::scratch_of(ps, split_kernel) : 0;
      if (!fits && !any_order) {
        if (std::max(o, q) + r > room) {
          alone.push_back(s.g);
          continue;
        }
        if (!runs.empty() && std::max(ro + o, rp + q) + rr + r > room) runs.emplace_back(), ro = rp = rr = 0;
      }
      if (runs.empty()) runs.emplace_back();
      runs.back().res.slots.push_back(s);
      if (slices) runs.back().fallback.slots.push_back(ps);
      ro += o;
      rp += q;
      rr += r;
    }
    needs_apart = runs.size() > 1 || !alone.empty();
    return 0;
  }

  int build() {
    const int s = deal();
    if (s) return s;
    empty = plain.slots.empty() && runs.empty();
    size_t o = 0;
    auto take = [&](size_t bytes) {
      const size_t at = o;
      o += align256(bytes);
      return at;
    };
    for (const Run &r : runs)
      if (!r.res.countable()) return MPGEMM_ERR_TOO_LARGE;
    plain.layout(take, split_kernel);
    size_t planes = 0;
    for (Run &r : runs) {
      r.fallback.layout(take, split_kernel);
      r.res.layout(take, sizeof(T), mode == MPGEMM_MODE_FLOAT);
      planes = std::max(planes, r.res.place_planes(r.fallback.scratch_bytes));
      for (size_t i = 0; i < r.res.slots.size(); ++i)
        for (auto &f : r.fallback.slots)
          if (f.g == r.res.slots[i].g) f.flag = r.res.off_flags + 4 * (i + 1);
      r.fallback.off_any = r.res.off_flags;
      r.fallback.off_ran = r.res.off_ran;
      r.res.shared = runs.size() > 1;
    }
    off_desc = take(0);
    desc_bytes = plain.stage_bytes();
    for (Run &r : runs) {
      r.off_fallback = desc_bytes;
      r.off_ops = r.off_fallback + r.fallback.stage_bytes();
      r.off_res = r.off_ops + r.res.ops_bytes(sizeof(ResidueOperand<T>));
      desc_bytes = r.off_res + r.res.slots.size() * sizeof(ResidueDesc);
    }
    take(desc_bytes);
    o = (o + 4095) & ~size_t(4095);  // the planes' blocks at multiples of their 1 KiB
    plain.scratch = take(plain.scratch_bytes);
    o = (o + 4095) & ~size_t(4095);
    const size_t scratch = take(planes);
    for (Run &r : runs) r.fallback.scratch = r.res.scratch = scratch;
    total = o;

    if (!allocate_device(&ws, total > 0 ? total : 256, device)) return MPGEMM_ERR_WORKSPACE;
    if (hipHostMalloc(&stage, desc_bytes > 0 ? desc_bytes : 64, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      stage = nullptr;
      return MPGEMM_ERR_WORKSPACE;
    }
    if (hipEventCreateWithFlags(&stage_done, hipEventDisableTiming) != hipSuccess) return MPGEMM_ERR_HIP;
    if (!plain.upload(ws)) return MPGEMM_ERR_HIP;
    for (const Run &r : runs)
      if (!r.fallback.upload(ws) || !r.res.upload(ws)) return MPGEMM_ERR_HIP;

    // capture the launch sequence on a private stream
    BatchCache &bc = cache();
    hipStream_t &cs = bc.capture[device & 63];
    if (!cs && hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) return MPGEMM_ERR_HIP;
    if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) != hipSuccess) return MPGEMM_ERR_HIP;
    // with one run every operand is read before the first C is written: C may be an operand
    hipError_t e = plain.launch_split(ws, off_desc, cs);
    for (size_t i = 0; i < runs.size(); ++i) {
      const Run &r = runs[i];
      if (e == hipSuccess) e = r.res.template launch_split<T, C>(ws, off_desc + r.off_ops, cs);
      if (e == hipSuccess) e = r.res.launch_gemm(ws, off_desc + r.off_res, cs);
      if (e == hipSuccess) e = r.fallback.launch_split(ws, off_desc + r.off_fallback, cs);
      if (e == hipSuccess) e = r.res.template launch_combine<T, C>(ws, off_desc + r.off_res, cs);
      if (e == hipSuccess) e = r.fallback.launch_products(ws, off_desc + r.off_fallback, layout, cs);
    }
    if (e == hipSuccess) e = plain.launch_products(ws, off_desc, layout, cs);
    hipGraph_t captured = nullptr;
    const hipError_t e2 = hipStreamEndCapture(cs, &captured);
    if (e != hipSuccess || e2 != hipSuccess || !captured) {
      if (captured) (void)hipGraphDestroy(captured);
      (void)hipGetLastError();
      return MPGEMM_ERR_HIP;
    }
    graph = captured;
    if (hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
      (void)hipGetLastError();
      return MPGEMM_ERR_HIP;
    }
    return 0;
  }

  // Descriptors carrying this call's pointers, into the pinned stage.
  void write(const T *const *A, const int *lda, const T *const *B, const int *ldb, T *const *Cm, const int *ldc) {
    char *to = static_cast<char *>(stage);
    plain.write(ws, to, last_slice, A, lda, B, ldb, Cm, ldc);
    for (const Run &r : runs) {
      r.fallback.write(ws, to + r.off_fallback, last_slice, A, lda, B, ldb, Cm, ldc);
      r.res.template write<T>(ws, reinterpret_cast<ResidueOperand<T> *>(to + r.off_ops),
                              reinterpret_cast<ResidueDesc *>(to + r.off_res), A, lda, B, ldb, Cm, ldc);
    }
  }
};

// Whether no C of the batch shares memory with an operand of it.
template <typename T, int C>
bool all_apart(int count, const int *m, const int *n, const int *k, const T *const *A, const int *lda,
               const T *const *B, const int *ldb, T *const *Cm, const int *ldc) {
  std::vector<std::pair<const T *, const T *>> ops;  // [begin, end)
  for (int g = 0; g < count; ++g) {
    if (m[g] <= 0 || n[g] <= 0 || k[g] <= 0) continue;
    ops.push_back({A[g], A[g] + (int64_t)C * lda[g] * k[g]});
    ops.push_back({B[g], B[g] + (int64_t)C * ldb[g] * n[g]});
  }
  std::sort(ops.begin(), ops.end());
  for (size_t i = 1; i < ops.size(); ++i) ops[i].second = std::max(ops[i].second, ops[i - 1].second);
  for (int g = 0; g < count; ++g) {
    if (m[g] <= 0 || n[g] <= 0) continue;
    const T *end = Cm[g] + (int64_t)C * ldc[g] * n[g];
    // of the operands that begin before C's end, the last end
    const auto it = std::lower_bound(ops.begin(), ops.end(), std::make_pair(end, (const T *)nullptr));
    if (it != ops.begin() && (it - 1)->second > Cm[g]) return false;
  }
  return true;
}

template <typename T, int C>
int run_batched(int fmt, int count, const int *m, const int *n, const int *k, const T *const *A, const int *lda,
                const T *const *B, const int *ldb, T *const *Cm, const int *ldc, hipStream_t st) {
  if (count < 0) return -1;
  if (count > 0 && (!m || !n || !k || !A || !lda || !B || !ldb || !Cm || !ldc)) {
    const void *args[] = {m, n, k, A, lda, B, ldb, Cm, ldc};
    for (int i = 0; i < 9; ++i)
      if (!args[i]) return -(i + 2);
  }
  for (int g = 0; g < count; ++g) {
    const int s = validate(m[g], n[g], k[g], A[g], lda[g], B[g], ldb[g], Cm[g], ldc[g]);
    if (s < 0) return s - 1;  // positions shifted by the leading count argument
    if (s > 0) return s;
  }
  int s;
  if ((s = check_device_cached())) return s;
  const int mode = thread_mode(fmt);
  if (mode != MPGEMM_MODE_FLOAT && (mode != MPGEMM_MODE_INT8 || sizeof(T) != 8)) return MPGEMM_ERR_UNSUPPORTED;
  const int layout = layout_for(fmt);
  const bool automatic = automatic_slices(fmt, mode);
  if (count == 0) return 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MPGEMM_ERR_HIP;

  std::vector<int> Ds(count);
  for (int g = 0; g < count; ++g) Ds[g] = slices_for(fmt, mode, k[g]);
  set_last_slices(Ds.empty() ? 0 : *std::max_element(Ds.begin(), Ds.end()));

  // products with k == 0 only need C cleared
  for (int g = 0; g < count; ++g)
    if (k[g] == 0 && m[g] > 0 && n[g] > 0) {
      if (launch_zero_matrix(Cm[g], sizeof(T), C, m[g], n[g], ldc[g], (int64_t)ldc[g] * n[g], st) != hipSuccess)
        return MPGEMM_ERR_HIP;
    }

  BatchCache &bc = cache();
  FormatPlan<T, C> *plan = nullptr;
  // The plan of this shape (any_order as in FormatPlan), built if there is none.
  auto plan_of = [&](bool any_order) -> int {
    for (BatchPlan *p : bc.plans)
      if (p->device == dev && p->stream == st && p->fmt == fmt && p->mode == mode && p->layout == layout &&
          p->int8_tile == int8_tile_override() && p->split_kernel == split_kernel_override() &&
          p->last_slice == last_slice_option() && p->automatic == automatic && p->any_order == any_order &&
          (int)p->m.size() == count &&
          std::equal(p->m.begin(), p->m.end(), m) && std::equal(p->n.begin(), p->n.end(), n) &&
          std::equal(p->k.begin(), p->k.end(), k) && p->D == Ds) {
        plan = static_cast<FormatPlan<T, C> *>(p);  // the format decides T and C
        return 0;
      }
    if ((int)bc.plans.size() >= kMaxPlans) {
      auto oldest = std::min_element(bc.plans.begin(), bc.plans.end(),
                                     [](const BatchPlan *a, const BatchPlan *b) { return a->last_use < b->last_use; });
      (void)hipDeviceSynchronize();  // its workspace may still be in use
      (*oldest)->release();
      delete *oldest;
      bc.plans.erase(oldest);
    }
    auto *made = new FormatPlan<T, C>();
    made->device = dev;
    made->stream = st;
    made->fmt = fmt;
    made->mode = mode;
    made->layout = layout;
    made->int8_tile = int8_tile_override();
    made->split_kernel = split_kernel_override();
    made->last_slice = last_slice_option();
    made->automatic = automatic;
    made->any_order = any_order;
    made->m.assign(m, m + count);
    made->n.assign(n, n + count);
    made->k.assign(k, k + count);
    made->D = Ds;
    const int status = made->build();
    if (status) {
      made->release();
      delete made;
      return status;
    }
    bc.plans.push_back(made);
    plan = made;
    return 0;
  };
  auto apart = [&] { return all_apart<T, C>(count, m, n, k, A, lda, B, ldb, Cm, ldc); };
  auto product = [&](int g) {
    return run_product<T, C>(fmt, mode, Ds[g], automatic, m[g], n[g], k[g], A[g], lda[g], B[g], ldb[g], Cm[g], ldc[g],
                             st);
  };
  s = plan_of(false);
  if (s == MPGEMM_ERR_WORKSPACE) {
    // the device has not that much left: one product after the other, each in its
    // own workspace, or all by slices
    if (apart()) {
      for (int g = 0; g < count; ++g)
        if (m[g] > 0 && n[g] > 0 && k[g] > 0 && (s = product(g)) != 0) return s;
      set_last_slices(*std::max_element(Ds.begin(), Ds.end()));
      return 0;
    }
    s = plan_of(true);
  }
  if (s == 0 && plan->needs_apart && !apart()) s = plan_of(true);
  if (s) return s;
  plan->last_use = ++bc.clock;
  for (int g : plan->alone)
    if ((s = product(g)) != 0) return s;
  if (!plan->alone.empty()) set_last_slices(*std::max_element(Ds.begin(), Ds.end()));
  if (plan->empty) return 0;

  // the stage may still feed the previous launch's descriptor copy
  if (hipEventSynchronize(plan->stage_done) != hipSuccess) return MPGEMM_ERR_HIP;
  plan->write(A, lda, B, ldb, Cm, ldc);
  hipEvent_t ev[3];
  profile_mark3(ev);
  if (ev[0]) (void)hipEventRecord(ev[0], st);
  if (hipMemcpyAsync(plan->ws + plan->off_desc, plan->stage, plan->desc_bytes, hipMemcpyHostToDevice, st) !=
          hipSuccess ||
      hipEventRecord(plan->stage_done, st) != hipSuccess)
    return MPGEMM_ERR_HIP;
  if (ev[1]) (void)hipEventRecord(ev[1], st);
  const hipError_t e = hipGraphLaunch(plan->exec, st);
  if (ev[2]) (void)hipEventRecord(ev[2], st);
  profile_commit(ev);
  return hip_status(e);
}

}  // namespace
}  // namespace host
}  // namespace mp

using namespace mp::host;

extern "C" {

int mpgemm_dd_batched(int count, const int *m, const int *n, const int *k, const double *const *A, const int *lda,
                      const double *const *B, const int *ldb, double *const *C, const int *ldc, hipStream_t stream) {
  return run_batched<double, 2>(MPGEMM_DD, count, m, n, k, A, lda, B, ldb, C, ldc, stream);
}
int mpgemm_td_batched(int count, const int *m, const int *n, const int *k, const double *const *A, const int *lda,
                      const double *const *B, const int *ldb, double *const *C, const int *ldc, hipStream_t stream) {
  return run_batched<double, 3>(MPGEMM_TD, count, m, n, k, A, lda, B, ldb, C, ldc, stream);
}
int mpgemm_qd_batched(int count, const int *m, const int *n, const int *k, const double *const *A, const int *lda,
                      const double *const *B, const int *ldb, double *const *C, const int *ldc, hipStream_t stream) {
  return run_batched<double, 4>(MPGEMM_QD, count, m, n, k, A, lda, B, ldb, C, ldc, stream);
}
int mpgemm_ts_batched(int count, const int *m, const int *n, const int *k, const float *const *A, const int *lda,
                      const float *const *B, const int *ldb, float *const *C, const int *ldc, hipStream_t stream) {
  return run_batched<float, 3>(MPGEMM_TS, count, m, n, k, A, lda, B, ldb, C, ldc, stream);
}

int mpgemm_batched_cache_clear(void) {
  if (!g_batch) return 0;
  const hipError_t e = hipDeviceSynchronize();
  for (BatchPlan *p : g_batch->plans) {
    p->release();
    delete p;
  }
  g_batch->plans.clear();
  return e == hipSuccess ? 0 : MPGEMM_ERR_HIP;
}

}  // extern "C"
