// Host side of the C ABI, part 2: contraction plans (label analysis, offset tables, screening
// setup, work decomposition), grouped persistent execution with hipGraph replay, and the
// autotuner that picks kernel configurations by measurement.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <queue>
#include <sstream>
#include <string>
#include <tuple>
#include <vector>

#include "host.h"
#include "mixed.h"

using namespace tamm;

namespace {

struct Label {
  char c;
  int od = -1, ad = -1, bd = -1;  // dimension in out, A, B (-1 if absent)
  std::shared_ptr<SpaceData> sp;
  std::vector<int32_t> cls;       // size class per tile
  std::vector<int64_t> cls_size;  // tile size of each class
};

int32_t pool_push(std::vector<int32_t>& pool, const std::vector<int64_t>& v) {
  int32_t start = (int32_t)pool.size();
  for (int64_t x : v) pool.push_back((int32_t)x);
  return start;
}

// An offset table followed by its padding of invalid entries (read by the gathers past the end).
static int32_t pool_push_table(std::vector<int32_t>& pool, const std::vector<int64_t>& v) {
  const int32_t start = pool_push(pool, v);
  pool.insert(pool.end(), kTablePad, kTableInvalid);
  return start;
}

// True when entries 2j and 2j+1 of a table are adjacent elements for every j (even length).
static bool pairs_adjacent(const std::vector<int64_t>& t) {
  if (t.size() % 2) return false;
  for (size_t j = 0; j + 1 < t.size(); j += 2)
    if (t[j + 1] != t[j] + 1) return false;
  return true;
}

// Offset table of one label group inside blocks of one operand shape: flattened index (mixed
// radix over `group`, last fastest) -> element offset in the row-major block.
std::vector<int64_t> group_table(const std::vector<int>& group, const std::vector<int64_t>& lab_ext,
                                 const std::vector<int64_t>& lab_stride) {
  int64_t n = 1;
  for (int l : group) n *= lab_ext[l];
  std::vector<int64_t> tab(n, 0);
  for (int64_t i = 0; i < n; ++i) {
    int64_t rem = i, off = 0;
    for (int q = (int)group.size() - 1; q >= 0; --q) {
      const int l = group[q];
      off += (rem % lab_ext[l]) * lab_stride[l];
      rem /= lab_ext[l];
    }
    tab[i] = off;
  }
  return tab;
}

uint64_t fnv(uint64_t h, const void* data, size_t n) {
  const unsigned char* p = (const unsigned char*)data;
  for (size_t i = 0; i < n; ++i) {
    h ^= p[i];
    h *= 0x100000001B3ULL;
  }
  return h;
}

// Device regions of one contraction's static tables and screened pair lists, relative to a base.
struct Layout {
  size_t pool = 0, atile = 0, btile = 0, blocks = 0, pairs = 0, counts = 0, end = 0;
};

}  // namespace

namespace {

// What the choice of a configuration needs of an output block: extents, surviving pairs, their
// summed K extent, and the chunks of 16 and of 32 summed indices that they take.
struct BlockShape {
  int64_t mext = 0, next = 0, pairs = 0, chunks16 = 0, chunks32 = 0;
  double kext = 0;
  int64_t count = 1;  // blocks of this shape
  bool same(const BlockShape& o) const {
    return mext == o.mext && next == o.next && pairs == o.pairs && chunks16 == o.chunks16 && chunks32 == o.chunks32 && kext == o.kext;
  }
  bool operator<(const BlockShape& o) const {
    return std::tie(mext, next, pairs, chunks16, chunks32, kext) < std::tie(o.mext, o.next, o.pairs, o.chunks16, o.chunks32, o.kext);
  }
};

// Equal shapes together.
void merge_shapes(std::vector<BlockShape>& v) {
  std::sort(v.begin(), v.end());
  size_t n = 0;
  for (size_t i = 0; i < v.size(); ++i) {
    if (n > 0 && v[n - 1].same(v[i])) v[n - 1].count += v[i].count;
    else v[n++] = v[i];
  }
  v.resize(n);
}

// What launches of one plan share in its workspace, and how they are kept apart when they overlap.
// Counter sets of persistent launches: the later one's clearing would hand items of the earlier one
// out again.  Eager launches take the first kEagerSets in turn, each after the last launch on its set
// (an event, so that any stream may come next).  A captured launch replays with its set whenever the
// graph runs, so it gets one of the others for good; when those are used up it runs as a plain launch.
// Partial sums, of which there is one set: eager launches come one after another (`serial`).
constexpr int kEagerSets = 8, kCapturedSets = 24;
struct SharedSets {
  std::mutex mu;                     // launches of one plan from several threads
  hipEvent_t done[kEagerSets] = {};  // end of the last eager launch on the set
  int device = -1;                   // of the events
  int next = 0, captured = 0;

  ~SharedSets() { drop_events(); }
  void drop_events() {
    for (hipEvent_t& e : done) {
      if (e) (void)hipEventDestroy(e);
      e = nullptr;
    }
  }
  // The counter set of a launch on s, which may run when s gets there; -1: none is left.
  int take(hipStream_t s, bool counters, bool serial, int* set) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) != hipSuccess) {
      (void)hipGetLastError();
      *set = -1;
      return TAMM_OK;
    }
    if (status != hipStreamCaptureStatusNone) {
      *set = counters && captured < kCapturedSets ? kEagerSets + captured++ : -1;
      return TAMM_OK;
    }
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != device) drop_events();  // the workspace moved to another device
    device = dev;
    *set = serial ? 0 : next;
    next = (*set + 1) % kEagerSets;
    if (done[*set]) HIP_TRY(hipStreamWaitEvent(s, done[*set], 0));
    else HIP_TRY(hipEventCreateWithFlags(&done[*set], hipEventDisableTiming));
    return TAMM_OK;
  }
  int launched(int set, hipStream_t s) {
    if (set >= 0 && set < kEagerSets) HIP_TRY(hipEventRecord(done[set], s));
    return TAMM_OK;
  }
};

}  // namespace

struct tamm_plan {
  tamm_tensor* out = nullptr;
  const tamm_tensor* lhs = nullptr;
  const tamm_tensor* rhs = nullptr;
  const tamm_tensor* A = nullptr;  // the operand whose labels are M + K
  const tamm_tensor* B = nullptr;
  bool swapped = false;
  tamm_precision prec = TAMM_PREC_F64;
  std::vector<Label> labels;
  std::vector<int> M, N, K;        // label indices in flattening order (last fastest)
  std::vector<int> k_lhs_order;    // for each K label in lhs order: its position in K
  bool a_kc = true, b_kc = true;
  bool pairs = false;              // every gathered pair of table entries is adjacent (16-byte loads)
  bool planes = false;             // split-bfloat16 operands in the planes layout
  std::vector<int32_t> pool;
  ScreenDesc sd{};                 // device pointers filled when bound
  int64_t n_kt = 1;
  std::vector<OutBlockDesc> blocks;
  std::vector<double> block_cost;  // sum of K extents of the surviving pairs of each block
  std::vector<BlockShape> block_shapes;  // of each block
  std::vector<BlockShape> shapes;  // the distinct ones and how many blocks have each
  uint64_t signature = 0;
  // split-bfloat16 precisions: per stored operand block, the split work description
  std::vector<PrepBlock> prepA, prepB;
  int64_t prepA_items = 0, prepB_items = 0;
  // operands the caller declared constant (tamm_plan_set_constant): their split is reused while
  // it is valid -- taken from the same storage into the current workspace
  bool const_A = false, const_B = false;
  const void* split_src_A = nullptr;  // storage the split of A in the workspace was taken from
  const void* split_src_B = nullptr;
  // kernel configuration and work decomposition
  int config = -1;
  int k_splits = 1;
  int xcd_chunk = -1;              // work items per die chunk (xcd_order); -1: the library default
  int tile_order = 0;              // 0: tiles of a block row by row; 1: grouped by B column panel
  std::vector<WorkItem> work;
  bool queued = false;             // persistent launch over the dies' queues (float64, more items than resident workgroups)
  size_t ws_limit = 0;             // the caller's workspace, when it is fixed (tamm_contract_noalloc); 0: any size
  int32_t queue_begin[kQueues + 1] = {};
  bool serial = false;             // eager launches one after another: they share partial sums
  int queue_grid = 0;              // workgroups of a persistent launch on the device it is bound on
  SharedSets sets;
  std::vector<ReduceItem> reduce;
  tamm_plan_stats stats{};
  // workspace: static layout, then work list, reduce list, partial tiles
  Layout lay;
  size_t off_work = 0, off_reduce = 0, off_queue = 0, off_partial = 0, off_prepA = 0, off_prepB = 0, off_xA = 0, off_xB = 0, ws_size = 0;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  bool ws_bound = false;
  bool screened = false;
  bool executed = false;
};

static int configure_work(tamm_plan* p, int config, int k_splits);

// Gather layout index of a plan's kernels: bit 1 = A k-contiguous, bit 0 = B k-contiguous,
// bit 2 = 16-byte (two-element) gathers.
static int gather_layout(const tamm_plan* p) {
  return 2 * (p->a_kc ? 1 : 0) + (p->b_kc ? 1 : 0) + (p->pairs ? 4 : 0) + (p->planes ? 8 : 0);
}
constexpr int kLayouts = 8;
constexpr int kComputeUnits = 256;  // MI355X

static Layout make_layout(const tamm_plan* p, size_t base) {
  Layout L;
  size_t off = align256(base);
  L.pool = off;
  off = align256(off + p->pool.size() * sizeof(int32_t));
  L.atile = off;
  off = align256(off + p->A->tile_off.size() * sizeof(int64_t));
  L.btile = off;
  off = align256(off + p->B->tile_off.size() * sizeof(int64_t));
  L.blocks = off;
  off = align256(off + p->blocks.size() * sizeof(OutBlockDesc));
  L.pairs = off;
  off = align256(off + p->blocks.size() * (size_t)p->n_kt * sizeof(PairDesc));
  L.counts = off;
  off = align256(off + p->blocks.size() * sizeof(int32_t));
  L.end = off;
  return L;
}

static int upload_static(const tamm_plan* p, char* ws, const Layout& L) {
  HIP_TRY(hipMemcpy(ws + L.pool, p->pool.data(), p->pool.size() * sizeof(int32_t), hipMemcpyHostToDevice));
  HIP_TRY(hipMemcpy(ws + L.atile, p->A->tile_off.data(), p->A->tile_off.size() * sizeof(int64_t), hipMemcpyHostToDevice));
  HIP_TRY(hipMemcpy(ws + L.btile, p->B->tile_off.data(), p->B->tile_off.size() * sizeof(int64_t), hipMemcpyHostToDevice));
  if (!p->blocks.empty())
    HIP_TRY(hipMemcpy(ws + L.blocks, p->blocks.data(), p->blocks.size() * sizeof(OutBlockDesc), hipMemcpyHostToDevice));
  return TAMM_OK;
}

static ScreenDesc screen_desc(const tamm_plan* p, char* ws, const Layout& L) {
  ScreenDesc s = p->sd;
  s.a_tile_off = (const int64_t*)(ws + L.atile);
  s.b_tile_off = (const int64_t*)(ws + L.btile);
  s.blocks = (const OutBlockDesc*)(ws + L.blocks);
  s.pairs = (PairDesc*)(ws + L.pairs);
  s.counts = (int32_t*)(ws + L.counts);
  s.pool = (const int32_t*)(ws + L.pool);
  s.a_base = 0;
  s.b_base = 0;
  s.pool_base = 0;
  s.pair_stride = (int32_t)p->n_kt;
  s.next_seg = -1;
  s.n_blocks = (int32_t)p->blocks.size();
  return s;
}

static ProblemDesc problem_desc(const tamm_plan* p, char* ws, const Layout& L, double* partial, int k_splits, double alpha,
                                double beta) {
  ProblemDesc d{};
  d.A = p->A->dev;
  d.B = p->B->dev;
  d.C = p->out->dev;
  d.blocks = (const OutBlockDesc*)(ws + L.blocks);
  d.pairs = (const PairDesc*)(ws + L.pairs);
  d.counts = (const int32_t*)(ws + L.counts);
  d.pool = (const int32_t*)(ws + L.pool);
  d.partial = partial;
  d.alpha = alpha;
  d.beta = beta;
  d.k_splits = k_splits;
  d.a_kc = p->a_kc ? 1 : 0;
  d.b_kc = p->b_kc ? 1 : 0;
  return d;
}

extern "C" int tamm_plan_create(tamm_tensor* out, const char* out_lbl, const tamm_tensor* lhs, const char* lhs_lbl,
                                const tamm_tensor* rhs, const char* rhs_lbl, tamm_precision precision, tamm_plan** plan) {
  if (!plan) return fail(TAMM_ERR_ARG, "null output pointer");
  *plan = nullptr;
  if (!out || !lhs || !rhs || !out_lbl || !lhs_lbl || !rhs_lbl) return fail(TAMM_ERR_ARG, "null tensor or label string");
  if (precision != TAMM_PREC_F64 && precision != TAMM_PREC_F32 && precision != TAMM_PREC_BF16X3 &&
      precision != TAMM_PREC_BF16X4_ALIGNED)
    return fail(TAMM_ERR_ARG, "unknown precision %d", (int)precision);
  const tamm_tensor* ts[3] = {out, lhs, rhs};
  const char* ls[3] = {out_lbl, lhs_lbl, rhs_lbl};
  for (int x = 0; x < 3; ++x) {
    const size_t n = strlen(ls[x]);
    if ((int)n != ts[x]->rank)
      return fail(TAMM_ERR_SHAPE, "label string '%s' has %zu letters for a rank-%d tensor", ls[x], n, ts[x]->rank);
    for (size_t i = 0; i < n; ++i) {
      const char c = ls[x][i];
      if (!((c >= 'a' && c <= 'z') || (c >= 'A' && c <= 'Z'))) return fail(TAMM_ERR_LABEL, "label '%c' is not a letter", c);
      for (size_t j = 0; j < i; ++j)
        if (ls[x][j] == c) return fail(TAMM_ERR_LABEL, "label '%c' repeats inside '%s'", c, ls[x]);
    }
  }
  auto p = std::make_unique<tamm_plan>();
  p->out = out;
  p->lhs = lhs;
  p->rhs = rhs;
  p->prec = precision;
  // orientation: the operand holding out's last label becomes B, so output stores run along N
  const char last = out_lbl[out->rank - 1];
  p->swapped = strchr(lhs_lbl, last) != nullptr;
  p->A = p->swapped ? rhs : lhs;
  p->B = p->swapped ? lhs : rhs;
  const char* a_lbl = p->swapped ? rhs_lbl : lhs_lbl;
  const char* b_lbl = p->swapped ? lhs_lbl : rhs_lbl;
  std::map<char, int> idx;
  auto touch = [&](char c) -> Label& {
    auto it = idx.find(c);
    if (it == idx.end()) {
      idx[c] = (int)p->labels.size();
      p->labels.push_back(Label{c});
      return p->labels.back();
    }
    return p->labels[it->second];
  };
  for (int d = 0; d < out->rank; ++d) touch(out_lbl[d]).od = d;
  for (int d = 0; d < p->A->rank; ++d) touch(a_lbl[d]).ad = d;
  for (int d = 0; d < p->B->rank; ++d) touch(b_lbl[d]).bd = d;
  for (auto& L : p->labels) {
    const int n = (L.od >= 0) + (L.ad >= 0) + (L.bd >= 0);
    if (n != 2) return fail(TAMM_ERR_LABEL, "label '%c' appears in %d tensors; each label must appear in exactly two", L.c, n);
    std::shared_ptr<SpaceData> s[3] = {L.od >= 0 ? out->dims[L.od] : nullptr, L.ad >= 0 ? p->A->dims[L.ad] : nullptr,
                                       L.bd >= 0 ? p->B->dims[L.bd] : nullptr};
    for (int x = 0; x < 3; ++x)
      if (s[x]) {
        if (!L.sp) L.sp = s[x];
        else if (!L.sp->same(*s[x])) return fail(TAMM_ERR_LABEL, "label '%c' binds two different tiled spaces", L.c);
      }
    for (int t = 0; t < L.sp->ntiles(); ++t) {
      auto it = std::find(L.cls_size.begin(), L.cls_size.end(), L.sp->size[t]);
      if (it == L.cls_size.end()) {
        L.cls.push_back((int32_t)L.cls_size.size());
        L.cls_size.push_back(L.sp->size[t]);
      } else {
        L.cls.push_back((int32_t)(it - L.cls_size.begin()));
      }
    }
  }
  const int nl = (int)p->labels.size();
  // flattening orders: M and N follow the operand's own dimension order; K follows the operand
  // whose stride-1 label is a K label (A first), so that gathers run along memory.
  std::vector<int> a_dim_label(p->A->rank), b_dim_label(p->B->rank), o_dim_label(out->rank);
  for (int l = 0; l < nl; ++l) {
    if (p->labels[l].ad >= 0) a_dim_label[p->labels[l].ad] = l;
    if (p->labels[l].bd >= 0) b_dim_label[p->labels[l].bd] = l;
    if (p->labels[l].od >= 0) o_dim_label[p->labels[l].od] = l;
  }
  for (int d = 0; d < p->A->rank; ++d)
    if (p->labels[a_dim_label[d]].od >= 0) p->M.push_back(a_dim_label[d]);
  for (int d = 0; d < p->B->rank; ++d)
    if (p->labels[b_dim_label[d]].od >= 0) p->N.push_back(b_dim_label[d]);
  const int a_last = a_dim_label[p->A->rank - 1], b_last = b_dim_label[p->B->rank - 1];
  p->a_kc = p->labels[a_last].od < 0;
  p->b_kc = p->labels[b_last].od < 0;
  if (p->a_kc || !p->b_kc) {
    for (int d = 0; d < p->A->rank; ++d)
      if (p->labels[a_dim_label[d]].od < 0) p->K.push_back(a_dim_label[d]);
  } else {
    for (int d = 0; d < p->B->rank; ++d)
      if (p->labels[b_dim_label[d]].od < 0) p->K.push_back(b_dim_label[d]);
  }
  if (p->K.size() > (size_t)kMaxRank) return fail(TAMM_ERR_UNSUPPORTED, "too many contracted labels");
  for (int i = 0; lhs_lbl[i]; ++i) {
    const int l = idx[lhs_lbl[i]];
    if (p->labels[l].od < 0) p->k_lhs_order.push_back((int)(std::find(p->K.begin(), p->K.end(), l) - p->K.begin()));
  }

  // ---- offset tables per operand shape class ------------------------------------------------
  auto& pool = p->pool;
  struct OpInfo {
    const tamm_tensor* t;
    std::vector<int> dim_label;
    std::vector<int64_t> cstride;  // class-id stride per dim
    int64_t ncls = 1;
  };
  auto op_info = [&](const tamm_tensor* t, const std::vector<int>& dl) {
    OpInfo o{t, dl, std::vector<int64_t>(t->rank, 1), 1};
    for (int d = t->rank - 1; d >= 0; --d) {
      o.cstride[d] = o.ncls;
      o.ncls *= (int64_t)p->labels[dl[d]].cls_size.size();
    }
    return o;
  };
  OpInfo ai = op_info(p->A, a_dim_label), bi = op_info(p->B, b_dim_label), oi = op_info(out, o_dim_label);
  if (ai.ncls + bi.ncls + oi.ncls > 100000) return fail(TAMM_ERR_UNSUPPORTED, "too many distinct block shapes");
  auto build_tables = [&](const OpInfo& o, const std::vector<int>& g1, const std::vector<int>& g2,
                          std::vector<int64_t>& start1, std::vector<int64_t>& start2, bool& pairs1, bool& pairs2) {
    start1.assign(o.ncls, 0);
    start2.assign(o.ncls, 0);
    pairs1 = pairs2 = true;
    std::vector<int64_t> lab_ext(nl, 1), lab_stride(nl, 0);
    for (int64_t c = 0; c < o.ncls; ++c) {
      int64_t stride = 1;
      for (int d = o.t->rank - 1; d >= 0; --d) {
        const Label& L = p->labels[o.dim_label[d]];
        const int64_t cl = (c / o.cstride[d]) % (int64_t)L.cls_size.size();
        lab_ext[o.dim_label[d]] = L.cls_size[cl];
        lab_stride[o.dim_label[d]] = stride;
        stride *= L.cls_size[cl];
      }
      if (stride > INT32_MAX) return false;
      const std::vector<int64_t> t1 = group_table(g1, lab_ext, lab_stride), t2 = group_table(g2, lab_ext, lab_stride);
      pairs1 = pairs1 && pairs_adjacent(t1);
      pairs2 = pairs2 && pairs_adjacent(t2);
      start1[c] = pool_push_table(pool, t1);
      start2[c] = pool_push_table(pool, t2);
      if (pool.size() > (size_t)INT32_MAX / 2) return false;
    }
    return true;
  };
  if (p->A->max_block >= kTableInvalid || p->B->max_block >= kTableInvalid)
    return fail(TAMM_ERR_UNSUPPORTED, "operand blocks of 2^27 or more elements are not supported");
  std::vector<int64_t> aM, aK, bK, bN, oM, oN;
  bool aM_pairs, aK_pairs, bK_pairs, bN_pairs, oM_pairs, oN_pairs;
  if (!build_tables(ai, p->M, p->K, aM, aK, aM_pairs, aK_pairs) || !build_tables(bi, p->K, p->N, bK, bN, bK_pairs, bN_pairs) ||
      !build_tables(oi, p->M, p->N, oM, oN, oM_pairs, oN_pairs))
    return fail(TAMM_ERR_UNSUPPORTED, "a block has more than 2^31 elements or the offset tables are too large");
  // 16-byte gathers pair consecutive k of a k-contiguous operand, consecutive rows otherwise
  p->pairs = (p->a_kc ? aK_pairs : aM_pairs) && (p->b_kc ? bK_pairs : bN_pairs);
  if (precision == TAMM_PREC_BF16X3 || precision == TAMM_PREC_BF16X4_ALIGNED) {
    // split work per stored operand block: rows (M for A, N for B) x K windows
    auto prep_list = [&](const OpInfo& o, const std::vector<int64_t>& rowtab, const std::vector<int64_t>& ktab,
                         const std::vector<int>& rowgroup, bool kc, std::vector<PrepBlock>& list, int64_t& items) {
      const tamm_tensor* t = o.t;
      items = 0;
      for (size_t b = 0; b < t->block_off.size(); ++b) {
        const int32_t* tt = &t->block_tiles[b * t->rank];
        int64_t cls = 0, rows = 1, kext = 1;
        for (int d = 0; d < t->rank; ++d) {
          const Label& L = p->labels[o.dim_label[d]];
          cls += L.cls[tt[d]] * o.cstride[d];
          const bool is_row = std::find(rowgroup.begin(), rowgroup.end(), o.dim_label[d]) != rowgroup.end();
          (is_row ? rows : kext) *= L.sp->size[tt[d]];
        }
        PrepBlock pb{};
        pb.off = t->block_off[b];
        pb.item0 = items;
        pb.rows = (int32_t)rows;
        pb.kext = (int32_t)kext;
        pb.tab_row = (int32_t)rowtab[cls];
        pb.tab_k = (int32_t)ktab[cls];
        pb.nwin = (int32_t)((kext + kSplitWindow - 1) / kSplitWindow);
        items += (kc ? rows : (rows + 63) / 64) * pb.nwin;
        list.push_back(pb);
      }
    };
    prep_list(ai, aM, aK, p->M, p->a_kc, p->prepA, p->prepA_items);
    prep_list(bi, bN, bK, p->N, p->b_kc, p->prepB, p->prepB_items);
    // planes layout (16-byte gathers of 8 consecutive k) when every block's K extent is a
    // multiple of 8; otherwise the packed layout at the float64 offsets
    p->planes = true;
    for (const auto* list : {&p->prepA, &p->prepB})
      for (const PrepBlock& pb : *list) p->planes = p->planes && pb.kext % 8 == 0;
  }
  ScreenDesc& sd = p->sd;
  memset(&sd, 0, sizeof(sd));
  sd.a_cls_tabM = pool_push(pool, aM);
  sd.a_cls_tabK = pool_push(pool, aK);
  sd.b_cls_tabK = pool_push(pool, bK);
  sd.b_cls_tabN = pool_push(pool, bN);
  sd.nk = (int)p->K.size();
  p->n_kt = 1;
  for (int q = 0; q < sd.nk; ++q) {
    const Label& L = p->labels[p->K[q]];
    sd.k_ntiles[q] = L.sp->ntiles();
    p->n_kt *= L.sp->ntiles();
    sd.a_tstride[q] = (int32_t)p->A->tstride[L.ad];
    sd.b_tstride[q] = (int32_t)p->B->tstride[L.bd];
    sd.a_cstride[q] = (int32_t)ai.cstride[L.ad];
    sd.b_cstride[q] = (int32_t)bi.cstride[L.bd];
    sd.k_size_tab[q] = pool_push(pool, L.sp->size);
    std::vector<int64_t> cls(L.cls.begin(), L.cls.end());
    sd.k_cls_tab[q] = pool_push(pool, cls);
  }
  if (p->n_kt > (1 << 20)) return fail(TAMM_ERR_UNSUPPORTED, "too many contracted tile tuples");
  sd.n_kt = (int32_t)p->n_kt;

  // ---- output blocks and host structural screening statistics ------------------------------
  const int64_t nob = (int64_t)out->block_off.size();
  if (nob * p->n_kt > (int64_t)1 << 28) return fail(TAMM_ERR_UNSUPPORTED, "pair capacity too large");
  p->blocks.resize(nob);
  p->block_cost.assign(nob, 0.0);
  double flops = 0;
  int64_t tasks = 0;
  p->shapes.resize(nob);
  for (int64_t b = 0; b < nob; ++b) {
    const int32_t* ot = &out->block_tiles[b * out->rank];
    OutBlockDesc& d = p->blocks[b];
    memset(&d, 0, sizeof(d));
    d.c_off = out->block_off[b];
    int64_t mext = 1, next = 1, ocls = 0;
    for (int l : p->M) mext *= p->labels[l].sp->size[ot[p->labels[l].od]];
    for (int l : p->N) next *= p->labels[l].sp->size[ot[p->labels[l].od]];
    for (int dd = 0; dd < out->rank; ++dd) ocls += p->labels[o_dim_label[dd]].cls[ot[dd]] * oi.cstride[dd];
    d.mext = (int32_t)mext;
    d.next = (int32_t)next;
    d.c_tabM = (int32_t)oM[ocls];
    d.c_tabN = (int32_t)oN[ocls];
    int64_t atb = 0, btb = 0, acb = 0, bcb = 0;
    for (int l : p->M) {
      const Label& L = p->labels[l];
      atb += ot[L.od] * p->A->tstride[L.ad];
      acb += L.cls[ot[L.od]] * ai.cstride[L.ad];
    }
    for (int l : p->N) {
      const Label& L = p->labels[l];
      btb += ot[L.od] * p->B->tstride[L.bd];
      bcb += L.cls[ot[L.od]] * bi.cstride[L.bd];
    }
    d.a_tbase = (int32_t)atb;
    d.b_tbase = (int32_t)btb;
    d.a_cbase = (int32_t)acb;
    d.b_cbase = (int32_t)bcb;
    d.pair_base = (int32_t)(b * p->n_kt);
    // host count of surviving pairs (statistics and scheduling cost; the kernels use the pair
    // list produced by the GPU screen)
    for (int64_t kt = 0; kt < p->n_kt; ++kt) {
      int64_t rem = kt, alin = atb, blin = btb, kext = 1;
      for (int q = sd.nk - 1; q >= 0; --q) {
        const int t = (int)(rem % sd.k_ntiles[q]);
        rem /= sd.k_ntiles[q];
        alin += (int64_t)t * sd.a_tstride[q];
        blin += (int64_t)t * sd.b_tstride[q];
        kext *= p->labels[p->K[q]].sp->size[t];
      }
      if (p->A->tile_off[alin] >= 0 && p->B->tile_off[blin] >= 0) {
        ++tasks;
        flops += 2.0 * (double)mext * (double)next * (double)kext;
        p->block_cost[b] += (double)kext;
        BlockShape& sh = p->shapes[b];
        ++sh.pairs;
        sh.chunks16 += (kext + 15) / 16;
        sh.chunks32 += (kext + 31) / 32;
      }
    }
    p->shapes[b].mext = mext;
    p->shapes[b].next = next;
    p->shapes[b].kext = p->block_cost[b];
  }
  p->block_shapes = p->shapes;
  merge_shapes(p->shapes);
  // dropped pairs: surviving pairs whose output block is not stored (user predicates only)
  int64_t dropped = 0;
  {
    std::vector<int32_t> ot(out->rank);
    const int64_t ntup = (int64_t)out->tile_off.size();
    for (int64_t lin = 0; lin < ntup; ++lin) {
      if (out->tile_off[lin] >= 0) continue;
      int64_t rem = lin;
      for (int dd = out->rank - 1; dd >= 0; --dd) {
        ot[dd] = (int32_t)(rem % out->dims[dd]->ntiles());
        rem /= out->dims[dd]->ntiles();
      }
      int64_t atb = 0, btb = 0;
      for (int l : p->M) atb += ot[p->labels[l].od] * p->A->tstride[p->labels[l].ad];
      for (int l : p->N) btb += ot[p->labels[l].od] * p->B->tstride[p->labels[l].bd];
      for (int64_t kt = 0; kt < p->n_kt; ++kt) {
        int64_t r2 = kt, alin = atb, blin = btb;
        for (int q = sd.nk - 1; q >= 0; --q) {
          const int t = (int)(r2 % sd.k_ntiles[q]);
          r2 /= sd.k_ntiles[q];
          alin += (int64_t)t * sd.a_tstride[q];
          blin += (int64_t)t * sd.b_tstride[q];
        }
        if (p->A->tile_off[alin] >= 0 && p->B->tile_off[blin] >= 0) ++dropped;
      }
    }
  }
  tamm_plan_stats& st = p->stats;
  st.out_blocks = nob;
  st.candidates = nob * p->n_kt;
  st.tasks = tasks;
  st.dropped = dropped;
  st.useful_flops = flops;
  st.algorithmic_bytes = 8.0 * ((double)lhs->numel + (double)rhs->numel + 2.0 * (double)out->numel);
  // structural signature (autotuner cache key)
  uint64_t h = 0xCBF29CE484222325ULL;
  const int32_t hdr[6] = {(int32_t)p->M.size(), (int32_t)p->N.size(), (int32_t)p->K.size(), (int32_t)p->a_kc,
                          (int32_t)p->b_kc, (int32_t)precision};
  h = fnv(h, hdr, sizeof(hdr));
  for (int l : p->M) h = fnv(h, p->labels[l].sp->size.data(), p->labels[l].sp->size.size() * 8);
  for (int l : p->N) h = fnv(h, p->labels[l].sp->size.data(), p->labels[l].sp->size.size() * 8);
  for (int l : p->K) h = fnv(h, p->labels[l].sp->size.data(), p->labels[l].sp->size.size() * 8);
  h = fnv(h, &tasks, sizeof(tasks));
  h = fnv(h, &nob, sizeof(nob));
  h = fnv(h, p->block_cost.data(), p->block_cost.size() * sizeof(double));
  p->signature = h;
  int rc = configure_work(p.get(), -1, 0);
  if (rc != TAMM_OK) return rc;
  *plan = p.release();
  return ok();
}

// Kernel configuration tables by precision.
struct TileCfg {
  int mt, nt, kt, threads;
  int um, un;  // rows and columns of one step of the tile size (16 per wave along the dimension)
  int resident;  // workgroups that fit on a compute unit
  double rate;   // flop/s of the whole chip on large blocks (of the products asked for, not of their slices)
  const char* name;
};

static int cfg_count(int prec) { return prec == TAMM_PREC_F64 ? f64_config_count() : mixed_config_count(prec); }

// planes: rates of the split-bfloat16 kernels on the planes layout, else on the packed one
static TileCfg cfg_get(int prec, int c, bool planes = false) {
  if (prec == TAMM_PREC_F64) {
    const F64Config& f = f64_config(c);
    return TileCfg{f.mt, f.nt, f.kt, 64 * f.wgm * f.wgn, 16 * f.wgm, 16 * f.wgn, f.resident, f.tflops * 1e12, f.name};
  }
  const MixedConfig& f = mixed_config(prec, c);
  // three slices multiply 6 pairs instead of 10, on the same gathers
  const double rate = (planes ? f.tflops_planes : f.tflops) * (prec == TAMM_PREC_BF16X3 ? 1.35e12 : 1e12);
  return TileCfg{f.mt, f.nt, f.kt, 64 * f.wgm * f.wgn, f.mt, f.nt, f.resident, rate, f.name};
}

// Number of output tiles of one configuration.
static int64_t tiles_for(const tamm_plan* p, int c) {
  const TileCfg f = cfg_get(p->prec, c);
  int64_t n = 0;
  for (const auto& b : p->blocks) n += (int64_t)((b.mext + f.mt - 1) / f.mt) * ((b.next + f.nt - 1) / f.nt);
  return n;
}

// K splits of a block's tiles: in proportion to its summed K extent, the heaviest blocks' get
// k_splits parts, lighter ones fewer (at least one), so that the parts cost about the same.
static int block_splits(int k_splits, double kext, double max_kext) {
  if (k_splits <= 1 || max_kext <= 0) return 1;
  return (int)std::min<double>(k_splits, std::max(1.0, std::floor(k_splits * kext / max_kext + 0.5)));
}

// Estimated time in microseconds of a contraction over blocks of these shapes: the larger of
// the longest item and the items' sum over the resident workgroups plus part of an item for the
// tail, at least the time of the unavoidable traffic.  An item takes, per chunk of summed
// indices, its products at the configuration's rate or one memory round trip, whichever is longer;
// per pair and per item a few dependent loads, and an epilogue that grows with the tile.  The constants
// were fitted to 108 contractions (3 kF to 6 TF, tiles of 3 to 64) timed with every configuration and
// 1 to 16 K splits: taking the configuration with the least estimate costs 4 % against the best one
// of each on average (up to 20 %), the rule before it (largest tile, no padding, two tiles per
// compute unit) 14 % (up to 63 %).  The reduced precisions share them but for split bfloat16's
// tail, whose few large workgroups leave more of it; over 26 contractions in each of them the least
// estimate costs 2-3 %, the rule before it 15 % in float32 and 20-40 % in split bfloat16, which it ran
// on four-wave tiles.
constexpr double kRoundTrip16 = 0.60, kRoundTrip32 = 0.70, kRoundTripWave = 0.78;  // a chunk of 16, of 32, of a one-wave workgroup
constexpr double kPair = 0.137, kItem = 3.84, kPer1024 = 0.63, kTail = 0.42, kTailSplit = 0.7;
constexpr double kReduce = 5.6, kReduceBytes = 5.0e6;  // launch, bytes per microsecond

static double item_us(const BlockShape& b, const TileCfg& f, double area, double parts) {
  const double rate = f.rate * 1e-6 / ((double)f.resident * kComputeUnits);  // flop per microsecond of a resident workgroup
  const double lat = f.threads == 64 ? kRoundTripWave : (f.kt == 32 ? kRoundTrip32 : kRoundTrip16);
  const double chunks = (double)(f.kt == 32 ? b.chunks32 : b.chunks16);
  return (chunks * std::max(2.0 * area * f.kt / rate, lat) + (double)b.pairs * kPair) / parts + kItem + kPer1024 * area / 1024.0;
}

// Tiles of at most tm x tn of the blocks of one shape: fn(rows, columns, how many).
template <typename F>
static void for_tiles(const BlockShape& b, const TileCfg& f, int64_t tm, int64_t tn, F&& fn) {
  const int64_t nm = (b.mext + tm - 1) / tm, um = (b.mext + f.um - 1) / f.um;  // tiles and units of the rows
  const int64_t nn = (b.next + tn - 1) / tn, un = (b.next + f.un - 1) / f.un;
  for (int hm = 0; hm < 2; ++hm)  // tiles of um / nm units, and the um % nm tiles of one more
    for (int hn = 0; hn < 2; ++hn) {
      const double n = (double)((hm ? um % nm : nm - um % nm) * (hn ? un % nn : nn - un % nn) * b.count);
      if (n > 0) fn((double)((um / nm + hm) * f.um), (double)((un / nn + hn) * f.un), n);
    }
}

static double estimate_us(const std::vector<BlockShape>& shapes, const TileCfg& f, int k_splits, double bytes, double tail) {
  const double slots = (double)f.resident * kComputeUnits;
  double max_kext = 0, total = 0, longest = 0, items = 0, partial = 0;
  for (const BlockShape& b : shapes) max_kext = std::max(max_kext, b.kext);
  for (const BlockShape& b : shapes) {
    const int ns = block_splits(k_splits, b.kext, max_kext);
    const double parts = (double)std::min<int64_t>(ns, std::max<int64_t>(1, b.pairs));  // a pair is never cut
    for_tiles(b, f, f.mt, f.nt, [&](double rows, double cols, double n) {
      const double t = item_us(b, f, rows * cols, parts);
      total += t * n * parts;
      items += n * parts;
      longest = std::max(longest, t);
    });
    if (ns > 1) partial += (double)(b.mext * b.next * b.count) * ns;
  }
  double t = items > slots ? std::max(longest, total / slots + tail * longest) : longest;
  t = std::max(t, bytes / (f.resident > 2 ? 4.8e6 : 3.8e6));  // what copies reach with many and with few workgroups in flight
  return t + (partial > 0 ? kReduce + partial * 16.0 / kReduceBytes : 0.0);
}

// Groups run without K splits, so a member with few output elements and long sums (the hole-hole
// intermediate) would hold a launch up with a handful of long items.  Its tiles are cut smaller: the
// largest tile, halved along its longer side down to 32 or one unit, whose item takes at most `limit`
// us.  (No more tiles than the 32 x 32 configuration has, which the workspace has room for.)
static std::pair<int32_t, int32_t> group_tile(const BlockShape& b, const TileCfg& f, double limit) {
  int32_t tm = f.mt, tn = f.nt;
  while (item_us(b, f, (double)std::min<int64_t>(tm, b.mext) * (double)std::min<int64_t>(tn, b.next), 1.0) > limit) {
    const int32_t um = std::max(f.um, 32), un = std::max(f.un, 32);
    const bool rows = (tm > um && (tm >= tn || tn <= un));
    if (!rows && tn <= un) break;
    int32_t& side = rows ? tm : tn;
    const int32_t unit = rows ? um : un;
    side = std::max(unit, side / 2 / unit * unit);
  }
  return std::make_pair(tm, tn);
}

// The limit of group_tile for the members of one launch: the launch's time if evenly spread.  (Of
// 0.4, 0.7 and 1 times that, 1 gave the best mean over 17 schedules and groups.  Whole tiles leave the
// hole-hole intermediate's launch 1.4 times as long at O=26, V=102, and make the ladder's at O=29,
// V=135 in tiles of 19 and 37 5 % shorter: group_default_config estimates both.)
static double group_limit_us(const std::vector<BlockShape>& shapes, const TileCfg& f) {
  double total = 0;
  for (const BlockShape& b : shapes)
    for_tiles(b, f, f.mt, f.nt, [&](double rows, double cols, double n) { total += item_us(b, f, rows * cols, 1.0) * n; });
  return total / ((double)f.resident * kComputeUnits);
}

// End of a launch whose slots take the items, longest first, one after another.  Items and slots are
// counted by classes of equal time.
struct ItemClass {
  double us, n;
};
static double longest_first_us(std::vector<ItemClass>& items, double slots) {
  std::sort(items.begin(), items.end(), [](const ItemClass& x, const ItemClass& y) { return x.us > y.us; });
  using Slots = std::pair<double, double>;  // when they are free, how many
  std::priority_queue<Slots, std::vector<Slots>, std::greater<Slots>> free;
  free.push(Slots(0.0, slots));
  double end = 0;
  for (const ItemClass& c : items)
    for (double left = c.n; left > 0;) {
      const Slots s = free.top();
      const double n = std::min(left, s.second);
      free.pop();
      if (s.second > n) free.push(Slots(s.first, s.second - n));
      free.push(Slots(s.first + c.us, n));
      end = std::max(end, s.first + c.us);
      left -= n;
    }
  return end;
}

// Estimated time of a group's launch over blocks of these shapes, whole tiles or cut ones.  A launch
// without K splits has few rounds of items, and cut tiles are slower than their area says, which the
// plans' estimate (sum over the slots plus part of an item) does not see: with it one contraction in a
// group lost 10 % to the best configuration and cut (78 contractions, 16 choices each), up to 72 %, and 20 of
// 48 were slower than with the rule of least padding before it (ladder at O=31, V=126 in tiles of 16 and 42
// 1.55 -> 2.29 ms).  Here the products' rate falls with a tile's perimeter over its area, the items are
// dealt out longest first, and slots that fall idle leave their share of the compute unit to the others
// (kGroupShare of the idle time): 3.5 % lost, up to 40 %.  Constants fitted to the same measurements.
constexpr double kGroupArea = 0.0124, kGroupPerimeter = 0.240;  // us per MFLOP of the chip, times 1 and perimeter / 2 / area
constexpr double kGroupTrip16 = 0.54, kGroupTrip32 = 0.60, kGroupTripWave = 0.92;
constexpr double kGroupPair = 0.151, kGroupItem = 2.09, kGroupPer1024 = 0.735, kGroupShare = 0.58;
static double group_estimate_us(const std::vector<BlockShape>& shapes, const TileCfg& f, double bytes, bool cut) {
  const double slots = (double)f.resident * kComputeUnits, limit = cut ? group_limit_us(shapes, f) : 1e300;
  const double trip = f.threads == 64 ? kGroupTripWave : (f.kt == 32 ? kGroupTrip32 : kGroupTrip16);
  double total = 0, n_items = 0, alone = 0, longest = 0;  // alone: the longest item with a compute unit to itself
  std::vector<ItemClass> items;
  for (const BlockShape& b : shapes) {
    const auto tile = group_tile(b, f, limit);
    const double chunks = (double)(f.kt == 32 ? b.chunks32 : b.chunks16);
    for_tiles(b, f, tile.first, tile.second, [&](double rows, double cols, double n) {
      const double area = rows * cols;
      const double unit = 2.0 * area * f.kt * (kGroupArea + kGroupPerimeter * (rows + cols) / area) * 1e-6 * kComputeUnits;
      const double rest = (double)b.pairs * kGroupPair + kGroupItem + kGroupPer1024 * area / 1024.0;
      const double t = chunks * std::max(unit * f.resident, trip) + rest;
      items.push_back(ItemClass{t, n});
      total += t * n;
      n_items += n;
      longest = std::max(longest, t);
      alone = std::max(alone, chunks * std::max(unit, trip) + rest);
    });
  }
  double t = alone;
  if (n_items > kComputeUnits) {
    // of many rounds the last leaves half an item's time on average
    const double even = total / slots, end = n_items > 16 * slots ? even + 0.5 * longest : longest_first_us(items, slots);
    t = std::max(alone, end - kGroupShare * (end - even));
  }
  return std::max(t, bytes / (f.resident > 2 ? 4.8e6 : 3.8e6));
}

// Workspace layout of a plan: static tables and pair lists, work list, reduce list, queue counters,
// partial tiles, and for the split-bfloat16 precisions the split operands.
static void layout_workspace(tamm_plan* p, const TileCfg& f, size_t items, size_t reduces, size_t partials, bool queued) {
  p->lay = make_layout(p, 0);
  size_t off = p->lay.end;
  p->off_work = off;
  off = align256(off + items * sizeof(WorkItem));
  p->off_reduce = off;
  off = align256(off + reduces * sizeof(ReduceItem));
  p->off_queue = off;
  if (queued) off = align256(off + (kEagerSets + kCapturedSets) * kQueues * sizeof(int32_t));
  p->off_partial = off;
  if (partials > 0) off = align256(off + partials * f.mt * f.nt * sizeof(double));
  if (p->prec == TAMM_PREC_BF16X3 || p->prec == TAMM_PREC_BF16X4_ALIGNED) {
    p->off_prepA = off;
    off = align256(off + p->prepA.size() * sizeof(PrepBlock));
    p->off_prepB = off;
    off = align256(off + p->prepB.size() * sizeof(PrepBlock));
    p->off_xA = off;
    off = align256(off + (size_t)p->A->numel * sizeof(uint64_t));
    p->off_xB = off;
    off = align256(off + (size_t)p->B->numel * sizeof(uint64_t));
  }
  p->ws_size = std::max<size_t>(off, 256);
}

// Workspace sizes of a plan's configurations, without building their work lists.
struct WorkspaceSizes {
  tamm_plan size_only;
  const std::vector<BlockShape>& shapes;
  double max_kext = 0;

  explicit WorkspaceSizes(const tamm_plan* p) : shapes(p->shapes) {
    size_only.A = p->A;
    size_only.B = p->B;
    size_only.prec = p->prec;
    size_only.pool.resize(p->pool.size());
    size_only.blocks.resize(p->blocks.size());
    size_only.n_kt = p->n_kt;
    size_only.prepA.resize(p->prepA.size());
    size_only.prepB.resize(p->prepB.size());
    for (const BlockShape& b : shapes) max_kext = std::max(max_kext, b.kext);
  }
  // 0: configure_work refuses it
  size_t bytes(const TileCfg& f, int k_splits, bool queued) {
    size_t items = 0, reduces = 0, partials = 0;
    for (const BlockShape& b : shapes) {
      const int ns = block_splits(k_splits, b.kext, max_kext);
      const size_t tiles = (size_t)(((b.mext + f.mt - 1) / f.mt) * ((b.next + f.nt - 1) / f.nt) * b.count);
      items += tiles * ns;
      if (ns > 1) reduces += tiles;
      if (ns > 1) partials += tiles * ns;
    }
    if (partials > (size_t)INT32_MAX / 2 || items > (size_t)INT32_MAX / 2) return 0;
    layout_workspace(&size_only, f, items, reduces, partials, queued);
    return size_only.ws_size;
  }
};

// The largest workspace of any configuration with 1, 2, .. max_splits K splits.
size_t tamm::plan_candidate_workspace(const tamm_plan* p, int max_splits) {
  WorkspaceSizes sizes(p);
  size_t most = 0;
  for (int c = 0; c < cfg_count(p->prec); ++c) {
    if (p->prec == TAMM_PREC_F64 && f64_config_canonical(c) != c) continue;
    const TileCfg f = cfg_get(p->prec, c);
    for (int ks = 1; ks <= max_splits; ks *= 2) most = std::max(most, sizes.bytes(f, ks, p->prec == TAMM_PREC_F64));
  }
  return most;
}

// Default configuration and K splits of a plan: the least estimate.  More splits only where they are
// estimated to gain 3 %, and in float64 8 % above a millisecond: of long launches the estimate tells the
// splits that gain from those that lose too poorly, since the dies' queues fill part of the tail (128 x 128
// tiles in 1, 2 and 4 parts: ladder at O=40, V=200 13.1, 12.6 and 13.3 ms; at O=32, V=160 3.07, 3.11 and
// 3.38, its gradients 3.26, 4.22 and 8.26 and 3.09, 3.12 and 3.45; ring at O=40, V=200 2.49, 2.66 and 2.73).
// Never of sums shorter than eight chunks in float64 and float32: what they gain is what ordering
// overlapping executions costs, see `starved` (ring at O=5, V=45 16 us in four parts, 19 in one, 20 in four
// with the event; in split bfloat16 at O=9, V=37 35, 43 and 38).  The partial tiles take at most an eighth
// of the tensors' bytes or 64 MiB, and the whole workspace no more than the plan's limit.
static std::pair<int, int> default_work(const tamm_plan* p, int config, int k_splits) {
  const bool f64 = p->prec == TAMM_PREC_F64, split_bf16 = !f64 && p->prec != TAMM_PREC_F32;
  const double bytes = p->stats.algorithmic_bytes, budget = std::max(bytes / 8, (double)(64 << 20));
  double best = 1e300, max_kext = 0;
  std::pair<int, int> pick(std::max(config, 0), std::max(k_splits, 1));
  for (const BlockShape& b : p->shapes) max_kext = std::max(max_kext, b.kext);
  const bool short_sums = !split_bf16 && max_kext < 8 * 16;
  std::unique_ptr<WorkspaceSizes> sizes;
  if (p->ws_limit > 0) sizes = std::make_unique<WorkspaceSizes>(p);
  size_t smallest = SIZE_MAX;
  for (int ks : {1, 2, 4, 8, 16}) {
    if (ks > 1 && (k_splits > 0 || short_sums)) break;
    const int splits = k_splits > 0 ? k_splits : ks;
    double least = 1e300;
    int at = -1;
    for (int c = 0; c < cfg_count(p->prec); ++c) {
      if (config >= 0 ? c != config : f64 && f64_config_canonical(c) != c) continue;
      const TileCfg f = cfg_get(p->prec, c, p->planes);
      double need = 0;
      for (const BlockShape& b : p->shapes) {
        const int ns = block_splits(splits, b.kext, max_kext);
        if (ns > 1) need += 8.0 * f.mt * f.nt * ns * (double)(((b.mext + f.mt - 1) / f.mt) * ((b.next + f.nt - 1) / f.nt) * b.count);
      }
      if (k_splits <= 0 && need > budget) continue;
      if (sizes) {  // a fixed workspace: what fits, or the smallest (the caller refuses it)
        const size_t n = sizes->bytes(f, splits, false);
        if (n == 0 || n > p->ws_limit) {
          if (n > 0 && best == 1e300 && n < smallest) {
            smallest = n;
            pick = std::make_pair(c, splits);
          }
          continue;
        }
      }
      const double t = estimate_us(p->shapes, f, splits, bytes, split_bf16 ? kTailSplit : kTail);
      if (t < least) {
        least = t;
        at = c;
      }
    }
    if (at >= 0 && least < (f64 && best > 1000.0 ? 0.92 : 0.97) * best) {
      best = least;
      pick = std::make_pair(at, splits);
    }
  }
  return pick;
}

// Extents of the tiles that cover `ext` rows (or columns): as many as whole tiles of `tile` would
// take, of even sizes in whole `unit`s (16 rows for every wave along the dimension, the step in
// which the float64 kernels' tile bodies come), the last one ending with the block.  A sliver of a
// tile left at the end of a block would cost the loads, barriers and epilogue of a whole one.
static void cut_extent(int32_t ext, int32_t tile, int32_t unit, std::vector<int32_t>& out) {
  out.clear();
  const int32_t n = (ext + tile - 1) / tile, units = (ext + unit - 1) / unit;
  int32_t at = 0;
  for (int32_t i = 0; i < n; ++i) {
    const int32_t end = std::min(ext, (int32_t)((int64_t)units * (i + 1) / n) * unit);
    out.push_back(end - at);
    at = end;
  }
}

// Launch order of the work items for the chip's eight accelerator dies (XCDs), each with its own
// L2: the dispatcher hands workgroup b to die b % 8.  The longest-first list is cut into chunks of
// `chunk` consecutive items (neighbouring tiles of one output block, which share operand panels)
// and chunk c goes to die c % 8, so every die works through whole chunks in longest-first order
// and tiles that read the same rows of A or columns of B run together behind one L2.  Slots left
// empty by dies with fewer items are squeezed out, which only moves a few tail items to another
// die.  A chunk of 0 or 1 keeps the list as it is.
static void xcd_order(std::vector<WorkItem>& work, size_t first, int chunk) {  // items from `first` on
  constexpr int kDies = 8;
  const size_t n = work.size() - first;
  if (chunk <= 1 || n <= (size_t)kDies) return;
  const size_t nchunks = (n + chunk - 1) / chunk;
  std::vector<size_t> len(kDies, 0);
  for (size_t c = 0; c < nchunks; ++c) len[c % kDies] += std::min<size_t>(chunk, n - c * chunk);
  const size_t rows = *std::max_element(len.begin(), len.end());
  std::vector<int64_t> slot(rows * kDies, -1);
  for (int x = 0; x < kDies; ++x)
    for (size_t i = 0; i < len[x]; ++i) {
      const size_t c = (size_t)x + kDies * (i / chunk);  // the die's (i / chunk)-th chunk
      slot[i * kDies + x] = (int64_t)(c * chunk + i % chunk);
    }
  std::vector<WorkItem> out;
  out.reserve(n);
  for (int64_t l : slot)
    if (l >= 0) out.push_back(work[first + (size_t)l]);
  std::copy(out.begin(), out.end(), work.begin() + first);
}

// The same chunks as the queues of a persistent launch: chunk c of the longest-first list goes to
// queue c % 8, each queue's chunks in list order (chunks of 0 or 1: item by item).  A workgroup takes its next item when it has ended
// the last, so unequal items leave no slot empty until the queues run dry; the dispatcher, handing
// out one workgroup per item in a fixed rotation, kept 76-92 % of the slots busy (ladder at O=40,
// V=200, K splits 4 and 1).
static void queue_order(std::vector<WorkItem>& work, size_t first, int chunk, int32_t* begin) {
  const size_t n = work.size() - first, step = std::max(1, chunk);
  std::vector<WorkItem> out;
  out.reserve(n);
  for (int x = 0; x < kQueues; ++x) {
    begin[x] = (int32_t)out.size();
    for (size_t c = x * step; c < n; c += kQueues * step)
      for (size_t i = c; i < std::min(n, c + step); ++i) out.push_back(work[first + i]);
  }
  begin[kQueues] = (int32_t)out.size();
  std::copy(out.begin(), out.end(), work.begin() + first);
}

// Whether a persistent launch pays: more items than resident workgroups, and items long enough.
// Taking an item costs two barriers and an atomic that goes past the dies' L2s, about 2 us; items of
// a few microseconds lost a factor of two and more by it (the T1 terms at O=40, V=200: 0.10 -> 0.24
// and 0.28 -> 0.43 ms), items of 190 us and more gained (hh 0.62 -> 0.57, ring 2.76 -> 2.53 ms).
static bool queue_pays(double flops, size_t items, const TileCfg& f) {
  const size_t slots = (size_t)f.resident * kComputeUnits;
  return items > slots && flops / (double)items / (f.rate / (double)slots) >= 40e-6;
}

static int xcd_chunk() {
  static const int v = [] {
    const char* e = getenv("TAMM_XCD_CHUNK");
    return e ? std::max(0, atoi(e)) : 32;
  }();
  return v;
}

// An output of fewer than two 128 x 128 tiles per compute unit, and sums of eight chunks and more: only
// K splits fill the chip, and executions that overlap are the caller's to order.  Other plans gain by
// splits, too, but their executions are ordered by an event (3 us of 56 and more for float64 gradients
// at O=13, V=81 and larger contractions): a program may run them on several streams, with out bound to
// other storage in between, and need not know of the partial sums.
static bool starved(const tamm_plan* p) {
  int64_t tiles = 0;
  double max_kext = 0;
  for (const BlockShape& b : p->shapes) {
    tiles += ((b.mext + 127) / 128) * ((b.next + 127) / 128) * b.count;
    max_kext = std::max(max_kext, b.kext);
  }
  return tiles < 2 * kComputeUnits && max_kext >= 8 * (p->prec <= TAMM_PREC_F32 ? 16 : 32);
}

// Work decomposition for one kernel configuration: macro-tiles of every stored output block,
// heaviest first (longest-processing-time order), with the K splits of a tile adjacent, then laid
// out for the dies (xcd_order).
static int configure_work(tamm_plan* p, int config, int k_splits) {
  const int ncfg = cfg_count(p->prec);
  const int64_t nob = (int64_t)p->blocks.size();
  if (config >= ncfg) return fail(TAMM_ERR_ARG, "kernel configuration %d does not exist (%d available)", config, ncfg);
  if (config < 0 || k_splits <= 0) std::tie(config, k_splits) = default_work(p, config, k_splits);
  const TileCfg f = cfg_get(p->prec, config);
  const int64_t ntiles = tiles_for(p, config);
  if (k_splits > 64) return fail(TAMM_ERR_ARG, "k_splits must be in [1, 64]");
  struct Tile {
    double cost;
    int32_t ob, m0, n0, rows, cols;
  };
  std::vector<Tile> tiles;
  tiles.reserve(ntiles);
  std::vector<int32_t> cm, cn;
  for (int64_t b = 0; b < nob; ++b) {
    const auto& d = p->blocks[b];
    cut_extent(d.mext, f.mt, f.um, cm);
    cut_extent(d.next, f.nt, f.un, cn);
    int32_t m0 = 0;
    for (int32_t rows : cm) {
      int32_t n0 = 0;
      for (int32_t cols : cn) {
        tiles.push_back(Tile{p->block_cost[b] * rows * cols, (int32_t)b, m0, n0, rows, cols});
        n0 += cols;
      }
      m0 += rows;
    }
  }
  double max_cost = 0;
  for (const Tile& t : tiles) max_cost = std::max(max_cost, p->block_cost[t.ob]);
  struct Part {
    double cost;
    WorkItem w;
  };
  std::vector<Part> parts;
  p->reduce.clear();
  int64_t slots = 0;
  for (const Tile& t : tiles) {
    const int ns = block_splits(k_splits, p->block_cost[t.ob], max_cost);
    for (int s = 0; s < ns; ++s)
      parts.push_back(Part{t.cost / ns, WorkItem{0, t.ob, t.m0, t.n0, item_shape(s, ns, t.rows, t.cols), (int32_t)slots}});
    if (ns > 1) {
      p->reduce.push_back(ReduceItem{0, t.ob, t.m0, t.n0, (int32_t)slots, item_shape(0, ns, t.rows, t.cols)});
      slots += ns;
    }
    if (slots > INT32_MAX / 2) return fail(TAMM_ERR_UNSUPPORTED, "too many partial tiles");
  }
  // longest processing time first; the parts of a tile stay adjacent when their costs tie.  Order
  // 0 keeps the tiles of one block row by row (neighbours share A row panels); order 1 puts the
  // tiles that read the same B column panel -- the same N tiles of their blocks, the same first
  // column -- next to each other across the blocks and rows (for operations whose B panels are the
  // large ones, such as a few output rows against long columns)
  const std::vector<OutBlockDesc>& bd = p->blocks;
  if (p->tile_order == 1)
    std::stable_sort(parts.begin(), parts.end(), [&bd](const Part& x, const Part& y) {
      if (x.cost != y.cost) return x.cost > y.cost;
      const int32_t bx = bd[x.w.ob].b_tbase, by = bd[y.w.ob].b_tbase;
      if (bx != by) return bx < by;
      if (x.w.n0 != y.w.n0) return x.w.n0 < y.w.n0;
      if (x.w.ob != y.w.ob) return x.w.ob < y.w.ob;
      return x.w.m0 < y.w.m0;
    });
  else
    std::stable_sort(parts.begin(), parts.end(), [](const Part& x, const Part& y) { return x.cost > y.cost; });
  p->work.clear();
  for (const Part& q : parts) p->work.push_back(q.w);
  if (p->work.size() > (size_t)INT32_MAX / 2) return fail(TAMM_ERR_UNSUPPORTED, "too many work items");
  const int chunk = p->xcd_chunk >= 0 ? p->xcd_chunk : xcd_chunk();
  p->queued = p->prec == TAMM_PREC_F64 && queue_pays(p->stats.useful_flops, p->work.size(), f);
  if (p->queued && p->ws_limit > 0) {  // the counters must not be what a fixed workspace lacks room for
    layout_workspace(p, f, p->work.size(), p->reduce.size(), (size_t)slots, true);
    p->queued = p->ws_size <= p->ws_limit;
  }
  if (p->queued) queue_order(p->work, 0, chunk, p->queue_begin);
  else xcd_order(p->work, 0, chunk);
  p->serial = k_splits > 1 && !starved(p);
  p->config = config;
  p->k_splits = k_splits;
  p->stats.work_items = (int64_t)p->work.size();
  p->stats.kernel_config = config;
  p->stats.k_splits = k_splits;
  p->stats.xcd_chunk = p->xcd_chunk >= 0 ? p->xcd_chunk : xcd_chunk();
  p->stats.tile_order = p->tile_order;
  p->stats.gather_layout = gather_layout(p);
  p->stats.persistent = p->queued ? 1 : 0;
  layout_workspace(p, f, p->work.size(), p->reduce.size(), (size_t)slots, p->queued);
  p->ws_bound = false;
  p->screened = false;
  p->executed = false;
  return TAMM_OK;
}

extern "C" int tamm_plan_workspace_size(const tamm_plan* p, size_t* bytes) {
  if (!p || !bytes) return fail(TAMM_ERR_ARG, "null argument");
  *bytes = p->ws_size;
  return ok();
}

// Workgroups of a persistent launch: every resident slot of the device (compute units x resident
// workgroups of the configuration), at most one per item.
static int persistent_grid(int config, int layout, int n_work) {
  int dev = 0, cus = kComputeUnits;
  if (hipGetDevice(&dev) == hipSuccess) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
  }
  return std::max(1, std::min<int>(f64_occupancy(config, layout) * cus, n_work));
}

static int bind_plan(tamm_plan* p, void* dev_ptr, size_t bytes) {
  if (!dev_ptr || ((uintptr_t)dev_ptr) % 256) return fail(TAMM_ERR_WORKSPACE, "workspace must be non-null and 256-byte aligned");
  if (bytes < p->ws_size) return fail(TAMM_ERR_WORKSPACE, "workspace of %zu bytes is smaller than the %zu needed", bytes, p->ws_size);
  char* ws = (char*)dev_ptr;
  int rc = upload_static(p, ws, p->lay);
  if (rc != TAMM_OK) return rc;
  if (!p->work.empty()) HIP_TRY(hipMemcpy(ws + p->off_work, p->work.data(), p->work.size() * sizeof(WorkItem), hipMemcpyHostToDevice));
  if (!p->reduce.empty())
    HIP_TRY(hipMemcpy(ws + p->off_reduce, p->reduce.data(), p->reduce.size() * sizeof(ReduceItem), hipMemcpyHostToDevice));
  if (!p->prepA.empty()) HIP_TRY(hipMemcpy(ws + p->off_prepA, p->prepA.data(), p->prepA.size() * sizeof(PrepBlock), hipMemcpyHostToDevice));
  if (!p->prepB.empty()) HIP_TRY(hipMemcpy(ws + p->off_prepB, p->prepB.data(), p->prepB.size() * sizeof(PrepBlock), hipMemcpyHostToDevice));
  if (p->queued) p->queue_grid = persistent_grid(p->config, gather_layout(p), (int)p->work.size());
  p->ws = ws;
  p->ws_bytes = bytes;
  p->ws_bound = true;
  p->screened = false;
  p->executed = false;
  p->split_src_A = p->split_src_B = nullptr;  // the workspace holds no split yet
  return TAMM_OK;
}

extern "C" int tamm_plan_bind_workspace(tamm_plan* p, void* dev_ptr, size_t bytes) {
  if (!p) return fail(TAMM_ERR_ARG, "null plan");
  const int rc = bind_plan(p, dev_ptr, bytes);
  return rc == TAMM_OK ? ok() : rc;
}

extern "C" int tamm_plan_stats_get(const tamm_plan* p, tamm_plan_stats* s) {
  if (!p || !s) return fail(TAMM_ERR_ARG, "null argument");
  *s = p->stats;
  return ok();
}

extern "C" int tamm_plan_config_count(const tamm_plan* p, int32_t* count) {
  if (!p || !count) return fail(TAMM_ERR_ARG, "null argument");
  *count = cfg_count(p->prec);
  return ok();
}

extern "C" int tamm_plan_set_config(tamm_plan* p, int32_t config, int32_t k_splits) {
  if (!p) return fail(TAMM_ERR_ARG, "null plan");
  if (config < 0 || config >= cfg_count(p->prec)) return fail(TAMM_ERR_ARG, "configuration %d does not exist", config);
  if (k_splits < 0 || k_splits > 64) return fail(TAMM_ERR_ARG, "k_splits must be in [0, 64]");
  const int rc = configure_work(p, config, k_splits);
  if (rc != TAMM_OK) return rc;
  return ok();
}

extern "C" int tamm_plan_set_constant(tamm_plan* p, int32_t which, int32_t constant) {
  if (!p || (which != 0 && which != 1)) return fail(TAMM_ERR_ARG, "null plan or operand not 0 or 1");
  const bool is_a = (which == 0) != p->swapped;  // lhs is A unless it holds out's last label
  (is_a ? p->const_A : p->const_B) = constant != 0;
  (is_a ? p->split_src_A : p->split_src_B) = nullptr;  // split again at the next execution
  return ok();
}

extern "C" int tamm_plan_set_order(tamm_plan* p, int32_t tile_order, int32_t chunk) {
  if (!p) return fail(TAMM_ERR_ARG, "null plan");
  if (tile_order != 0 && tile_order != 1) return fail(TAMM_ERR_ARG, "tile order must be 0 or 1");
  if (chunk < -1 || chunk > (1 << 20)) return fail(TAMM_ERR_ARG, "chunk must be -1, 0 or a positive item count");
  p->tile_order = tile_order;
  p->xcd_chunk = chunk;
  const int rc = configure_work(p, p->config, p->k_splits);
  return rc == TAMM_OK ? ok() : rc;
}

extern "C" const char* tamm_config_name(int32_t precision, int32_t config) {
  if (precision < TAMM_PREC_F64 || precision > TAMM_PREC_BF16X4_ALIGNED) return "";
  if (config < 0 || config >= cfg_count(precision)) return "";
  return cfg_get(precision, config).name;
}

static bool overlaps(const tamm_tensor* a, const tamm_tensor* b) {
  if (a->numel == 0 || b->numel == 0) return false;
  const char* a0 = (const char*)a->dev;
  const char* b0 = (const char*)b->dev;
  return a0 < b0 + b->numel * 8 && b0 < a0 + a->numel * 8;
}

static int check_tensors(const tamm_plan* p) {
  const tamm_tensor* ts[3] = {p->out, p->lhs, p->rhs};
  const char* nm[3] = {"out", "lhs", "rhs"};
  for (int x = 0; x < 3; ++x)
    if (!ts[x]->bound) return fail(TAMM_ERR_UNBOUND, "%s tensor has no bound storage", nm[x]);
  if (overlaps(p->out, p->lhs) || overlaps(p->out, p->rhs)) return fail(TAMM_ERR_ARG, "out storage overlaps an operand");
  return TAMM_OK;
}

static int check_bound(const tamm_plan* p) {
  if (!p->ws_bound) return fail(TAMM_ERR_UNBOUND, "plan workspace is not bound (or the configuration changed since binding)");
  return check_tensors(p);
}

static int screen_launch(tamm_plan* p, int32_t* queue_next, hipStream_t s) {
  ScreenParams sp{};
  sp.single = screen_desc(p, p->ws, p->lay);
  sp.n_items = sp.single.n_blocks;
  sp.queue_next = queue_next;
  sp.n_queues = queue_next ? kQueues : 0;
  HIP_TRY(launch_screen(sp, s));
  p->screened = true;
  return TAMM_OK;
}

extern "C" int tamm_plan_screen(tamm_plan* p, void* stream) {
  if (!p) return fail(TAMM_ERR_ARG, "null plan");
  int rc = check_bound(p);
  if (rc == TAMM_OK) rc = screen_launch(p, nullptr, (hipStream_t)stream);
  return rc == TAMM_OK ? ok() : rc;
}

// The contraction, after the screening if `screen` (which then clears the queue counters).
static int contract_launch(tamm_plan* p, double alpha, double beta, bool screen, hipStream_t s) {
  ContractParams cp{};
  cp.single = problem_desc(p, p->ws, p->lay, p->k_splits > 1 ? (double*)(p->ws + p->off_partial) : nullptr, p->k_splits,
                           alpha, beta);
  cp.probs = nullptr;
  cp.work = (const WorkItem*)(p->ws + p->off_work);
  cp.n_work = (int32_t)p->work.size();
  const int layout = gather_layout(p);
  std::unique_lock<std::mutex> lock(p->sets.mu, std::defer_lock);
  const bool shared = p->queued || p->serial;
  int set = -1, rc = TAMM_OK;
  if (shared) {
    lock.lock();
    if ((rc = p->sets.take(s, p->queued, p->serial, &set)) != TAMM_OK) return rc;
  }
  if (p->queued && set >= 0) {
    cp.queue_next = (int32_t*)(p->ws + p->off_queue) + set * kQueues;
    std::copy(p->queue_begin, p->queue_begin + kQueues + 1, cp.queue_begin);
    if (!screen) HIP_TRY(launch_clear_queues(cp.queue_next, s));
  }
  if (screen && (rc = screen_launch(p, cp.queue_next, s)) != TAMM_OK) return rc;
  if (p->prec == TAMM_PREC_F64) {
    HIP_TRY(launch_contract_f64(p->config, layout, cp, cp.queue_next ? p->queue_grid : 0, s));
  } else {
    if (p->prec != TAMM_PREC_F32) {
      // operand split into packed bfloat16 slices, then the contraction reads the split copies
      PrepParams pa{};
      pa.x = p->A->dev;
      pa.out = (uint64_t*)(p->ws + p->off_xA);
      pa.blocks = (const PrepBlock*)(p->ws + p->off_prepA);
      pa.pool = (const int32_t*)(p->ws + p->lay.pool);
      pa.n_items = p->prepA_items;
      pa.n_blocks = (int32_t)p->prepA.size();
      pa.aligned = p->prec == TAMM_PREC_BF16X4_ALIGNED ? 1 : 0;
      pa.planes = p->planes ? 1 : 0;
      pa.plane_stride = p->A->numel;
      // a constant operand keeps the split of an earlier execution from the same storage
      if (!(p->const_A && p->split_src_A == p->A->dev)) HIP_TRY(launch_prep_split(pa, !p->a_kc, s));
      p->split_src_A = p->const_A ? (const void*)p->A->dev : nullptr;
      PrepParams pbp = pa;
      pbp.x = p->B->dev;
      pbp.out = (uint64_t*)(p->ws + p->off_xB);
      pbp.blocks = (const PrepBlock*)(p->ws + p->off_prepB);
      pbp.n_items = p->prepB_items;
      pbp.n_blocks = (int32_t)p->prepB.size();
      pbp.plane_stride = p->B->numel;
      if (!(p->const_B && p->split_src_B == p->B->dev)) HIP_TRY(launch_prep_split(pbp, !p->b_kc, s));
      p->split_src_B = p->const_B ? (const void*)p->B->dev : nullptr;
      cp.single.A = (const double*)(p->ws + p->off_xA);
      cp.single.B = (const double*)(p->ws + p->off_xB);
      if (p->planes) {
        cp.single.a_plane = p->A->numel;
        cp.single.b_plane = p->B->numel;
      }
    }
    const bool planes = p->planes && p->prec != TAMM_PREC_F32;
    HIP_TRY(launch_contract_mixed(p->prec, p->config, planes ? kPlanesLayout : (layout & 3), cp, s));
  }
  if (p->k_splits > 1) {
    const TileCfg f = cfg_get(p->prec, p->config);
    ReduceParams r{};
    r.single = cp.single;
    r.probs = nullptr;
    r.items = (const ReduceItem*)(p->ws + p->off_reduce);
    r.n_items = (int32_t)p->reduce.size();
    r.tile_m = f.mt;
    r.tile_n = f.nt;
    HIP_TRY(launch_reduce(r, s));
  }
  return shared ? p->sets.launched(set, s) : TAMM_OK;
}

extern "C" int tamm_plan_contract(tamm_plan* p, double alpha, double beta, void* stream) {
  if (!p) return fail(TAMM_ERR_ARG, "null plan");
  int rc = check_bound(p);
  if (rc != TAMM_OK) return rc;
  if (!p->screened) return fail(TAMM_ERR_UNBOUND, "the plan has not been screened on its bound workspace");
  rc = contract_launch(p, alpha, beta, false, (hipStream_t)stream);
  if (rc != TAMM_OK) return rc;
  p->executed = true;
  return ok();
}

extern "C" int tamm_plan_execute(tamm_plan* p, double alpha, double beta, void* stream) {
  if (!p) return fail(TAMM_ERR_ARG, "null plan");
  int rc = check_bound(p);
  if (rc != TAMM_OK) return rc;
  rc = contract_launch(p, alpha, beta, true, (hipStream_t)stream);
  if (rc != TAMM_OK) return rc;
  p->executed = true;
  return ok();
}

extern "C" int tamm_plan_screen_result(tamm_plan* p, void* stream, int32_t* counts, int32_t* k_tiles) {
  if (!p || !counts) return fail(TAMM_ERR_ARG, "null argument");
  if (!p->ws_bound || !p->screened) return fail(TAMM_ERR_UNBOUND, "plan has not been screened on a bound workspace");
  const size_t nob = p->blocks.size();
  HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
  HIP_TRY(hipMemcpy(counts, p->ws + p->lay.counts, nob * sizeof(int32_t), hipMemcpyDeviceToHost));
  if (k_tiles) {
    std::vector<PairDesc> pairs((size_t)nob * p->n_kt);
    HIP_TRY(hipMemcpy(pairs.data(), p->ws + p->lay.pairs, pairs.size() * sizeof(PairDesc), hipMemcpyDeviceToHost));
    const int nk = p->sd.nk;
    std::vector<int> t(nk);
    size_t w = 0;
    for (size_t b = 0; b < nob; ++b)
      for (int i = 0; i < counts[b]; ++i) {
        int rem = pairs[b * p->n_kt + i].kt;
        for (int q = nk - 1; q >= 0; --q) {
          t[q] = rem % p->sd.k_ntiles[q];
          rem /= p->sd.k_ntiles[q];
        }
        for (int j = 0; j < nk; ++j) k_tiles[w++] = t[p->k_lhs_order[j]];
      }
  }
  return ok();
}

extern "C" int tamm_plan_split_operand(const tamm_plan* p, int32_t which, void* out_dev, size_t bytes, void* stream) {
  if (!p || !out_dev || (which != 0 && which != 1)) return fail(TAMM_ERR_ARG, "null plan or buffer, or operand not 0 or 1");
  if (p->prec != TAMM_PREC_BF16X3 && p->prec != TAMM_PREC_BF16X4_ALIGNED)
    return fail(TAMM_ERR_UNSUPPORTED, "the plan's precision splits no operand");
  const int rc = check_bound(p);
  if (rc != TAMM_OK) return rc;
  const bool is_a = (which == 0) != p->swapped;  // lhs is A unless it holds out's last label
  const tamm_tensor* t = is_a ? p->A : p->B;
  if (bytes < (size_t)t->numel * sizeof(uint64_t))
    return fail(TAMM_ERR_WORKSPACE, "output buffer of %zu bytes is smaller than %lld words", bytes, (long long)t->numel);
  PrepParams pa{};
  pa.x = t->dev;
  pa.out = out_dev;
  pa.blocks = (const PrepBlock*)(p->ws + (is_a ? p->off_prepA : p->off_prepB));
  pa.pool = (const int32_t*)(p->ws + p->lay.pool);
  pa.n_items = is_a ? p->prepA_items : p->prepB_items;
  pa.n_blocks = (int32_t)(is_a ? p->prepA.size() : p->prepB.size());
  pa.aligned = p->prec == TAMM_PREC_BF16X4_ALIGNED ? 1 : 0;
  pa.planes = 0;  // packed words at the float64 element offsets
  HIP_TRY(launch_prep_split(pa, is_a ? !p->a_kc : !p->b_kc, (hipStream_t)stream));
  return ok();
}

extern "C" int tamm_plan_destroy(tamm_plan* p) {
  delete p;
  return ok();
}

// ---------------------------------------------------------------------------------------------
// one-shot contraction: plans cached inside the library, keyed by tensor handles and labels
// ---------------------------------------------------------------------------------------------
namespace {

struct ContractKey {
  const tamm_tensor* out;
  const tamm_tensor* lhs;
  const tamm_tensor* rhs;
  std::string labels;  // out, lhs and rhs labels joined by '/'
  int32_t precision;
  size_t limit;  // of the workspace, 0: none
  bool operator<(const ContractKey& o) const {
    return std::tie(out, lhs, rhs, labels, precision, limit) < std::tie(o.out, o.lhs, o.rhs, o.labels, o.precision, o.limit);
  }
};

struct ContractCache {
  std::mutex mu;
  std::map<ContractKey, std::unique_ptr<tamm_plan>> plans;
  struct Holder {
    const tamm_plan* plan;  // the plan whose tables the workspace holds
    size_t bytes;           // the workspace's length
  };
  std::map<const void*, Holder> holder;  // workspace start -> its holder
};

// Never destroyed: tensor handles may be released from other static destructors at exit.
ContractCache& contract_cache() {
  static ContractCache* c = new ContractCache;
  return *c;
}

// The cached plan for a contraction, created on first use.  The caller holds the cache lock.  With a
// limit of the workspace: the plan without one if that fits, else a plan of its own.
int cached_plan(ContractCache& c, tamm_tensor* out, const char* ol, const tamm_tensor* lhs, const char* ll,
                const tamm_tensor* rhs, const char* rl, int32_t precision, size_t limit, tamm_plan** plan) {
  if (limit > 0) {
    const int rc = cached_plan(c, out, ol, lhs, ll, rhs, rl, precision, 0, plan);
    if (rc != TAMM_OK || (*plan)->ws_size <= limit) return rc;
  }
  if (!out || !lhs || !rhs || !ol || !ll || !rl) return fail(TAMM_ERR_ARG, "null tensor or label string");
  ContractKey key{out, lhs, rhs, std::string(ol) + "/" + ll + "/" + rl, precision, limit};
  auto it = c.plans.find(key);
  if (it != c.plans.end()) {
    *plan = it->second.get();
    return TAMM_OK;
  }
  tamm_plan* p = nullptr;
  int rc = tamm_plan_create(out, ol, lhs, ll, rhs, rl, (tamm_precision)precision, &p);
  if (rc != TAMM_OK) return rc;
  if (limit > 0) {
    p->ws_limit = limit;
    if ((rc = configure_work(p, -1, 0)) != TAMM_OK) {
      delete p;
      return rc;
    }
  }
  c.plans.emplace(std::move(key), std::unique_ptr<tamm_plan>(p));
  *plan = p;
  return TAMM_OK;
}

}  // namespace

void tamm::contract_cache_evict(const tamm_tensor* t) {
  ContractCache& c = contract_cache();
  std::lock_guard<std::mutex> lock(c.mu);
  for (auto it = c.plans.begin(); it != c.plans.end();) {
    if (it->first.out != t && it->first.lhs != t && it->first.rhs != t) {
      ++it;
      continue;
    }
    for (auto h = c.holder.begin(); h != c.holder.end();) h = h->second.plan == it->second.get() ? c.holder.erase(h) : std::next(h);
    it = c.plans.erase(it);
  }
}

extern "C" int tamm_contract_workspace_size(tamm_tensor* out, const char* out_lbl, const tamm_tensor* lhs,
                                            const char* lhs_lbl, const tamm_tensor* rhs, const char* rhs_lbl,
                                            int32_t precision, size_t* bytes) {
  if (!bytes) return fail(TAMM_ERR_ARG, "null argument");
  ContractCache& c = contract_cache();
  std::lock_guard<std::mutex> lock(c.mu);
  tamm_plan* p = nullptr;
  const int rc = cached_plan(c, out, out_lbl, lhs, lhs_lbl, rhs, rhs_lbl, precision, 0, &p);
  if (rc != TAMM_OK) return rc;
  *bytes = p->ws_size;
  return ok();
}

// Workspace that a caller with `limit` bytes needs.
int tamm::contract_workspace_within(tamm_tensor* out, const char* out_lbl, const tamm_tensor* lhs, const char* lhs_lbl,
                                    const tamm_tensor* rhs, const char* rhs_lbl, int32_t precision, size_t limit, size_t* bytes) {
  ContractCache& c = contract_cache();
  std::lock_guard<std::mutex> lock(c.mu);
  tamm_plan* p = nullptr;
  const int rc = cached_plan(c, out, out_lbl, lhs, lhs_lbl, rhs, rhs_lbl, precision, limit, &p);
  if (rc != TAMM_OK) return rc;
  *bytes = p->ws_size;
  if (p->ws_size > limit)  // to be refused: the plan made for the limit is of no use
    for (auto it = c.plans.begin(); it != c.plans.end(); ++it)
      if (it->second.get() == p) {
        c.plans.erase(it);
        break;
      }
  return TAMM_OK;
}

extern "C" int tamm_contract(tamm_tensor* out, const char* out_lbl, const tamm_tensor* lhs, const char* lhs_lbl,
                             const tamm_tensor* rhs, const char* rhs_lbl, int32_t precision, double alpha, double beta,
                             void* workspace, size_t bytes, void* stream) {
  return contract_within(out, out_lbl, lhs, lhs_lbl, rhs, rhs_lbl, precision, 0, alpha, beta, workspace, bytes, stream);
}

// tamm_contract with the plan for a caller whose workspace is `limit` bytes (0: tamm_contract's own).
int tamm::contract_within(tamm_tensor* out, const char* out_lbl, const tamm_tensor* lhs, const char* lhs_lbl,
                          const tamm_tensor* rhs, const char* rhs_lbl, int32_t precision, size_t limit, double alpha, double beta,
                          void* workspace, size_t bytes, void* stream) {
  ContractCache& c = contract_cache();
  std::lock_guard<std::mutex> lock(c.mu);
  tamm_plan* p = nullptr;
  int rc = cached_plan(c, out, out_lbl, lhs, lhs_lbl, rhs, rhs_lbl, precision, limit, &p);
  if (rc != TAMM_OK) return rc;
  const auto h = c.holder.find(workspace);
  const bool holds = p->ws_bound && p->ws == (char*)workspace && p->ws_bytes == bytes && h != c.holder.end() &&
                     h->second.plan == p && h->second.bytes == bytes;
  if (!holds) {
    if (!workspace || ((uintptr_t)workspace) % 256)
      return fail(TAMM_ERR_WORKSPACE, "workspace must be non-null and 256-byte aligned");
    if (bytes < p->ws_size)
      return fail(TAMM_ERR_WORKSPACE, "workspace of %zu bytes is smaller than the %zu needed", bytes, p->ws_size);
    // Earlier calls, on any stream, may still read tables in the range this upload overwrites:
    // drain the device before replacing them (a rare path: it runs when a workspace changes hands).
    const char* lo = (const char*)workspace;
    bool busy = false;
    for (auto it = c.holder.begin(); it != c.holder.end();) {
      const char* o = (const char*)it->first;
      if (o < lo + bytes && lo < o + it->second.bytes) {
        busy = true;
        it = c.holder.erase(it);
      } else {
        ++it;
      }
    }
    if (busy) HIP_TRY(hipDeviceSynchronize());
    rc = bind_plan(p, workspace, bytes);
    if (rc != TAMM_OK) return rc;
    c.holder[workspace] = ContractCache::Holder{p, bytes};
  }
  return tamm_plan_execute(p, alpha, beta, stream);
}

extern "C" int tamm_contract_cache_count(int64_t* plans) {
  if (!plans) return fail(TAMM_ERR_ARG, "null argument");
  ContractCache& c = contract_cache();
  std::lock_guard<std::mutex> lock(c.mu);
  *plans = (int64_t)c.plans.size();
  return ok();
}

extern "C" int tamm_contract_cache_clear(void) {
  ContractCache& c = contract_cache();
  std::lock_guard<std::mutex> lock(c.mu);
  c.holder.clear();
  c.plans.clear();
  return ok();
}

// ---------------------------------------------------------------------------------------------
// autotuner (plans)
// ---------------------------------------------------------------------------------------------
namespace {

struct CacheEntry {
  int config, k_splits, grid;
  double ms;
};

// The two timing events of an autotuner, destroyed on every exit path (HIP_TRY returns early).
struct TimerEvents {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int create() {
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    return TAMM_OK;
  }
  ~TimerEvents() {
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
  }
};

bool cache_lookup(const char* path, uint64_t sig, const char* kind, CacheEntry& e) {
  if (!path || !*path) return false;
  std::ifstream f(path);
  std::string line;
  bool found = false;
  while (std::getline(f, line)) {
    std::istringstream is(line);
    std::string s, k;
    CacheEntry c{};
    if (!(is >> s >> k >> c.config >> c.k_splits >> c.grid >> c.ms)) continue;
    if (k == kind && std::strtoull(s.c_str(), nullptr, 16) == sig) {
      e = c;
      found = true;  // the last entry wins
    }
  }
  return found;
}

void cache_store(const char* path, uint64_t sig, const char* kind, const CacheEntry& e) {
  if (!path || !*path) return;
  std::ofstream f(path, std::ios::app);
  char buf[160];
  snprintf(buf, sizeof(buf), "%016llx %s %d %d %d %.6f\n", (unsigned long long)sig, kind, e.config, e.k_splits, e.grid, e.ms);
  f << buf;
}

}  // namespace

extern "C" int tamm_plan_autotune_workspace_size(const tamm_plan* p, size_t* bytes) {
  if (!p || !bytes) return fail(TAMM_ERR_ARG, "null argument");
  *bytes = plan_candidate_workspace(p, 8);
  return ok();
}

extern "C" int tamm_plan_autotune(tamm_plan* p, void* workspace, size_t bytes, void* stream, const char* cache_path,
                                  int32_t reps) {
  if (!p) return fail(TAMM_ERR_ARG, "null plan");
  int rc = check_tensors(p);
  if (rc != TAMM_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  // cache entries of kind "plan2" hold the configuration, K splits and die chunk (grid field)
  CacheEntry best{-1, 1, -1, 1e30};
  if (!cache_lookup(cache_path, p->signature, "plan2", best)) {
    if (reps <= 0) reps = 3;
    TimerEvents ev;
    if ((rc = ev.create()) != TAMM_OK) return rc;
    hipEvent_t e0 = ev.e0, e1 = ev.e1;
    // one candidate: configure, bind, warm up, fastest of reps (alpha = 0, beta = 1 leaves out
    // unchanged for finite operands while doing the full work)
    auto trial = [&](int c, int ks, float* ms) -> int {
      *ms = 1e30f;
      if (configure_work(p, c, ks) != TAMM_OK || p->ws_size > bytes) return TAMM_OK;
      int r = bind_plan(p, workspace, bytes);
      if (r != TAMM_OK) return r;
      if ((r = tamm_plan_execute(p, 0.0, 1.0, stream)) != TAMM_OK) return r;
      for (int i = 0; i < reps; ++i) {
        HIP_TRY(hipEventRecord(e0, s));
        if ((r = tamm_plan_execute(p, 0.0, 1.0, stream)) != TAMM_OK) return r;
        HIP_TRY(hipEventRecord(e1, s));
        HIP_TRY(hipEventSynchronize(e1));
        float one = 0;
        HIP_TRY(hipEventElapsedTime(&one, e0, e1));
        *ms = std::min(*ms, one);
      }
      return TAMM_OK;
    };
    const int chunk0 = p->xcd_chunk;
    const int64_t ntiles_max = tiles_for(p, 0);
    std::vector<CacheEntry> ranked;  // every (configuration, K splits) at the current launch order
    for (int c = 0; c < cfg_count(p->prec) && rc == TAMM_OK; ++c) {
      if (p->prec == TAMM_PREC_F64 && f64_config_canonical(c) != c) continue;  // another id of a kernel already timed
      const int64_t nt = tiles_for(p, c);
      for (int ks : {1, 2, 4, 8}) {
        if (ks > 1 && nt * ks > 4 * std::max<int64_t>(ntiles_max, 2048)) continue;
        float ms = 0;
        if ((rc = trial(c, ks, &ms)) != TAMM_OK) break;
        if (ms < 1e29f) ranked.push_back(CacheEntry{c, ks, chunk0, ms});
        if (ms < best.ms) best = CacheEntry{c, ks, chunk0, ms};
      }
    }
    // tile orders and die chunks (they change only the launch order) for the three fastest
    // (configuration, K splits) of the first pass, since a configuration that loses at one order
    // can win at another; the cache's grid field holds chunk + order * 2^24
    if (rc == TAMM_OK && best.config >= 0) {
      best.grid = (chunk0 < 0 ? xcd_chunk() : chunk0) + (p->tile_order << 24);
      std::stable_sort(ranked.begin(), ranked.end(), [](const CacheEntry& x, const CacheEntry& y) { return x.ms < y.ms; });
      if (ranked.size() > 3) ranked.resize(3);
      std::vector<CacheEntry> finals{best};  // every candidate with its launch order
      for (const CacheEntry& cand : ranked)
        for (int order : {0, 1})
          for (int ch : {0, 16, 32, 64, 128}) {
            if (rc != TAMM_OK) break;  // a failed trial ends the search with its error
            p->xcd_chunk = ch;
            p->tile_order = order;
            float ms = 0;
            if ((rc = trial(cand.config, cand.k_splits, &ms)) != TAMM_OK) break;
            if (ms < 1e29f) finals.push_back(CacheEntry{cand.config, cand.k_splits, ch + (order << 24), ms});
            if (ms < best.ms) best = CacheEntry{cand.config, cand.k_splits, ch + (order << 24), ms};
          }
      // confirmation: the fastest single trial among candidates within a few per cent of each
      // other is partly chance, so the three fastest are timed again in turn, three rounds, and
      // the lowest median kept
      std::stable_sort(finals.begin(), finals.end(), [](const CacheEntry& x, const CacheEntry& y) { return x.ms < y.ms; });
      std::vector<CacheEntry> top;
      for (const CacheEntry& f : finals) {
        bool dup = false;
        for (const CacheEntry& t : top)
          dup = dup || (t.config == f.config && t.k_splits == f.k_splits && t.grid == f.grid);
        if (!dup) top.push_back(f);
        if (top.size() == 3) break;
      }
      if (rc == TAMM_OK && top.size() > 1) {
        std::vector<std::vector<float>> times(top.size());
        for (int round = 0; round < 3 && rc == TAMM_OK; ++round)
          for (size_t t = 0; t < top.size() && rc == TAMM_OK; ++t) {
            p->xcd_chunk = top[t].grid & 0xFFFFFF;
            p->tile_order = (top[t].grid >> 24) & 1;
            float ms = 0;
            if ((rc = trial(top[t].config, top[t].k_splits, &ms)) != TAMM_OK) break;
            times[t].push_back(ms);
          }
        if (rc == TAMM_OK) {
          size_t pick = 0;
          float pick_ms = 1e30f;
          for (size_t t = 0; t < top.size(); ++t) {
            std::vector<float> v = times[t];
            std::sort(v.begin(), v.end());
            if (v[v.size() / 2] < pick_ms) {
              pick_ms = v[v.size() / 2];
              pick = t;
            }
          }
          best = CacheEntry{top[pick].config, top[pick].k_splits, top[pick].grid, pick_ms};
        }
      }
    }
    if (rc != TAMM_OK) return rc;
    if (best.config < 0) return fail(TAMM_ERR_WORKSPACE, "no configuration fits the %zu-byte workspace", bytes);
    cache_store(cache_path, p->signature, "plan2", best);
  }
  p->xcd_chunk = best.grid < 0 ? -1 : (best.grid & 0xFFFFFF);
  p->tile_order = best.grid < 0 ? 0 : (best.grid >> 24) & 1;
  rc = configure_work(p, best.config, best.k_splits);
  if (rc != TAMM_OK) return rc;
  if (p->ws_size > bytes) return fail(TAMM_ERR_WORKSPACE, "cached configuration needs %zu bytes", p->ws_size);
  rc = bind_plan(p, workspace, bytes);
  return rc == TAMM_OK ? ok() : rc;
}

// ---------------------------------------------------------------------------------------------
// groups: contraction nodes executed together -- one screening launch and one persistent
// contraction launch per gather layout class (each with its own configuration), optionally
// captured once into a hipGraph and replayed.  A node is one plan, or several plans that write
// the same output tiles (a fused node, built by the scheduler): their pair lists are screened
// into one list per output block and one output tile's K loop runs over all of them.
// ---------------------------------------------------------------------------------------------
constexpr int kGroupChunk = 8;  // items per die chunk of a group's queues, or of its plain launches
struct tamm_group {
  std::vector<std::vector<tamm_plan*>> nodes;  // member plans of each node
  std::vector<tamm_plan*> plans;               // every member plan, node by node
  std::vector<int32_t> node_first;             // index in `plans` (and segment index) of each node's first plan
  std::vector<Layout> lays;                    // static tables of each plan
  struct Fused {
    size_t blocks = 0, pairs = 0, counts = 0;  // regions of a fused node's own output descriptors and pair list
    int32_t stride = 0;                        // pair capacity per output block (sum over the members)
  };
  std::vector<Fused> fused;                    // per node (fused nodes only)
  size_t off_sdesc = 0, off_pdesc = 0, off_sitems = 0, off_work = 0, off_counter = 0, ws_size = 0;
  std::vector<int32_t> sitem_prob, sitem_block;  // screening items: first segment of the node, output block
  std::vector<WorkItem> work;       // grouped by gather layout class, each class longest first (prob = node)
  size_t work_capacity = 0;         // work items of the largest mix of per-class configurations
  int32_t queue_begin[kLayouts][kQueues + 1] = {};  // each class's queues, relative to its work range
  bool queued[kLayouts] = {};            // a persistent launch pays (queue_pays)
  int auto_grid[kLayouts] = {};          // its workgroups on the device the group is bound on
  int32_t cls_begin[kLayouts + 1] = {};  // work range of gather layout c: [cls_begin[c], cls_begin[c+1])
  int cfg[kLayouts] = {};   // kernel configuration of each layout class (its tile shape)
  int grid[kLayouts] = {};  // persistent grid of each layout class (0: automatic)
  uint64_t signature = 0;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  bool bound = false;
  std::vector<ProblemDesc> pdesc;   // host copy per node (alpha/beta updated per execute)
  std::vector<ScreenDesc> sdesc;    // host copy per plan (segment)
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  std::vector<double> g_alpha, g_beta;
  // side streams (default priority) and events that run the layout classes' launches
  // concurrently, forked after the screening launch and joined back into the caller's stream
  hipStream_t side[kLayouts] = {};
  hipEvent_t ev_fork = nullptr;
  hipEvent_t ev_join[kLayouts] = {};
  bool ran = false;  // launched outside a capture
};

static void group_drop_graph(tamm_group* g) {
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (g->graph) (void)hipGraphDestroy(g->graph);
  g->exec = nullptr;
  g->graph = nullptr;
}

// Gather layout of a node: its plans share the operand orientations; 16-byte gathers only when
// every member's tables allow them.
static int node_layout(const tamm_group* g, size_t q) {
  int lay = gather_layout(g->nodes[q][0]) & 3;
  bool pairs = true;
  for (const tamm_plan* p : g->nodes[q]) pairs = pairs && p->pairs;
  return lay | (pairs ? 4 : 0);
}

// Summed K extent of the surviving pairs of output block b over the node's plans.
static double node_block_cost(const tamm_group* g, size_t q, size_t b) {
  double c = 0;
  for (const tamm_plan* p : g->nodes[q]) c += p->block_cost[b];
  return c;
}

// Shape of output block b of a node: of its plan, or of the plans that share its output tiles, their
// pairs one after another.
static BlockShape node_block_shape(const tamm_group* g, size_t q, size_t b) {
  BlockShape sh = g->nodes[q][0]->block_shapes[b];
  for (size_t i = 1; i < g->nodes[q].size(); ++i) {
    const BlockShape& o = g->nodes[q][i]->block_shapes[b];
    sh.pairs += o.pairs;
    sh.chunks16 += o.chunks16;
    sh.chunks32 += o.chunks32;
    sh.kext += o.kext;
  }
  return sh;
}

// The distinct block shapes of the nodes of one layout class, and the bytes of their tensors.
static std::vector<BlockShape> class_shapes(const tamm_group* g, int layout, double* bytes) {
  std::vector<BlockShape> shapes;
  *bytes = 0;
  for (size_t q = 0; q < g->nodes.size(); ++q) {
    if (node_layout(g, q) != layout) continue;
    if (g->nodes[q].size() == 1) shapes.insert(shapes.end(), g->nodes[q][0]->shapes.begin(), g->nodes[q][0]->shapes.end());
    else
      for (size_t b = 0; b < g->nodes[q][0]->blocks.size(); ++b) shapes.push_back(node_block_shape(g, q, b));
    for (const tamm_plan* p : g->nodes[q]) *bytes += p->stats.algorithmic_bytes;
  }
  merge_shapes(shapes);
  return shapes;
}

// Default configuration of the nodes of one layout class, and whether long items are cut: the least
// estimated time of its launch.
static int group_default_config(const tamm_group* g, int layout, bool* cut) {
  double bytes = 0;
  const std::vector<BlockShape> shapes = class_shapes(g, layout, &bytes);
  int config = 0;
  double best = 1e300;
  for (int c = 0; c < f64_config_count(); ++c) {
    if (f64_config_canonical(c) != c) continue;
    for (bool with_cut : {true, false}) {
      const double t = group_estimate_us(shapes, cfg_get(TAMM_PREC_F64, c), bytes, with_cut);
      if (t < best) {
        best = t;
        config = c;
        *cut = with_cut;
      }
    }
  }
  return config;
}

// Work lists of every layout class with the class's configuration cfgs[c] (< 0: the class's
// default; others cut long items), each heaviest first, and the workspace layout.
static int group_configure_classes(tamm_group* g, const int* cfgs, const int* grids) {
  bool cut[kLayouts];
  std::fill(cut, cut + kLayouts, true);
  for (int c = 0; c < kLayouts; ++c) {
    const int k = cfgs[c] < 0 ? group_default_config(g, c, &cut[c]) : cfgs[c];
    if (k >= f64_config_count()) return fail(TAMM_ERR_ARG, "configuration %d does not exist", k);
    g->cfg[c] = k;
  }
  std::copy(grids, grids + kLayouts, g->grid);
  struct Tile {
    double cost;
    WorkItem w;
  };
  g->work.clear();
  for (int c = 0; c < kLayouts; ++c) {
    std::vector<Tile> tiles;
    std::vector<int32_t> cm, cn;
    const TileCfg tc = cfg_get(TAMM_PREC_F64, g->cfg[c]);
    double bytes = 0;
    const double limit = cut[c] ? group_limit_us(class_shapes(g, c, &bytes), tc) : 1e300;
    for (size_t q = 0; q < g->nodes.size(); ++q) {
      if (node_layout(g, q) != c) continue;
      const tamm_plan* p = g->nodes[q][0];
      int32_t t = 0;
      for (size_t b = 0; b < p->blocks.size(); ++b) {
        const auto& d = p->blocks[b];
        const double bc = node_block_cost(g, q, b);
        const auto tile = group_tile(node_block_shape(g, q, b), tc, limit);
        cut_extent(d.mext, tile.first, tc.um, cm);
        cut_extent(d.next, tile.second, tc.un, cn);
        int32_t m0 = 0;
        for (int32_t rows : cm) {
          int32_t n0 = 0;
          for (int32_t cols : cn) {
            tiles.push_back(Tile{bc * rows * cols, WorkItem{(int32_t)q, (int32_t)b, m0, n0, item_shape(0, 1, rows, cols), t++}});
            n0 += cols;
          }
          m0 += rows;
        }
      }
    }
    std::stable_sort(tiles.begin(), tiles.end(), [](const Tile& x, const Tile& y) { return x.cost > y.cost; });
    g->cls_begin[c] = (int32_t)g->work.size();
    for (auto& t : tiles) g->work.push_back(t.w);
    double flops = 0;
    for (const Tile& t : tiles) flops += 2.0 * t.cost;
    g->queued[c] = queue_pays(flops, tiles.size(), cfg_get(TAMM_PREC_F64, g->cfg[c]));
    if (g->grid[c] > 0 || g->queued[c]) queue_order(g->work, g->cls_begin[c], kGroupChunk, g->queue_begin[c]);
    else xcd_order(g->work, g->cls_begin[c], kGroupChunk);
  }
  g->cls_begin[kLayouts] = (int32_t)g->work.size();
  size_t off = 0;
  g->lays.clear();
  for (auto* p : g->plans) {
    g->lays.push_back(make_layout(p, off));
    off = g->lays.back().end;
  }
  g->fused.assign(g->nodes.size(), tamm_group::Fused{});
  for (size_t q = 0; q < g->nodes.size(); ++q) {
    if (g->nodes[q].size() < 2) continue;
    tamm_group::Fused& F = g->fused[q];
    const size_t nob = g->nodes[q][0]->blocks.size();
    int64_t stride = 0;
    for (const tamm_plan* p : g->nodes[q]) stride += p->n_kt;
    F.stride = (int32_t)stride;
    F.blocks = align256(off);
    off = align256(F.blocks + nob * sizeof(OutBlockDesc));
    F.pairs = off;
    off = align256(off + nob * (size_t)stride * sizeof(PairDesc));
    F.counts = off;
    off = align256(off + nob * sizeof(int32_t));
  }
  g->off_sdesc = off;
  off = align256(off + g->plans.size() * sizeof(ScreenDesc));
  g->off_pdesc = off;
  off = align256(off + g->nodes.size() * sizeof(ProblemDesc));
  g->off_sitems = off;
  off = align256(off + g->sitem_prob.size() * 2 * sizeof(int32_t));
  g->off_work = off;
  // room for any mix of per-class configurations, so the autotuner's choice always fits the
  // workspace sized for the candidates
  off = align256(off + std::max(g->work.size(), g->work_capacity) * sizeof(WorkItem));
  g->off_counter = off;  // the queue counters of every gather layout
  off = align256(off + kLayouts * kQueues * sizeof(int32_t));
  g->ws_size = off;
  g->bound = false;
  group_drop_graph(g);
  return TAMM_OK;
}

// One configuration (< 0: each class's default) and persistent grid (0: automatic) for every class.
static int group_configure(tamm_group* g, int config, int grid) {
  int cfgs[kLayouts], grids[kLayouts];
  std::fill(cfgs, cfgs + kLayouts, config);
  std::fill(grids, grids + kLayouts, grid);
  return group_configure_classes(g, cfgs, grids);
}

// Plans that can share output tiles: float64, the same output tensor, the same flattening of the
// output's labels into rows (M) and columns (N), and the same operand orientations.
static int check_fusable(const std::vector<tamm_plan*>& node) {
  const tamm_plan* p0 = node[0];
  auto out_dims = [](const tamm_plan* p, const std::vector<int>& grp) {
    std::vector<int> d;
    for (int l : grp) d.push_back(p->labels[l].od);
    return d;
  };
  for (size_t i = 1; i < node.size(); ++i) {
    const tamm_plan* p = node[i];
    if (p->out != p0->out) return fail(TAMM_ERR_ARG, "fused plans must write the same output tensor");
    if (out_dims(p, p->M) != out_dims(p0, p0->M) || out_dims(p, p->N) != out_dims(p0, p0->N) || p->a_kc != p0->a_kc ||
        p->b_kc != p0->b_kc)
      return fail(TAMM_ERR_UNSUPPORTED, "fused plans must split the output into the same rows and columns");
  }
  int64_t stride = 0;
  for (const tamm_plan* p : node) stride += p->n_kt;
  if ((int64_t)p0->blocks.size() * stride > (int64_t)1 << 28) return fail(TAMM_ERR_UNSUPPORTED, "fused pair capacity too large");
  return TAMM_OK;
}

namespace tamm {

// Create a group of nodes (each node one plan, or several fusable plans writing the same output).
int group_create_nodes(const std::vector<std::vector<tamm_plan*>>& nodes, tamm_group** out) {
  *out = nullptr;
  if (nodes.empty()) return fail(TAMM_ERR_ARG, "a group needs at least one plan");
  auto g = std::make_unique<tamm_group>();
  uint64_t h = 0xCBF29CE484222325ULL;
  for (size_t q = 0; q < nodes.size(); ++q) {
    if (nodes[q].empty()) return fail(TAMM_ERR_ARG, "node %zu is empty", q);
    for (tamm_plan* p : nodes[q]) {
      if (!p) return fail(TAMM_ERR_ARG, "a member plan is null");
      if (p->prec != TAMM_PREC_F64) return fail(TAMM_ERR_UNSUPPORTED, "groups run float64 plans only");
    }
    int rc = check_fusable(nodes[q]);
    if (rc != TAMM_OK) return rc;
    for (size_t r = 0; r < q; ++r)
      if (nodes[r][0]->out == nodes[q][0]->out)
        return fail(TAMM_ERR_ARG, "members %zu and %zu write the same output tensor", r, q);
    g->nodes.push_back(nodes[q]);
    g->node_first.push_back((int32_t)g->plans.size());
    const uint32_t sz = (uint32_t)nodes[q].size();
    h = fnv(h, &sz, sizeof(sz));
    for (tamm_plan* p : nodes[q]) {
      g->plans.push_back(p);
      h = fnv(h, &p->signature, sizeof(uint64_t));
    }
    for (size_t b = 0; b < nodes[q][0]->blocks.size(); ++b) {
      g->sitem_prob.push_back(g->node_first.back());
      g->sitem_block.push_back((int32_t)b);
    }
  }
  g->signature = h;
  for (int c = 0; c < kLayouts; ++c) {
    size_t most = 0;
    for (int k = 0; k < f64_config_count(); ++k) {
      if (f64_config_canonical(k) != k) continue;
      const F64Config& f = f64_config(k);
      size_t n = 0;
      for (size_t q = 0; q < g->nodes.size(); ++q)
        if (node_layout(g.get(), q) == c)
          for (const auto& b : g->nodes[q][0]->blocks)
            n += (size_t)((b.mext + f.mt - 1) / f.mt) * ((b.next + f.nt - 1) / f.nt);
      most = std::max(most, n);
    }
    g->work_capacity += most;
  }
  const int rc = group_configure(g.get(), -1, 0);
  if (rc != TAMM_OK) return rc;
  *out = g.release();
  return TAMM_OK;
}

}  // namespace tamm

extern "C" int tamm_group_create(tamm_plan* const* plans, int32_t n, tamm_group** out) {
  if (!out) return fail(TAMM_ERR_ARG, "null output pointer");
  *out = nullptr;
  if (!plans || n <= 0) return fail(TAMM_ERR_ARG, "a group needs at least one plan");
  std::vector<std::vector<tamm_plan*>> nodes;
  for (int32_t i = 0; i < n; ++i) {
    if (!plans[i]) return fail(TAMM_ERR_ARG, "plan %d is null", i);
    nodes.push_back({plans[i]});
  }
  const int rc = group_create_nodes(nodes, out);
  return rc == TAMM_OK ? ok() : rc;
}

extern "C" int tamm_group_workspace_size(const tamm_group* g, size_t* bytes) {
  if (!g || !bytes) return fail(TAMM_ERR_ARG, "null argument");
  *bytes = g->ws_size;
  return ok();
}

// Screening descriptors of every plan (segment) and problem descriptors of every node for the
// current tensor bindings and coefficients.
static void group_descs(const tamm_group* g, char* ws, const double* alpha, const double* beta, std::vector<ScreenDesc>& sds,
                        std::vector<ProblemDesc>& pds) {
  sds.clear();
  pds.clear();
  for (size_t q = 0; q < g->nodes.size(); ++q) {
    const int first = g->node_first[q];
    const tamm_plan* p0 = g->nodes[q][0];
    const Layout& L0 = g->lays[first];
    ProblemDesc pd = problem_desc(p0, ws, L0, nullptr, 1, alpha[q], beta[q]);
    const bool fused = g->nodes[q].size() > 1;
    const tamm_group::Fused& F = g->fused[q];
    if (fused) {
      pd.blocks = (const OutBlockDesc*)(ws + F.blocks);
      pd.pairs = (const PairDesc*)(ws + F.pairs);
      pd.counts = (const int32_t*)(ws + F.counts);
    }
    pds.push_back(pd);
    for (size_t i = 0; i < g->nodes[q].size(); ++i) {
      const tamm_plan* p = g->nodes[q][i];
      const Layout& L = g->lays[first + i];
      ScreenDesc s = screen_desc(p, ws, L);
      if (fused) {
        s.pairs = (PairDesc*)(ws + F.pairs);
        s.counts = (int32_t*)(ws + F.counts);
        s.pair_stride = F.stride;
        // element offsets and table starts relative to the first member's operands and pool
        s.a_base = (int64_t)((const double*)p->A->dev - (const double*)p0->A->dev);
        s.b_base = (int64_t)((const double*)p->B->dev - (const double*)p0->B->dev);
        s.pool_base = (int32_t)(((int64_t)L.pool - (int64_t)L0.pool) / (int64_t)sizeof(int32_t));
        s.next_seg = i + 1 < g->nodes[q].size() ? first + (int32_t)i + 1 : -1;
      }
      sds.push_back(s);
    }
  }
}

static int group_bind(tamm_group* g, void* dev_ptr, size_t bytes) {
  if (!dev_ptr || ((uintptr_t)dev_ptr) % 256) return fail(TAMM_ERR_WORKSPACE, "workspace must be non-null and 256-byte aligned");
  if (bytes < g->ws_size) return fail(TAMM_ERR_WORKSPACE, "workspace of %zu bytes is smaller than the %zu needed", bytes, g->ws_size);
  char* ws = (char*)dev_ptr;
  for (size_t q = 0; q < g->plans.size(); ++q) {
    int rc = upload_static(g->plans[q], ws, g->lays[q]);
    if (rc != TAMM_OK) return rc;
  }
  for (size_t q = 0; q < g->nodes.size(); ++q) {
    if (g->nodes[q].size() < 2) continue;
    std::vector<OutBlockDesc> d = g->nodes[q][0]->blocks;  // the first member's tables, the node's pair list
    for (size_t b = 0; b < d.size(); ++b) d[b].pair_base = (int32_t)(b * (size_t)g->fused[q].stride);
    if (!d.empty()) HIP_TRY(hipMemcpy(ws + g->fused[q].blocks, d.data(), d.size() * sizeof(OutBlockDesc), hipMemcpyHostToDevice));
  }
  std::vector<double> one(g->nodes.size(), 1.0), zero(g->nodes.size(), 0.0);
  group_descs(g, ws, one.data(), zero.data(), g->sdesc, g->pdesc);
  HIP_TRY(hipMemcpy(ws + g->off_sdesc, g->sdesc.data(), g->sdesc.size() * sizeof(ScreenDesc), hipMemcpyHostToDevice));
  HIP_TRY(hipMemcpy(ws + g->off_pdesc, g->pdesc.data(), g->pdesc.size() * sizeof(ProblemDesc), hipMemcpyHostToDevice));
  std::vector<int32_t> items(g->sitem_prob);
  items.insert(items.end(), g->sitem_block.begin(), g->sitem_block.end());
  if (!items.empty()) HIP_TRY(hipMemcpy(ws + g->off_sitems, items.data(), items.size() * sizeof(int32_t), hipMemcpyHostToDevice));
  if (!g->work.empty()) HIP_TRY(hipMemcpy(ws + g->off_work, g->work.data(), g->work.size() * sizeof(WorkItem), hipMemcpyHostToDevice));
  for (int c = 0; c < kLayouts; ++c) {
    const int n = g->cls_begin[c + 1] - g->cls_begin[c];
    g->auto_grid[c] = n > 0 && g->queued[c] ? persistent_grid(g->cfg[c], c, n) : 0;
  }
  g->ws = ws;
  g->ws_bytes = bytes;
  g->bound = true;
  group_drop_graph(g);
  return TAMM_OK;
}

extern "C" int tamm_group_bind_workspace(tamm_group* g, void* dev_ptr, size_t bytes) {
  if (!g) return fail(TAMM_ERR_ARG, "null group");
  const int rc = group_bind(g, dev_ptr, bytes);
  return rc == TAMM_OK ? ok() : rc;
}

extern "C" int tamm_group_set_config(tamm_group* g, int32_t config, int32_t grid) {
  if (!g) return fail(TAMM_ERR_ARG, "null group");
  if (grid < 0) return fail(TAMM_ERR_ARG, "grid must be >= 0");
  const int rc = group_configure(g, config, grid);
  return rc == TAMM_OK ? ok() : rc;
}

// The contraction launch of one layout class, persistent on the tuned grid or, for long items, on every
// resident slot of the device; nothing for an empty class.  Consumes the last screening results;
// `cleared`: the screening has just cleared the queue counters.
static int group_enqueue_class(tamm_group* g, int c, bool cleared, hipStream_t s) {
  const int n = g->cls_begin[c + 1] - g->cls_begin[c];
  if (n <= 0) return TAMM_OK;
  ContractParams cp{};
  int grid = 0;
  if (g->grid[c] > 0 || g->queued[c]) {
    grid = g->grid[c] > 0 ? std::min<int>(g->grid[c], n) : g->auto_grid[c];
    cp.queue_next = (int32_t*)(g->ws + g->off_counter) + c * kQueues;
    std::copy(g->queue_begin[c], g->queue_begin[c] + kQueues + 1, cp.queue_begin);
    if (!cleared) HIP_TRY(launch_clear_queues(cp.queue_next, s));
  }
  cp.probs = (const ProblemDesc*)(g->ws + g->off_pdesc);
  cp.work = (const WorkItem*)(g->ws + g->off_work) + g->cls_begin[c];
  cp.n_work = n;
  HIP_TRY(launch_contract_f64(g->cfg[c], c, cp, grid, s));
  return TAMM_OK;
}

namespace tamm {

// TAMM_GROUP_SERIAL: the layout classes' launches one after another.
static bool group_serial() {
  static const bool v = [] {
    const char* e = getenv("TAMM_GROUP_SERIAL");
    return e && atoi(e) != 0;
  }();
  return v;
}

// Whether the group may be captured.  Several groups of several layout classes, captured before their
// first launch outside a capture, alive together and replayed in turn, have ended in a segmentation
// fault on the host whose cause is not known; that order is refused.
int group_check_capture(const tamm_group* g) {
  int present = 0;
  for (int c = 0; c < kLayouts; ++c) present += g->cls_begin[c + 1] > g->cls_begin[c] ? 1 : 0;
  if (present > 1 && !g->ran && !group_serial())
    return fail(TAMM_ERR_UNSUPPORTED, "a group of several gather layouts must be executed once before it is captured");
  return TAMM_OK;
}

// Enqueue the group's kernels (screening, which clears the queue counters, then each class's
// contraction), consuming the descriptors in the workspace.
int group_enqueue(tamm_group* g, hipStream_t s) {
  if (!g->ran) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) != hipSuccess) (void)hipGetLastError();  // the launches will say it
    else if (status == hipStreamCaptureStatusNone) g->ran = true;
    else if (const int rc = group_check_capture(g)) return rc;
  }
  ScreenParams sp{};
  sp.probs = (const ScreenDesc*)(g->ws + g->off_sdesc);
  sp.item_prob = (const int32_t*)(g->ws + g->off_sitems);
  sp.item_block = sp.item_prob + g->sitem_prob.size();
  sp.n_items = (int32_t)g->sitem_prob.size();
  sp.queue_next = (int32_t*)(g->ws + g->off_counter);
  sp.n_queues = kLayouts * kQueues;
  static_assert(kLayouts * kQueues <= 64, "one counter per lane of a screening workgroup");
  HIP_TRY(launch_screen(sp, s));
  // one persistent launch per gather layout present in the group.  With several, they run
  // concurrently: the first on the caller's stream, the others on side streams that wait for the
  // screening and that the caller's stream then waits for, so the workgroups of one class take
  // the compute units the tail of another leaves free (each workgroup only pulls work items
  // from its own class's counter, so no launch waits on another)
  int present[kLayouts], np = 0;
  for (int c = 0; c < kLayouts; ++c)
    if (g->cls_begin[c + 1] > g->cls_begin[c]) present[np++] = c;
  if (np <= 1 || group_serial()) {
    for (int i = 0; i < np; ++i) {
      const int rc = group_enqueue_class(g, present[i], true, s);
      if (rc != TAMM_OK) return rc;
    }
    return TAMM_OK;
  }
  if (!g->ev_fork) HIP_TRY(hipEventCreateWithFlags(&g->ev_fork, hipEventDisableTiming));
  HIP_TRY(hipEventRecord(g->ev_fork, s));
  for (int i = 1; i < np; ++i) {
    const int c = present[i];
    if (!g->side[c]) HIP_TRY(hipStreamCreateWithFlags(&g->side[c], hipStreamNonBlocking));
    if (!g->ev_join[c]) HIP_TRY(hipEventCreateWithFlags(&g->ev_join[c], hipEventDisableTiming));
    HIP_TRY(hipStreamWaitEvent(g->side[c], g->ev_fork, 0));
    const int rc = group_enqueue_class(g, c, true, g->side[c]);
    if (rc != TAMM_OK) return rc;
    HIP_TRY(hipEventRecord(g->ev_join[c], g->side[c]));
  }
  const int rc = group_enqueue_class(g, present[0], true, s);
  if (rc != TAMM_OK) return rc;
  for (int i = 1; i < np; ++i) HIP_TRY(hipStreamWaitEvent(s, g->ev_join[present[i]], 0));
  return TAMM_OK;
}

}  // namespace tamm

static int group_check(tamm_group* g) {
  if (!g->bound) return fail(TAMM_ERR_UNBOUND, "group workspace is not bound (or the configuration changed since binding)");
  for (auto* p : g->plans) {
    int rc = check_tensors(p);
    if (rc != TAMM_OK) return rc;
  }
  // nodes must be independent: no node writes storage that another node reads or writes
  for (size_t i = 0; i < g->nodes.size(); ++i)
    for (size_t j = 0; j < g->nodes.size(); ++j) {
      if (i == j) continue;
      const tamm_tensor* out = g->nodes[i][0]->out;
      for (const tamm_plan* b : g->nodes[j])
        if (overlaps(out, b->out) || overlaps(out, b->lhs) || overlaps(out, b->rhs))
          return fail(TAMM_ERR_ARG, "group members %zu and %zu are not independent (member %zu writes storage member %zu uses)",
                      i, j, i, j);
    }
  return TAMM_OK;
}

namespace tamm {

// Refresh the device descriptors when storage bindings or coefficients changed (after draining
// the stream: earlier launches may still read the old ones).
int group_update_desc(tamm_group* g, const double* alpha, const double* beta, hipStream_t s, bool* changed) {
  std::vector<ScreenDesc> sds;
  std::vector<ProblemDesc> pds;
  group_descs(g, g->ws, alpha, beta, sds, pds);
  const bool sc = memcmp(sds.data(), g->sdesc.data(), sds.size() * sizeof(ScreenDesc)) != 0;
  const bool pc = memcmp(pds.data(), g->pdesc.data(), pds.size() * sizeof(ProblemDesc)) != 0;
  *changed = sc || pc;
  if (*changed) {
    HIP_TRY(hipStreamSynchronize(s));
    if (sc) HIP_TRY(hipMemcpy(g->ws + g->off_sdesc, sds.data(), sds.size() * sizeof(ScreenDesc), hipMemcpyHostToDevice));
    if (pc) HIP_TRY(hipMemcpy(g->ws + g->off_pdesc, pds.data(), pds.size() * sizeof(ProblemDesc), hipMemcpyHostToDevice));
    g->sdesc.swap(sds);
    g->pdesc.swap(pds);
  }
  return TAMM_OK;
}

int group_check_bound(tamm_group* g) { return group_check(g); }
size_t group_node_count(const tamm_group* g) { return g->nodes.size(); }

}  // namespace tamm

// Whether the descriptors in the workspace match the current bindings and these coefficients.
static bool group_desc_current(const tamm_group* g, const double* alpha, const double* beta) {
  std::vector<ScreenDesc> sds;
  std::vector<ProblemDesc> pds;
  group_descs(g, g->ws, alpha, beta, sds, pds);
  return memcmp(sds.data(), g->sdesc.data(), sds.size() * sizeof(ScreenDesc)) == 0 &&
         memcmp(pds.data(), g->pdesc.data(), pds.size() * sizeof(ProblemDesc)) == 0;
}

extern "C" int tamm_group_execute(tamm_group* g, const double* alpha, const double* beta, void* stream) {
  if (!g || !alpha || !beta) return fail(TAMM_ERR_ARG, "null argument");
  int rc = group_check(g);
  if (rc != TAMM_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  bool changed = false;
  if (g->exec) {
    const size_t n = g->nodes.size();
    const bool same = std::equal(alpha, alpha + n, g->g_alpha.begin()) && std::equal(beta, beta + n, g->g_beta.begin());
    if (same && group_desc_current(g, alpha, beta)) {  // the captured graph used these descriptors
      HIP_TRY(hipGraphLaunch(g->exec, s));
      return ok();
    }
    group_drop_graph(g);
  }
  // eager path: descriptor refresh when something changed (after the stream drained, so that
  // earlier launches that read the old descriptors are finished), then the launches
  rc = group_update_desc(g, alpha, beta, s, &changed);
  if (rc != TAMM_OK) return rc;
  rc = group_enqueue(g, s);
  return rc == TAMM_OK ? ok() : rc;
}

extern "C" int tamm_group_capture(tamm_group* g, const double* alpha, const double* beta, void* stream) {
  if (!g || !alpha || !beta) return fail(TAMM_ERR_ARG, "null argument");
  int rc = group_check(g);
  if (rc == TAMM_OK) rc = group_check_capture(g);
  if (rc != TAMM_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  bool changed = false;
  rc = group_update_desc(g, alpha, beta, s, &changed);
  if (rc != TAMM_OK) return rc;
  group_drop_graph(g);
  hipStream_t cs;
  HIP_TRY(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
  hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) {
    (void)hipStreamDestroy(cs);
    return fail(TAMM_ERR_HIP, "hipStreamBeginCapture: %s", hipGetErrorString(e));
  }
  rc = group_enqueue(g, cs);
  hipGraph_t graph = nullptr;
  e = hipStreamEndCapture(cs, &graph);
  (void)hipStreamDestroy(cs);
  if (rc != TAMM_OK) {
    if (graph) (void)hipGraphDestroy(graph);
    return rc;
  }
  if (e != hipSuccess) return fail(TAMM_ERR_HIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
  hipGraphExec_t exec = nullptr;
  e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    (void)hipGraphDestroy(graph);
    return fail(TAMM_ERR_HIP, "hipGraphInstantiate: %s", hipGetErrorString(e));
  }
  g->graph = graph;
  g->exec = exec;
  g->g_alpha.assign(alpha, alpha + g->nodes.size());
  g->g_beta.assign(beta, beta + g->nodes.size());
  return ok();
}

namespace tamm {

// Autotuner of a group (see tamm_group_autotune): per gather layout class, the fastest
// (configuration, grid) of the class's own launch, timed with alpha = 0, beta = 1.
int group_autotune(tamm_group* g, hipStream_t s, const char* cache_path, int32_t reps) {
  int rc = group_check(g);
  if (rc != TAMM_OK) return rc;
  void* ws = g->ws;
  const size_t bytes = g->ws_bytes;
  CacheEntry best[kLayouts];
  char tag[kLayouts][16];
  bool cached = true;
  for (int c = 0; c < kLayouts; ++c) {
    best[c] = CacheEntry{-1, 1, 0, 1e30};
    snprintf(tag[c], sizeof(tag[c]), "group%d", c);
    cached = cache_lookup(cache_path, g->signature, tag[c], best[c]) && cached;
  }
  if (!cached) {
    if (reps <= 0) reps = 3;
    for (int c = 0; c < kLayouts; ++c) best[c] = CacheEntry{-1, 1, 0, 1e30};
    std::vector<double> a0(g->nodes.size(), 0.0), b1(g->nodes.size(), 1.0);
    TimerEvents ev;
    if ((rc = ev.create()) != TAMM_OK) return rc;
    hipEvent_t e0 = ev.e0, e1 = ev.e1;
    int cus = 256, dev = 0;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    for (int k = 0; k < f64_config_count() && rc == TAMM_OK; ++k) {
      if (f64_config_canonical(k) != k) continue;  // another id of a kernel already timed
      for (int mult : {0, 1, 2, 4}) {  // 0: every resident slot (occupancy-sized grid)
        if (rc != TAMM_OK) break;  // a failed launch ends the search with its error
        if ((rc = group_configure(g, k, mult * cus)) != TAMM_OK) break;
        if (g->ws_size > bytes) continue;
        if ((rc = group_bind(g, ws, bytes)) != TAMM_OK) break;
        // screening and a warm-up; alpha = 0, beta = 1 leaves every output unchanged (finite
        // operands), and the classes' launches below reuse that screening
        bool changed = false;
        if ((rc = group_update_desc(g, a0.data(), b1.data(), s, &changed)) != TAMM_OK) break;
        if ((rc = group_enqueue(g, s)) != TAMM_OK) break;
        for (int c = 0; c < kLayouts && rc == TAMM_OK; ++c) {
          if (g->cls_begin[c + 1] == g->cls_begin[c]) continue;
          HIP_TRY(hipEventRecord(e0, s));
          for (int r = 0; r < reps && rc == TAMM_OK; ++r) rc = group_enqueue_class(g, c, false, s);
          HIP_TRY(hipEventRecord(e1, s));
          HIP_TRY(hipEventSynchronize(e1));
          float ms = 0;
          HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
          ms /= reps;
          if (ms < best[c].ms) best[c] = CacheEntry{k, 1, mult * cus, ms};
        }
      }
    }
    if (rc != TAMM_OK) return rc;
    for (int c = 0; c < kLayouts; ++c)
      if (g->cls_begin[c + 1] != g->cls_begin[c] && best[c].config < 0)
        return fail(TAMM_ERR_WORKSPACE, "no configuration fits the bound workspace");
    for (int c = 0; c < kLayouts; ++c) cache_store(cache_path, g->signature, tag[c], best[c]);
  }
  int cfgs[kLayouts], grids[kLayouts];
  for (int c = 0; c < kLayouts; ++c) {
    cfgs[c] = best[c].config;  // < 0 (empty class): default
    grids[c] = best[c].config >= 0 ? best[c].grid : 0;
  }
  rc = group_configure_classes(g, cfgs, grids);
  if (rc != TAMM_OK) return rc;
  if (g->ws_size > bytes) return fail(TAMM_ERR_WORKSPACE, "cached configuration needs %zu bytes", g->ws_size);
  return group_bind(g, ws, bytes);
}

size_t group_workspace_size(const tamm_group* g) { return g->ws_size; }

// The largest workspace any configuration of the group needs: its layout reserves room for the work
// lists of any mix of them.
size_t group_autotune_workspace_size(tamm_group* g) { return g->ws_size; }

int group_bind_ws(tamm_group* g, void* ws, size_t bytes) { return group_bind(g, ws, bytes); }

}  // namespace tamm

extern "C" int tamm_group_autotune(tamm_group* g, void* stream, const char* cache_path, int32_t reps) {
  if (!g) return fail(TAMM_ERR_ARG, "null group");
  const int rc = group_autotune(g, (hipStream_t)stream, cache_path, reps);
  return rc == TAMM_OK ? ok() : rc;
}

extern "C" int tamm_group_stats(const tamm_group* g, int32_t* config, int32_t* grid, int64_t* work_items) {
  if (!g) return fail(TAMM_ERR_ARG, "null group");
  // the class with the most work items speaks for the group
  int big = 0;
  for (int c = 1; c < kLayouts; ++c)
    if (g->cls_begin[c + 1] - g->cls_begin[c] > g->cls_begin[big + 1] - g->cls_begin[big]) big = c;
  if (config) *config = g->cfg[big];
  if (grid) *grid = g->grid[big];
  if (work_items) *work_items = (int64_t)g->work.size();
  return ok();
}

extern "C" int tamm_group_destroy(tamm_group* g) {
  if (g) {
    group_drop_graph(g);
    for (int c = 0; c < kLayouts; ++c) {
      if (g->side[c]) (void)hipStreamDestroy(g->side[c]);
      if (g->ev_join[c]) (void)hipEventDestroy(g->ev_join[c]);
    }
    if (g->ev_fork) (void)hipEventDestroy(g->ev_fork);
  }
  delete g;
  return ok();
}

namespace tamm {

void plan_io(const tamm_plan* p, tamm_tensor** out, const tamm_tensor** lhs, const tamm_tensor** rhs, int* precision) {
  *out = p->out;
  *lhs = p->lhs;
  *rhs = p->rhs;
  *precision = p->prec;
}

bool plans_fusable(tamm_plan* a, tamm_plan* b) {
  const std::vector<tamm_plan*> node{a, b};
  return a->prec == TAMM_PREC_F64 && b->prec == TAMM_PREC_F64 && check_fusable(node) == TAMM_OK;
}

}  // namespace tamm
