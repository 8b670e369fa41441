// HIP kernels for gfx950: tile-pair screening, the FP64 block-sparse contraction (index-permuted
// LDS gathers feeding v_mfma_f64_16x16x4_f64, atomic-free epilogue), the ordered K-split
// reduction and the orbital-energy denominator update.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "internal.h"

// Part of the file to compile: 0 = all but the float64 contraction kernels, n = those of
// TAMM_F64_KERNELS_n (they take most of the compile time and are built side by side).
#ifndef TAMM_F64_PART
#define TAMM_F64_PART 0
#endif

namespace tamm {

typedef double d4_t __attribute__((ext_vector_type(4)));

#if TAMM_F64_PART == 0
// ---------------------------------------------------------------------------------------------
// Tile-pair screening (the block non-zero analysis).  One wave per stored output block walks the
// K tile tuples in lexicographic order, keeps a pair when both operand blocks are stored, and
// compacts the survivors in order with a wave ballot (deterministic, no atomics).  A fused node
// (several contractions into the same output tiles) walks its segments one after another and
// appends to one list, so that one output tile's K loop later runs over every segment's pairs.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_screen(ScreenParams P) {
  const int item = blockIdx.x;
  if (item >= P.n_items) return;
  const ScreenDesc* S = P.probs ? P.probs + P.item_prob[item] : &P.single;
  const int ob = P.probs ? P.item_block[item] : item;
  const int lane = threadIdx.x;
  if (item == 0 && lane < P.n_queues) P.queue_next[lane] = 0;
  PairDesc* __restrict__ out = S->pairs + (int64_t)ob * S->pair_stride;
  int32_t* counts = S->counts;
  int count = 0;
  while (true) {  // segments of a fused node append to one list, in order
    const OutBlockDesc blk = S->blocks[ob];
    for (int kt0 = 0; kt0 < S->n_kt; kt0 += 64) {
      const int kt = kt0 + lane;
      bool keep = false;
      int64_t aoff = -1, boff = -1;
      int kext = 1, acls = blk.a_cbase, bcls = blk.b_cbase;
      if (kt < S->n_kt) {
        int rem = kt, alin = blk.a_tbase, blin = blk.b_tbase;
        for (int k = S->nk - 1; k >= 0; --k) {
          const int t = rem % S->k_ntiles[k];
          rem /= S->k_ntiles[k];
          alin += t * S->a_tstride[k];
          blin += t * S->b_tstride[k];
          const int c = S->pool[S->k_cls_tab[k] + t];
          acls += c * S->a_cstride[k];
          bcls += c * S->b_cstride[k];
          kext *= S->pool[S->k_size_tab[k] + t];
        }
        aoff = S->a_tile_off[alin];
        boff = S->b_tile_off[blin];
        keep = aoff >= 0 && boff >= 0;
      }
      const unsigned long long mask = __ballot(keep);
      if (keep) {
        const int rank = __popcll(mask & ((1ull << lane) - 1ull));
        PairDesc d;
        d.a_off = aoff + S->a_base;
        d.b_off = boff + S->b_base;
        d.kext = kext;
        d.a_tabM = S->pool[S->a_cls_tabM + acls] + S->pool_base;
        d.a_tabK = S->pool[S->a_cls_tabK + acls] + S->pool_base;
        d.b_tabK = S->pool[S->b_cls_tabK + bcls] + S->pool_base;
        d.b_tabN = S->pool[S->b_cls_tabN + bcls] + S->pool_base;
        d.kt = kt;
        out[count + rank] = d;
      }
      count += __popcll(mask);
    }
    if (S->next_seg < 0) break;
    S = P.probs + S->next_seg;
  }
  if (lane == 0) counts[ob] = count;
}

hipError_t launch_screen(const ScreenParams& p, hipStream_t s) {
  if (p.n_items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_screen, dim3(p.n_items), dim3(64), 0, s, p);
  return hipGetLastError();
}
#endif  // TAMM_F64_PART == 0

// ---------------------------------------------------------------------------------------------
// FP64 contraction.
//
// A workgroup owns one output macro-tile (MT x NT of the flattened M x N of one stored output
// block) and, with K splits, one contiguous range of that block's surviving pairs.  The K loop
// runs over the pairs and, inside a pair, over chunks of KT flattened K indices.  Each chunk is
// gathered from the operand blocks through the plan's offset tables straight into LDS; the
// thread-to-element mapping follows the operand's stride-1 label (lanes along k when it is a
// summed label, along m/n otherwise) so that global reads coalesce.  Each operand chunk sits in
// LDS in the layout LdsLayout chooses for its orientation and size, which keeps the MFMA operand
// reads and the gather stores free of bank conflicts.  There is no separate permutation pass.
//
// Software pipeline with one barrier per chunk: LDS holds two chunk buffers.  While the MFMAs
// of chunk c run from one buffer, the registers holding chunk c+1 (loaded during the previous
// chunk's MFMAs) are stored into the other buffer, the global loads of chunk c+2 are issued into
// the same registers, and the offset-table entries of chunk c+3 are fetched; these and the operand
// reads of k-step s+1 are spread between the products of step s, and the barrier comes before the
// last step's.  A tile takes the body compiled for its own number of 16 x 16 fragments per wave
// (the planner cuts a block into tiles of even size), so no branch sits in the MFMA stream and no
// fragment past a block's end is multiplied.
//
// v_mfma_f64_16x16x4_f64 lane layout (gfx950, checked on the device): A[m][k] comes from lane
// m + 16k, B[k][n] from lane n + 16k, and D[m][n] lands in lane n + 16*(m%4), register m/4.
//
// The epilogue writes beta*C + alpha*acc through out's offset tables; every element is written
// by exactly one workgroup (beta == 0 never reads C).  With K splits, partial tiles go to the
// workspace and k_reduce sums them in split order.  Results are bitwise reproducible.
//
// Launch modes: one workgroup per work item, or a persistent grid whose workgroups take items
// from the queue of the die they run on (long items, queue_pays in the planner); the item order is
// the plan's.  The operands' gather
// layouts (A_KC, B_KC) are template parameters: "layout" = 2*A_KC + B_KC.
// ---------------------------------------------------------------------------------------------
// LDS layout of one operand chunk (ROWS rows x KT summed indices, float64), chosen by the LDS's
// measured service pattern on gfx950 (8-byte reads: 32 lanes per cycle over 64 four-byte banks;
// 8-byte writes: 16 lanes per cycle over 32 banks; 16-byte writes: 8 lanes per cycle over 32
// banks) for the MFMA operand reads (8 bytes per lane: lanes 16q + r read row R0 + r at k-step
// position q) and the gather's stores:
//   kind 0, an operand whose stride-1 label is summed (lanes gather along k), up to 128 rows:
//     [row][k] with a row stride of KT + 2 doubles -- half the stride is odd, so the 16 rows x 2 k
//     of a read cycle land on 32 distinct 8-byte bank pairs, and a lane's two adjacent k go in
//     one aligned 16-byte store;
//   kind 1, the other operands with rows = 16 mod 32 or at least 128 rows: [k][row] with a k
//     stride of rows + pad (16 mod 32 doubles) -- 16 consecutive rows of one k fill half the
//     banks and the next k the other half, and a lane's two adjacent rows go in one store;
//   kind 2, otherwise (where that padding would cost LDS occupancy): [row][k] with an odd row
//     stride KT + 1, reads two-way conflicted.
template <int ROWS, int KT, bool KC>
struct LdsLayout {
  static constexpr int KIND = KC ? (ROWS <= 128 ? 0 : 2) : ((ROWS % 32 == 16 || ROWS >= 128) ? 1 : 2);
  static constexpr int LDR = ROWS + ((48 - ROWS % 32) % 32);  // kind 1: k stride, 16 mod 32
  static constexpr int RS = KIND == 1 ? 1 : (KIND == 0 ? KT + 2 : KT + 1);  // element stride between rows
  static constexpr int KS = KIND == 1 ? LDR : 1;                            // ... between k positions
  static constexpr int SIZE = KIND == 1 ? KT * LDR : ROWS * RS;             // doubles per buffer
  static constexpr int PAIR = KC ? KS : RS;  // distance of the two elements of a 16-byte gather load
  static constexpr bool STORE16 = PAIR == 1 && (KC ? RS : KS) % 2 == 0;  // they go in one aligned store
  static_assert(KIND != 1 || LDR % 32 == 16, "kind 1 stride");
  static_assert(KIND != 0 || (RS / 2) % 2 == 1, "kind 0 stride");
  static_assert(SIZE % 2 == 0, "16-byte aligned buffers");
  __device__ static constexpr int at(int row, int k) { return row * RS + k * KS; }
};

// A gather load's VEC elements into LDS: one 16-byte store when they are adjacent and aligned,
// else one store each, PAIR elements apart
template <int VEC, int PAIR, bool STORE16>
__device__ __forceinline__ void lds_store(double* dst, const double* v) {
  if constexpr (VEC == 2 && STORE16) {
    typedef double d2_t __attribute__((ext_vector_type(2)));
    *reinterpret_cast<d2_t*>(dst) = (d2_t){v[0], v[1]};
  } else {
    dst[0] = v[0];
    if constexpr (VEC == 2) dst[PAIR] = v[1];
  }
}

// The register that holds the die (XCC) a wave runs on: id 20, offset 0, 4 bits.
constexpr int kXccIdReg = 20 | (0 << 6) | ((4 - 1) << 11);

// One work item whose tile takes FM x FN fragments of 16 x 16 per wave: at most (16 WGM FM) x
// (16 WGN FN) elements, the last ones possibly past the item's rows or columns.  FMX, FNX: the
// configuration's largest fragment counts (the layout of the partial tiles).
template <int FM, int FN, int FMX, int FNX, int KT, int WGM, int WGN, bool A_KC, bool B_KC, int VEC>
__device__ __forceinline__ void contract_tile(const ProblemDesc& pr, const WorkItem& w, const OutBlockDesc& blk, double* smem) {
  constexpr int NTHR = 64 * WGM * WGN;
  constexpr int WM = 16 * FM, WN = 16 * FN, MT = WM * WGM, NT = WN * WGN;
  constexpr int MT_MAX = 16 * FMX * WGM, NT_MAX = 16 * FNX * WGN;
  constexpr int NS = KT / 4;  // MFMA k-steps per chunk
  static_assert(KT % 8 == 0, "an even number of k-steps");
  // 16-byte gathers where this tile's chunks split into them
  constexpr bool VEC_FITS = gather_pairs_fit<MT, KT, NTHR, A_KC>() && gather_pairs_fit<NT, KT, NTHR, B_KC>();
  constexpr int V = VEC == 2 && VEC_FITS ? 2 : 1;
  using G = Gather<MT, NT, KT, NTHR, A_KC, B_KC, double, V>;
  using LA = LdsLayout<MT, KT, A_KC>;
  using LB = LdsLayout<NT, KT, B_KC>;
  static_assert(LA::SIZE <= LdsLayout<MT_MAX, KT, A_KC>::SIZE && LB::SIZE <= LdsLayout<NT_MAX, KT, B_KC>::SIZE,
                "a smaller tile fits the configuration's buffers");
  double* const As = smem;
  double* const Bs = smem + 2 * LA::SIZE;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // keeps the addresses of one tile size out of the registers of the others
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int lr = lane & 15, lq = lane >> 4;
  const int a_frag = LA::at(wm * WM + lr, lq);  // this lane's operand reads at k-step 0
  const int b_frag = LB::at(wn * WN + lr, lq);
  G g;
  g.init(tid);
  const int32_t* __restrict__ pool = pr.pool;
  const PairDesc* __restrict__ pairs = pr.pairs + blk.pair_base;
  const int cnt = wave_uniform(gload(pr.counts + w.ob));
  const int nsplit = shape_nsplit(w.shape), split = shape_split(w.shape);
  const int pb = (int)(((int64_t)cnt * split) / nsplit), pe = (int)(((int64_t)cnt * (split + 1)) / nsplit);

  d4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = (d4_t){0.0, 0.0, 0.0, 0.0};

  if (pb < pe) {
    double af[2][FM], bf[2][FN];  // operands of two k-steps
    constexpr int NF = FM * FN, NR = FM + FN, AL = G::MA::L, NL = AL + G::MB::L, NP = NF * (NS - 1);
    constexpr int RPP = (NR + NF - 1) / NF;  // operand reads beside one product
    // operand r (A fragments, then B fragments) of k-step st of the chunk in buffer b, into set f
    auto fetch = [&](int b, auto st, auto r, auto f) {
      if constexpr (r() < FM) af[f()][r()] = As[b * LA::SIZE + a_frag + r() * 16 * LA::RS + 4 * st() * LA::KS];
      else bf[f()][r() - FM] = Bs[b * LB::SIZE + b_frag + (r() - FM) * 16 * LB::RS + 4 * st() * LB::KS];
    };
    // staged load y of the chunk (A's, then B's): to LDS buffer b, and from memory again
    auto restage = [&](int b, auto y) {
      constexpr int e = (y() < AL ? y() : y() - AL) * V;
      if constexpr (y() < AL)
        lds_store<V, LA::PAIR, LA::STORE16>(&As[b * LA::SIZE + LA::at(g.a_lds_row(e), g.a_lds_k(e))], &g.ra[e]);
      else
        lds_store<V, LB::PAIR, LB::STORE16>(&Bs[b * LB::SIZE + LB::at(g.b_lds_row(e), g.b_lds_k(e))], &g.rb[e]);
      g.load_one(y());
    };
    // the operand reads beside product x of a k-step: of k-step st of buffer b, into set f
    auto fetch_beside = [&](int b, auto st, auto x, auto f) {
      static_for<RPP>([&](auto q) {
        if constexpr (x() * RPP + q() < NR) fetch(b, st, int_c<x() * RPP + q()>{}, f);
      });
    };
    ChunkWalk<KT, G, double> walk(g, pairs, pb, pe, pool, pr.A, pr.B, w, blk.mext, blk.next);
    walk.setup();
    g.load_tables(walk.d, pool, 0);
    g.load_data();
    bool inflight = walk.next_tables();  // the chunk staged during this one is real
    static_for<NL>([&](auto y) { restage(0, y); });
    bool tabs = inflight && walk.next_tables();  // so is the one after it
    __syncthreads();
    static_for<NR>([&](auto r) { fetch(0, int_c<0>{}, r, int_c<0>{}); });
    for (int buf = 0;; buf ^= 1) {
      // Every k-step but the last: beside each product the wave issues a little of what feeds the
      // later ones -- an operand read of the next k-step, and in the first half now and then the LDS
      // store of one staged load and the load that refills its registers (early, so that they
      // arrive before the next chunk stores them).  Left to itself the compiler issues all stores
      // and loads of the chunk in one run, during which the wave multiplies nothing: dense 4D on
      // 1024-row blocks 66.0 TF/s, against 69.3 with the stores spread and 70.9 with the barrier
      // before the last step's products as well (128 x 128 tiles).
      __builtin_amdgcn_s_setprio(1);  // MFMA phase first when waves of two workgroups compete
      static_for<NP>([&](auto x) {
        constexpr int st = x() / NF, i = x() % NF / FN, j = x() % FN;
        fetch_beside(buf, int_c<st + 1>{}, int_c<x() % NF>{}, int_c<(st + 1) & 1>{});
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[st & 1][i], bf[st & 1][j], acc[i][j], 0, 0, 0);
        constexpr int y0 = min_c(2 * x() * NL / NP, NL), y1 = min_c(2 * (x() + 1) * NL / NP, NL);
        static_for<y1 - y0>([&](auto y) { restage(buf ^ 1, int_c<y0 + y()>{}); });
        __builtin_amdgcn_sched_barrier(0);
      });
      // Here every wave holds the operands of the chunk's last k-step and has stored its part of
      // the next chunk: the buffers change hands, and the next chunk's first operands are read
      // under the last step's products.
      __syncthreads();
      static_for<NF>([&](auto x) {
        constexpr int i = x() / FN, j = x() % FN;
        fetch_beside(buf ^ 1, int_c<0>{}, x, int_c<0>{});
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[1][i], bf[1][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_s_setprio(0);
      const bool tabs_next = tabs && walk.next_tables();
      if (!inflight) break;
      inflight = tabs;
      tabs = tabs_next;
    }
  }

  // epilogue: lane holds D[m][n] for m = 4r + lane/16 (register r), n = lane%16
  const int mb = wm * WM + lq, nb = wn * WN + lr;  // this lane's first row and column in the tile
  if (nsplit > 1) {
    double* part = pr.partial + ((int64_t)w.tile + split) * (MT_MAX * NT_MAX);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(mb + i * 16 + 4 * r) * NT_MAX + nb + j * 16] = acc[i][j][r];
  } else {
    // through out's offset tables: every table entry first (the tables are padded, so rows and
    // columns past the block read in bounds), then per row block the old values (beta != 0),
    // then the results, so that no load waits behind the use of another
    const double alpha = pr.alpha, beta = pr.beta;
    __attribute__((address_space(1))) double* __restrict__ Cg = (__attribute__((address_space(1))) double*)pr.C;
    const int rows = shape_rows(w.shape), cols = shape_cols(w.shape);
    int32_t rt[FM][4], ct[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) rt[i][r] = gload(pool + blk.c_tabM + w.m0 + mb + i * 16 + 4 * r);
#pragma unroll
    for (int j = 0; j < FN; ++j) ct[j] = gload(pool + blk.c_tabN + w.n0 + nb + j * 16);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      double old[4][FN];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const bool live = mb + i * 16 + 4 * r < rows && nb + j * 16 < cols;
          old[r][j] = (beta != 0.0 && live) ? Cg[blk.c_off + rt[i][r] + ct[j]] : 0.0;
        }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const bool live = mb + i * 16 + 4 * r < rows && nb + j * 16 < cols;
          const double v = alpha * acc[i][j][r];
          if (live) Cg[blk.c_off + rt[i][r] + ct[j]] = (beta == 0.0) ? v : beta * old[r][j] + v;
        }
    }
  }
}

// The tile body for the item's fragment counts (um x un per wave), each compiled for its own
// counts: the chunk loop has no branch in its product stream whatever the tile's size.
template <int FM, int FN, int FMX, int FNX, int KT, int WGM, int WGN, bool A_KC, bool B_KC, int VEC>
__device__ __forceinline__ void contract_any(int um, int un, const ProblemDesc& pr, const WorkItem& w, const OutBlockDesc& blk,
                                             double* smem) {
  if (FN > 1 && un < FN) {
    if constexpr (FN > 1) contract_any<FM, FN - 1, FMX, FNX, KT, WGM, WGN, A_KC, B_KC, VEC>(um, un, pr, w, blk, smem);
  } else if (FM > 1 && um < FM) {
    if constexpr (FM > 1) contract_any<FM - 1, FN, FMX, FNX, KT, WGM, WGN, A_KC, B_KC, VEC>(um, FN, pr, w, blk, smem);
  } else {
    contract_tile<FM, FN, FMX, FNX, KT, WGM, WGN, A_KC, B_KC, VEC>(pr, w, blk, smem);
  }
}

template <int MT, int NT, int KT, int WGM, int WGN, int OCC, bool A_KC, bool B_KC, int VEC>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(OCC))) void k_contract_f64(ContractParams P) {
  constexpr int FM = MT / WGM / 16, FN = NT / WGN / 16;
  static_assert(MT == FM * WGM * 16 && NT == FN * WGN * 16, "wave tile must be a multiple of 16");
  __shared__ __attribute__((aligned(16))) double smem[2 * (LdsLayout<MT, KT, A_KC>::SIZE + LdsLayout<NT, KT, B_KC>::SIZE)];
  __shared__ int s_next;
  // A launch with one workgroup per item runs its own; a persistent one takes items from its die's
  // queue and, when that is empty, from the queue with the most items left (counters only grow, so
  // every workgroup ends).
  const bool queued = P.queue_next != nullptr;
  int queue = queued ? (int)__builtin_amdgcn_s_getreg(kXccIdReg) & (kQueues - 1) : 0;
  int item = blockIdx.x;
  while (true) {
    if (queued) {
      __syncthreads();  // s_next and the tile buffers are free
      if (threadIdx.x < kQueues) {  // one lane per queue
        const int lane = threadIdx.x, begin = P.queue_begin[lane], len = P.queue_begin[lane + 1] - begin;
        int found = -1;
        while (true) {
          int i = len;
          if (lane == queue && len > 0) i = atomicAdd(P.queue_next + lane, 1);
          found = __shfl(i < len ? begin + i : -1, queue);
          if (found >= 0) break;
          const int left = len - __hip_atomic_load(P.queue_next + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          int most = left;
#pragma unroll
          for (int o = kQueues / 2; o > 0; o /= 2) most = max(most, __shfl_xor(most, o));
          if (most <= 0) break;  // nothing is left anywhere
          queue = __ffsll(__ballot(left == most)) - 1;
        }
        if (lane == 0) s_next = found;
      }
      queue = __shfl(queue, 0);
      __syncthreads();
      item = s_next;
      if (item < 0) break;
    } else if (item >= P.n_work) {
      break;
    }
    // work-item descriptors are the same for the whole wave: keep them in scalar registers
    const WorkItem w = wave_uniform(sload(P.work + wave_uniform(item)));
    const ProblemDesc pr = wave_uniform(P.probs ? sload(P.probs + w.prob) : P.single);
    const OutBlockDesc blk = wave_uniform(sload(pr.blocks + w.ob));
    contract_any<FM, FN, FM, FN, KT, WGM, WGN, A_KC, B_KC, VEC>((shape_rows(w.shape) + 16 * WGM - 1) / (16 * WGM),
                                                                 (shape_cols(w.shape) + 16 * WGN - 1) / (16 * WGN), pr, w, blk,
                                                                 smem);
    if (!queued) break;
  }
}

#if TAMM_F64_PART == 0
__global__ void k_clear_queues(int32_t* queue_next) {
  if (threadIdx.x < kQueues) queue_next[threadIdx.x] = 0;
}

hipError_t launch_clear_queues(int32_t* queue_next, hipStream_t s) {
  hipLaunchKernelGGL(k_clear_queues, dim3(1), dim3(64), 0, s, queue_next);
  return hipGetLastError();
}

// Ordered reduction of K-split partial tiles (split 0, 1, ... in order) and the epilogue.  A
// workgroup takes kReduceUnroll elements per thread of one tile (grid: tiles x parts of a tile) and
// issues all their loads (table entries, then the partials and old values) before any use.  A
// workgroup per tile walked its 4096 elements four rounds one after another, each a memory round
// trip: 10.7 us for 96 tiles of 25 x 25, six splits.
constexpr int kReduceUnroll = 4, kReduceThreads = 256;

__global__ __launch_bounds__(kReduceThreads) void k_reduce(ReduceParams P) {
  const int t = blockIdx.x;
  if (t >= P.n_items) return;
  const ReduceItem it = P.items[t];
  const int rows = shape_rows(it.shape), cols = shape_cols(it.shape), nsplit = shape_nsplit(it.shape);
  const int e0 = (int)blockIdx.y * kReduceUnroll * kReduceThreads + (int)threadIdx.x;
  if (e0 >= rows * cols) return;
  const ProblemDesc& pr = P.probs ? P.probs[it.prob] : P.single;
  const OutBlockDesc blk = pr.blocks[it.ob];
  const int tile = P.tile_m * P.tile_n;
  const double* part = pr.partial + (int64_t)it.tile * tile;
  const double alpha = pr.alpha, beta = pr.beta;
  __attribute__((address_space(1))) double* __restrict__ Cg = (__attribute__((address_space(1))) double*)pr.C;
  int64_t idx[kReduceUnroll];
  int src[kReduceUnroll];
  bool live[kReduceUnroll];
#pragma unroll
  for (int u = 0; u < kReduceUnroll; ++u) {
    const int e = e0 + u * kReduceThreads, m = e / cols, n = e - m * cols;
    live[u] = e < rows * cols;
    src[u] = live[u] ? m * P.tile_n + n : 0;
    idx[u] = live[u] ? blk.c_off + pr.pool[blk.c_tabM + it.m0 + m] + pr.pool[blk.c_tabN + it.n0 + n] : 0;
  }
  double s[kReduceUnroll], old[kReduceUnroll];
#pragma unroll
  for (int u = 0; u < kReduceUnroll; ++u) {
    old[u] = (beta != 0.0 && live[u]) ? Cg[idx[u]] : 0.0;
    s[u] = 0.0;
  }
#pragma unroll 4
  for (int k = 0; k < nsplit; ++k) {  // split order; the elements' loads of one split together
#pragma unroll
    for (int u = 0; u < kReduceUnroll; ++u) s[u] += part[(int64_t)k * tile + src[u]];
  }
#pragma unroll
  for (int u = 0; u < kReduceUnroll; ++u) {
    const double v = alpha * s[u];
    if (live[u]) Cg[idx[u]] = (beta == 0.0) ? v : beta * old[u] + v;
  }
}

hipError_t launch_reduce(const ReduceParams& p, hipStream_t s) {
  if (p.n_items <= 0) return hipSuccess;
  const int per = kReduceUnroll * kReduceThreads, parts = (p.tile_m * p.tile_n + per - 1) / per;
  hipLaunchKernelGGL(k_reduce, dim3(p.n_items, parts), dim3(kReduceThreads), 0, s, p);
  return hipGetLastError();
}
#endif  // TAMM_F64_PART == 0

// ---------------------------------------------------------------------------------------------
// Configurations and dispatch.  X(kernel, MT, NT, KT, WGM, WGN, OCC, RES, TF): OCC is the minimum number
// of waves per SIMD the register allocation must allow (1 = no constraint), RES the workgroups that
// then fit on a compute unit, TF the TFLOP/s measured on large blocks (dense 4D, extents of 128 in
// tiles of 32).  This file is compiled once for part 0 (everything but these kernels) and once for
// every other part, a few kernels each.
// ---------------------------------------------------------------------------------------------
#define TAMM_F64_KERNELS_1(X) X(m128n128k16, 128, 128, 16, 2, 2, 2, 2, 70.0)
#define TAMM_F64_KERNELS_2(X) X(m128n64k16, 128, 64, 16, 2, 2, 1, 2, 63.0)
#define TAMM_F64_KERNELS_3(X) X(m64n128k16, 64, 128, 16, 2, 2, 1, 2, 62.0)
#define TAMM_F64_KERNELS_4(X)          \
  X(m64n64k16, 64, 64, 16, 2, 2, 1, 4, 57.0)    \
  X(m32n64k16, 32, 64, 16, 2, 2, 1, 5, 47.0)    \
  X(m32n32k16, 32, 32, 16, 1, 1, 1, 8, 46.0)
#define TAMM_F64_KERNELS_5(X)          \
  X(m64n80k32, 64, 80, 32, 4, 1, 1, 2, 56.5)    \
  X(m64n64k32, 64, 64, 32, 2, 2, 1, 2, 57.0)
#define TAMM_F64_KERNELS(X) \
  TAMM_F64_KERNELS_1(X) TAMM_F64_KERNELS_2(X) TAMM_F64_KERNELS_3(X) TAMM_F64_KERNELS_4(X) TAMM_F64_KERNELS_5(X)

#define TAMM_F64_DECLARE(k, mt, nt, kt, wgm, wgn, occ, res, tf)                                           \
  hipError_t f64_launch_##k(int layout, const ContractParams& p, int grid, hipStream_t s);       \
  int f64_resident_##k(int layout);
TAMM_F64_KERNELS(TAMM_F64_DECLARE)
#undef TAMM_F64_DECLARE

#if TAMM_F64_PART > 0
// Gather layout index: bit 1 = A k-contiguous, bit 0 = B k-contiguous, bit 2 = 16-byte gathers.
// A tile whose chunks do not split into pairs runs the 8-byte gather for bit 2 as well.
template <int MT, int NT, int KT, int WGM, int WGN, int OCC, int LAYOUT>
static constexpr auto contract_kernel() {
  return k_contract_f64<MT, NT, KT, WGM, WGN, OCC, (LAYOUT & 2) != 0, (LAYOUT & 1) != 0, (LAYOUT & 4) != 0 ? 2 : 1>;
}

template <int MT, int NT, int KT, int WGM, int WGN, int OCC>
static auto contract_kernel_for(int layout) {
  using K = decltype(contract_kernel<MT, NT, KT, WGM, WGN, OCC, 0>());
  static const K table[8] = {contract_kernel<MT, NT, KT, WGM, WGN, OCC, 0>(), contract_kernel<MT, NT, KT, WGM, WGN, OCC, 1>(),
                             contract_kernel<MT, NT, KT, WGM, WGN, OCC, 2>(), contract_kernel<MT, NT, KT, WGM, WGN, OCC, 3>(),
                             contract_kernel<MT, NT, KT, WGM, WGN, OCC, 4>(), contract_kernel<MT, NT, KT, WGM, WGN, OCC, 5>(),
                             contract_kernel<MT, NT, KT, WGM, WGN, OCC, 6>(), contract_kernel<MT, NT, KT, WGM, WGN, OCC, 7>()};
  return table[layout & 7];
}

#define TAMM_F64_DEFINE(k, mt, nt, kt, wgm, wgn, occ, res, tf)                                                               \
  hipError_t f64_launch_##k(int layout, const ContractParams& p, int grid, hipStream_t s) {                         \
    const auto kernel = contract_kernel_for<mt, nt, kt, wgm, wgn, occ>(layout);                                     \
    hipLaunchKernelGGL(kernel, dim3(grid > 0 ? grid : p.n_work), dim3(64 * wgm * wgn), 0, s, p);                    \
    return hipGetLastError();                                                                                       \
  }                                                                                                                 \
  int f64_resident_##k(int layout) {                                                                                \
    int n = 0;                                                                                                      \
    const auto kernel = contract_kernel_for<mt, nt, kt, wgm, wgn, occ>(layout);                                     \
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, 64 * wgm * wgn, 0);               \
    return e == hipSuccess && n > 0 ? n : 1;                                                                        \
  }
#define TAMM_F64_PART_KERNELS_(n) TAMM_F64_KERNELS_##n
#define TAMM_F64_PART_KERNELS(n) TAMM_F64_PART_KERNELS_(n)
TAMM_F64_PART_KERNELS(TAMM_F64_PART)(TAMM_F64_DEFINE)
#endif  // TAMM_F64_PART > 0

#if TAMM_F64_PART == 0
struct F64Kernel {
  F64Config cfg;
  hipError_t (*launch)(int layout, const ContractParams& p, int grid, hipStream_t s);
  int (*resident)(int layout);
};
#define TAMM_F64_ENTRY(k, mt, nt, kt, wgm, wgn, occ, res, tf)                                                       \
  static const F64Kernel kF64_##k = {{mt, nt, kt, wgm, wgn, occ, res, tf, "f64_" #k "_w" #wgm "x" #wgn "_o" #occ}, \
                                     f64_launch_##k, f64_resident_##k};
TAMM_F64_KERNELS(TAMM_F64_ENTRY)
#undef TAMM_F64_ENTRY

// Configuration ids, as tuning files hold them; their number is fixed.  Ids whose own tile shape became a
// size of another kernel's tiles (80 and 256 wide, 128 x 128 at one wave per SIMD or in chunks of 32) name
// the kernel that runs them; 9, once 256 x 32 for outputs of few columns, names the 32 x 32 kernel.
static const F64Kernel* const kF64Configs[] = {
    &kF64_m64n64k16,   &kF64_m128n64k16, &kF64_m64n128k16, &kF64_m128n128k16, &kF64_m32n64k16,
    &kF64_m128n64k16,  &kF64_m64n128k16, &kF64_m64n64k16,  &kF64_m64n128k16,  &kF64_m32n32k16,
    &kF64_m128n128k16, &kF64_m128n64k16, &kF64_m64n80k32,  &kF64_m64n64k32,   &kF64_m128n128k16};

int f64_config_count() { return (int)(sizeof(kF64Configs) / sizeof(kF64Configs[0])); }
const F64Config& f64_config(int id) { return kF64Configs[id]->cfg; }
int f64_config_canonical(int id) {
  int c = 0;
  while (kF64Configs[c] != kF64Configs[id]) ++c;
  return c;
}

int f64_occupancy(int config, int layout) { return kF64Configs[config]->resident(layout); }

hipError_t launch_contract_f64(int config, int layout, const ContractParams& p, int grid, hipStream_t s) {
  if (p.n_work <= 0) return hipSuccess;
  if (config < 0 || config >= f64_config_count()) return hipErrorInvalidValue;
  return kF64Configs[config]->launch(layout, p, grid, s);
}

// ---------------------------------------------------------------------------------------------
// Orbital-energy denominator update.  Each workgroup handles `chunk` consecutive elements of one
// stored block; IEEE float64 division; the denominator is summed in the documented order (the
// energies of the +1 dimensions in dimension order, then minus those of the -1 dimensions).
// A thread splits its first element into per-dimension indices once and then steps by the
// workgroup size with a mixed-radix add, so no integer division runs per element.  Elements go in
// batches of kDenomUnroll per thread whose loads are all issued before any division, so each wave
// keeps that many coalesced loads in flight.
// ---------------------------------------------------------------------------------------------
constexpr int kDenomUnroll = 4;

template <int RANK>
__device__ __forceinline__ void denominator_block(const DenomParams& P, int b, int e0, int e1) {
  int lo[RANK], ext[RANK], idx[RANK], step[RANK];
#pragma unroll
  for (int d = 0; d < RANK; ++d) {
    const int t = P.block_tiles[(int64_t)b * RANK + d];
    lo[d] = (int)P.tile_offset[P.dim_tile_base[d] + t];
    ext[d] = (int)P.tile_size[P.dim_tile_base[d] + t];
  }
  int rem = e0 + (int)threadIdx.x, srem = (int)blockDim.x;
#pragma unroll
  for (int d = RANK - 1; d >= 0; --d) {
    idx[d] = rem % ext[d];
    rem /= ext[d];
    step[d] = srem % ext[d];
    srem /= ext[d];
  }
  const double* __restrict__ in = P.in + P.block_off[b];
  double* __restrict__ out = P.out + P.block_off[b];
  for (int e = e0 + (int)threadIdx.x; e < e1; e += kDenomUnroll * (int)blockDim.x) {
    // all loads of the batch first (the element and its energies), then the arithmetic: no
    // load waits behind another's use
    double x[kDenomUnroll], ev[kDenomUnroll][RANK];
#pragma unroll
    for (int u = 0; u < kDenomUnroll; ++u) {
      const int eu = e + u * (int)blockDim.x;
      x[u] = eu < e1 ? in[eu] : 1.0;
#pragma unroll
      for (int d = 0; d < RANK; ++d) ev[u][d] = P.sign[d] != 0 ? P.energy[d][lo[d] + idx[d]] : 0.0;
      int carry = 0;  // idx += step in the block's mixed radix (each digit stays below 2*ext)
#pragma unroll
      for (int d = RANK - 1; d >= 0; --d) {
        idx[d] += step[d] + carry;
        carry = idx[d] >= ext[d] ? 1 : 0;
        idx[d] -= carry ? ext[d] : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < kDenomUnroll; ++u) {
      double den = 0.0;  // 0 + v and 0 - v are exact: the first term enters unchanged
#pragma unroll
      for (int d = 0; d < RANK; ++d)
        if (P.sign[d] > 0) den += ev[u][d];
#pragma unroll
      for (int d = 0; d < RANK; ++d)
        if (P.sign[d] < 0) den -= ev[u][d];
      const int eu = e + u * (int)blockDim.x;
      if (eu < e1) out[eu] = x[u] / den;
    }
  }
}

template <int RANK>
__global__ __launch_bounds__(256) void k_denominator(DenomParams P) {
  const int64_t it = blockIdx.x;
  if (it >= P.n_items) return;
  const int b = P.item_block[it];
  int n = 1;
#pragma unroll
  for (int d = 0; d < RANK; ++d) n *= (int)P.tile_size[P.dim_tile_base[d] + P.block_tiles[(int64_t)b * RANK + d]];
  const int e0 = P.item_start[it];
  denominator_block<RANK>(P, b, e0, min(n, e0 + P.chunk));
}

hipError_t launch_denominator(const DenomParams& p, hipStream_t s) {
  if (p.n_items <= 0) return hipSuccess;
  const dim3 g((unsigned)p.n_items), blk(256);
  switch (p.rank) {
    case 1: hipLaunchKernelGGL(k_denominator<1>, g, blk, 0, s, p); break;
    case 2: hipLaunchKernelGGL(k_denominator<2>, g, blk, 0, s, p); break;
    case 3: hipLaunchKernelGGL(k_denominator<3>, g, blk, 0, s, p); break;
    case 4: hipLaunchKernelGGL(k_denominator<4>, g, blk, 0, s, p); break;
    case 5: hipLaunchKernelGGL(k_denominator<5>, g, blk, 0, s, p); break;
    case 6: hipLaunchKernelGGL(k_denominator<6>, g, blk, 0, s, p); break;
    case 7: hipLaunchKernelGGL(k_denominator<7>, g, blk, 0, s, p); break;
    case 8: hipLaunchKernelGGL(k_denominator<8>, g, blk, 0, s, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#endif  // TAMM_F64_PART == 0

}  // namespace tamm
