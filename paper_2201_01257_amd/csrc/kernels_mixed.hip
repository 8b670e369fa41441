// Mixed-precision contraction kernels for gfx950: the bulk products run on float32 or bfloat16
// matrix cores with float32 accumulation inside K windows of 256, and every window's partial
// sums are promoted into float64 accumulators; the epilogue (beta*C + alpha*acc) is float64.
//
//   float32 (v_mfma_f32_16x16x4_f32): operands rounded to float32 (round to nearest even) while
//       they are gathered into LDS.
//   split bfloat16 (v_mfma_f32_16x16x32_bf16): each operand is first split by k_prep_split into
//       bfloat16 slices, stored either as slice planes (plane s holds slice s of every element,
//       each block [row][k]; used when every block's K extent is a multiple of 8) or as one packed
//       64-bit word per element (slice s in bits 16s..16s+15) at the float64 element offsets; the
//       contraction then multiplies selected slice pairs.
//         - three plain slices (x ~ b0 + b1 + b2, b_i = bf16(x - b_0 - ... - b_{i-1})), the six
//           products b_i*b_j with i + j <= 2; b0*b0 in one float32 accumulator per window, the
//           five smaller products in another;
//         - aligned lead: slice 0 is x rounded to a fixed-point grid of 8 bits below the maximum
//           exponent of its (row, window) -- an integer of magnitude <= 256 times a power of two,
//           exact in bfloat16 -- and slices 1..3 are bfloat16 slices of the residual; the ten
//           products of slice order i + j <= 3.  Within one 256-long window every lead*lead
//           product is an integer of at most 16 bits times the same power of two for a given
//           (m, n), so their sum (at most 2^24 in magnitude) is exact in float32; it is kept in
//           its own accumulator, and only the small residual products see float32 rounding.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "internal.h"
#include "mixed.h"

namespace tamm {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------------
// operand split
// ---------------------------------------------------------------------------------------------
// Round to nearest even at 8 significant bits (the bfloat16 precision), on the float64 bit pattern:
// adding half a unit of the kept part (less one ulp when the kept part is even) and clearing the
// 45 dropped mantissa bits rounds to nearest even; a carry out of the mantissa steps the exponent,
// which is the correctly rounded result.  Magnitudes below 2^-100 are flushed to zero (far below
// anything the slices can carry).  Finite inputs only.
__device__ __forceinline__ double round_bf16(double x) {
  uint64_t u = __builtin_bit_cast(uint64_t, x);
  if (((u >> 52) & 0x7FF) < 1023 - 100) return 0.0;
  u += 0x00000FFFFFFFFFFFull + ((u >> 45) & 1u);
  u &= ~0x00001FFFFFFFFFFFull;
  return __builtin_bit_cast(double, u);
}

// Bits of a value that is exactly representable in bfloat16.
__device__ __forceinline__ uint64_t bf16_bits(double y) {
  const float f = (float)y;  // exact: y has at most 8 significant bits and a float exponent
  return (uint64_t)(__float_as_uint(f) >> 16);
}

__device__ __forceinline__ uint64_t split_plain(double x) {
  const double b0 = round_bf16(x);
  const double r1 = x - b0;
  const double b1 = round_bf16(r1);
  const double b2 = round_bf16(r1 - b1);
  return bf16_bits(b0) | (bf16_bits(b1) << 16) | (bf16_bits(b2) << 32);
}

// 2^p for -1022 <= p <= 1023
__device__ __forceinline__ double pow2(int p) { return __builtin_bit_cast(double, (uint64_t)(p + 1023) << 52); }

// Grid of a (row, window) with maximum magnitude mx: the exponent e with 2^(e-1) <= mx < 2^e
// (taken as -1000 for smaller maxima, whose slices are all zero in bfloat16 anyway); the lead
// slice is x rounded to multiples of 2^(e-8).
__device__ __forceinline__ int window_exponent(double mx) {
  const int bexp = (int)((__builtin_bit_cast(uint64_t, mx) >> 52) & 0x7FF);
  return max(bexp - 1022, -1000);
}

__device__ __forceinline__ uint64_t split_aligned(double x, int e) {
  const double lead = rint(x * pow2(8 - e)) * pow2(e - 8);  // an integer of magnitude <= 256 times 2^(e-8)
  const double r = x - lead;                                // exact
  const double s1 = round_bf16(r);
  const double r2 = r - s1;
  const double s2 = round_bf16(r2);
  const double s3 = round_bf16(r2 - s2);
  return bf16_bits(lead) | (bf16_bits(s1) << 16) | (bf16_bits(s2) << 32) | (bf16_bits(s3) << 48);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Block of a wave's item (the same for the whole wave), through scalar loads: the search is a chain
// of dependent ones.
__device__ __forceinline__ int find_block(const PrepBlock* blocks, int n, int64_t item) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sload(&blocks[mid].item0) <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Lanes along k (the operand's stride-1 label is summed): a wave converts kPrepUnroll consecutive
// (block, row, window) items, the maximum of a window is a wave reduction.  Planes layout: 4
// consecutive k of one row per lane and item; packed: k = lane + 64 j.  The loads of all its items
// are issued before any of them is converted, so each wave keeps that many windows of reads in flight
// (one in the packed layout, whose K extents are mostly far below a window: four rows of a dozen
// elements after one another only made the chain of descriptor loads longer, 23 -> 30 us for the
// T1 occupied term at O=13, V=102).
template <bool PLANES>
constexpr int kPrepUnroll = PLANES ? 4 : 1;

template <bool PLANES>
__device__ __forceinline__ void prep_k_along_lanes(const PrepParams& P, int64_t first, int lane) {
  static_assert(kSplitWindow == 4 * 64, "a wave converts one window, 4 k per lane");
  typedef double d2_t __attribute__((ext_vector_type(2)));
  constexpr int U = kPrepUnroll<PLANES>;
  if (first >= P.n_items) return;
  const int32_t* __restrict__ pool = P.pool;
  double x[U][4];
  int64_t pos[U];   // planes: element of the first k; packed: the row
  int32_t t[U][4];  // table entries
  int nk[U];        // k of this lane in the window (planes: 0 or 4)
  int b = find_block(P.blocks, P.n_blocks, first);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t item = first + u;
    nk[u] = 0;
    pos[u] = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[u][i] = 0.0;
    if (item >= P.n_items) continue;  // wave-uniform
    while (b + 1 < P.n_blocks && sload(&P.blocks[b + 1].item0) <= item) ++b;
    const PrepBlock pb = sload(P.blocks + b);
    const int64_t local = item - pb.item0;
    const int k0 = (int)(local % pb.nwin) * kSplitWindow, row = (int)(local / pb.nwin);
    const int k1 = min(pb.kext, k0 + kSplitWindow);
    const int64_t rowoff = pb.off + sload(pool + pb.tab_row + row);
    if constexpr (PLANES) {
      const int k = k0 + 4 * lane;
      pos[u] = pb.off + (int64_t)row * pb.kext + k;
      if (k >= k1) continue;  // k1 is a multiple of 8: all four k are inside or all outside
      nk[u] = 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) t[u][i] = pool[pb.tab_k + k + i];
      const int64_t a = rowoff + t[u][0];
      if (t[u][1] == t[u][0] + 1 && t[u][2] == t[u][0] + 2 && t[u][3] == t[u][0] + 3 && (a & 1) == 0) {
        // four consecutive elements at a 16-byte boundary: two 16-byte loads
        const d2_t lo = *reinterpret_cast<const d2_t*>(P.x + a), hi = *reinterpret_cast<const d2_t*>(P.x + a + 2);
        x[u][0] = lo[0];
        x[u][1] = lo[1];
        x[u][2] = hi[0];
        x[u][3] = hi[1];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[u][i] = P.x[rowoff + t[u][i]];
      }
    } else {
      pos[u] = rowoff;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k0 + lane + 64 * i < k1) {
          nk[u] = i + 1;
          t[u][i] = pool[pb.tab_k + k0 + lane + 64 * i];
          x[u][i] = P.x[rowoff + t[u][i]];
        }
    }
  }
  const int ns = P.aligned ? 4 : 3;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (first + u >= P.n_items) break;  // wave-uniform
    double mx = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) mx = fmax(mx, fabs(x[u][i]));
    const int e = window_exponent(wave_max(mx));
    if (nk[u] == 0) continue;
    uint64_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = P.aligned ? split_aligned(x[u][i], e) : split_plain(x[u][i]);
    if constexpr (PLANES) {
      for (int sl = 0; sl < ns; ++sl) {
        uint64_t v = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) v |= ((w[i] >> (16 * sl)) & 0xFFFFull) << (16 * i);
        *reinterpret_cast<uint64_t*>(static_cast<unsigned short*>(P.out) + sl * P.plane_stride + pos[u]) = v;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < nk[u]) static_cast<uint64_t*>(P.out)[pos[u] + t[u][i]] = w[i];
    }
  }
}

// Lanes along the rows (the operand's stride-1 label is not summed): a workgroup converts one (block,
// 64 rows, window) item, its four waves a quarter of the window each.  A lane holds its row's 64
// elements in registers: all of them are in flight at once and read once.  (One wave walking the
// window, twice for the maximum, took 2.0 ms for the 157 million doubles of the amplitudes at O=64,
// V=320, where this takes 1.3, and most of the time of a small contraction: three-slice ladder at
// O=12, V=67 in tiles of 11, 192 -> 122 us in all.)
template <bool PLANES>
__device__ __forceinline__ void prep_rows_along_lanes(const PrepParams& P, double (&maxima)[4][64]) {
  constexpr int KW = kSplitWindow / 4;  // k per wave
  const int lane = threadIdx.x & 63, wave = wave_uniform((int)threadIdx.x >> 6);
  const int64_t item = blockIdx.x + (int64_t)blockIdx.y * gridDim.x;
  if (item >= P.n_items) return;
  const PrepBlock pb = sload(P.blocks + find_block(P.blocks, P.n_blocks, item));
  const int64_t local = item - pb.item0;
  const int k0 = (int)(local % pb.nwin) * kSplitWindow + wave * KW;  // this wave's first k
  const int n = min(KW, min(pb.kext, k0 - wave * KW + kSplitWindow) - k0);  // and how many
  const int row = (int)(local / pb.nwin) * 64 + lane;
  const int32_t* __restrict__ pool = P.pool;
  const int64_t rowoff = pb.off + pool[pb.tab_row + min(row, pb.rows - 1)];
  const int32_t* __restrict__ tab = pool + pb.tab_k + k0;
  double x[KW];
#pragma unroll
  for (int i = 0; i < KW; ++i) x[i] = 0.0;
  if (n == KW) {
#pragma unroll
    for (int i = 0; i < KW; ++i) x[i] = P.x[rowoff + sload(tab + i)];
  } else {
#pragma unroll
    for (int g = 0; g < KW / 8; ++g) {
      if (8 * g >= n) continue;  // wave-uniform
#pragma unroll
      for (int i = 8 * g; i < 8 * g + 8; ++i) x[i] = P.x[rowoff + sload(tab + min(i, n - 1))];  // past the end: the last again
    }
  }
  int e = 0;
  if (P.aligned) {
    double mx = 0.0;
#pragma unroll
    for (int i = 0; i < KW; ++i) mx = fmax(mx, fabs(x[i]));
    maxima[wave][lane] = mx;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) mx = fmax(mx, maxima[q][lane]);
    e = window_exponent(mx);
  }
  if (row >= pb.rows) return;
  const int ns = P.aligned ? 4 : 3;
#pragma unroll
  for (int g = 0; g < KW / 8; ++g) {
    if (8 * g >= n) continue;  // wave-uniform
    uint64_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = P.aligned ? split_aligned(x[8 * g + i], e) : split_plain(x[8 * g + i]);
    if constexpr (PLANES) {  // every K extent is a multiple of 8
      const int64_t pos = pb.off + (int64_t)row * pb.kext + k0 + 8 * g;
      for (int sl = 0; sl < ns; ++sl) {
        u4_t v;
#pragma unroll
        for (int h = 0; h < 4; ++h)
          v[h] = (uint32_t)((w[2 * h] >> (16 * sl)) & 0xFFFFu) | ((uint32_t)((w[2 * h + 1] >> (16 * sl)) & 0xFFFFu) << 16);
        *reinterpret_cast<u4_t*>(static_cast<unsigned short*>(P.out) + sl * P.plane_stride + pos) = v;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (8 * g + i < n) static_cast<uint64_t*>(P.out)[rowoff + sload(tab + 8 * g + i)] = w[i];
    }
  }
}

template <bool ROWS_ALONG_LANES, bool PLANES>
__global__ __launch_bounds__(256) void k_prep_split(PrepParams P) {
  if constexpr (ROWS_ALONG_LANES) {
    __shared__ double maxima[4][64];
    prep_rows_along_lanes<PLANES>(P, maxima);
  } else {
    const int wave = wave_uniform((int)threadIdx.x >> 6);
    prep_k_along_lanes<PLANES>(P, ((int64_t)blockIdx.x * 4 + wave) * kPrepUnroll<PLANES>, threadIdx.x & 63);
  }
}

hipError_t launch_prep_split(const PrepParams& p, bool rows_along_lanes, hipStream_t s) {
  if (p.n_items <= 0) return hipSuccess;
  const int64_t per_block = rows_along_lanes ? 1 : 4 * (p.planes ? kPrepUnroll<true> : kPrepUnroll<false>);  // items per workgroup
  // a grid dimension holds fewer than 2^32 threads: long item lists take two
  const int64_t blocks = (p.n_items + per_block - 1) / per_block, wide = rows_along_lanes ? std::min<int64_t>(blocks, 1 << 20) : blocks;
  const dim3 g((unsigned)wide, (unsigned)((blocks + wide - 1) / wide)), b(256);
  if (rows_along_lanes && p.planes) hipLaunchKernelGGL((k_prep_split<true, true>), g, b, 0, s, p);
  else if (rows_along_lanes) hipLaunchKernelGGL((k_prep_split<true, false>), g, b, 0, s, p);
  else if (p.planes) hipLaunchKernelGGL((k_prep_split<false, true>), g, b, 0, s, p);
  else hipLaunchKernelGGL((k_prep_split<false, false>), g, b, 0, s, p);
  return hipGetLastError();
}

// Epilogue shared by the mixed kernels: float64 accumulators in the float32 MFMA layout (D[m][n]
// in lane n + 16*(m/4), register m%4).
template <int MT, int NT, int WM, int WN, int FM, int FN>
__device__ __forceinline__ void epilogue_f32layout(const ProblemDesc& pr, const WorkItem& w, const OutBlockDesc& blk,
                                                   d4_t (&acc)[FM][FN], int wm, int wn, int lr, int lq) {
  if (shape_nsplit(w.shape) > 1) {
    double* part = pr.partial + ((int64_t)w.tile + shape_split(w.shape)) * (MT * NT);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(wm * WM + i * 16 + 4 * lq + r) * NT + wn * WN + j * 16 + lr] = acc[i][j][r];
    return;
  }
  // through out's offset tables: every table entry first (the tables are padded, so rows and
  // columns past the block read in bounds), then per row block the old values (beta != 0), then
  // the results, so that no load waits behind the use of another
  const double alpha = pr.alpha, beta = pr.beta;
  const int32_t* pool = pr.pool;
  __attribute__((address_space(1))) double* __restrict__ Cg = (__attribute__((address_space(1))) double*)pr.C;
  const int mb = w.m0 + wm * WM + 4 * lq, nb = w.n0 + wn * WN + lr;
  int32_t rt[FM][4], ct[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) rt[i][r] = pool[blk.c_tabM + mb + i * 16 + r];
#pragma unroll
  for (int j = 0; j < FN; ++j) ct[j] = pool[blk.c_tabN + nb + j * 16];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    double old[4][FN];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const bool live = mb + i * 16 + r < blk.mext && nb + j * 16 < blk.next;
        old[r][j] = (beta != 0.0 && live) ? Cg[blk.c_off + rt[i][r] + ct[j]] : 0.0;
      }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const bool live = mb + i * 16 + r < blk.mext && nb + j * 16 < blk.next;
        const double v = alpha * acc[i][j][r];
        if (live) Cg[blk.c_off + rt[i][r] + ct[j]] = (beta == 0.0) ? v : beta * old[r][j] + v;
      }
  }
}

// ---------------------------------------------------------------------------------------------
// float32 products (v_mfma_f32_16x16x4_f32), float32 window sums promoted to float64.
//
// Bound by the products on large blocks: float32 MFMAs take half the time of float64 ones on the
// same float64 traffic, so what a wave issues beside them weighs double.  LDS holds a row's chunk by
// lane quarter (slot), so that one 16-byte read gives a lane its operands of all four k-steps; the
// stores and loads of the staged chunk go between the products of the first k-steps, and the barrier
// comes before the last one's, under which the next chunk's operands are read.  Ladder at O=32,
// V=160, tiles of 32: 2.52 -> 2.12 ms (99 TFLOP/s; this card's library product of 8192 x 8192
// matrices reaches 153) on 128 x 128 with eight waves, 2.64 -> 2.35 on 128 x 64.
// ---------------------------------------------------------------------------------------------
template <int MT, int NT, int KT, int WGM, int WGN, bool A_KC, bool B_KC>
__global__ __launch_bounds__(64 * WGM * WGN, MT * NT <= 64 * 64 ? 4 : WGM * WGN / 4) void k_contract_f32(ContractParams P) {
  constexpr int NTHR = 64 * WGM * WGN;
  constexpr int WM = MT / WGM, WN = NT / WGN, FM = WM / 16, FN = WN / 16;
  constexpr int NS = KT / 4;  // MFMA k-steps per chunk
  constexpr int LD = KT + 4;  // floats: 16 rows' 16-byte operands start on distinct bank quadruples
  static_assert(kSplitWindow % KT == 0, "chunks tile the promotion window");
  static_assert(NS == 4, "a lane's operands of a chunk in one 16-byte read");
  // LDS position of k within a row: lane quarter k % 4 reads its operands of all k-steps at once
  auto slot = [](int k) { return k % 4 * NS + k / 4; };
  using G = Gather<MT, NT, KT, NTHR, A_KC, B_KC, double>;
  __shared__ __attribute__((aligned(16))) float As[2][MT * LD];
  __shared__ __attribute__((aligned(16))) float Bs[2][NT * LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM, lr = lane & 15, lq = lane >> 4;
  const int a_frag = (wm * WM + lr) * LD + lq * NS, b_frag = (wn * WN + lr) * LD + lq * NS;
  const int item = blockIdx.x;
  if (item >= P.n_work) return;
  const WorkItem w = wave_uniform(sload(P.work + item));
  const ProblemDesc pr = wave_uniform(P.probs ? sload(P.probs + w.prob) : P.single);
  const OutBlockDesc blk = wave_uniform(sload(pr.blocks + w.ob));
  const int32_t* __restrict__ pool = pr.pool;
  const PairDesc* __restrict__ pairs = pr.pairs + blk.pair_base;
  const int cnt = wave_uniform(gload(pr.counts + w.ob));
  const int nsplit = shape_nsplit(w.shape), split = shape_split(w.shape);
  const int pb = (int)(((int64_t)cnt * split) / nsplit), pe = (int)(((int64_t)cnt * (split + 1)) / nsplit);
  G g;
  g.init(tid);
  d4_t acc[FM][FN];
  f4_t part[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      acc[i][j] = (d4_t){0.0, 0.0, 0.0, 0.0};
      part[i][j] = (f4_t){0.f, 0.f, 0.f, 0.f};
    }
  if (pb < pe) {
    constexpr int NF = FM * FN, NR = FM + FN, AL = G::MA::L, NL = AL + G::MB::L;
    constexpr int NX = NF * NS, NP = NF * (NS - 1);  // products of a chunk, of all its k-steps but the last
    // A chunk's operands, k-step s in component s: A fragments, then B fragments.  Two sets, so that
    // the next chunk's are read under the last products of this one; one on 64 x 64 tiles, where 32
    // registers less let four workgroups share a compute unit, whose products cover each other's reads.
    constexpr int SETS = NF <= 4 ? 1 : 2;
    f4_t op[SETS][NR];
    auto fetch = [&](int b, auto set, auto r) {
      if constexpr (r() < FM) op[set() % SETS][r()] = *reinterpret_cast<const f4_t*>(&As[b][a_frag + r() * 16 * LD]);
      else op[set() % SETS][r()] = *reinterpret_cast<const f4_t*>(&Bs[b][b_frag + (r() - FM) * 16 * LD]);
    };
    auto restage = [&](int b, auto y) {  // staged load y (A's, then B's): to LDS, and from memory again
      constexpr int e = y() < AL ? y() : y() - AL;
      if constexpr (y() < AL) As[b][g.a_lds_row(e) * LD + slot(g.a_lds_k(e))] = (float)g.ra[e];
      else Bs[b][g.b_lds_row(e) * LD + slot(g.b_lds_k(e))] = (float)g.rb[e];
      g.load_one(y());
    };
    ChunkWalk<KT, G, double> walk(g, pairs, pb, pe, pool, pr.A, pr.B, w, blk.mext, blk.next);
    uint32_t flushes = 0;  // of the chunks fetched and not yet multiplied, the oldest in bit 0
    int ahead = 0;
    auto note = [&]() {
      const int kend = walk.k + KT;
      flushes |= (kend >= walk.d.kext || kend % kSplitWindow == 0 ? 1u : 0u) << ahead;
      ++ahead;
    };
    auto next_chunk = [&]() {
      const bool more = walk.next_tables();
      if (more) note();
      return more;
    };
    walk.setup();
    g.load_tables(walk.d, pool, 0);
    note();
    g.load_data();
    bool inflight = next_chunk();  // the chunk staged during this one is real
    static_for<NL>([&](auto y) { restage(0, y); });
    bool tabs = inflight && next_chunk();  // so is the one after it
    __syncthreads();
    static_for<NR>([&](auto r) { fetch(0, int_c<0>{}, r); });
    // one chunk, its operands in set SET; false after the last one
    auto chunk = [&](auto set) {
      constexpr int SET = set();
      const bool flush = (flushes & 1u) != 0;
      flushes >>= 1;
      --ahead;
      __builtin_amdgcn_s_setprio(1);  // MFMA phase first when waves of two workgroups compete
      static_for<NX>([&](auto x) {  // zeros beyond a ragged chunk's K extent
        constexpr int st = x() / NF, i = x() % NF / FN, j = x() % FN;
        if constexpr (x() == NP) __syncthreads();
        part[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(op[SET % SETS][i][st], op[SET % SETS][FM + j][st], part[i][j], 0, 0, 0);
        if constexpr (x() < NP) {
          constexpr int y0 = min_c(x() * NL * 4 / (NP * 3), NL), y1 = min_c((x() + 1) * NL * 4 / (NP * 3), NL);
          static_for<y1 - y0>([&](auto y) { restage(SET ^ 1, int_c<y0 + y()>{}); });
        } else if constexpr (SETS == 2) {
          constexpr int r0 = (x() - NP) * NR / NF, r1 = (x() - NP + 1) * NR / NF;
          static_for<r1 - r0>([&](auto r) { fetch(SET ^ 1, int_c<SET ^ 1>{}, int_c<r0 + r()>{}); });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_s_setprio(0);
      if constexpr (SETS == 1) static_for<NR>([&](auto r) { fetch(SET ^ 1, set, r); });
      const bool tabs_next = tabs && next_chunk();
      if (flush) {  // end of a promotion window or of a pair: float32 sums into float64
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              acc[i][j][r] += (double)part[i][j][r];
              part[i][j][r] = 0.f;
            }
      }
      const bool more = inflight;
      inflight = tabs;
      tabs = tabs_next;
      return more;
    };
    while (chunk(int_c<0>{}) && chunk(int_c<1>{})) {}
  }
  epilogue_f32layout<MT, NT, WM, WN, FM, FN>(pr, w, blk, acc, wm, wn, lr, lq);
}

// ---------------------------------------------------------------------------------------------
// Gather of split operands in the planes layout: plane s holds bfloat16 slice s of every element,
// each block as [row][k] (flattened M or N rows, flattened K, k fastest) at the block's element
// offset.  A lane moves 8 consecutive k of one row and plane with one 16-byte load and one
// 16-byte LDS store.  The planner uses this layout only when every operand block's K extent is a
// multiple of 8, so a group of 8 is either inside the block or wholly past its K extent; groups
// past the rows or the K extent read zeros (offset beyond the buffer resource).
// Same interface as Gather, for ChunkWalk.
// ---------------------------------------------------------------------------------------------
// LDS layout of a chunk in the planes layout: per plane, the 16-byte units (8 k of one row) are
// stored k-group major, unit (k-group q, row r) at q*ROWS + (r ^ 2q).  An MFMA operand read (16
// rows, one k-group per 16 lanes) is then a permutation of one aligned 256-byte block per 16
// lanes, which the LDS serves without bank conflicts; the gather's stores (4 lanes per row, one
// k-group each) put every 8 consecutive lanes on 8 distinct 16-byte bank groups.
template <int ROWS>
__device__ __forceinline__ int lds_unit(int r, int q) { return q * ROWS + (r ^ (2 * q)); }

template <int MT, int NT, int KT, int NTHR, int NS>
struct PlaneGather {
  static constexpr int KG = KT / 8;           // 16-byte groups per row of a chunk
  static constexpr int AJ = (MT * KG + NTHR - 1) / NTHR;  // loads per plane and thread
  static constexpr int BJ = (NT * KG + NTHR - 1) / NTHR;
  static_assert(KT % 8 == 0 && (MT * KG % NTHR == 0 || NTHR % (MT * KG) == 0) &&
                    (NT * KG % NTHR == 0 || NTHR % (NT * KG) == 0), "plane gather mapping");
  // a load slot past the tile (fewer 16-byte groups than threads): whole waves skip it
  __device__ static bool a_live(int p) { return MT * KG % NTHR == 0 || p < MT * KG; }
  __device__ static bool b_live(int p) { return NT * KG % NTHR == 0 || p < NT * KG; }
  static constexpr uint32_t kPast = 0x80000000u;  // byte offset beyond every block

  int tid;
  int64_t a_plane, b_plane;
  const __bf16* a_base;
  const __bf16* b_base;
  int m0, n0, mext, next, kext, kbase;
  u4_t ra[NS][AJ], rb[NS][BJ];

  __device__ void init(int t, int64_t ap, int64_t bp) {
    tid = t;
    a_plane = ap;
    b_plane = bp;
  }
  __device__ void setup_pair(const PairDesc& d, const int32_t*, const __bf16* A, const __bf16* B, int m0_, int n0_,
                             int mext_, int next_, int, int) {
    a_base = A + d.a_off;
    b_base = B + d.b_off;
    m0 = m0_;
    n0 = n0_;
    mext = mext_;
    next = next_;
    kext = d.kext;
  }
  __device__ void load_tables(const PairDesc&, const int32_t*, int kb) { kbase = kb; }
  // load y of the chunk: slice y / (AJ + BJ), A's loads before B's
  static constexpr int kLoads = NS * (AJ + BJ);
  __device__ void load_one(int y) {
    const int sl = y / (AJ + BJ), j = y % (AJ + BJ);
    if (j < AJ) {
      const int p = tid + j * NTHR, r = m0 + p / KG, k = kbase + 8 * (p % KG);
      if (!a_live(p)) return;
      const __amdgpu_buffer_rsrc_t ar = block_rsrc(a_base + sl * a_plane, (uint32_t)mext * (uint32_t)kext * 2u);
      const uint32_t off = (r < mext && k < kext) ? (uint32_t)(r * kext + k) * 2u : kPast;
      ra[sl][j] = __builtin_bit_cast(u4_t, __builtin_amdgcn_raw_buffer_load_b128(ar, (int)off, 0, 0));
    } else {
      const int jb = j - AJ, p = tid + jb * NTHR, r = n0 + p / KG, k = kbase + 8 * (p % KG);
      if (!b_live(p)) return;
      const __amdgpu_buffer_rsrc_t br = block_rsrc(b_base + sl * b_plane, (uint32_t)next * (uint32_t)kext * 2u);
      const uint32_t off = (r < next && k < kext) ? (uint32_t)(r * kext + k) * 2u : kPast;
      rb[sl][jb] = __builtin_bit_cast(u4_t, __builtin_amdgcn_raw_buffer_load_b128(br, (int)off, 0, 0));
    }
  }
  __device__ void load_data() {
#pragma unroll
    for (int y = 0; y < kLoads; ++y) load_one(y);
  }
  // LDS position (row, first k) of load j
  __device__ int lds_row(int j) const { return (tid + j * NTHR) / KG; }
  __device__ int lds_k(int j) const { return 8 * ((tid + j * NTHR) % KG); }
};

// ---------------------------------------------------------------------------------------------
// split bfloat16 products (v_mfma_f32_16x16x32_bf16).  LDS holds NS slice planes per operand: in
// the planes layout as 16-byte units placed by lds_unit; in the packed layout as [row][k] bfloat16
// with a row stride of KT+8 elements (an odd number of 16-byte units).
// ---------------------------------------------------------------------------------------------
template <int MT, int NT, int KT, int WGM, int WGN, bool ALIGNED, bool A_KC, bool B_KC, bool PLANES>
__global__ __launch_bounds__(64 * WGM * WGN) void k_contract_bf16s(ContractParams P) {
  constexpr int NTHR = 64 * WGM * WGN;
  constexpr int WM = MT / WGM, WN = NT / WGN, FM = WM / 16, FN = WN / 16;
  constexpr int NS = ALIGNED ? 4 : 3;
  // LDS rows of KT bfloat16.  Packed layout: padded to an odd number of 16-byte units.  Planes
  // layout: a plane of MT (NT) rows x KT holds MT*KT elements, unit (q, r) at lds_unit.
  constexpr int LD = PLANES ? KT : KT + 8;
  static_assert(KT % 32 == 0 && kSplitWindow % KT == 0, "chunks of whole MFMA k-steps tile the window");
  static_assert(PLANES ? KT == 32 : ((LD * 2) / 16) % 2 == 1, "LDS row layout");
  using G = std::conditional_t<PLANES, PlaneGather<MT, NT, KT, NTHR, NS>, Gather<MT, NT, KT, NTHR, A_KC, B_KC, uint64_t>>;
  using E = std::conditional_t<PLANES, __bf16, uint64_t>;  // element type of the split operands
  __shared__ __attribute__((aligned(16))) __bf16 As[2][NS * MT * LD];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[2][NS * NT * LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM, lr = lane & 15, lq = lane >> 4;
  // operand read offsets of this lane (row block i / j, MFMA k-step 0)
  int a_frag[FM], b_frag[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int r = wm * WM + i * 16 + lr;
    a_frag[i] = PLANES ? 8 * lds_unit<MT>(r, lq) : r * LD + 8 * lq;
  }
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int r = wn * WN + j * 16 + lr;
    b_frag[j] = PLANES ? 8 * lds_unit<NT>(r, lq) : r * LD + 8 * lq;
  }
  const int item = blockIdx.x;
  if (item >= P.n_work) return;
  const WorkItem w = wave_uniform(sload(P.work + item));
  const ProblemDesc pr = wave_uniform(P.probs ? sload(P.probs + w.prob) : P.single);
  const OutBlockDesc blk = wave_uniform(sload(pr.blocks + w.ob));
  const int32_t* __restrict__ pool = pr.pool;
  const PairDesc* __restrict__ pairs = pr.pairs + blk.pair_base;
  const E* Ap = reinterpret_cast<const E*>(pr.A);
  const E* Bp = reinterpret_cast<const E*>(pr.B);
  const int cnt = wave_uniform(gload(pr.counts + w.ob));
  const int nsplit = shape_nsplit(w.shape), split = shape_split(w.shape);
  const int pb = (int)(((int64_t)cnt * split) / nsplit), pe = (int)(((int64_t)cnt * (split + 1)) / nsplit);
  G g;
  if constexpr (PLANES) g.init(tid, pr.a_plane, pr.b_plane);
  else g.init(tid);
  d4_t acc[FM][FN];
  f4_t lead[FM][FN], rest[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      acc[i][j] = (d4_t){0.0, 0.0, 0.0, 0.0};
      lead[i][j] = (f4_t){0.f, 0.f, 0.f, 0.f};
      rest[i][j] = (f4_t){0.f, 0.f, 0.f, 0.f};
    }
  auto flush_window = [&]() {  // end of a promotion window or of a pair: float32 sums into float64
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[i][j][r] += (double)lead[i][j][r] + (double)rest[i][j][r];
          lead[i][j][r] = 0.f;
          rest[i][j][r] = 0.f;
        }
  };
  if constexpr (PLANES) {
    if (pb < pe) {
      // products of one output fragment, in order: slice pairs (a, b) of the accumulators; product 0
      // goes to the lead sum, the others to the residual's
      constexpr int NP = ALIGNED ? 10 : 6;
      constexpr int PA[10] = {0, 0, 1, 0, 2, 1, 0, 3, 1, 2}, PB[10] = {0, 1, 0, 2, 0, 1, 3, 0, 2, 1};
      // The operand with more fragments per wave is streamed one fragment at a time (two register
      // sets), the other stays in registers for the chunk: 64 + 32 registers of operands at most.
      constexpr bool SA = FM > FN;                       // A streamed, else B
      constexpr int FR = SA ? FN : FM, FS = SA ? FM : FN;
      constexpr int NX = NP * FR;                        // products of one streamed fragment
      constexpr int NL = G::kLoads, NSTAGE = NX * (FS - 1);  // products that the staging spreads over
      static_assert(FS % 2 == 0, "the first and last streamed fragment use different register sets");
      bf8_t res[NS][FR], str[2][NS];
      auto fetch = [&](int b, bool a, int s, int f) {
        return a ? *reinterpret_cast<const bf8_t*>(&As[b][s * MT * LD + a_frag[f]])
                 : *reinterpret_cast<const bf8_t*>(&Bs[b][s * NT * LD + b_frag[f]]);
      };
      auto fetch_resident = [&](int b, auto s, auto f) { res[s()][f()] = fetch(b, !SA, s(), f()); };
      auto fetch_streamed = [&](int b, auto s, auto f) { str[f() & 1][s()] = fetch(b, SA, s(), f()); };
      // the last product that uses resident slice s
      constexpr auto last_use = [](int s) {
        constexpr int qa[10] = {0, 0, 1, 0, 2, 1, 0, 3, 1, 2}, qb[10] = {0, 1, 0, 2, 0, 1, 3, 0, 2, 1};
        int at = -1;
        for (int p = 0; p < NP; ++p)
          if ((SA ? qb[p] : qa[p]) == s) at = p;
        return at;
      };
      auto stage_one = [&](int b, auto y) {
        constexpr int sl = y() / (G::AJ + G::BJ), j = y() % (G::AJ + G::BJ);
        if constexpr (j < G::AJ) {
          if (G::a_live(tid + j * NTHR))
            *reinterpret_cast<u4_t*>(&As[b][sl * MT * LD + 8 * lds_unit<MT>(g.lds_row(j), g.lds_k(j) / 8)]) = g.ra[sl][j];
        } else {
          constexpr int jb = j - G::AJ;
          if (G::b_live(tid + jb * NTHR))
            *reinterpret_cast<u4_t*>(&Bs[b][sl * NT * LD + 8 * lds_unit<NT>(g.lds_row(jb), g.lds_k(jb) / 8)]) = g.rb[sl][jb];
        }
        g.load_one(y());
      };
      ChunkWalk<KT, G, E> walk(g, pairs, pb, pe, pool, Ap, Bp, w, blk.mext, blk.next);
      uint32_t flushes = 0;  // of the chunks fetched and not yet multiplied, the oldest in bit 0
      int ahead = 0;
      auto note = [&]() {
        const int kend = walk.k + KT;
        flushes |= (kend >= walk.d.kext || kend % kSplitWindow == 0 ? 1u : 0u) << ahead;
        ++ahead;
      };
      auto next_chunk = [&]() {
        const bool more = walk.next_tables();
        if (more) note();
        return more;
      };
      walk.setup();
      g.load_tables(walk.d, pool, 0);
      note();
      g.load_data();
      bool inflight = next_chunk();  // the chunk staged during this one is real
      static_for<NL>([&](auto y) { stage_one(0, y); });
      bool tabs = inflight && next_chunk();  // so is the one after it
      __syncthreads();
      static_for<NS>([&](auto s) {
        static_for<FR>([&](auto f) { fetch_resident(0, s, f); });
        fetch_streamed(0, s, int_c<0>{});
      });
      for (int buf = 0;; buf ^= 1) {
        const bool flush = (flushes & 1u) != 0;
        flushes >>= 1;
        --ahead;
        // One streamed fragment after another; beside the products, the next one's operands are read
        // and the staged chunk is stored and loaded again, a little at a time (all reads of a chunk
        // in one run after the barrier left the matrix pipe idle meanwhile: both waves of a SIMD come
        // from one workgroup and wait at the same barrier).  The barrier comes before the last
        // fragment's products: by then every wave holds its operands of this chunk and has stored
        // its part of the next one, whose first operands are read under those products as soon as
        // their registers are free.  Aligned ladder at O=64, V=320 on 128 x 128 tiles: 113 -> 109 ms,
        // 1234 TFLOP/s of bfloat16 products, where this card's library product of 8192 x 8192
        // matrices reaches 1319: the board's power bounds both.
        __builtin_amdgcn_s_setprio(1);
        static_for<FS>([&](auto f) {
          if constexpr (f() == FS - 1) __syncthreads();
          static_for<NX>([&](auto x) {
            constexpr int p = x() / FR, fr = x() % FR, i = SA ? f() : fr, j = SA ? fr : f();
            f4_t& sum = p == 0 ? lead[i][j] : rest[i][j];
            sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(SA ? str[f() & 1][PA[p]] : res[PA[p]][fr],
                                                           SA ? res[PB[p]][fr] : str[f() & 1][PB[p]], sum, 0, 0, 0);
            if constexpr (f() + 1 < FS) {
              if constexpr (x() < NS) fetch_streamed(buf, x, int_c<f() + 1>{});
              constexpr int at = f() * NX + x(), y0 = at * NL / NSTAGE, y1 = (at + 1) * NL / NSTAGE;
              static_for<y1 - y0>([&](auto y) { stage_one(buf ^ 1, int_c<y0 + y()>{}); });
            } else {
              if constexpr (x() < NS) fetch_streamed(buf ^ 1, x, int_c<0>{});
              static_for<NS>([&](auto s) {
                if constexpr (p == last_use(s())) fetch_resident(buf ^ 1, s, int_c<fr>{});
              });
            }
            __builtin_amdgcn_sched_barrier(0);
          });
        });
        __builtin_amdgcn_s_setprio(0);
        const bool tabs_next = tabs && next_chunk();
        if (flush) flush_window();
        if (!inflight) break;
        inflight = tabs;
        tabs = tabs_next;
      }
    }
  } else if (pb < pe) {
    auto store = [&](int b) {  // one packed element: its NS slices to NS planes
      unsigned short* As16 = reinterpret_cast<unsigned short*>(As[b]);
      unsigned short* Bs16 = reinterpret_cast<unsigned short*>(Bs[b]);
#pragma unroll
      for (int e = 0; e < G::AE; ++e) {
        const int o = g.a_lds_row(e) * LD + g.a_lds_k(e);
#pragma unroll
        for (int s = 0; s < NS; ++s) As16[s * MT * LD + o] = (unsigned short)(g.ra[e] >> (16 * s));
      }
#pragma unroll
      for (int e = 0; e < G::BE; ++e) {
        const int o = g.b_lds_row(e) * LD + g.b_lds_k(e);
#pragma unroll
        for (int s = 0; s < NS; ++s) Bs16[s * NT * LD + o] = (unsigned short)(g.rb[e] >> (16 * s));
      }
    };
    auto compute = [&](int b, bool flush, auto&& stage, auto&& post) {
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int st = 0; st < KT / 32; ++st) {  // zeros beyond a ragged chunk's K extent
        bf8_t af[NS][FM], bfr[NS][FN];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
          for (int i = 0; i < FM; ++i)
            af[s][i] = *reinterpret_cast<const bf8_t*>(&As[b][s * MT * LD + a_frag[i] + 32 * st]);
#pragma unroll
          for (int j = 0; j < FN; ++j)
            bfr[s][j] = *reinterpret_cast<const bf8_t*>(&Bs[b][s * NT * LD + b_frag[j] + 32 * st]);
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            f4_t r = rest[i][j];
            if (ALIGNED) {
              // lead x lead is exact in float32 and kept apart; nine residual products
              lead[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][i], bfr[0][j], lead[i][j], 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][i], bfr[1][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[1][i], bfr[0][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][i], bfr[2][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[2][i], bfr[0][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[1][i], bfr[1][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][i], bfr[NS - 1][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[NS - 1][i], bfr[0][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[1][i], bfr[2][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[2][i], bfr[1][j], r, 0, 0, 0);
            } else {
              // b0 x b0 carries almost all of the sum: its own accumulator, so that its running
              // sum is rounded once per k-step rather than once per product plane
              lead[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][i], bfr[0][j], lead[i][j], 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][i], bfr[1][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[1][i], bfr[0][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][i], bfr[2][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[2][i], bfr[0][j], r, 0, 0, 0);
              r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[1][i], bfr[1][j], r, 0, 0, 0);
            }
            rest[i][j] = r;
          }
        if (st == 0) stage();
      }
      __builtin_amdgcn_s_setprio(0);
      post();  // bookkeeping of the next chunk while the MFMAs drain
      if (flush) flush_window();
    };
    chunk_pipeline<KT, kSplitWindow>(g, pairs, pb, pe, pool, Ap, Bp, w, blk.mext, blk.next, store, compute);
  }
  epilogue_f32layout<MT, NT, WM, WN, FM, FN>(pr, w, blk, acc, wm, wn, lr, lq);
}

// ---------------------------------------------------------------------------------------------
// configurations and dispatch
// ---------------------------------------------------------------------------------------------
static const MixedConfig kF32Configs[] = {
    {64, 64, 16, 2, 2, 4, 86, 86, "f32_m64n64k16_w2x2"},
    {128, 64, 16, 2, 2, 2, 93, 93, "f32_m128n64k16_w2x2"},
    {64, 128, 16, 2, 2, 2, 92, 92, "f32_m64n128k16_w2x2"},
    {128, 128, 16, 2, 2, 1, 83, 83, "f32_m128n128k16_w2x2"},
    {128, 128, 16, 4, 2, 1, 95, 95, "f32_m128n128k16_w4x2"},
    {128, 128, 16, 2, 4, 1, 95, 95, "f32_m128n128k16_w2x4"},
};
// Eight waves where one workgroup fills a compute unit's LDS (two waves per SIMD): four on the same
// tile were slower on both layouts (aligned ladder at O=24, V=104 1.04 against 0.88 ms; at O=64,
// V=320 139 against 109, on 128 x 128).  4 x 2 waves read the planes best, 2 x 4 the packed words.
static const MixedConfig kBf16Configs[] = {
    {64, 64, 32, 2, 2, 2, 61, 100, "bf16s_m64n64k32_w2x2"},
    {128, 64, 32, 2, 2, 1, 55, 97, "bf16s_m128n64k32_w2x2"},
    {64, 128, 32, 2, 2, 1, 50, 97, "bf16s_m64n128k32_w2x2"},
    {128, 64, 32, 4, 2, 1, 73, 110, "bf16s_m128n64k32_w4x2"},
    {64, 128, 32, 2, 4, 1, 64, 110, "bf16s_m64n128k32_w2x4"},
    {128, 128, 32, 4, 2, 1, 50, 125, "bf16s_m128n128k32_w4x2"},
    {128, 128, 32, 2, 4, 1, 92, 120, "bf16s_m128n128k32_w2x4"},
};

int mixed_config_count(int precision) {
  if (precision == TAMM_PREC_F32) return (int)(sizeof(kF32Configs) / sizeof(kF32Configs[0]));
  return (int)(sizeof(kBf16Configs) / sizeof(kBf16Configs[0]));
}

const MixedConfig& mixed_config(int precision, int id) {
  return precision == TAMM_PREC_F32 ? kF32Configs[id] : kBf16Configs[id];
}

template <int MT, int NT, int KT, int WGM, int WGN>
static hipError_t launch_f32(int layout, const ContractParams& p, hipStream_t s) {
  const dim3 g(p.n_work), b(64 * WGM * WGN);
  switch (layout) {
    case 3: hipLaunchKernelGGL((k_contract_f32<MT, NT, KT, WGM, WGN, true, true>), g, b, 0, s, p); break;
    case 2: hipLaunchKernelGGL((k_contract_f32<MT, NT, KT, WGM, WGN, true, false>), g, b, 0, s, p); break;
    case 1: hipLaunchKernelGGL((k_contract_f32<MT, NT, KT, WGM, WGN, false, true>), g, b, 0, s, p); break;
    default: hipLaunchKernelGGL((k_contract_f32<MT, NT, KT, WGM, WGN, false, false>), g, b, 0, s, p); break;
  }
  return hipGetLastError();
}

template <int MT, int NT, int KT, int WGM, int WGN, bool AL>
static hipError_t launch_bf(int layout, const ContractParams& p, hipStream_t s) {
  const dim3 g(p.n_work), b(64 * WGM * WGN);
  switch (layout) {
    case kPlanesLayout: hipLaunchKernelGGL((k_contract_bf16s<MT, NT, KT, WGM, WGN, AL, false, false, true>), g, b, 0, s, p); break;
    case 3: hipLaunchKernelGGL((k_contract_bf16s<MT, NT, KT, WGM, WGN, AL, true, true, false>), g, b, 0, s, p); break;
    case 2: hipLaunchKernelGGL((k_contract_bf16s<MT, NT, KT, WGM, WGN, AL, true, false, false>), g, b, 0, s, p); break;
    case 1: hipLaunchKernelGGL((k_contract_bf16s<MT, NT, KT, WGM, WGN, AL, false, true, false>), g, b, 0, s, p); break;
    default: hipLaunchKernelGGL((k_contract_bf16s<MT, NT, KT, WGM, WGN, AL, false, false, false>), g, b, 0, s, p); break;
  }
  return hipGetLastError();
}

hipError_t launch_contract_mixed(int precision, int config, int layout, const ContractParams& p, hipStream_t s) {
  if (p.n_work <= 0) return hipSuccess;
  if (precision == TAMM_PREC_F32) {
    switch (config) {
      case 0: return launch_f32<64, 64, 16, 2, 2>(layout, p, s);
      case 1: return launch_f32<128, 64, 16, 2, 2>(layout, p, s);
      case 2: return launch_f32<64, 128, 16, 2, 2>(layout, p, s);
      case 3: return launch_f32<128, 128, 16, 2, 2>(layout, p, s);
      case 4: return launch_f32<128, 128, 16, 4, 2>(layout, p, s);
      case 5: return launch_f32<128, 128, 16, 2, 4>(layout, p, s);
      default: return hipErrorInvalidValue;
    }
  }
  const bool al = precision == TAMM_PREC_BF16X4_ALIGNED;
  switch (config) {
    case 0: return al ? launch_bf<64, 64, 32, 2, 2, true>(layout, p, s) : launch_bf<64, 64, 32, 2, 2, false>(layout, p, s);
    case 1: return al ? launch_bf<128, 64, 32, 2, 2, true>(layout, p, s) : launch_bf<128, 64, 32, 2, 2, false>(layout, p, s);
    case 2: return al ? launch_bf<64, 128, 32, 2, 2, true>(layout, p, s) : launch_bf<64, 128, 32, 2, 2, false>(layout, p, s);
    case 3: return al ? launch_bf<128, 64, 32, 4, 2, true>(layout, p, s) : launch_bf<128, 64, 32, 4, 2, false>(layout, p, s);
    case 4: return al ? launch_bf<64, 128, 32, 2, 4, true>(layout, p, s) : launch_bf<64, 128, 32, 2, 4, false>(layout, p, s);
    case 5: return al ? launch_bf<128, 128, 32, 4, 2, true>(layout, p, s) : launch_bf<128, 128, 32, 4, 2, false>(layout, p, s);
    case 6: return al ? launch_bf<128, 128, 32, 2, 4, true>(layout, p, s) : launch_bf<128, 128, 32, 2, 4, false>(layout, p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tamm
