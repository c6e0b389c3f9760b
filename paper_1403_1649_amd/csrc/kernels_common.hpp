// Generic launch skeletons of the solve phase: a CSR row kernel (L lanes per
// row, wave64 sub-groups) and an elementwise kernel, both with an optional
// fused reduction.  Reductions are deterministic: each block reduces in a
// fixed order and writes one partial per block; the partials are then summed
// in block order (by a one-block finalize kernel, or for grids of at most
// kTailBlocks blocks by the last block of the kernel itself) and handed to
// the operation's finalizer, which writes device scalars and flags.  Every operation carries an `active` flag read at
// kernel entry, so branches of the K-cycle and the outer iteration are
// decided on the device.
#pragma once
#include <atomic>
#include <type_traits>

#include "amg_internal.hpp"
#include "device_utils.hpp"

namespace amg {

constexpr int kBlock = 256;

// Grids of at most kTailBlocks blocks finish their reduction in the kernel:
// the last block to arrive (a ticket counter) sums the partials in block
// order, exactly as k_finalize does, and runs the finalizer; larger grids use
// the separate finalize kernel.  The limit is set by the release fence each
// block needs before taking its ticket: at device scope it writes back the
// XCD's L2, which grows expensive when many blocks of a large kernel do it.
constexpr int kTailBlocks = 64;


template <int NV, class Op>
__device__ __forceinline__ void write_partials(double (&acc)[NV], RedCtx rc, const Op& op, bool tail) {
  static_assert(NV <= kMaxReduce, "the partials buffer holds kMaxReduce values per block");
  __shared__ double red[NV * (kBlock / kWave)];
  __shared__ int s_last;
  block_sum<NV>(acc, red);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) rc.part[k * gridDim.x + blockIdx.x] = acc[k];
  }
  if (!tail) return;
  if (threadIdx.x == 0) {
    __threadfence();   // the partial is visible before the ticket is taken
    s_last = atomicAdd(rc.ticket, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (!s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const int nb = gridDim.x;
  double v[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double t = 0.0;
    for (int b = threadIdx.x; b < nb; b += kBlock) t += rc.part[k * nb + b];
    v[k] = t;
  }
  block_sum<NV>(v, red);
  if (threadIdx.x == 0) {
    op.finalize(v);
    *rc.ticket = 0u;
  }
}

// The one-block finalize reads the partials with 1024 threads (2048 blocks x
// up to 3 values: a few loads per thread): on the 128^3 Poisson solve, 15
// finalizes per iteration, 9.51 -> 9.25 ms against 256 threads.  Five values of
// 2048 blocks: 7.1 us when each value's loads waited for the last one's, 5.6.
constexpr int kFinBlock = 1024;
template <class Op>
__global__ void __launch_bounds__(kFinBlock) k_finalize(Op op, const double* __restrict__ part, int nb) {
  if (!op.active()) return;
  constexpr int NV = Op::NV;
  __shared__ double red[NV * (kFinBlock / kWave)];
  static_assert(kMaxPartialBlocks <= 2 * kFinBlock, "two loads per thread and value");
  double v[NV], w[NV];   // all loads in flight together
  const int b0 = threadIdx.x, b1 = b0 + kFinBlock;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    v[k] = b0 < nb ? part[k * nb + b0] : 0.0;
    w[k] = b1 < nb ? part[k * nb + b1] : 0.0;
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += w[k];
  block_sum<NV>(v, red);
  if (threadIdx.x == 0) op.finalize(v);
}

// y-side of a sparse row operation: Op provides
//   static constexpr int NV;           number of fused reductions
//   void begin();                      optional: device scalars read once, into the operation itself
//   bool active() const;               kernel-wide enable
//   void idle() const;                 run by thread 0 of block 0 when inactive
//   T x(int j) const;                  the gathered operand
//   void row(int i, T ax, double* acc) the epilogue of row i
//   void finalize(const double* v)     totals of the reductions

template <class Op>
__device__ __forceinline__ auto op_begin(Op& op, int) -> decltype(op.begin(), void()) {
  op.begin();
}
template <class Op>
__device__ __forceinline__ void op_begin(Op&, long) {}

// Blocks are dispatched round-robin over the 8 XCDs (each with its own L2).
// The logical block index gives every XCD a contiguous run of blocks, and
// each logical block a contiguous chunk of the work, so the neighbouring rows
// whose x entries overlap share one L2.
__device__ __forceinline__ int xcd_logical_block() {
  const int g = gridDim.x, b = blockIdx.x;
  if (g < 8 || (g & 7)) return b;
  return (b & 7) * (g >> 3) + (b >> 3);
}

// Schedules of the slice kernels, whose unit of work is a step of 4 slices
// (one per wave of a block).  sched:
//    0   contiguous: each logical block a run of ceil(steps / grid) steps;
//   > 0  plane-ordered over planes of sched steps (a grid plane of rows, the
//        largest column offset of the level; steps a multiple of it): logical
//        step u of that run executes step (u % planes) * sched + u / planes,
//        so a block walks the same rows plane after plane and finds what it
//        gathers from the next plane in the cache;
//   -1   XCD sweep: each XCD a contiguous eighth of the steps, which its B
//        blocks take together (its block j: steps j, j + B, j + 2B, ... of
//        that eighth), so what the XCD reads at a time is one run of
//        adjacent rows and their neighbours (grids that are not a multiple
//        of 8: block j takes steps j, j + grid, ...).
struct Steps {
  int u, end, inc, planes, pstep;
  __device__ int step() const { return pstep > 0 ? (u % planes) * pstep + u / planes : u; }
};

__device__ __forceinline__ Steps block_steps(int steps, int sched) {
  Steps r;
  r.inc = 1;
  r.pstep = sched > 0 ? sched : 0;
  r.planes = sched > 0 ? steps / sched : 1;
  const int g = gridDim.x;
  if (sched == -1) {
    if (g >= 8 && !(g & 7)) {
      const int per8 = (steps + 7) / 8, x = blockIdx.x & 7;
      r.u = x * per8 + (blockIdx.x >> 3);
      r.end = min(steps, (x + 1) * per8);
      r.inc = g >> 3;
    } else {
      r.u = blockIdx.x;
      r.end = steps;
      r.inc = g;
    }
    return r;
  }
  const int per = (steps + g - 1) / g;
  r.u = xcd_logical_block() * per;
  r.end = min(steps, r.u + per);
  return r;
}

// D16: the columns come as 16-bit offsets col - row (Level::ci16).
template <typename T, int LPR, class Op, bool D16 = false>
__global__ void __launch_bounds__(kBlock) k_rows(int n, const int* __restrict__ rp,
                                                 const void* __restrict__ cols,
                                                 const T* __restrict__ av, Op op, RedCtx rc) {
  if (!op.active()) {
    if (blockIdx.x == 0 && threadIdx.x == 0) op.idle();
    return;
  }
  op_begin(op, 0);
  constexpr int RPB = kBlock / LPR;
  const int lane = threadIdx.x & (LPR - 1);
  double acc[Op::NV > 0 ? Op::NV : 1];
#pragma unroll
  for (int k = 0; k < (Op::NV > 0 ? Op::NV : 1); ++k) acc[k] = 0.0;
  const int groups = (n + RPB - 1) / RPB;
  const int per = (groups + gridDim.x - 1) / gridDim.x;
  const int g0 = xcd_logical_block() * per;
  const int g1 = min(groups, g0 + per);
  for (int g = g0; g < g1; ++g) {
    const int row = g * RPB + threadIdx.x / LPR;
    T sum = T(0);
    if (row < n) {
      const int s = rp[row], e = rp[row + 1];
      // a lane's entries four at a time: the column and value loads, then the
      // gathers, then the products in entry order (the same sum as one entry
      // at a time), so four gathers are in flight instead of one
      for (int k0 = s + lane; k0 < e; k0 += 4 * LPR) {
        int c[4];
        T v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = k0 + q * LPR;
          if constexpr (D16) c[q] = k < e ? row + (int)static_cast<const int16_t*>(cols)[k] : 0;
          else c[q] = k < e ? static_cast<const int*>(cols)[k] : 0;
          v[q] = k < e ? av[k] : T(0);
        }
        T xv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) xv[q] = k0 + q * LPR < e ? op.x(c[q]) : T(0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (k0 + q * LPR < e) sum += v[q] * xv[q];
      }
    }
    sum = group_sum<LPR>(sum);
    if (row < n && lane == 0) op.row(row, sum, acc);
  }
  if constexpr (Op::NV > 0) write_partials<Op::NV>(acc, rc, op, rc.ticket != nullptr);
}

// Orders a wave's own LDS writes before its later reads of other lanes' words
// (and the reads before the next writes): the wave runs in step, so only the
// compiler has to be held back.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Operands of row i that an operation wants loaded with the gathers (Op::Pre).
template <class Op, class = void>
struct RowPre {
  struct type {};
  __device__ static type load(const Op&, int) { return type{}; }
  template <typename T>
  __device__ static void row(const Op& op, int i, T sum, const type&, double* acc) { op.row(i, sum, acc); }
};
template <class Op>
struct RowPre<Op, std::void_t<typename Op::Pre>> {
  using type = typename Op::Pre;
  __device__ static type load(const Op& op, int i) { return op.pre(i); }
  template <typename T>
  __device__ static void row(const Op& op, int i, T sum, const type& p, double* acc) { op.row(i, sum, p, acc); }
};

// The row sums of a streamed group that exceeds the LDS: as many rows at a time
// as fit it, their products (entry(k)) by coalesced loads; a row of more than
// kLongRow entries is summed by the whole wave.  The sum of row l % R, whose
// entries are beg .. end, in lane l.
constexpr int kLongRow = 64;
template <typename T, int R, int Q, class Entry>
__device__ __forceinline__ T long_group_sum(int beg, int end, T* prod, Entry entry) {
  constexpr int LPR = kWave / R;
  constexpr uint64_t kRows = R == kWave ? ~0ull : (1ull << R) - 1;
  const int lane = threadIdx.x & (kWave - 1), rl = lane & (R - 1), part = lane / R;
  const uint64_t longs = __ballot(end - beg > kLongRow) & kRows;
  T sum = T(0);
  for (int i0 = 0; i0 < R;) {
    const int base = __builtin_amdgcn_readlane(beg, i0);
    const uint64_t after = longs >> i0;
    if (after & 1) {
      const int e = __builtin_amdgcn_readlane(end, i0);
      T t = T(0);
      for (int k = base + lane; k < e; k += kWave) t += entry(k);
      t = wave_sum(t);
      if (lane == i0) sum = t;
      ++i0;
      continue;
    }
    const int upto = after ? i0 + __ffsll((unsigned long long)after) - 1 : R;
    const int take = __popcll(__ballot(rl >= i0 && rl < upto && end - base <= kWave * Q) & kRows);
    const int total = __builtin_amdgcn_readlane(end, i0 + take - 1) - base;
    T p[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) p[q] = q * kWave + lane < total ? entry(base + q * kWave + lane) : T(0);
#pragma unroll
    for (int q = 0; q < Q; ++q) prod[q * kWave + lane] = p[q];
    wave_lds_order();
    if (rl >= i0 && rl < i0 + take)
      for (int k = beg - base + part; k < end - base; k += LPR) sum += prod[k];
    wave_lds_order();
    i0 += take;
  }
  if constexpr (LPR == 2) sum += __shfl_xor(sum, 32, kWave);
  return sum;
}

// CSR rows streamed through LDS.  A wave takes groups of R consecutive rows of
// about 64 Q entries together; a larger group takes several turns
// (long_group_sum).  A group's entries are one contiguous run, loaded coalesced,
// Q per lane; the products go to the wave's LDS, and 64/R lanes sum each row there.  So there is no padding, no
// idle lane on short rows, and every load instruction covers whole lines.
// What bounds it otherwise is the chain row pointers -> columns -> gathers ->
// sum: the loop keeps three groups in flight (the gathers of one, the columns
// and values of the next, the row pointers of the one after, and the row
// operands, Op::Pre, with the gathers), so a group costs one round trip.  All
// loads are unconditional, at clamped positions, for the same reason.
// Groups go to the XCDs in contiguous eighths, swept by the blocks of the XCD
// side by side (block_steps, -1).
// D16: columns as 16-bit offsets from the group's base column gbase[g].
template <typename T, class Op, int R, int Q, bool D16>
__global__ void __launch_bounds__(kBlock) k_stream(int n, const int* __restrict__ rp, const void* __restrict__ cols,
                                                   const int* __restrict__ gbase, const T* __restrict__ av, Op op,
                                                   RedCtx rc) {
  static_assert(R == 64 || R == 32, "rows per group");
  if (!op.active()) {
    if (blockIdx.x == 0 && threadIdx.x == 0) op.idle();
    return;
  }
  op_begin(op, 0);
  constexpr int SPB = kBlock / kWave;
  constexpr int LPR = kWave / R;
  __shared__ T s_prod[SPB][kWave * Q];
  double acc[Op::NV > 0 ? Op::NV : 1];
#pragma unroll
  for (int k = 0; k < (Op::NV > 0 ? Op::NV : 1); ++k) acc[k] = 0.0;
  const int lane = threadIdx.x & (kWave - 1);
  const int rl = lane & (R - 1), part = lane / R;   // this lane's row in the group, and its share of it
  const int wv = threadIdx.x / kWave;
  T* prod = s_prod[wv];
  const int ngroups = (n + R - 1) / R;
  const int steps = (ngroups + SPB - 1) / SPB;
  const Steps st = block_steps(steps, -1);
  struct Rows { int beg, end, cbase; };
  struct Entries { int c[Q]; T v[Q]; };
  auto rows_of = [&](int u) {   // groups past the end: an empty run at the matrix's end
    Rows w;
    const int grp = u < st.end ? min(u * SPB + wv, ngroups) : ngroups;
    const int row = grp * R + rl;
    w.beg = rp[min(row, n)];
    w.end = rp[min(row + 1, n)];
    w.cbase = D16 ? gbase[min(grp, ngroups - 1)] : 0;
    return w;
  };
  auto entries_of = [&](const Rows& w) {
    Entries t;
    const int base = __builtin_amdgcn_readfirstlane(w.beg);
    const int last = max(__builtin_amdgcn_readlane(w.end, R - 1) - 1, 0);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = min(base + q * kWave + lane, last);
      if constexpr (D16) t.c[q] = w.cbase + (int)static_cast<const int16_t*>(cols)[k];
      else t.c[q] = static_cast<const int*>(cols)[k];
      t.v[q] = av[k];
    }
    return t;
  };
  Rows r0 = rows_of(st.u), r1 = rows_of(st.u + st.inc);
  Entries e0 = entries_of(r0);
  for (int u = st.u; u < st.end; u += st.inc) {
    const int row = (u * SPB + wv) * R + rl;
    T xv[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) xv[q] = op.x(e0.c[q]);
    const typename RowPre<Op>::type pre = RowPre<Op>::load(op, min(row, n - 1));
    const Entries e1 = entries_of(r1);
    const Rows r2 = rows_of(u + 2 * st.inc);
    const int base = __builtin_amdgcn_readfirstlane(r0.beg);
    const int total = __builtin_amdgcn_readlane(r0.end, R - 1) - base;
    T sum = T(0);
    if (total <= kWave * Q) {
#pragma unroll
      for (int q = 0; q < Q; ++q) prod[q * kWave + lane] = e0.v[q] * xv[q];
      wave_lds_order();
      for (int k = r0.beg - base + part; k < r0.end - base; k += LPR) sum += prod[k];
      wave_lds_order();
      if constexpr (LPR == 2) sum += __shfl_xor(sum, 32, kWave);
    } else {
      sum = long_group_sum<T, R, Q>(r0.beg, r0.end, prod, [&](int k) {
        int c;
        if constexpr (D16) c = r0.cbase + (int)static_cast<const int16_t*>(cols)[k];
        else c = static_cast<const int*>(cols)[k];
        return av[k] * op.x(c);
      });
    }
    if (row < n && part == 0) RowPre<Op>::row(op, row, sum, pre, acc);
    r0 = r1;
    r1 = r2;
    e0 = e1;
  }
  if constexpr (Op::NV > 0) write_partials<Op::NV>(acc, rc, op, rc.ticket != nullptr);
}

// Sliced ELL with slices of H rows (H = 64, 32 or 16): slice s holds the rows
// of slots s*H .. s*H + H - 1 column-major, element (slot s*H + l, k) at
// sl_ptr[s] + H k + l, padded with zero values that point at the row itself.
// Slot i holds row perm[i] (perm null: row i); the copies in shorter slices
// order the rows of each 256-row window by decreasing length, so a slice's
// rows are of nearly equal length and the padding small.  One wave per slice
// and G = 64/H lanes per row: lane j*H + l takes entries j, j + G, ... of the
// row in slot l, so every value and column load of a wave is one contiguous
// run of 64 elements; the G partial sums are added by lane exchange (lane xor
// H, 2H, ...).
// D16: the columns come as 16-bit offsets col - row (128 bytes per wave and
// entry instead of 256), for levels whose couplings all lie within 32767
// rows, as on the lexicographically ordered grids.
// pstep: the schedule of the block steps (block_steps).
template <typename T, class Op, bool D16, int H = kWave>
__global__ void __launch_bounds__(kBlock) k_sell(int n, int nslices, const int* __restrict__ sl_ptr,
                                                 const void* __restrict__ sl_cols, const T* __restrict__ sl_val,
                                                 const int* __restrict__ perm, Op op, RedCtx rc, int pstep) {
  static_assert(H == 64 || H == 32 || H == 16, "slice height");
  constexpr int G = kWave / H;   // lanes per row
  if (!op.active()) {
    if (blockIdx.x == 0 && threadIdx.x == 0) op.idle();
    return;
  }
  op_begin(op, 0);
  double acc[Op::NV > 0 ? Op::NV : 1];
#pragma unroll
  for (int k = 0; k < (Op::NV > 0 ? Op::NV : 1); ++k) acc[k] = 0.0;
  constexpr int SPB = kBlock / kWave;   // slices per block step
  const int lane = threadIdx.x & (kWave - 1);
  const int j = lane / H;               // this lane's entries: j, j + G, j + 2G, ...
  const int wv = threadIdx.x / kWave;
  const int steps = (nslices + SPB - 1) / SPB;
  for (Steps st = block_steps(steps, pstep); st.u < st.end; st.u += st.inc) {
    const int sl = st.step() * SPB + wv;
    if (sl >= nslices) continue;
    const int slot = sl * H + (lane & (H - 1));
    const int row = perm ? perm[slot] : slot;
    const int base = __builtin_amdgcn_readfirstlane(sl_ptr[sl]);   // wave-uniform
    const int w = (__builtin_amdgcn_readfirstlane(sl_ptr[sl + 1]) - base) / H;
    T sum = T(0);
    const int* cp = static_cast<const int*>(sl_cols) + base + lane;
    const int16_t* dp = static_cast<const int16_t*>(sl_cols) + base + lane;
    const T* vp = sl_val + base + lane;
    // chunks of 8 entries per lane: all column and value loads of a chunk,
    // then all gathers, then the FMAs in entry order, so a chunk costs one
    // round trip.  Entry k0 + G q + j of the row sits at H k0 + 64 q + lane.
    for (int k0 = 0; k0 < w; k0 += 8 * G) {
      int c[8];
      T v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const bool in = k0 + G * q + j < w;
        const int off = H * k0 + kWave * q;
        if constexpr (D16) c[q] = in ? row + (int)dp[off] : 0;
        else c[q] = in ? cp[off] : 0;
        // the values stream through once per pass: non-temporal loads keep
        // them from displacing what the next kernels reuse from the caches
        // (the coarse levels' data in the Infinity Cache); 128^3 Poisson
        // solve 9.20 -> 8.92 ms
        v[q] = in ? __builtin_nontemporal_load(vp + off) : T(0);
      }
      T xv[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) xv[q] = k0 + G * q + j < w ? op.x(c[q]) : T(0);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (k0 + G * q + j < w) sum += v[q] * xv[q];
    }
    if constexpr (G > 1) {
#pragma unroll
      for (int o = H; o < kWave; o <<= 1) sum += __shfl_xor(sum, o, kWave);
    }
    if (row < n && j == 0) op.row(row, sum, acc);
  }
  if constexpr (Op::NV > 0) write_partials<Op::NV>(acc, rc, op, rc.ticket != nullptr);
}

// Symmetric diagonals: the main diagonal and those above it, one vector over the
// rows each (offsets d, ascending, the same for every row); row i takes
// a_{i, i-d} from where row i-d stores it, in the L2 or, for the largest offset,
// mostly in the Infinity Cache (160^3: 423 MB cross the L2s per pre-smoothing,
// 467 with sliced diagonals; the format's own bytes are 262 MB).  Bound by
// memory: a structured seven-point level moves 32 bytes of values per row
// instead of 56 (sliced diagonals).  160^3 in FP64, pre-smoothing 83.7 -> 71.2
// us, FCG product 75.1 -> 56.4, plain residual 70.5 -> 51.2.  Products are
// summed in ascending columns, as in the other layouts.
template <int U>
struct SymOff {
  int d[U];
};
// An operation of its own (Op::kOnce: a product outside the cycle) finds nothing
// of the matrix in the caches and leaves nothing there worth keeping, so its
// values are loaded non-temporally.  After a gigabyte of other writes 160^3
// takes 61 us (77 without the hint, 69 with sliced diagonals), 128^3 34 (44, 38),
// a 2000^2 five-point grid 45 (58); back to back, all of it in the Infinity
// Cache, 52 (39, 59), which is why the cycle's kernels have no hint.
template <class Op, class = void>
struct OnceOp : std::false_type {};
template <class Op>
struct OnceOp<Op, std::enable_if_t<Op::kOnce>> : std::true_type {};
template <typename T, int U, class Op>
__global__ void __launch_bounds__(kBlock) k_sym_dia_rows(int n, long ld, SymOff<U> off, const T* __restrict__ val,
                                                         Op op, RedCtx rc, int pstep) {
  if (!op.active()) {
    if (blockIdx.x == 0 && threadIdx.x == 0) op.idle();
    return;
  }
  op_begin(op, 0);
  double acc[Op::NV > 0 ? Op::NV : 1];
#pragma unroll
  for (int k = 0; k < (Op::NV > 0 ? Op::NV : 1); ++k) acc[k] = 0.0;
  const int steps = (int)((ld + kBlock - 1) / kBlock);
  for (Steps st = block_steps(steps, pstep); st.u < st.end; st.u += st.inc) {
    const int row = st.step() * kBlock + (int)threadIdx.x;
    if (row >= n) continue;
    T lo[U], up[U], xl[U], xu[U];
#pragma unroll
    for (int t = 0; t < U; ++t) {
      const T* d = val + t * ld;
      const int j = row - off.d[t] < 0 ? 0 : row - off.d[t];
      if constexpr (OnceOp<Op>::value) {
        up[t] = __builtin_nontemporal_load(d + row);
        lo[t] = t > 0 ? __builtin_nontemporal_load(d + j) : T(0);
      } else {
        up[t] = d[row];
        lo[t] = t > 0 ? d[j] : T(0);
      }
    }
#pragma unroll
    for (int t = 0; t < U; ++t) {   // past either end: clamped, and not taken
      const int j = row - off.d[t], k = row + off.d[t];
      xu[t] = op.x(k < n ? k : n - 1);
      xl[t] = t > 0 ? op.x(j < 0 ? 0 : j) : T(0);
    }
    // where the row has no entry the stored zero is left out, not multiplied:
    // x there may hold an infinity (the compares cost nothing beside the loads)
    T sum = T(0);
#pragma unroll
    for (int t = U - 1; t > 0; --t)
      if (row >= off.d[t] && lo[t] != T(0)) sum += lo[t] * xl[t];
    sum += up[0] * xu[0];
#pragma unroll
    for (int t = 1; t < U; ++t)
      if (up[t] != T(0)) sum += up[t] * xu[t];
    op.row(row, sum, acc);
  }
  if constexpr (Op::NV > 0) write_partials<Op::NV>(acc, rc, op, rc.ticket != nullptr);
}

// Sliced diagonals: slices of 64 rows (one wave), each with its own short
// list of diagonal offsets d (col = row + d, ascending): slice s holds
// offsets dg_off[dg_ptr[s] .. dg_ptr[s+1]) and, for the q-th of them, the
// value of row s*64 + l at (dg_ptr[s] + q) * 64 + l (zero where the row has no
// entry on that diagonal).  No column is stored: the offset is one scalar per
// wave and diagonal, so a level from a structured grid moves 8 bytes per entry
// (4 in FP32) plus the vectors.  pstep: the schedule (block_steps).
template <typename T, class Op>
__global__ void __launch_bounds__(kBlock) k_sdia(int n, int nslices, const int* __restrict__ dg_ptr,
                                                 const int* __restrict__ dg_off, const T* __restrict__ dg_val,
                                                 Op op, RedCtx rc, int pstep) {
  if (!op.active()) {
    if (blockIdx.x == 0 && threadIdx.x == 0) op.idle();
    return;
  }
  op_begin(op, 0);
  double acc[Op::NV > 0 ? Op::NV : 1];
#pragma unroll
  for (int k = 0; k < (Op::NV > 0 ? Op::NV : 1); ++k) acc[k] = 0.0;
  constexpr int SPB = kBlock / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  const int steps = (nslices + SPB - 1) / SPB;
  for (Steps st = block_steps(steps, pstep); st.u < st.end; st.u += st.inc) {
    const int sl = st.step() * SPB + wv;
    if (sl >= nslices) continue;
    const int row = sl * kWave + lane;
    // wave-uniform: the offsets come by scalar loads and the entry loop needs
    // no lane masks (so no wait between the loads of a chunk)
    const int base = __builtin_amdgcn_readfirstlane(dg_ptr[sl]);
    const int w = __builtin_amdgcn_readfirstlane(dg_ptr[sl + 1]) - base;
    const T* vp = dg_val + (size_t)base * kWave + lane;
    T sum = T(0);
    for (int k0 = 0; k0 < w; k0 += 8) {
      int c[8];
      T v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        // the chunk's offsets unconditionally (scalar loads; slots past the
        // slice repeat its last offset); padding may point past either end
        // of the rows: clamp (its value is zero)
        const int col = row + dg_off[base + min(k0 + q, w - 1)];
        c[q] = col < 0 ? 0 : (col >= n ? n - 1 : col);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = k0 + q < w ? __builtin_nontemporal_load(vp + (size_t)(k0 + q) * kWave) : T(0);
      T xv[8];   // padding slots gather their slice's last column again (a cache hit)
#pragma unroll
      for (int q = 0; q < 8; ++q) xv[q] = op.x(c[q]);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (k0 + q < w) sum += v[q] * xv[q];
    }
    if (row < n) op.row(row, sum, acc);
  }
  if constexpr (Op::NV > 0) write_partials<Op::NV>(acc, rc, op, rc.ticket != nullptr);
}

// Elementwise operation over [0, n): Op provides NV, active(), idle(),
// elem(int i, double* acc), finalize(const double*).
template <class Op>
__global__ void __launch_bounds__(kBlock) k_elem(int n, Op op, RedCtx rc) {
  if (!op.active()) {
    if (blockIdx.x == 0 && threadIdx.x == 0) op.idle();
    return;
  }
  op_begin(op, 0);
  double acc[Op::NV > 0 ? Op::NV : 1];
#pragma unroll
  for (int k = 0; k < (Op::NV > 0 ? Op::NV : 1); ++k) acc[k] = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) op.elem(i, acc);
  if constexpr (Op::NV > 0) write_partials<Op::NV>(acc, rc, op, rc.ticket != nullptr);
}

// Grid of the row kernels: one block per 256-row (or RPB-row) group up to a
// cap of 2048 resident blocks (8 per CU); a multiple of 8 above 8 blocks so
// that the XCD-aware mapping is a bijection.
inline int rows_grid(int n, int lpr, bool reduce) {
  (void)reduce;
  long rpb = kBlock / lpr;
  long g = (n + rpb - 1) / rpb;
  const long cap = kMaxPartialBlocks;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  if (g > 8) g &= ~7L;
  return (int)g;
}

inline int elem_grid(int n, bool reduce) {
  long g = ((long)n + kBlock - 1) / kBlock;
  long cap = reduce ? kMaxPartialBlocks : 65536;
  if (g < 1) g = 1;
  return (int)(g < cap ? g : cap);
}

// Blocks of kernel k that the device holds at once, at most
// kMaxPartialBlocks: a slice kernel gives each block a fixed share of the
// steps, so a grid larger than what is resident would run its last blocks
// in a second, mostly empty round (kernels whose registers allow fewer than
// 8 blocks of 256 threads per CU).  Per kernel instance, taken once (host
// threads that race on the first launch compute the same value).
template <class K>
int resident_blocks(K k) {
  static std::atomic<int> cached{0};
  int g = cached.load(std::memory_order_relaxed);
  if (g == 0) {
    int per = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, kBlock, 0) != hipSuccess || per < 1) per = 8;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 256;
    const long r = (long)per * cus;
    g = (int)(r < kMaxPartialBlocks ? r : kMaxPartialBlocks);
    cached.store(g, std::memory_order_relaxed);
  }
  return g;
}

// Grid of a slice kernel over `steps` steps: one block per step up to the
// resident cap, a multiple of 8 above 8 blocks (the XCD mapping).
inline int step_grid(int steps, int resident) {
  long g = steps;
  if (g < 1) g = 1;
  if (g > resident) g = resident;
  if (g > 8) g &= ~7L;
  return (int)g;
}

template <typename T, int LPR, class Op, bool D16 = false>
void launch_rows_l(int n, const int* rp, const void* ci, const T* av, const Op& op, RedCtx rc, hipStream_t s) {
  int g = rows_grid(n, LPR, Op::NV > 0);
  const int cap = resident_blocks(k_rows<T, LPR, Op, D16>);
  if (g > cap) g = cap > 8 ? cap & ~7 : cap;
  const bool tail = Op::NV > 0 && g <= kTailBlocks && rc.ticket != nullptr;
  const RedCtx r2{rc.part, tail ? rc.ticket : nullptr};
  k_rows<T, LPR, Op, D16><<<g, kBlock, 0, s>>>(n, rp, ci, av, op, r2);
  if constexpr (Op::NV > 0)
    if (!tail) k_finalize<Op><<<1, kFinBlock, 0, s>>>(op, rc.part, g);
}

// The streamed kernel (a step is four groups of R rows).  gbase non-null:
// cols are 16-bit offsets.
template <typename T, class Op, int R, int Q, bool D16>
void launch_stream_l(int n, const int* rp, const void* cols, const int* gbase, const T* av, const Op& op, RedCtx rc,
                     hipStream_t s) {
  constexpr int rows = R * (kBlock / kWave);
  const int g = step_grid((n + rows - 1) / rows, resident_blocks(k_stream<T, Op, R, Q, D16>));
  const bool tail = Op::NV > 0 && g <= kTailBlocks && rc.ticket != nullptr;
  k_stream<T, Op, R, Q, D16><<<g, kBlock, 0, s>>>(n, rp, cols, gbase, av, op,
                                                      RedCtx{rc.part, tail ? rc.ticket : nullptr});
  if constexpr (Op::NV > 0)
    if (!tail) k_finalize<Op><<<1, kFinBlock, 0, s>>>(op, rc.part, g);
}

// Streamed rows of a CSR matrix with short rows: groups of 64 rows up to 7.5
// entries a row, of 32 up to 15 (the group's entries then fill eight loads per
// lane).  Longer rows: lanes per row.
inline bool stream_rows(int n, long nnz) { return nnz <= 15L * n; }
template <typename T, class Op>
void launch_stream(int n, long nnz, const int* rp, const int* ci, const T* av, const Op& op, RedCtx rc,
                   hipStream_t s) {
  if (2 * nnz <= 15L * n) launch_stream_l<T, Op, 64, 8, false>(n, rp, ci, nullptr, av, op, rc, s);
  else launch_stream_l<T, Op, 32, 8, false>(n, rp, ci, nullptr, av, op, rc, s);
}

// 2 to 64 lanes per row (one lane: the caller's products alone, spmv_f64)
template <typename T, class Op>
void launch_rows(int n, int lpr, const int* rp, const int* ci, const T* av, const Op& op, RedCtx rc,
                 hipStream_t s) {
  switch (lpr) {
    case 2: launch_rows_l<T, 2>(n, rp, ci, av, op, rc, s); break;
    case 4: launch_rows_l<T, 4>(n, rp, ci, av, op, rc, s); break;
    case 8: launch_rows_l<T, 8>(n, rp, ci, av, op, rc, s); break;
    case 16: launch_rows_l<T, 16>(n, rp, ci, av, op, rc, s); break;
    case 32: launch_rows_l<T, 32>(n, rp, ci, av, op, rc, s); break;
    default: launch_rows_l<T, 64>(n, rp, ci, av, op, rc, s); break;
  }
}

// The same with the columns as 16-bit offsets (2 to 32 lanes per row).
template <typename T, class Op>
void launch_rows16(int n, int lpr, const int* rp, const int16_t* ci16, const T* av, const Op& op, RedCtx rc,
                   hipStream_t s) {
  switch (lpr) {
    case 2: launch_rows_l<T, 2, Op, true>(n, rp, ci16, av, op, rc, s); break;
    case 4: launch_rows_l<T, 4, Op, true>(n, rp, ci16, av, op, rc, s); break;
    case 8: launch_rows_l<T, 8, Op, true>(n, rp, ci16, av, op, rc, s); break;
    case 16: launch_rows_l<T, 16, Op, true>(n, rp, ci16, av, op, rc, s); break;
    default: launch_rows_l<T, 32, Op, true>(n, rp, ci16, av, op, rc, s); break;
  }
}


// sl_dcol non-null: the kernel reads the 16-bit column offsets instead of sl_col.


template <typename T, class Op, bool D16, int H>
void launch_sell_h(int n, int nslices, const int* sl_ptr, const void* cols, const T* sl_val, const int* perm,
                   const Op& op, RedCtx rc, hipStream_t s, int pstep, int cap) {
  const int g = step_grid((nslices + kBlock / kWave - 1) / (kBlock / kWave),
                          std::min(cap, resident_blocks(k_sell<T, Op, D16, H>)));
  const bool tail = Op::NV > 0 && g <= kTailBlocks && rc.ticket != nullptr;
  const RedCtx r2{rc.part, tail ? rc.ticket : nullptr};
  k_sell<T, Op, D16, H><<<g, kBlock, 0, s>>>(n, nslices, sl_ptr, cols, sl_val, perm, op, r2, pstep);
  if constexpr (Op::NV > 0)
    if (!tail) k_finalize<Op><<<1, kFinBlock, 0, s>>>(op, rc.part, g);
}

// slice_h: the slice height of the copy (64, 32 or 16 rows); perm: its row
// order (null: rows in order)
template <typename T, class Op>
void launch_sell(int n, int nslices, const int* sl_ptr, const int* sl_col, const T* sl_val, const Op& op,
                 RedCtx rc, hipStream_t s, const int16_t* sl_dcol = nullptr, int pstep = 0, int slice_h = kWave,
                 const int* perm = nullptr, int cap = kMaxPartialBlocks) {   // cap: blocks at most
  if (slice_h != kWave) pstep = 0;
  const void* cols = sl_dcol ? static_cast<const void*>(sl_dcol) : static_cast<const void*>(sl_col);
  if (sl_dcol) {
    if (slice_h == 32) launch_sell_h<T, Op, true, 32>(n, nslices, sl_ptr, cols, sl_val, perm, op, rc, s, pstep, cap);
    else if (slice_h == 16) launch_sell_h<T, Op, true, 16>(n, nslices, sl_ptr, cols, sl_val, perm, op, rc, s, pstep, cap);
    else launch_sell_h<T, Op, true, 64>(n, nslices, sl_ptr, cols, sl_val, perm, op, rc, s, pstep, cap);
  } else {
    if (slice_h == 32) launch_sell_h<T, Op, false, 32>(n, nslices, sl_ptr, cols, sl_val, perm, op, rc, s, pstep, cap);
    else if (slice_h == 16) launch_sell_h<T, Op, false, 16>(n, nslices, sl_ptr, cols, sl_val, perm, op, rc, s, pstep, cap);
    else launch_sell_h<T, Op, false, 64>(n, nslices, sl_ptr, cols, sl_val, perm, op, rc, s, pstep, cap);
  }
}

template <typename T, class Op>
void launch_sym_dia(int n, const Level::SymDia& q, const T* val, const Op& op, RedCtx rc, hipStream_t s,
                    int pstep = 0, int cap = kMaxPartialBlocks) {
  const int steps = (int)(q.ld / kBlock) + (q.ld % kBlock != 0);
  auto go = [&](auto u) {
    constexpr int U = decltype(u)::value;
    SymOff<U> o;
    for (int t = 0; t < U; ++t) o.d[t] = q.off[t];
    const int g = step_grid(steps, std::min(cap, resident_blocks(k_sym_dia_rows<T, U, Op>)));
    const bool tail = Op::NV > 0 && g <= kTailBlocks && rc.ticket != nullptr;
    k_sym_dia_rows<T, U, Op><<<g, kBlock, 0, s>>>(n, q.ld, o, val, op, RedCtx{rc.part, tail ? rc.ticket : nullptr},
                                                  pstep);
    if constexpr (Op::NV > 0)
      if (!tail) k_finalize<Op><<<1, kFinBlock, 0, s>>>(op, rc.part, g);
  };
  static_assert(kSymDiaMin == 3 && kSymDiaMax == 5, "one kernel per number of stored diagonals");
  if (q.u == 3) go(std::integral_constant<int, 3>());
  else if (q.u == 4) go(std::integral_constant<int, 4>());
  else go(std::integral_constant<int, 5>());
}

template <typename T, class Op>
void launch_sdia(int n, int nslices, const int* dg_ptr, const int* dg_off, const T* dg_val, const Op& op,
                 RedCtx rc, hipStream_t s, int pstep = 0, int cap = kMaxPartialBlocks) {
  const int g = step_grid((nslices + kBlock / kWave - 1) / (kBlock / kWave),
                          std::min(cap, resident_blocks(k_sdia<T, Op>)));
  const bool tail = Op::NV > 0 && g <= kTailBlocks && rc.ticket != nullptr;
  const RedCtx r2{rc.part, tail ? rc.ticket : nullptr};
  k_sdia<T, Op><<<g, kBlock, 0, s>>>(n, nslices, dg_ptr, dg_off, dg_val, op, r2, pstep);
  if constexpr (Op::NV > 0)
    if (!tail) k_finalize<Op><<<1, kFinBlock, 0, s>>>(op, rc.part, (int)g);
}

template <class Op>
void launch_elem(int n, const Op& op, RedCtx rc, hipStream_t s) {
  const int g = elem_grid(n, Op::NV > 0);
  const bool tail = Op::NV > 0 && g <= kTailBlocks && rc.ticket != nullptr;
  k_elem<Op><<<g, kBlock, 0, s>>>(n, op, RedCtx{rc.part, tail ? rc.ticket : nullptr});
  if constexpr (Op::NV > 0)
    if (!tail) k_finalize<Op><<<1, kFinBlock, 0, s>>>(op, rc.part, g);
}

// Lanes per row from the average row length: about two entries per lane, as a
// lane keeps four in flight (7 entries a row, 28.5 M entries: 4 lanes 100 us,
// 8 lanes 125; 13.4 a row, 4.9 M entries: 8 lanes 19.8 us, 16 lanes 22.2).
inline int pick_lpr(int n, int nnz) {
  double avg = n > 0 ? (double)nnz / n : 1.0;
  int l = 1;
  while (2 * l < avg && l < 64) l <<= 1;
  return l < 2 ? 2 : l;
}

}  // namespace amg
