// Gradient pass by records: gradT_b += W_b^T S_b (columns) / S_b W_b^T (rows), S holding one non-zero per (line, group) at
// the group's arg-max (paper Sec. 4.1: gradient of the surrogate through the transformed weights; Sec. 4.2: of the
// LogSumExp surrogate).  Row j of a block's gradient is the sum of coefficient x line over the lines whose arg-max is j,
// so where a block meets one group per line (groups no shorter than the block) every line adds to ONE of the block's K
// rows: K multiply-adds a line and not the K^2 of the product with the matrix of zeros, in float32 without any splitting.
//
// Two launches.  sort_records_kernel: per unit -- the K rows of a block, or the rows of one of its groups where groups are
// shorter -- the records that fall into it, sorted by row (stable: the sums' order is the lines', run to run); the loss
// reduction, which a pair's coefficients wait for, and a single matrix' middle factor ride in it.
// grad_gather_kernel: a workgroup owns a few rows of a unit, its waves take equal shares of the rows' entries, whatever the
// distribution of the arg-max over the rows is.  A wave works on one line at a time -- row, coefficient and address in scalar
// registers, sixteen to 64 lines in flight (gather_ring) -- and a row that several waves share is put together in the waves' order.
// No partials: the rows leave in their final place.  The lines come from the matrix itself (columns: a line's inputs lie
// side by side) or from the line-major copy among the prepared weights (rows).
//
// Bound: memory, 4 K (2 K) bytes per line and block, once.
#include "cafeq_internal.hpp"
#include "loss_reduce.hpp"
#include "mmid.hpp"

namespace cafeq {
namespace {

constexpr int kGgThreads = 256, kGgWaves = kGgThreads / kWave;
constexpr int kGgFlight = 8;                         // a wave requests this many lines at a time ...
// ... and has this many requests in flight (registers: K / 64 a line.  20 blocks of 64, a wave's 50 to 500 lines: 2 deep 37 us, 8 deep 29;
// 27B-shaped pair in bfloat16 147, 142)
constexpr int gather_ring(int K) { return K == 256 ? 2 : K == 128 ? 3 : 8; }
constexpr int kGsThreads = 512, kGsWaves = kGsThreads / kWave;
constexpr int kGsFlight = 9;                         // records in flight per lane: those of 4608 lines stay in registers
constexpr int kGsList = 5120;                        // entries of a list that is put together in LDS (40 KB)
constexpr int kGatherLineBits = 24;                  // an entry: (row of the unit << 24 | line, the value at the arg-max)

struct GatherMember {
  const void* W;
  int64_t line_stride, seg_stride;   // elements: from line to line, from 128 inputs to the next
  const float2* rec;                 // [axis group][line]: (signed value at the arg-max, index inside the group)
  const float* rG;                   // kLossSur: [axis group]
  float* out;                        // [nb][K][K]
  uint2* sorted;                     // [unit][line]
  int* start;                        // [unit][unit_rows + 1]: the rows' first entries
  int64_t nlines;
  int bf16, grp, rep, unit_rows, transpose_out;
  int rows;                          // per workgroup of the gather
  unsigned nunit, nwg;               // of all row-blocks; workgroups of the gather
};
struct GatherArgs {
  GatherMember m[2];
  int nmem, loss_kind;
  float beta, lse_t;
  LossArgs la;                       // the call's loss reduction
  unsigned ntail;                    // single matrices: kMmidParts workgroups per block for the middle factor, or 0
  VArgs va;
  RhoGroups rho;                     // sums of rho over groups that span segments, a workgroup each (ngroups 0: none)
};

// ---------------------------------------------------------------------------------------------------
// records sorted by row
// ---------------------------------------------------------------------------------------------------
// BITS: log2 of the unit's rows.  A wave owns a contiguous share of the lines; its records are counted per row, then placed:
// the lanes of a batch of 64 that hold the same row find each other by ballots over the row's bits.  The list is put together
// in LDS (`list`; null: more lines than it holds) and leaves in whole vectors: entries stored where they belong one by one
// took 14 of the 22 us of the 27B-shaped pair's 576 units.
template <int BITS>
__device__ __forceinline__ void sort_unit(const GatherMember& M, const unsigned unit, int* smem, uint2* list) {
  constexpr int UR = 1 << BITS, NB = UR / 64 > 0 ? UR / 64 : 1;   // rows; rows a lane scans
  int* hist = smem;                                   // [wave][UR], then every wave's next place per row
  int* total = smem + kGsWaves * UR;                  // [UR]: all waves' records per row
  int* first_of = total + UR;                         // [UR + 1]: the rows' first places
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ax0 = int64_t(unit) * UR, gidx = ax0 / M.grp;
  const int lo = int(ax0 - gidx * M.grp);             // the unit's first row inside its group
  const float2* rec = M.rec + gidx * M.nlines;
  const int64_t share = ((M.nlines + kGsWaves - 1) / kGsWaves + 63) / 64 * 64;
  const int64_t l0 = wave * share, l1 = l0 + share < M.nlines ? l0 + share : M.nlines;
  int* mine = hist + wave * UR;

#pragma unroll
  for (int i = 0; i < NB; ++i) if (UR >= 64 || lane < UR) mine[i * 64 + lane] = 0;
  auto load = [&](float2 (&rc)[kGsFlight], int64_t at) {
#pragma unroll
    for (int u = 0; u < kGsFlight; ++u) {
      const int64_t line = at + 64 * u + lane;
      rc[u] = line < l1 ? rec[line] : make_float2(0.f, __int_as_float(-1));
    }
  };
  auto row_of = [&](float2 r) { const int i = __float_as_int(r.y); return i >= lo && i - lo < UR ? i - lo : -1; };
  float2 rc[kGsFlight];
  for (int64_t at = l0; at < l1; at += 64 * kGsFlight) {
    load(rc, at);
#pragma unroll
    for (int u = 0; u < kGsFlight; ++u) {
      const int r = row_of(rc[u]);
      if (r >= 0) atomicAdd(&mine[r], 1);
    }
  }
  __syncthreads();
  // the waves' counts per row into first places: per row over the waves, then over the rows
  for (int r = tid; r < UR; r += kGsThreads) {
    int s = 0;
#pragma unroll
    for (int w = 0; w < kGsWaves; ++w) {
      const int c = hist[w * UR + r];
      hist[w * UR + r] = s;
      s += c;
    }
    total[r] = s;
  }
  __syncthreads();
  if (wave == 0) {
    int carry = 0;
    int* start = M.start + int64_t(unit) * (UR + 1);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int c = UR >= 64 || lane < UR ? total[i * 64 + lane] : 0;
      int s = c;
#pragma unroll
      for (int o = 1; o < 64; o *= 2) {
        const int t = __shfl_up(s, o);
        if (lane >= o) s += t;
      }
      if (UR >= 64 || lane < UR) {
        first_of[i * 64 + lane] = carry + s - c;
        start[i * 64 + lane] = carry + s - c;
      }
      carry += __builtin_amdgcn_readlane(s, 63);
    }
    if (lane == 0) first_of[UR] = start[UR] = carry;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NB; ++i) if (UR >= 64 || lane < UR) mine[i * 64 + lane] += first_of[i * 64 + lane];
  __builtin_amdgcn_wave_barrier();
  uint2* sorted = M.sorted + int64_t(unit) * M.nlines;
  for (int64_t at = l0; at < l1; at += 64 * kGsFlight) {
    if (share > 64 * kGsFlight) load(rc, at);
#pragma unroll
    for (int u = 0; u < kGsFlight; ++u) {
      const int r = row_of(rc[u]);
      const uint64_t any = __ballot(r >= 0);
      if (!any) continue;                             // (uniform)
      uint32_t lo32 = uint32_t(any), hi32 = uint32_t(any >> 32);
#pragma unroll
      for (int bit = 0; bit < BITS; ++bit) {
        const uint32_t set = uint32_t(-((r >> bit) & 1));
        const uint64_t v = __ballot(set != 0);
        lo32 &= ~(uint32_t(v) ^ set);
        hi32 &= ~(uint32_t(v >> 32) ^ set);
      }
      if (r >= 0) {
        const int rank = __builtin_amdgcn_mbcnt_hi(hi32, __builtin_amdgcn_mbcnt_lo(lo32, 0u));
        const int place = mine[r] + rank;
        const uint2 e = make_uint2(uint32_t(r) << kGatherLineBits | uint32_t(at + 64 * u + lane), __float_as_uint(rc[u].x));
        if (list) list[place] = e;
        else sorted[place] = e;
        __builtin_amdgcn_wave_barrier();
        if (rank == 0) mine[r] = place + __popc(lo32) + __popc(hi32);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  if (list) {
    __syncthreads();
    const int n = first_of[UR];
    for (int i = tid; i < n; i += kGsThreads) sorted[i] = list[i];
  }
}

__global__ __launch_bounds__(kGsThreads, 6) void sort_records_kernel(const GatherArgs a) {
  extern __shared__ __align__(16) uint2 gsl[];        // [kGsList] if the members' lines fit
  __shared__ int smem[(kGsWaves + 2) * 256 + 1];
  __shared__ double red[5 * kGsWaves];
  unsigned id = blockIdx.x;
  // the losses (a chain of its own: first in the grid), the middle factor's parts, the units
  if (id == 0) {
    double m, s;
    reduce_losses_body<kGsThreads>(a.la, red, true, &m, &s);
    return;
  }
  if (--id < a.ntail) {
    build_mmid_body(a.va, int(id) / kMmidParts, int(id) % kMmidParts, kMmidParts);
    return;
  }
  id -= a.ntail;
  if (id < a.rho.ngroups) {
    // (what the gather takes its coefficients from; the addends' order: a thread's, the wave's, the waves')
    double acc = 0;
#pragma unroll 8
    for (int e = int(threadIdx.x); e < a.rho.G; e += kGsThreads) {
      const int64_t ax = int64_t(id) * a.rho.G + e;
      acc += a.rho.rho[((ax >> a.rho.lk) / a.rho.rep << a.rho.lk) + (ax & ((1 << a.rho.lk) - 1))];
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < kGsWaves; ++w) acc += red[w];
      a.rho.rG[id] = float(acc);
    }
    return;
  }
  id -= a.rho.ngroups;
  const int mi = id >= a.m[0].nunit ? 1 : 0;
  const GatherMember& M = a.m[mi];
  if (mi) id -= a.m[0].nunit;
  uint2* list = M.nlines <= kGsList ? gsl : nullptr;
  switch (M.unit_rows) {
    case 32: sort_unit<5>(M, id, smem, list); break;
    case 64: sort_unit<6>(M, id, smem, list); break;
    case 128: sort_unit<7>(M, id, smem, list); break;
    default: sort_unit<8>(M, id, smem, list); break;
  }
}

// ---------------------------------------------------------------------------------------------------
// lines gathered
// ---------------------------------------------------------------------------------------------------
__host__ __device__ constexpr int gather_row_floats(int K) { return K + 4; }   // (rows a few banks apart: read by columns, too)
__host__ __device__ constexpr size_t gather_lds(int K, int rows) {
  return (size_t(rows) * gather_row_floats(K) + size_t(kGgWaves) * K) * sizeof(float);
}

// a lane's inputs of a line, as they come from memory: K / 64 of them (blocks of 32: one, the upper lanes repeat the lower
// ones'); converted when they are used, so that a request does not wait for the one before it
template <int K> constexpr int lane_inputs() { return K / 64 > 0 ? K / 64 : 1; }
template <typename T> using GlobalPtr = const __attribute__((address_space(1))) T*;
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
template <int K, typename E> struct Raw;
template <int K> struct Raw<K, float> { typedef float V; V v; __device__ __forceinline__ float get(int) const { return v; } };
template <> struct Raw<128, float> { typedef floatx2 V; V v; __device__ __forceinline__ float get(int x) const { return v[x]; } };
template <> struct Raw<256, float> { typedef floatx4 V; V v; __device__ __forceinline__ float get(int x) const { return v[x]; } };
template <int K> struct Raw<K, uint16_t> { typedef uint16_t V; V v; __device__ __forceinline__ float get(int) const { return bf16_bits_to_f32(v); } };
template <> struct Raw<128, uint16_t> {
  typedef uint32_t V;
  V v;
  __device__ __forceinline__ float get(int x) const { return x ? bf16_hi_f32(v) : bf16_lo_f32(v); }
};
template <> struct Raw<256, uint16_t> {
  typedef uintx2 V;
  V v;
  __device__ __forceinline__ float get(int x) const { return x & 1 ? bf16_hi_f32(v[x / 2]) : bf16_lo_f32(v[x / 2]); }
};

// what an entry's value becomes: its coefficient in the gradient
struct CoefRule {
  float scale, t, mstar;                              // surrogate (t = 0): scale z; LogSumExp: sign(z) scale exp(t (|z| - mstar))
  __device__ __forceinline__ float operator()(float z) const {
    if (t == 0.f) return scale * z;
    const float e = __expf(t * (fabsf(z) - mstar)) * scale;
    return z < 0.f ? -e : e;
  }
};
// A wave's share [s0, s1) of the unit's list: runs of lines that belong to one row, each run's sum added to its row -- or,
// where a wave before this one began the row, left in `part` (the row is returned; -1: none).  e0: the workgroup's first entry.
// ONCE: no line is read by another unit as well.  Such lines pass the caches by: 9B-shaped pair 87 -> 81 us, Adam on the
// 2B-shaped pair 41.5 -> 35.5, and its loss pass, which then finds its own copy of the weights in the memory-side cache,
// 62 -> 57; blocks of 256 with groups of 64, whose lines four units read, 63 us from the caches, 82 past them.
template <int K, typename E, bool ONCE>
__device__ __forceinline__ int gather_share(const uint2* __restrict__ sorted, const int e0, const int s0, const int s1, const int j0,
                                            const uint64_t lines, const uint32_t stride, const uint32_t loff, float* tile,
                                            float* part, const int m0, const CoefRule rule) {
  constexpr int NX = lane_inputs<K>(), LDT = gather_row_floats(K);
  const int lane = threadIdx.x & 63;
  // (lanes past the share's end: its last line with a coefficient of zero)
  uint2 nx = sorted[s0 + lane < s1 ? s0 + lane : s1 - 1];
  int before = -1;                                    // the row of the entry before the batch
  if (s0 > e0) before = __builtin_amdgcn_readfirstlane(int(sorted[s0 - 1].x >> kGatherLineBits));
  int cur = __builtin_amdgcn_readfirstlane(int(nx.x >> kGatherLineBits));
  const int first = before == cur ? cur : -1;
  before = cur;
  float acc[NX];
#pragma unroll
  for (int x = 0; x < NX; ++x) acc[x] = 0.f;
  auto put = [&]() {
    float* t = (cur == first ? part : tile + (cur - j0) * LDT) + m0;
    const bool add = cur != first;
    if (K > 32 || lane < 32) {
#pragma unroll
      for (int x = 0; x < NX; ++x) t[x] = add ? t[x] + acc[x] : acc[x];
    }
#pragma unroll
    for (int x = 0; x < NX; ++x) acc[x] = 0.f;
  };
  for (int i0 = s0; i0 < s1; i0 += 64) {
    const int cnt = s1 - i0 < 64 ? s1 - i0 : 64;
    const uint2 e = nx;
    if (i0 + 64 < s1) nx = sorted[i0 + 64 + lane < s1 ? i0 + 64 + lane : s1 - 1];
    const uint64_t off = uint64_t(e.x & ((1u << kGatherLineBits) - 1u)) * stride;
    const uint32_t off_lo = uint32_t(off), off_hi = uint32_t(off >> 32);
    const float coef = lane < cnt ? rule(__uint_as_float(e.y)) : 0.f;
    const int row = int(e.x >> kGatherLineBits);
    int prev = __shfl_up(row, 1);
    if (lane == 0) prev = before;
    const uint64_t turn = __ballot(row != prev);      // entries that begin another row
    before = __builtin_amdgcn_readlane(row, 63);
    // eight lines at a time, the requests of RING of them ahead of their use
    constexpr int RING = gather_ring(K);
    Raw<K, E> v[RING][kGgFlight];
    auto request = [&](int grp) {
#pragma unroll
      for (int u = 0; u < kGgFlight; ++u) {
        // (a scalar base and the lane's offset, kept apart: no address to compute per lane)
        const int i = grp * kGgFlight + u;
        uint64_t at = lines + (uint64_t(uint32_t(__builtin_amdgcn_readlane(off_hi, i))) << 32 |
                               uint32_t(__builtin_amdgcn_readlane(off_lo, i)));
        uint32_t own = loff;
        asm("" : "+s"(at), "+v"(own));
        const auto src = reinterpret_cast<GlobalPtr<typename Raw<K, E>::V>>(reinterpret_cast<GlobalPtr<unsigned char>>(at) + own);
        if constexpr (ONCE) v[grp % RING][u].v = __builtin_nontemporal_load(src);
        else v[grp % RING][u].v = *src;
      }
    };
    auto consume = [&](int grp) {
      const uint32_t turns = __builtin_amdgcn_readfirstlane(uint32_t(turn >> (grp * kGgFlight)));
#pragma unroll
      for (int u = 0; u < kGgFlight; ++u) {
        const int i = grp * kGgFlight + u;
        if (turns >> u & 1) { put(); cur = __builtin_amdgcn_readlane(row, i); }
        const float c = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(coef), i));
#pragma unroll
        for (int x = 0; x < NX; ++x) acc[x] = fmaf(c, v[grp % RING][u].get(x), acc[x]);
      }
    };
#pragma unroll
    for (int g = 0; g < 64 / kGgFlight + RING - 1; ++g) {
      if (g * kGgFlight < cnt && g < 64 / kGgFlight) request(g);
      if (g >= RING - 1 && (g - RING + 1) * kGgFlight < cnt) consume(g - RING + 1);
    }
  }
  put();
  return first;
}

// Workgroup `id` of a member -> its block and which of the block's shares of rows.  Lines that several units read: the readers behind one L2
// (9B-shaped (V, O) pair, blocks of 256 and groups of 64 57 -> 41 us); lines that are read once spread over the chip as they come (blocks of 32,
// pair 2000 x 2048, the evaluation 55.7 us, behind one L2 57.2).
template <bool ONCE>
__device__ __forceinline__ void gather_place(unsigned id, unsigned per, unsigned total, int* b, int* share) {
  if constexpr (ONCE) {
    *b = int(id / per);
    *share = int(id % per);
  } else {
    block_and_part(id, per, total, b, share);
  }
}

// The products with S's zeros that the gather leaves out matter where a weight is infinite or not a number: there they are not
// numbers, in all rows of the block.  Such a weight spoils the member's sum of squared rounding errors -- every transformed
// value of its line and block is not a number -- which the launch before this one has reduced: a finite sum rules them out,
// and only otherwise are the block's lines read once more, whole.
// (The kernel's arguments are fetched anew, block and member worked out anew: kept until here -- the compiler would -- they take
// blocks of 256 from 94 registers to 97, i.e. a wave per SIMD.)
template <int K, bool ONCE>
__device__ __forceinline__ void spoiled_inputs(float* tile) {
  unsigned id = blockIdx.x;
  auto args = (const __attribute__((address_space(4))) GatherArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(id), "+s"(args));
  const auto& a = *args;
  const int mi = (a.nmem > 1 && id >= a.m[0].nwg) ? 1 : 0;
  if (fabsf(a.la.losses[a.loss_kind == kLossSur ? 1 : mi]) < INFINITY) return;   // (uniform)
  const auto& M = a.m[mi];
  int b, part;
  gather_place<ONCE>(mi ? id - a.m[0].nwg : id, unsigned(K / M.rows), M.nwg, &b, &part);
  const int m = int(threadIdx.x) % K;
  bool bad = false;
  for (int q = b * M.rep; q < (b + 1) * M.rep; ++q) {
    const int64_t ax = int64_t(q) * K + m, at = (ax >> 7) * M.seg_stride + (ax & 127);
#pragma unroll 1
    for (int64_t line = int(threadIdx.x) / K; line < M.nlines; line += kGgThreads / K) {
      const int64_t i = at + line * M.line_stride;
      const float w = M.bf16 ? bf16_bits_to_f32(static_cast<const uint16_t*>(M.W)[i]) : static_cast<const float*>(M.W)[i];
      bad |= !(fabsf(w) < INFINITY);
    }
  }
  if (bad)
    for (int r = 0; r < M.rows; ++r) tile[r * gather_row_floats(K) + m] = NAN;
  __syncthreads();
}

template <int K, bool ONCE>
__global__ __launch_bounds__(kGgThreads) void grad_gather_kernel(const GatherArgs a) {
  constexpr int NX = lane_inputs<K>(), LDT = gather_row_floats(K), LW = K / 4;
  extern __shared__ __align__(16) float gsm[];
  __shared__ int shared_row[kGgWaves];                // the row of `part`, -1: none
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned id = blockIdx.x;
  const int mi = (a.nmem > 1 && id >= a.m[0].nwg) ? 1 : 0;
  const GatherMember& M = a.m[mi];
  if (mi) id -= a.m[0].nwg;
  const int rows = M.rows, per = K / rows;
  int b, share;
  gather_place<ONCE>(id, unsigned(per), M.nwg, &b, &share);
  const int j0 = share * rows;                                                   // block, first row
  const int upb = K / M.unit_rows, u0 = j0 / M.unit_rows, r0 = j0 % M.unit_rows; // units per block, the rows' unit, first row in it
  float* tile = gsm;                                  // [rows][LDT]
  float* part = tile + rows * LDT + wave * K;         // [wave][K]: a share's first row, begun by a wave before
  for (int i = tid; i < rows * LDT; i += kGgThreads) tile[i] = 0.f;
  const int m0 = NX * (K == 32 ? lane & 31 : lane), es = M.bf16 ? 2 : 4;
  const uint32_t stride = uint32_t(M.line_stride) * uint32_t(es);
  // (within a line, the segment of 128 inputs matters for blocks of 256)
  const uint32_t loff = (uint32_t((m0 >> 7) * M.seg_stride) + uint32_t(m0 & 127)) * uint32_t(es);

  CoefRule rule{1.f, 0.f, 0.f};
  if (a.loss_kind == kLossLse) rule = CoefRule{float(1.0 / a.la.lse_ms[1]), a.lse_t, float(a.la.lse_ms[0])};
  for (int q = b * M.rep; q < (b + 1) * M.rep; ++q) {
    if (a.loss_kind == kLossSur) rule.scale = 2.f * a.beta * M.rG[(int64_t(q) * K + j0) / M.grp];
    const int64_t unit = int64_t(q) * upb + u0;
    const uint2* sorted = M.sorted + unit * M.nlines;
    const int* start = M.start + unit * (M.unit_rows + 1) + r0;
    const int e0 = start[0], n = start[rows] - e0;
    const int64_t aq = int64_t(q) * K;
    const uint64_t lines = reinterpret_cast<uint64_t>(M.W) + uint64_t((aq >> 7) * M.seg_stride + (aq & 127)) * es;
    const int s0 = e0 + int(int64_t(wave) * n / kGgWaves), s1 = e0 + int(int64_t(wave + 1) * n / kGgWaves);
    __syncthreads();                                  // (the tile is cleared; the row-block before is put together)
    int first = -1;
    if (s0 < s1)
      first = M.bf16 ? gather_share<K, uint16_t, ONCE>(sorted, e0, s0, s1, r0, lines, stride, loff, tile, part, m0, rule)
                     : gather_share<K, float, ONCE>(sorted, e0, s0, s1, r0, lines, stride, loff, tile, part, m0, rule);
    if (lane == 0) shared_row[wave] = first;
    __syncthreads();
    // rows that several waves share: the later waves' sums, in their order
    for (int m = tid; m < K; m += kGgThreads) {
#pragma unroll
      for (int w = 1; w < kGgWaves; ++w)
        if (shared_row[w] >= 0) tile[(shared_row[w] - r0) * LDT + m] += tile[rows * LDT + w * K + m];
    }
  }
  __syncthreads();
  spoiled_inputs<K, ONCE>(tile);
  float* dst = M.out + size_t(b) * K * K;
  if (M.transpose_out) {
    const int rq = rows / 4;
    for (int i = tid; i < K * rq; i += kGgThreads) {
      const int m = i / rq, r = 4 * (i % rq);
      const float* t = tile + r * LDT + m;
      *reinterpret_cast<float4*>(dst + size_t(m) * K + j0 + r) = make_float4(t[0], t[LDT], t[2 * LDT], t[3 * LDT]);
    }
  } else {
    for (int i = tid; i < rows * LW; i += kGgThreads) {
      const int r = i / LW, m = 4 * (i % LW);
      *reinterpret_cast<float4*>(dst + size_t(j0 + r) * K + m) = *reinterpret_cast<const float4*>(tile + r * LDT + m);
    }
  }
}

template <int K>
int launch_k(const GatherArgs& a, unsigned nwg, int rows, hipStream_t st) {
  const bool once = a.m[0].grp >= K && (a.nmem == 1 || a.m[1].grp >= K);
  if (once) hipLaunchKernelGGL((grad_gather_kernel<K, true>), dim3(nwg), dim3(kGgThreads), gather_lds(K, rows), st, a);
  else hipLaunchKernelGGL((grad_gather_kernel<K, false>), dim3(nwg), dim3(kGgThreads), gather_lds(K, rows), st, a);
  CAFEQ_CHECK_LAUNCH();
  return CAFEQ_OK;
}

}  // namespace

bool grad_gather_fits(int64_t nlines, int64_t line_stride, int64_t seg_stride, int dtype) {
  const int64_t es = dtype == CAFEQ_BF16 ? 2 : 4, most = int64_t(1) << 31;
  return nlines < (int64_t(1) << kGatherLineBits) && line_stride * es < most && seg_stride * es < most;
}
size_t grad_gather_entries(int K, int grp, int64_t naxis, int64_t nlines) {
  return size_t(naxis / std::min(K, grp)) * size_t(nlines);
}
size_t grad_gather_starts(int K, int grp, int64_t naxis) {
  const int ur = std::min(K, grp);
  return size_t(naxis / ur) * size_t(ur + 1);
}

int launch_grad_gather(int K, const GradGatherJob* jobs, int n, const LossArgs& la, const VArgs* va, hipStream_t st, const RhoGroups* rho) {
  if (n < 1 || n > 2 || !la.hdrA || !la.losses || (la.kind == kLossLse && !la.lse_ms)) return CAFEQ_ERR_INVALID_ARG;
  // rows per workgroup: three workgroups per compute unit keep the memory busy
  int64_t blocks = 0;
  for (int i = 0; i < n; ++i) blocks += jobs[i].nb;
  int rows = 32;
  while (rows > 4 && blocks * (K / rows) < 3 * int64_t(device_cu_count())) rows /= 2;
  GatherArgs a{};
  unsigned nwg = 0, nsort = 0;
  for (int i = 0; i < n; ++i) {
    const GradGatherJob& j = jobs[i];
    if (!j.W || !j.rec || !j.out || !j.sorted || !j.start || j.grp < 32 || j.grp % 32 != 0 || j.nb < 1 || j.rep < 1 || j.nlines < 1)
      return CAFEQ_ERR_INVALID_ARG;
    if ((j.grp < K ? K % j.grp : j.grp % K) != 0 || (la.kind == kLossSur && !j.rG)) return CAFEQ_ERR_INVALID_ARG;
    if (!grad_gather_fits(j.nlines, j.line_stride, j.seg_stride, j.dtype)) return CAFEQ_ERR_INVALID_ARG;
    GatherMember& m = a.m[i];
    m.W = j.W; m.bf16 = j.dtype == CAFEQ_BF16; m.line_stride = j.line_stride; m.seg_stride = j.seg_stride;
    m.rec = j.rec; m.rG = j.rG; m.out = j.out; m.sorted = j.sorted; m.start = j.start;
    m.nlines = j.nlines; m.grp = j.grp; m.rep = j.rep;
    m.unit_rows = std::min(K, j.grp); m.transpose_out = j.transpose_out; m.rows = rows;
    m.nunit = unsigned(j.nb) * unsigned(j.rep) * unsigned(K / m.unit_rows);
    m.nwg = unsigned(j.nb) * unsigned(K / rows);
    nwg += m.nwg;
    nsort += m.nunit;
  }
  a.nmem = n; a.loss_kind = la.kind; a.beta = la.beta; a.lse_t = la.t; a.la = la;
  if (va) {
    a.va = *va;
    a.ntail = unsigned(jobs[0].nb) * kMmidParts;
  }
  if (rho) a.rho = *rho;
  nsort += a.ntail + 1 + a.rho.ngroups;
  int64_t list = 0;
  for (int i = 0; i < n; ++i)
    if (jobs[i].nlines <= kGsList) list = std::max(list, jobs[i].nlines);
  hipLaunchKernelGGL(sort_records_kernel, dim3(nsort), dim3(kGsThreads), size_t(list) * sizeof(uint2), st, a);
  CAFEQ_CHECK_LAUNCH();
  switch (K) {
    case 32: return launch_k<32>(a, nwg, rows, st);
    case 64: return launch_k<64>(a, nwg, rows, st);
    case 128: return launch_k<128>(a, nwg, rows, st);
    case 256: return launch_k<256>(a, nwg, rows, st);
    default: return CAFEQ_ERR_UNSUPPORTED;
  }
}

}  // namespace cafeq
