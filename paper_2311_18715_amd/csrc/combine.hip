// Rollout / basis read-out: out[k] = U c_k for a block of coefficient
// columns, with U = S[:, :m] Q the logical basis (Q folded into the
// coefficients by the caller's coefficient kernel):
//     out[k*ldo + i] = sum_{j < m} S(i, j) * coefA[k*CMAX + j],
// S(i, j) stored at ((i/64)*ct + j)*64 + i%64 (64-row tiles).
// This is the O(N r) prediction of Sec. 2.3 (one read of the basis, one
// write per predicted state).
//
// As a product it is Out (K x n) = Coef (K x m) S^T (m x n) with a short
// contraction (m <= 72): 2 K n m flops against K n output writes.  It runs
// on the FP64 matrix cores (16x16x4): a wavefront takes 16 rows of one tile
// in the streaming pass's operand layout (lane l holds row l%16 of stored
// columns 4 kk + l/16, so one column of the unit is a 128-byte line for
// FP64) and multiplies them by 16-state blocks of coefficients staged in LDS
// in the operand layout; lane l then holds states 4 v + l/16 of the block
// at row l%16, so 16 lanes write 16 consecutive rows of one state.  The
// stored values convert exactly to FP64, the coefficients are FP64 and so
// are the sums; the output is rounded once, to its type.  A workgroup covers
// a contiguous share of the rows and 16 NS states; the stored columns are
// read once per 16 NS states.  FP32 states from FP32 or BF16 stored columns
// take the FP32 matrix cores instead (128-byte stores); a few states
// (K <= 4) take one row per lane.
//
// The products bound it as long as the writes merge; how they are made decides
// that.  A state's rows start at any multiple of the element size, so a
// wavefront's piece of a state is usually not whole 128-byte lines.  Streaming
// (nontemporal) stores send such pieces to memory as partial lines; ordinary
// ones merge neighbouring pieces in L2.  Only where every state starts on a
// line do streaming stores save time, and they are used only there.  Pieces
// merge when neighbours are written soon after each other, so few wavefronts
// write at a time: one workgroup per CU in all (two with streaming stores),
// each on a contiguous share of the rows.  The store addresses step by one
// 64-bit add each from an opaque start: left to itself the compiler held every
// state's address in registers (230 registers, two waves per SIMD, spills with
// the next unit's loads in flight).
// The whole read-out, kernel trace, 56 columns, us; "none" skips the stores:
//                                streaming  ordinary  none   before (streaming
//                                                            everywhere, two
//                                                            or more per CU)
//   500 FP64, n = 160,000 (lines)   192        212     180   219
//   500 FP64, n = 160,001           544        288     190   545
//   100 FP64, n = 160,001           112         57      54   114
//   100 FP32, n = 585,732           192        112     107   185
// and with two and three workgroups per CU, ordinary stores, 500 FP64 states
// at n = 160,001 337 and 338, 100 FP32 118 and 128.  The products of the first
// row run at 51 of 78.6 TFLOP/s, of the last at 78 of 157.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <map>
#include <mutex>

#include "odmd_internal.h"
#include "pass.h"
#include "storage.h"

namespace odmd {

typedef double d4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float to_float_value(float v) { return v; }
__device__ __forceinline__ float to_float_value(bf16 v) { return __uint_as_float((uint32_t)v.bits << 16); }

constexpr int CB_THREADS = 256;          // four wavefronts

// Wave-uniform base address of a unit's rows (scalar registers; each lane
// adds a constant 32-bit offset)
__device__ __forceinline__ gbytes uniform_base(const void* p) {
  const uint64_t b = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return (gbytes)(((uint64_t)hi << 32) | lo);
}

// Element at a byte address of global memory, by a streaming or an ordinary store
template <bool NT, typename TO>
__device__ __forceinline__ void put(uint64_t at, TO v) {
  typedef __attribute__((address_space(1))) TO* gptr;
  if constexpr (NT) __builtin_nontemporal_store(v, (gptr)at);
  else *(gptr)at = v;
}

// Workgroup bx of gx (a contiguous share of the 16-row units), states 16 NS by
// .. 16 NS (by + 1) - 1.  smem: combine_lds<RB, NS>() doubles.
template <int RB, int NS>
constexpr int combine_lds() { return NS * (RB / 4) * 64; }
template <typename TS, typename TO, int RB, int NS, bool NT>
__device__ __forceinline__ void combine_body(const CombineArgs& c, const int bx, const int gx, const int by,
                                             double* sC) {
  typedef Storage<TS> SC;
  constexpr int KK = RB / 4;                 // k-steps over the stored columns
  constexpr int NW = CB_THREADS / 64;
  typedef typename std::conditional<sizeof(TS) == 8, uint64_t, uint32_t>::type raw_t;
  const DevState* __restrict__ st = c.st;
  const int m = st->m;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int q = lane >> 4, l16 = lane & 15;
  const int k0 = by * (16 * NS);

  // coefficients of the workgroup's states in the A-operand layout: entry
  // [kk][s][lane] = coef(state k0 + 16 s + lane%16, column 4 kk + lane/16)
  for (int idx = threadIdx.x; idx < combine_lds<RB, NS>(); idx += CB_THREADS) {
    const int ln = idx & 63, s = (idx >> 6) % NS, kk = (idx >> 6) / NS;
    const int k = k0 + 16 * s + (ln & 15), col = 4 * kk + (ln >> 4);
    sC[idx] = (k < c.K && col < m) ? st->coefA[k * CMAX + col] : 0.0;
  }

  const int64_t units = (c.n + 15) / 16;
  const int64_t ub = (int64_t)bx * units / gx, ue = (int64_t)(bx + 1) * units / gx;
  const uint32_t loff = (uint32_t)((q * 64 + l16) * sizeof(TS));
  // 16-row units never straddle a tile; a k-step past the m live columns
  // re-reads the first (a cache hit; its coefficients are zero and stored
  // values are finite)
  auto load = [&](int64_t u, raw_t (&A)[KK]) {
    const gbytes base = uniform_base(static_cast<const TS*>(c.Us) + (u >> 2) * (int64_t)c.ct * 64 + 16 * (u & 3));
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      A[kk] = (raw_t)SC::row(base + (4 * kk < m ? kk : 0) * 256 * (int)sizeof(TS) + loff);
  };
  raw_t A[KK], An[KK];                       // the next unit's loads are in flight during the products
  int64_t u = ub + wave;
  load(u < ue ? u : ub, A);
  __syncthreads();
  const int full = min(NS, (c.K - k0) / 16); // blocks with 16 states
  for (; u < ue; u += NW) {
    load(u + NW < ue ? u + NW : u, An);
    // (opaque: the coefficients are read again for every unit, not held)
    int at = lane;
    asm volatile("" : "+v"(at));
    d4_t d[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) d[s] = d4_t{0.0, 0.0, 0.0, 0.0};
    // the NS accumulator chains are independent: k-steps outermost
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const double a = SC::to_double(SC::elem(A[kk], 0));
#pragma unroll
      for (int s = 0; s < NS; ++s)
        d[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(sC[(kk * NS + s) * 64 + at], a, d[s], 0, 0, 0);
    }
    const int64_t row = 16 * u + l16;
    if (row < c.n) {
      uint64_t p = reinterpret_cast<uint64_t>(static_cast<TO*>(c.out) + (int64_t)(k0 + q) * c.ldo + row);
      const uint64_t step = (uint64_t)c.ldo * 4 * sizeof(TO);
      asm volatile("" : "+v"(p));
#pragma unroll
      for (int e = 0; e < 4 * NS; ++e, p += step)
        if (e < 4 * full || k0 + 4 * e + q < c.K) put<NT>(p, (TO)d[e / 4][e % 4]);
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) A[kk] = An[kk];
  }
}

// FP32 states from FP32 or BF16 stored columns: the same product on the
// FP32 matrix cores (32x32x2, twice the FP64 rate), which also writes
// 128-byte pieces: a wavefront takes 32 consecutive rows of one tile
// (lane l supplies row l%32 of stored column 2 kk + l/32; 32 lanes read a
// 128-byte line of a column), and register r of lane l holds state
// 8 (r/4) + 4 (l/32) + r%4 of a 32-state block at row l%32, so 32 lanes
// write 32 consecutive rows of one state.  The stored values are exact in
// FP32; the coefficients are rounded to FP32 and the sums are FP32 (about
// m FP32 roundings per state against one for the FP64 path: the output is
// FP32 either way).  NS 32-state blocks per workgroup; with one block the
// k-steps alternate between two accumulators, so that two product chains
// are in flight.  smem: combine32_lds<RB, NS>() floats.
template <int RB, int NS>
constexpr int combine32_lds() { return NS * (RB / 2) * 64; }
template <typename TS, int RB, int NS, bool NT>
__device__ __forceinline__ void combine32_body(const CombineArgs& c, const int bx, const int gx, const int by,
                                               float* sC) {
  typedef Storage<TS> SC;
  constexpr int KK = RB / 2;                 // k-steps over the stored columns
  constexpr int NA = NS == 1 ? 2 : 1;        // accumulators per block
  constexpr int NW = CB_THREADS / 64;
  typedef float f16v __attribute__((ext_vector_type(16)));
  typedef typename std::conditional<sizeof(TS) == 4, uint32_t, uint16_t>::type raw_t;
  const DevState* __restrict__ st = c.st;
  const int m = st->m;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int h = lane >> 5, l32 = lane & 31;
  const int k0 = by * (32 * NS);

  // entry [kk][s][lane] = coef(state k0 + 32 s + lane%32, column 2 kk + lane/32)
  for (int idx = threadIdx.x; idx < combine32_lds<RB, NS>(); idx += CB_THREADS) {
    const int ln = idx & 63, s = (idx >> 6) % NS, kk = (idx >> 6) / NS;
    const int k = k0 + 32 * s + (ln & 31), col = 2 * kk + (ln >> 5);
    sC[idx] = (k < c.K && col < m) ? (float)st->coefA[k * CMAX + col] : 0.f;
  }

  const int64_t units = (c.n + 31) / 32;     // 32-row units (two per 64-row tile)
  const int64_t ub = (int64_t)bx * units / gx, ue = (int64_t)(bx + 1) * units / gx;
  const uint32_t loff = (uint32_t)((h * 64 + l32) * sizeof(TS));
  auto load = [&](int64_t u, raw_t (&B)[KK]) {
    const gbytes base = uniform_base(static_cast<const TS*>(c.Us) + (u >> 1) * (int64_t)c.ct * 64 + 32 * (u & 1));
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      B[kk] = (raw_t)SC::row(base + (2 * kk < m ? kk : 0) * 128 * (int)sizeof(TS) + loff);
  };
  raw_t B[KK], Bn[KK];
  int64_t u = ub + wave;
  load(u < ue ? u : ub, B);
  __syncthreads();
  const int full = min(NS, (c.K - k0) / 32); // blocks with 32 states
  for (; u < ue; u += NW) {
    load(u + NW < ue ? u + NW : u, Bn);
    int at = lane;
    asm volatile("" : "+v"(at));
    f16v d[NS][NA];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int a = 0; a < NA; ++a) d[s][a] = f16v{};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const float b = to_float_value(SC::elem(B[kk], 0));
#pragma unroll
      for (int s = 0; s < NS; ++s)
        d[s][kk % NA] = __builtin_amdgcn_mfma_f32_32x32x2f32(sC[(kk * NS + s) * 64 + at], b, d[s][kk % NA], 0, 0, 0);
    }
    if (NA == 2) d[0][0] += d[0][NA - 1];
    const int64_t row = 32 * u + l32;
    if (row < c.n) {
      uint64_t p = reinterpret_cast<uint64_t>(static_cast<float*>(c.out) + (int64_t)(k0 + 4 * h) * c.ldo + row);
      const uint64_t step = (uint64_t)c.ldo * sizeof(float);
      asm volatile("" : "+v"(p));
      // register r of a block: state 8 (r/4) + r%4 (+ 4 h)
#pragma unroll
      for (int e = 0; e < 16 * NS; ++e, p += e % 4 ? step : 5 * step)
        if (e < 16 * full || k0 + 8 * (e / 4) + e % 4 + 4 * h < c.K) put<NT>(p, d[e / 16][0][e % 16]);
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) B[kk] = Bn[kk];
  }
}

// A few states (a one-step prediction, Sec. 2.3's u(t + dt)): bound by the
// read of the stored columns, not by the flops.  One row per lane (a wave
// reads 64 consecutive rows of a column, one 64-row tile), the coefficients of
// each state uniform across the wave (scalar loads); the stored values are
// read once for all the states of the launch.  For FP32 and BF16 storage every
// column's load is issued before the first value is used, and without a test
// (a column past the m live ones re-reads column 0, a cache hit, against a
// zero coefficient; stored values are finite): with the load and its
// conversion under a test per column, each column waited for the one before.
// FP64, which needs no conversion, keeps the test (it skips the loads of a
// short bucket).  One state at n = 6M with 72 columns: FP32 929 -> 277 us, BF16
// 911 -> 143 us, FP64 558 us (6.2 TB/s).  Lanes of 8 bytes (two FP32, four BF16
// rows) were no faster for one state (279 and 156 us) and slower for more,
// each conversion made again for each state: four states of a BF16 basis of
// 72 columns, n = 6M 268 against 185 us, n = 20,000 33 against 19 us.
template <typename TS, typename TO, int RB>
__device__ __forceinline__ void combine_rows_body(const CombineArgs& c, const int64_t blk) {
  typedef Storage<TS> SC;
  typedef typename std::conditional<sizeof(TS) == 8, uint64_t, uint32_t>::type raw_t;
  const int m = c.st->m;
  const int64_t row = blk * CB_THREADS + threadIdx.x;
  if (row >= c.n) return;
  const gbytes T = (gbytes)(static_cast<const TS*>(c.Us) + (row >> 6) * (int64_t)c.ct * 64 + (row & 63));
  raw_t u[RB];
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    if constexpr (sizeof(TS) == 8) u[j] = j < m ? SC::row(T + j * 64 * (int)sizeof(TS)) : 0;
    else u[j] = (raw_t)SC::row(T + (j < m ? j : 0) * 64 * (int)sizeof(TS));
  }
  typedef const __attribute__((address_space(4))) double* cdp;
  cdp A = (cdp)c.st->coefA;
  TO* __restrict__ out = static_cast<TO*>(c.out);
  for (int k = 0; k < c.K; ++k) {
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < RB; ++j) acc = __builtin_fma(SC::to_double(SC::elem(u[j], 0)), A[k * CMAX + j], acc);
    out[(int64_t)k * c.ldo + row] = (TO)acc;
  }
}

enum { KIND_ROWS, KIND_FP64, KIND_FP32 };
template <int KIND, typename TS, typename TO, int RB, int NS, bool NT>
__device__ __forceinline__ void combine_block(const CombineArgs& c, int bx, int gx, int by) {
  if constexpr (KIND == KIND_ROWS) {
    combine_rows_body<TS, TO, RB>(c, bx);
  } else if constexpr (KIND == KIND_FP64) {
    __shared__ double smem[combine_lds<RB, NS>()];
    combine_body<TS, TO, RB, NS, NT>(c, bx, gx, by, smem);
  } else {
    __shared__ float smem[combine32_lds<RB, NS>()];
    combine32_body<TS, RB, NS, NT>(c, bx, gx, by, smem);
  }
}

template <int KIND, typename TS, typename TO, int RB, int NS, bool NT>
__global__ __launch_bounds__(CB_THREADS) void k_combine(CombineArgs c) {
  combine_block<KIND, TS, TO, RB, NS, NT>(c, blockIdx.x, gridDim.x, blockIdx.y);
}

// A few states of many streams in one launch: workgroup b belongs to the
// stream whose range from blk0 on holds b and does what workgroup b - blk0
// of that stream's own launch does.  One state of each of 256 FP32 streams
// of 1e4 to 1e6 rows: 4.4 ms with a launch each (8 us of reading and a start
// and an end for each), 2.1 ms in one per bucket.
template <typename TS, typename TO, int RB>
__global__ __launch_bounds__(CB_THREADS) void k_combine_few(const CombineDesc* __restrict__ d, int nd) {
  typedef const __attribute__((address_space(4))) CombineDesc* cdesc;
  cdesc D = (cdesc)d;
  const int b = blockIdx.x;
  int lo = 0, hi = nd - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (D[mid].blk0 <= b) lo = mid;
    else hi = mid - 1;
  }
  CombineArgs c{};
  c.st = D[lo].c.st;
  c.Us = D[lo].c.Us;
  c.out = D[lo].c.out;
  c.n = D[lo].c.n;
  c.ldo = D[lo].c.ldo;
  c.ct = D[lo].c.ct;
  c.K = D[lo].c.K;
  combine_rows_body<TS, TO, RB>(c, b - D[lo].blk0);
}

// Read-out class of a launch: the kernel and its states per workgroup.  A
// few states are read bound (rows); FP32 states of FP32 or BF16 columns go to
// the FP32 matrix cores in up to four 32-state blocks, the rest to the FP64
// ones in one, two, four or eight 16-state blocks: no more than a block of
// states is computed in vain, and a workgroup's accumulators fit its
// registers.  (More blocks per workgroup: more independent accumulator
// chains and fewer re-reads of the stored columns.)
struct CombineClass { int kind, ns, states; };   // states: per workgroup
static CombineClass combine_class(int basis, int out_f32, int K) {
  if (K <= COMBINE_FEW) return {KIND_ROWS, 1, K};
  if (out_f32 && basis != 0) {
    const int ns = std::min(4, (K + 31) / 32);
    return {KIND_FP32, ns, 32 * ns};
  }
  const int ns = K <= 16 ? 1 : (K <= 32 ? 2 : (K <= 64 ? 4 : 8));
  return {KIND_FP64, ns, 16 * ns};
}

static int cu_count() {
  static std::mutex mu;
  static std::map<int, int> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find(dev);
  if (it != cache.end()) return it->second;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) {
    (void)hipGetLastError();
    return 256;
  }
  return cache[dev] = cus;
}

int combine_few_blocks(int64_t n) { return (int)((n + CB_THREADS - 1) / CB_THREADS); }

// Grid of one read-out.  Rows: one thread per row.  Else one workgroup per CU
// in all (two with streaming stores; see the top of the file), shared by the
// launch's state blocks, with a unit per wavefront at least.  Up to 10 FP64
// states (16 with streaming stores) of many rows are read bound, not write
// bound, and want more loads in flight: one workgroup per CU and 32 units a
// wavefront, at most eight (5 states of 32 columns, n = 1,000,001: 65 us with
// one per CU, 52 with the two it gets; of 24 columns, n = 2,000,001: 123 and
// 97).  More of them cost smaller reads (5 of 56 columns, n = 400,001: 38.7 us
// with one, 44.4 with three) and ragged states beyond that count, which merge
// better from few writers (16 states of 32 columns, n = 5,000,001: a quarter
// less time with one than with eight).
// Workgroups go to the eight XCDs in turn by linear index x + g y; with g a
// multiple of 8 the state blocks of one row share run on the same XCD and read
// its stored columns through one L2.
static dim3 combine_grid(const CombineArgs& c, const CombineClass& k, bool nt) {
  if (k.kind == KIND_ROWS) return dim3((unsigned)combine_few_blocks(c.n), 1);
  const int waves = CB_THREADS / 64, ur = (k.kind == KIND_FP32 ? 32 : 16) * waves;
  const unsigned ys = (unsigned)((c.K + k.states - 1) / k.states);
  const int64_t most = (c.n + ur - 1) / ur;             // one unit a wavefront
  const int64_t cus = cu_count();
  int64_t per_cu = nt ? 2 : 1;
  if (k.kind == KIND_FP64 && (c.K <= 10 || (nt && c.K <= 16)))
    per_cu = std::max(per_cu, std::min<int64_t>(8, (most + 32 * cus - 1) / (32 * cus)));
  int64_t g = per_cu * cus;
  g = std::min<int64_t>(most, std::max<int64_t>(1, g / (int64_t)ys));
  if (ys > 1 && g > 8) g = g / 8 * 8;
  return dim3((unsigned)g, ys);
}

// every state starts on a 128-byte line
static bool whole_lines(const CombineArgs& c, int out_f32) {
  const int64_t es = out_f32 ? 4 : 8;
  return reinterpret_cast<uintptr_t>(c.out) % 128 == 0 && (c.K == 1 || c.ldo * es % 128 == 0);
}

template <int KIND, typename TS, typename TO, int NS, bool NT>
static hipError_t launch_rb(const CombineArgs& c, const dim3& grid, int rb, hipStream_t s) {
  switch (rb) {
#define ODMD_CASE(RB) \
  case RB: hipLaunchKernelGGL((k_combine<KIND, TS, TO, RB, NS, NT>), grid, dim3(CB_THREADS), 0, s, c); break;
    ODMD_CASE(8) ODMD_CASE(16) ODMD_CASE(24) ODMD_CASE(32) ODMD_CASE(40) ODMD_CASE(48)
    ODMD_CASE(56) ODMD_CASE(64) ODMD_CASE(72)
#undef ODMD_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename TS, typename TO, bool NT>
static hipError_t launch_t(const CombineArgs& c, int basis, int out_f32, int rb, hipStream_t s) {
  const CombineClass k = combine_class(basis, out_f32, c.K);
  const dim3 grid = combine_grid(c, k, NT);
  if (k.kind == KIND_ROWS) return launch_rb<KIND_ROWS, TS, TO, 1, false>(c, grid, rb, s);
  if constexpr (std::is_same<TO, float>::value && !std::is_same<TS, double>::value) {
    switch (k.ns) {
      case 1: return launch_rb<KIND_FP32, TS, TO, 1, NT>(c, grid, rb, s);
      case 2: return launch_rb<KIND_FP32, TS, TO, 2, NT>(c, grid, rb, s);
      case 3: return launch_rb<KIND_FP32, TS, TO, 3, NT>(c, grid, rb, s);
      default: return launch_rb<KIND_FP32, TS, TO, 4, NT>(c, grid, rb, s);
    }
  } else {
    switch (k.ns) {
      case 1: return launch_rb<KIND_FP64, TS, TO, 1, NT>(c, grid, rb, s);
      case 2: return launch_rb<KIND_FP64, TS, TO, 2, NT>(c, grid, rb, s);
      case 4: return launch_rb<KIND_FP64, TS, TO, 4, NT>(c, grid, rb, s);
      default: return launch_rb<KIND_FP64, TS, TO, 8, NT>(c, grid, rb, s);
    }
  }
}

hipError_t launch_combine(const CombineArgs& c, int basis, int out_f32, int rb, hipStream_t s) {
  const bool nt = whole_lines(c, out_f32);
  switch (2 * basis + (out_f32 ? 1 : 0)) {   // (an FP64 basis has FP64 states)
    case 0: return nt ? launch_t<double, double, true>(c, basis, 0, rb, s) : launch_t<double, double, false>(c, basis, 0, rb, s);
    case 2: return nt ? launch_t<float, double, true>(c, basis, 0, rb, s) : launch_t<float, double, false>(c, basis, 0, rb, s);
    case 3: return nt ? launch_t<float, float, true>(c, basis, 1, rb, s) : launch_t<float, float, false>(c, basis, 1, rb, s);
    case 4: return nt ? launch_t<bf16, double, true>(c, basis, 0, rb, s) : launch_t<bf16, double, false>(c, basis, 0, rb, s);
    case 5: return nt ? launch_t<bf16, float, true>(c, basis, 1, rb, s) : launch_t<bf16, float, false>(c, basis, 1, rb, s);
  }
  return hipErrorInvalidValue;
}

template <typename TS, typename TO>
static hipError_t launch_few(const CombineDesc* d, int nd, int nblocks, int rb, hipStream_t s) {
  switch (rb) {
#define ODMD_CASE(RB) \
  case RB: hipLaunchKernelGGL((k_combine_few<TS, TO, RB>), dim3(nblocks), dim3(CB_THREADS), 0, s, d, nd); break;
    ODMD_CASE(8) ODMD_CASE(16) ODMD_CASE(24) ODMD_CASE(32) ODMD_CASE(40) ODMD_CASE(48)
    ODMD_CASE(56) ODMD_CASE(64) ODMD_CASE(72)
#undef ODMD_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_combine_few(const CombineDesc* d, int nd, int nblocks, int basis, int out_f32, int rb,
                              hipStream_t s) {
  switch (2 * basis + (out_f32 ? 1 : 0)) {   // (an FP64 basis has FP64 states)
    case 0: return launch_few<double, double>(d, nd, nblocks, rb, s);
    case 2: return launch_few<float, double>(d, nd, nblocks, rb, s);
    case 3: return launch_few<float, float>(d, nd, nblocks, rb, s);
    case 4: return launch_few<bf16, double>(d, nd, nblocks, rb, s);
    case 5: return launch_few<bf16, float>(d, nd, nblocks, rb, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace odmd
