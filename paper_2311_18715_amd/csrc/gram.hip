// Gram matrix of a BF16 basis just rewritten by a refold.
//
// A refold rewrites S[:, :r] <- S Q (Brand's deferred rotation, Sec. 2.3's
// update held as stored columns times a small matrix) and rounds the new
// columns to BF16.  Their rounding (about 2^-9 of each entry) leaves the
// stored columns S' = fl(S Q) measurably non-orthogonal (||S'^T S' - I||_F
// about 1e-3), and the method's small problems assume an orthonormal basis.
// This kernel forms M = S'^T S' (FP64 sums of exact BF16 products), from
// which the small-state kernel takes the orthonormal basis S' M^-1/2 and
// carries the model over to it, before the update of that step.
//
// Layout: S' in 64-row tiles, column-major inside a tile, so four
// consecutive rows of a column are 8 contiguous bytes: exactly the operand
// of one lane of the 16x16x16 BF16 matrix-core product, which contracts over
// 16 rows.  A wavefront takes a tile and, 16 rows (a unit) at a time and for
// every pair of 16-column blocks I <= J, adds S'_I^T S'_J of those rows (lane
// l supplies rows 4 (l/16) .. 4 (l/16) + 3 of column 16 I + l%16 for both
// operands); the FP32 block sums of a unit are added into FP64 accumulators.
// A workgroup sums its waves in a fixed order and writes one record per
// workgroup; the small-state kernel adds the records in index order, so the
// result is bitwise reproducible.  The kernel returns at once unless the
// pass of this update refolded (the host launches it after every pass of a
// BF16 stream; only the refold passes need it).
#include <hip/hip_runtime.h>

#include "odmd_internal.h"
#include "pass.h"
#include "xlane.h"

namespace odmd {

typedef short s4_t __attribute__((ext_vector_type(4)));
typedef short h8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr int GRAM_THREADS = 512;
constexpr int GRAM_LD = 72;     // rows of a column in LDS: 64 and padding

__device__ __forceinline__ void gram_body(const GramArgs& g, int wg) {
  const DevState* __restrict__ st = g.st;
  if (!st->refold) return;                   // uniform: no refold in this update's pass
  const int r = st->r;
  const int nb = (r + 15) / 16;              // 16-column blocks of the refolded columns
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, l16 = lane & 15;
  constexpr int NW = GRAM_THREADS / 64;

  double acc[GRAM_PAIRS][4];
#pragma unroll
  for (int p = 0; p < GRAM_PAIRS; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[p][v] = 0.0;

  const int64_t tiles = (g.n + 63) / 64;
  const int64_t t0 = (int64_t)wg * tiles / g.nwg, t1 = (int64_t)(wg + 1) * tiles / g.nwg;
  const uint16_t* __restrict__ Us = static_cast<const uint16_t*>(g.Us);
  // The operands of a load would be 32 bytes of 16 lines, and the lines, not
  // the bytes, are what a load costs (about five cycles each: 731 us at
  // n = 6M, r = 64 on 64 compute units).  A tile's columns are contiguous,
  // so a wave reads its tile 1 KB a load and turns it in LDS of its own,
  // columns GRAM_LD apart (reads of 16 columns fall in distinct banks): 345
  // us, then bound by the conversion and FP64 addition of every element of
  // every block sum.
  __shared__ __attribute__((aligned(16))) uint16_t smem[NW * 16 * GRAM_BLOCKS * GRAM_LD];
  static_assert(sizeof(smem) >= GRAM_REC * sizeof(double), "the record takes the tiles' place");
  uint16_t* sw = smem + wave * 16 * GRAM_BLOCKS * GRAM_LD;
  // columns 8 i + lane / 8, rows 8 (lane % 8) .. + 7 (the rows of the last
  // tile past n are zero, never written); columns past the blocks in use
  // re-read the first ones and are not used
  constexpr int NL = 2 * GRAM_BLOCKS;
  auto load_tile = [&](int64_t t, h8_t (&v)[NL]) {
    const uint16_t* T = Us + t * (int64_t)g.ct * 64 + 8 * lane;
#pragma unroll
    for (int i = 0; i < NL; ++i) v[i] = *reinterpret_cast<const h8_t*>(T + (i < 2 * nb ? i * 512 : 0));
  };
  h8_t next[NL];
  int64_t t = t0 + wave;
  if (t < t1) load_tile(t, next);
  for (; t < t1; t += NW) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      *reinterpret_cast<h8_t*>(sw + (8 * i + (lane >> 3)) * GRAM_LD + 8 * (lane & 7)) = next[i];
    wave_lds_fence();                        // other lanes read them
    load_tile(t + NW < t1 ? t + NW : t, next);   // under this tile's products
#pragma unroll
    for (int j = 0; j < 4; ++j) {            // sixteen rows at a time
      s4_t op[GRAM_BLOCKS];
#pragma unroll
      for (int I = 0; I < GRAM_BLOCKS; ++I)
        op[I] = *reinterpret_cast<const s4_t*>(sw + (16 * I + l16) * GRAM_LD + 16 * j + 4 * q);
      int p = 0;
#pragma unroll
      for (int I = 0; I < GRAM_BLOCKS; ++I)
#pragma unroll
        for (int J = I; J < GRAM_BLOCKS; ++J, ++p) {
          if (J < nb) {                      // uniform
            const f4_t d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(op[I], op[J], f4_t{0.f, 0.f, 0.f, 0.f},
                                                                    0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[p][v] += (double)d[v];
          }
        }
    }
    wave_lds_fence();                        // the next tile takes their place
  }
  // waves in index order into one LDS record, then the record to memory:
  // entry p * 256 + 4 lane + v is the (4 (lane/16) + v, lane%16) element of
  // block pair p (I <= J, row-major over I then J)
  double* red = reinterpret_cast<double*>(smem);
  __syncthreads();
  for (int w = 0; w < NW; ++w) {
    if (wave == w) {
#pragma unroll
      for (int p = 0; p < GRAM_PAIRS; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int e = p * 256 + 4 * lane + v;
          red[e] = (w == 0 ? 0.0 : red[e]) + acc[p][v];
        }
    }
    __syncthreads();
  }
  double* __restrict__ out = g.rec + (int64_t)wg * GRAM_REC;
  for (int e = threadIdx.x; e < GRAM_REC; e += GRAM_THREADS) out[e] = red[e];
}

__global__ __launch_bounds__(GRAM_THREADS) void k_gram(GramArgs g) { gram_body(g, blockIdx.x); }

// Many streams in one launch: workgroup b belongs to the stream whose
// range [blk0, blk0 + nwg) contains b (a device-resident table sorted by blk0).
__global__ __launch_bounds__(GRAM_THREADS) void k_gram_batch(const GramArgs* __restrict__ d, int nd) {
  const int b = blockIdx.x;
  int lo = 0, hi = nd - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (d[mid].blk0 <= b) lo = mid;
    else hi = mid - 1;
  }
  const GramArgs g = d[lo];
  gram_body(g, b - g.blk0);
}

hipError_t launch_gram(const GramArgs& g, hipStream_t s) {
  hipLaunchKernelGGL(k_gram, dim3(g.nwg), dim3(GRAM_THREADS), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gram_batch(const GramArgs* d, int nd, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(k_gram_batch, dim3(nblocks), dim3(GRAM_THREADS), 0, s, d, nd);
  return hipGetLastError();
}

}  // namespace odmd
