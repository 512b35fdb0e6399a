// Feature map phi(x) for rows of coordinates (Sec. 2.4, "Efficient
// Computation"): each output is a monomial's weight times the product of its
// indices' coordinates.  The kernel is bound by the HBM writes of the
// float32 output, D / d times the input.
//
// A workgroup takes kRows rows and kThreads consecutive features (one per
// thread); workgroups that write the same rows run on one XCD (see the tile
// remap).  Each thread reads its feature's generation-program word once (x
// offset of the last index, the first two other indices, a flag for more, the
// weight; table.hpp build_gen_program), so a row costs three LDS reads, three
// multiplies and one store.  The rows' coordinates sit in LDS transposed,
// [index][row] with a stride of kRows + 1 floats (distinct banks for distinct
// indices), plus an index d held at 1 for features of lower degree, so every
// read of a given index takes an immediate row offset.  Consecutive threads
// write consecutive features of a row.
//
// What sets the rate of the writes is how soon a workgroup gets to them and how
// compact the region is that the workgroups in flight write: with 32 rows x
// 256 features, each waited for d / 8 loads of coordinates, one after another,
// and then for its program word.  Now the word is fetched first, the
// coordinates kStage loads at a time, and 16 rows x 512 features make the runs
// of a row 2 KB: 65536 rows of d = 32, P = 4 (1.7 GB) take 285 us in place of
// 390 (6.0 TB/s; 256 threads 349, 1024 threads 276 but slower at D < 1000), 8192
// rows of d = 64 274 in place of 376, 262144 rows of d = 16 173 in place of 197.
// Slower: 8 rows (403 / 384 / 250 us), several feature blocks per workgroup
// (508 / 462 / 312), nontemporal stores, and 16-byte stores, for which a
// workgroup takes every fourth row (311 / 291 / 196).
#include <hip/hip_runtime.h>

#include "device_common.hpp"
#include "kernels.hpp"

namespace sata {

namespace {

// kRows: rows per workgroup; kThreads: features per workgroup; kStage: loads of
// coordinates that a thread keeps in flight.
template <typename T, int kRows, int kThreads, int kStage>
__global__ void __launch_bounds__(kThreads)
feature_map_kernel(const T* __restrict__ x, int64_t rows, int d, const uint32_t* __restrict__ gen,
                   const uint64_t* __restrict__ packed, int64_t D, float* __restrict__ phi) {
  constexpr int kXT = kRows + 1;  // LDS floats per coordinate index
  extern __shared__ float xt[];  // [d + 1][kXT]
  // workgroups are dealt to the 8 XCDs in turn by linear index; with more
  // than one feature block per row, the remap gives each XCD a contiguous run
  // of (row block, feature block) tiles, so that the neighbouring feature
  // blocks of a row, which share the cache lines at their edges, are written
  // through the same L2 (one feature block writes whole rows: no remap)
  int64_t rb = blockIdx.y, fb = 0;
  if (gridDim.x > 1) {
    const int64_t nblk = (int64_t)gridDim.x * gridDim.y;
    const int64_t lin = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t per_xcd = nblk / 8;
    const int64_t tile = lin < 8 * per_xcd ? (lin % 8) * per_xcd + lin / 8 : lin;
    rb = tile / gridDim.x;
    fb = tile % gridDim.x;
  }
  const int64_t r0 = rb * kRows;
  const int nr = (int)min<int64_t>(kRows, rows - r0);
  const int tid = threadIdx.x;
  const int64_t f = fb * kThreads + tid;
  const uint2 g = *(const uint2*)(gen + 2 * min(f, D - 1));
  const T* const xr = x + r0 * d;
  for (int i0 = tid; i0 < kRows * d; i0 += kStage * kThreads) {
    T c[kStage];
#pragma unroll
    for (int j = 0; j < kStage; ++j) {
      const int i = i0 + j * kThreads;
      c[j] = i < nr * d ? xr[i] : T{};
    }
#pragma unroll
    for (int j = 0; j < kStage; ++j) {
      const int i = i0 + j * kThreads, r = i / d;
      if (i < kRows * d) xt[(i - r * d) * kXT + r] = to_f32(c[j]);
    }
  }
  for (int r = tid; r < kRows; r += kThreads) xt[d * kXT + r] = 1.f;
  __syncthreads();
  if (f >= D) return;
  const uint32_t w0 = g.x;
  const float w = __uint_as_float(g.y);
  const float* const xl = xt + (int)((w0 & 0x3ffu) >> 2) * kXT;   // last index
  const float* const x0 = xt + (int)((w0 >> 10) & 0xffu) * kXT;   // first other index (or d)
  const float* const x1 = xt + (int)((w0 >> 18) & 0xffu) * kXT;   // second other index (or d)
  // degrees above 3: the further indices come from the packed entry
  uint64_t e = 0;
  int p = 0;
  if ((w0 >> 30) & 1u) {
    e = packed[f];
    p = (int)(e >> 56);
  }
  // all rows' reads first (rows past the end read zeros), then the further
  // factors of high degrees, then the stores
  float v[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) v[r] = w * x0[r] * x1[r] * xl[r];
  for (int j = 2; j < p - 1; ++j) {
    const float* const xj = xt + (int)((e >> (8 * j)) & 0xff) * kXT;
#pragma unroll
    for (int r = 0; r < kRows; ++r) v[r] *= xj[r];
  }
  float* const out = phi + r0 * D + f;
  if (nr == kRows) {
#pragma unroll
    for (int r = 0; r < kRows; ++r) out[(int64_t)r * D] = v[r];
  } else {
#pragma unroll
    for (int r = 0; r < kRows; ++r)
      if (r < nr) out[(int64_t)r * D] = v[r];
  }
}

template <typename T, int kRows, int kThreads, int kStage>
hipError_t launch_rows(const T* x, int64_t rows, const DevTable& t, float* phi, hipStream_t s) {
  const size_t lds = sizeof(float) * (size_t)(t.d + 1) * (kRows + 1);
  const int64_t fblocks = (t.D + kThreads - 1) / kThreads;
  const int64_t total_rb = (rows + kRows - 1) / kRows;
  // at most 65535 row blocks per launch (the grid's y extent)
  for (int64_t rb = 0; rb < total_rb; rb += 65535) {
    const int64_t nrb = std::min<int64_t>(65535, total_rb - rb);
    const int64_t r0 = rb * kRows;
    const int64_t nrows = std::min<int64_t>(rows - r0, nrb * kRows);
    hipLaunchKernelGGL((feature_map_kernel<T, kRows, kThreads, kStage>), dim3((unsigned)fblocks, (unsigned)nrb),
                       dim3(kThreads), lds, s, x + r0 * t.d, nrows, t.d, t.gen, t.packed, t.D, phi + r0 * t.D);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Rows of up to 256 features: one feature block writes whole rows, so a
// workgroup's region is contiguous whatever its rows, and more threads would
// idle past the row's end (10^6 rows of D = 45: 31 us, with 16 rows x 512
// features 70; 300,000 rows of D = 165: 32.6 both).  From 257 on the wider
// blocks win (200,000 rows of D = 325: 73 us against 54).
template <typename T>
hipError_t launch_typed(const T* x, int64_t rows, const DevTable& t, float* phi, hipStream_t s) {
  return t.D <= 256 ? launch_rows<T, 32, 256, 1>(x, rows, t, phi, s) : launch_rows<T, 16, 512, 2>(x, rows, t, phi, s);
}

}  // namespace

hipError_t launch_feature_map(const void* x, bool bf16, int64_t rows, const DevTable& t, float* phi,
                              hipStream_t s) {
  return bf16 ? launch_typed((const bf16_t*)x, rows, t, phi, s) : launch_typed((const float*)x, rows, t, phi, s);
}

}  // namespace sata
