// Largest row norm per (batch, head): max_t ||x_t||_2 for x [BH, L, d].  The
// gate-aware skipping entry points bound every score s q.k by
// s ||q|| ||k||, and this kernel gives them ||k||'s maximum (or ||q||'s).
//
// A workgroup takes a chunk of rows; a group of d / 8 lanes (bf16) or d / 4
// lanes (fp32) reads one row with 16-byte loads (eight rows' loads are issued
// before their sums), the row sums are DPP butterflies, the groups reduce to
// the chunk's maximum in LDS, and the chunk maxima meet in an atomic maximum on
// the float's bit pattern (non-negative floats order like their bits).  The
// result is enlarged by 2^-10 relative so that it bounds the exact norm
// despite the fp32 rounding of the sum of squares.
#include "fox_device.h"
#include "fox_internal.h"

namespace fox {

// A workgroup takes kNormChunk rows, half as many where that leaves CUs idle; its passes
// are a chain of waits for memory, so it is as large as it gets (one or two passes).
// Smaller chunks for more workgroups do not pay: the chunk maxima of a head, and of its
// neighbours, meet in one cache line, whose atomics run one after the other (1024 of them
// took 17 us at B H = 16, L = 8192, more than reading the 33.5 MB).  Measured there, bf16
// at d = 128, 15.7 -> 8.8 us against 256 threads per 1024 rows; with 512 rows 8.9 us there,
// 28 against 24 at B H = 32, L = 16384, but 6.3 against 7.3 at B H = 2, L = 16384 (32
// workgroups).  bf16 at d = 64 loads 512 rows with four loads a lane group, not eight:
// B H = 2, L = 16384 5.3 -> 4.5 us, B H = 12, L = 2048 5.1 -> 4.3 (1024 rows 4.9 both).
// fp32 rows are twice as long, so a chunk has twice the passes, and where the chunks come
// near one per CU 256 threads, whose workgroups overlap, beat 1024 (us, 256 / 1024 threads,
// repeated on one buffer): d = 128, 192 chunks 18.2 / 19.3, 256 22.5 / 28.2, 512 41.6 / 49.0;
// d = 64, 256 chunks 13.7 / 14.7, 512 22.8 / 24.0; below, 144 chunks 15.7 / 15.1 and 9.3 /
// 8.2.  At d = 64 the fp32 loads are quick enough for the atomics of few heads to show (us,
// 512 / 1024 rows): B H = 12, L = 10240 10.5 / 7.3, B H = 4, L = 20480 8.6 / 6.9; alike at 72
// chunks (6.8 / 6.7), and with more heads 512 rows win (B H = 48, L = 2048 6.3 / 6.7).
constexpr int kNormThreads = 1024;
constexpr int kNormFewThreads = 256;
constexpr long long kNormFewChunks = 192;  // from which fp32 takes the few threads
constexpr int kNormChunk = 1024;
constexpr int kNormAhead = 8;

__global__ void zero_kernel(float* __restrict__ out, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = 0.0f;
}

template <typename Tt, int D, int ROWS, int THREADS>
__global__ __launch_bounds__(THREADS) void row_norm_max_kernel(const Tt* __restrict__ x,
                                                               float* __restrict__ out, int L,
                                                               int n_chunk) {
  constexpr int VEC = 16 / (int)sizeof(Tt);
  constexpr int LPR = D / VEC;                 // lanes per row
  constexpr int RPI = THREADS / LPR;      // rows per load
  // rows per lane group whose loads are in flight together, no more than the chunk has
  constexpr int AHEAD = ROWS / RPI < kNormAhead ? ROWS / RPI : kNormAhead;
  const int bh = blockIdx.x / n_chunk, chunk = blockIdx.x % n_chunk;
  const int tid = threadIdx.x, g = tid / LPR, lp = tid % LPR;
  const int r0 = chunk * ROWS, r1 = min(L, r0 + ROWS);
  const Tt* base = x + (size_t)bh * (size_t)L * D + lp * VEC;
  float best = 0.0f;
  for (int rb = r0 + g; rb < r1; rb += AHEAD * RPI) {
    float ss[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int r = min(rb + u * RPI, r1 - 1);  // rows past the chunk repeat its last row
      ss[u] = 0.0f;
      if constexpr (sizeof(Tt) == 2) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(base + (size_t)r * D);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss[u] += (float)v[e] * (float)v[e];
      } else {
        const f32x4 v = *reinterpret_cast<const f32x4*>(base + (size_t)r * D);
#pragma unroll
        for (int e = 0; e < 4; ++e) ss[u] += v[e] * v[e];
      }
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) best = fmaxf(best, row_sum<LPR>(ss[u]));
  }
  __shared__ float s_best[THREADS / 64];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) best = fmaxf(best, __shfl_xor(best, off));
  if ((tid & 63) == 0) s_best[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
    float m = 0.0f;
    for (int w = 0; w < THREADS / 64; ++w) m = fmaxf(m, s_best[w]);
    const float nrm = sqrtf(m) * (1.0f + 0x1p-10f);
    atomicMax(reinterpret_cast<unsigned int*>(out + bh), __float_as_uint(nrm));
  }
}

template <typename Tt, int ROWS, int THREADS>
static void row_norm_rows(const void* x, float* out, int BH, int L, int d, hipStream_t s) {
  const int n_chunk = (L + ROWS - 1) / ROWS;
  auto kern = d == 128 ? row_norm_max_kernel<Tt, 128, ROWS, THREADS>
                       : row_norm_max_kernel<Tt, 64, ROWS, THREADS>;
  // a part holds whole heads: the pointers advance
  launch_in_parts((unsigned)BH, (unsigned)(n_chunk * THREADS), [&](unsigned first, unsigned n) {
    hipLaunchKernelGGL(kern, dim3(n * (unsigned)n_chunk), dim3(THREADS), 0, s,
                       (const Tt*)x + (size_t)first * (size_t)L * d, out + first, L, n_chunk);
  });
}

template <typename Tt>
static void row_norm_t(const void* x, float* out, int BH, int L, int d, hipStream_t s) {
  const long long full = (long long)BH * ((L + kNormChunk - 1) / kNormChunk);
  if constexpr (sizeof(Tt) == 4) {
    if (full >= kNormFewChunks)
      return row_norm_rows<Tt, kNormChunk, kNormFewThreads>(x, out, BH, L, d, s);
  }
  const bool crowded = sizeof(Tt) == 4 && d == 64 && BH < 32 && full > 72;
  if (full >= 128 || crowded) row_norm_rows<Tt, kNormChunk, kNormThreads>(x, out, BH, L, d, s);
  else row_norm_rows<Tt, kNormChunk / 2, kNormThreads>(x, out, BH, L, d, s);
}

hipError_t launch_row_norm_max(bool bf16_, const void* x, float* out, int BH, int L, int d,
                               hipStream_t s) {
  hipLaunchKernelGGL(zero_kernel, dim3((BH + 255) / 256), dim3(256), 0, s, out, BH);
  if (bf16_) row_norm_t<bf16>(x, out, BH, L, d, s);
  else row_norm_t<float>(x, out, BH, L, d, s);
  return hipGetLastError();
}

}  // namespace fox
