// Forgetting Attention in fp32: forward (appendix, Alg. 1) and both halves of the
// backward (Alg. 2), on the fp32 matrix instruction v_mfma_f32_32x32x2_f32.
//
// The instruction multiplies and accumulates in fp32, so nothing is rounded to a
// shorter type: these kernels differ from a scalar fp32 loop only in the order of
// their sums.  It runs at twice the rate of the vector ALU's fma, and a tile's
// operands come from LDS once per 32 x 32 outputs.
//
// Shape, common to the three kernels.  A workgroup owns 32 rows (queries for the
// forward and dQ, keys for dK/dV) of one (batch, head); its waves share those rows
// and split the other axis: wave w takes the 32-row tiles w, w + NW, ... on its
// own, with a private slice of LDS for its two tiles, and the waves' partial
// results meet in LDS at the end.  So no wave waits for another inside the loop,
// a short sequence still fills the part (the longest chain is 1 / NW of the tiles),
// and the order of every sum is fixed.  Splitting instead the rows over the waves
// and sharing the tiles, as the bf16 kernels do, leaves 4 workgroups at
// B H = 2, L = 256 and chains of L / 32 tiles.
//     Measured (graph replay), against the kernels before, one lane per 32 dims on the
//     vector ALU with 128 or 64 rows and the whole key range per workgroup: B H = 24,
//     L = 1000, d = 64 forward / dK/dV / dQ 544 / 697 / 882 -> 45 / 77 / 59 us; B H = 2,
//     L = 256, d = 64 forward 128 -> 10 us.  At B H = 16, L = 8192, d = 64 the forward
//     reaches 118 TFLOP/s and dK/dV 131, of 157 the instruction can issue at 2.4 GHz
//     (a large fp32 library product reaches 153); what is left is the softmax between
//     the products, with two waves per SIMD to overlap it.
//   * Tiles move global -> LDS by DMA (16 bytes per lane, no registers; rows past L
//     read as zero).  Each tile's buffer is refilled as soon as its last reader of
//     the step is done, while the other tile is multiplied, so one buffer per tile
//     suffices and the waits count only the loads they need.
//   * A product contracts two elements per instruction, one per half-wave, and any
//     assignment of elements to steps serves if both operands use the same one.
//     Over the head dimension lane half h takes dims 8 s + 4 h .. + 3 of step group
//     s (one 16-byte LDS read per four instructions).  Over the rows of a tile it
//     takes the rows its accumulator registers hold (mfma_row), so P or dS feeds the
//     next product from the registers it was formed in, and the other operand is a
//     4-byte read of 32 consecutive floats per half.
//   * LDS rows keep their 16-byte chunks at chunk ^ f(row), f the row's low four
//     bits with bits 2 and 3 exchanged: 16 consecutive rows put one chunk in 16
//     different places (the 16-byte reads), and rows four apart use opposite halves
//     of the 64 banks (the 4-byte reads, whose half-waves read rows four apart).
//   * The gate bias c_i - c_j is formed in natural-log units before the change to
//     base 2, so the row maximum stays small and the logsumexp carries no
//     cancellation even when c changes by thousands within a block.
#include <algorithm>

#include "fox_device.h"
#include "fox_internal.h"

namespace fox {

constexpr int kF32Rows = 32;  // rows of a workgroup and of a tile
template <int D>
constexpr int f32_tile_bytes() { return kF32Rows * D * 4; }
template <int D>
constexpr int f32_tile_loads() { return f32_tile_bytes<D>() / 1024; }  // DMA loads of a wave
// More row blocks than this (2^31 lanes at 512 threads; a launch takes below 2^32) are
// walked by a loop.
constexpr long long kF32MaxGrid = 1LL << 22;

__device__ __forceinline__ f32x16 mfma32_f32(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__host__ __device__ constexpr int f32_swz(int r) {
  return (r & 3) | (((r >> 3) & 1) << 2) | (((r >> 2) & 1) << 3);
}

// Wait until at most N vector-memory operations of this wave are outstanding (the
// 6-bit count: low four bits, and two more above the LDS count's).
template <int N>
__device__ __forceinline__ void wait_vmem6() {
  static_assert(N >= 0 && N < 64, "vmcnt immediate");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Global byte offset, relative to a tile's first row, that this lane asks for in
// the tile's first DMA load (LDS position = lane); load i of 1 KB starts at row
// i * 256 / D, whose swizzle bits are disjoint from the lane's.
template <int D>
__device__ __forceinline__ uint32_t f32_dma_offset(int lane) {
  const int r = lane / (D / 4);
  return (uint32_t)(r * D * 4 + ((lane % (D / 4)) ^ f32_swz(r)) * 16);
}
template <int D>
__device__ __forceinline__ void f32_dma_tile(__amdgpu_buffer_rsrc_t rsrc, char* tile,
                                             uint32_t lane_off, int first_row) {
  const uint32_t base = (uint32_t)first_row * D * 4;
#pragma unroll
  for (int i = 0; i < f32_tile_loads<D>(); ++i)
    dma16(rsrc, tile + i * 1024,
          (lane_off ^ (uint32_t)(16 * f32_swz((i * 256 / D) & 15))) + uniform_u32(base + i * 1024));
}

// Per-lane LDS addresses of a tile's two kinds of operand reads (see above).
template <int D>
struct F32Reads {
  uint32_t row_at;  // dims 4 h .. + 3 of tile row col, swizzled
  uint32_t tr_at;   // row 4 h, dim col, swizzled
  __device__ F32Reads(const char* tile, int col, int h) {
    const uint32_t base = (uint32_t)(uintptr_t)lds_opaque(lds_ptr(tile));
    row_at = base + (uint32_t)(col * D * 4 + ((h ^ f32_swz(col & 15)) * 16));
    tr_at = base + (uint32_t)(4 * h * D * 4 + (((col >> 2) ^ (h << 3)) * 16) + (col & 3) * 4);
  }
  // dims 8 s + 4 h .. + 3 of row col
  __device__ f32x4 row(int s) const {
    return *(const lds_f32x4_t*)(const lds_byte*)(uintptr_t)(row_at ^ (uint32_t)(32 * s));
  }
  // dim col + 32 db of row mfma_row(r, h)
  __device__ float tr(int r, int db) const {
    const uint32_t x = 16u * (uint32_t)((8 * db) ^ f32_swz((r & 3) | ((r & 4) << 1)));
    return *(const lds_f32_t*)(const lds_byte*)(uintptr_t)(
        (tr_at ^ x) + (uint32_t)((8 * (r >> 2) + (r & 3)) * D * 4));
  }
};

// acc += X Y^T over the head dimension: X the tile (rows on the MFMA's rows), Y one
// row per lane in registers
template <int D>
__device__ __forceinline__ void f32_row_product(const F32Reads<D>& x, const f32x4 (&y)[D / 8],
                                                f32x16& acc) {
#pragma unroll
  for (int s = 0; s < D / 8; ++s) {
    const f32x4 a = x.row(s);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = mfma32_f32(a[e], y[s][e], acc);
  }
}
// acc[db] += X^T W over the tile's 32 rows: W the 16 registers of a product whose
// rows are the tile's
template <int D>
__device__ __forceinline__ void f32_tr_product(const F32Reads<D>& x, const float (&w)[16],
                                               f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int db = 0; db < D / 32; ++db) acc[db] = mfma32_f32(x.tr(r, db), w[r], acc[db]);
}

template <int D>
__device__ __forceinline__ void f32_load_row(const float* p, bool ok, int h, f32x4 (&y)[D / 8]) {
#pragma unroll
  for (int s = 0; s < D / 8; ++s)
    y[s] = ok ? *reinterpret_cast<const f32x4*>(p + 8 * s + 4 * h) : f32x4{0.f, 0.f, 0.f, 0.f};
}

// A wave's partial result acc (X^T: dims on MFMA rows, one of 32 rows per lane) as
// [32][D] floats in its LDS slice, 16-byte chunks swizzled by the row.
template <int D>
__device__ __forceinline__ void f32_put_partial(char* slice, const f32x16 (&acc)[D / 32], int col,
                                                int h) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 v;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) v[jj] = acc[db][4 * g + jj];
      *reinterpret_cast<f32x4*>(slice + col * D * 4 +
                                (((8 * db + 2 * g + h) ^ (col & 15)) * 16)) = v;
    }
}
template <int D>
__device__ __forceinline__ f32x4 f32_get_partial(const char* slice, int row, int chunk) {
  return *reinterpret_cast<const f32x4*>(slice + row * D * 4 + ((chunk ^ (row & 15)) * 16));
}

// ---------------------------------------------------------------------------
// Forward.
// ---------------------------------------------------------------------------
template <int D, int NW>
struct F32FwdSmem {
  alignas(1024) char tile[NW][2][f32_tile_bytes<D>()];  // a wave's K and V, then its O partial
  float c[NW][64];
  float m[NW][32], l[NW][32];
};

template <int D, bool FIXED, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1)))
void fwd_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                    const float* __restrict__ V, const float* __restrict__ gate,
                    float* __restrict__ O, float* __restrict__ LSE, int BH, int H, int L,
                    int n_blk, float scale_log2) {
  constexpr int NL = f32_tile_loads<D>();
  constexpr int NVC = NL + (FIXED ? 0 : 1);  // loads of a V tile and its prefix values
  __shared__ F32FwdSmem<D, NW> sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, col = lane & 31;
  const uint32_t dma_off = f32_dma_offset<D>(lane);
  const F32Reads<D> kt(sm.tile[wave][0], col, h), vt(sm.tile[wave][1], col, h);
  const lds_byte* c_at = lds_opaque(lds_ptr(&sm.c[wave][4 * h]));
  const long long n_all = (long long)n_blk * BH;

  for (long long blk = blockIdx.x; blk < n_all; blk += gridDim.x) {
    const int bh = (int)(blk % BH);
    const int mb = n_blk - 1 - (int)(blk / BH);  // longest rows first
    const size_t head = (size_t)bh * (size_t)L;
    const int q0 = mb * 32;
    const int qi = q0 + col;
    const bool q_valid = qi < L;
    const GateRow<FIXED> gr(gate, bh, H, head);
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(K + head * D, (uint32_t)L * D * 4);
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(V + head * D, (uint32_t)L * D * 4);
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(FIXED ? K : gate + head, (uint32_t)L * 4);

    f32x4 qf[D / 8];
    f32_load_row<D>(Q + (head + qi) * D, q_valid, h, qf);
    const float c_q0 = gr.raw(q0);
    const float cq = q_valid ? gr.diff(qi, q0) : 0.0f;
    f32x16 oacc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) oacc[db] = f32x16{};
    float m = -INFINITY, l = 0.0f;

    const int n_tiles = mb + 1;  // the last one holds the diagonal
    auto issue_k = [&](int j) { f32_dma_tile<D>(rk, sm.tile[wave][0], dma_off, 32 * j); };
    auto issue_vc = [&](int j) {
      f32_dma_tile<D>(rv, sm.tile[wave][1], dma_off, 32 * j);
      if constexpr (!FIXED) dma4(rc, &sm.c[wave][0], (uint32_t)(32 * j + lane) * 4);
    };
    if (wave < n_tiles) {
      issue_k(wave);
      issue_vc(wave);
    }
    for (int j = wave; j < n_tiles; j += NW) {
      const bool more = j + NW < n_tiles;
      wait_vmem6<NVC>();  // K of tile j
      f32x16 s = {};
      f32_row_product<D>(kt, qf, s);
      sched_fence();  // every read of the K tile is done
      if (more) {
        issue_k(j + NW);
        wait_vmem6<NL>();  // V and c of tile j
      } else {
        wait_vmem6<0>();
      }
      float p[16];
      float mt = -INFINITY;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 c4 = FIXED ? f32x4{} : *(const lds_f32x4_t*)(c_at + 32 * g);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int key = 32 * j + 8 * g + 4 * h + jj;
          float x = s[4 * g + jj] * scale_log2 +
                    (cq - gr.diff_raw(key, c4[jj], q0, c_q0)) * kLog2e;
          if (j == mb && key > qi) x = -INFINITY;
          p[4 * g + jj] = x;
          mt = fmaxf(mt, x);
        }
      }
      // -inf only where every score so far overflowed: a finite reference keeps the
      // exponents free of (-inf) - (-inf)
      const float m_new = fmaxf(m, wave_max_pair(mt));
      const float m_ref = m_new == -INFINITY ? 0.0f : m_new;
      const float alpha = exp2_fast(m - m_ref);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) oacc[db] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[r] = exp2_fast(p[r] - m_ref);
        l += p[r];
      }
      f32_tr_product<D>(vt, p, oacc);
      sched_fence();  // every read of the V tile and of c is done
      if (more) issue_vc(j + NW);
    }

    // merge the waves' partials: O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w
    f32_put_partial<D>(sm.tile[wave][0], oacc, col, h);
    const float l_wave = wave_sum_pair(l);
    if (h == 0) {
      sm.m[wave][col] = m;
      sm.l[wave][col] = l_wave;
    }
    __syncthreads();
    for (int item = tid; item < 32 * (D / 4); item += 64 * NW) {
      const int q = item / (D / 4), chunk = item % (D / 4);
      float M = sm.m[0][q];
#pragma unroll
      for (int w = 1; w < NW; ++w) M = fmaxf(M, sm.m[w][q]);
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
      float lt = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = exp2_fast(sm.m[w][q] - M);
        o += f * f32_get_partial<D>(sm.tile[w][0], q, chunk);
        lt += f * sm.l[w][q];
      }
      if (q0 + q < L) {
        *reinterpret_cast<f32x4*>(O + (head + q0 + q) * D + 4 * chunk) = o * (1.0f / lt);
        if (chunk == 0) LSE[head + q0 + q] = kLn2 * (M + log2f(lt));
      }
    }
    if (n_all > gridDim.x) __syncthreads();  // the next block reuses the slices
  }
}

// ---------------------------------------------------------------------------
// dQ and dc^q: query-stationary, dQ^T += K^T dS^T with dS^T = P^T o (V dO^T - Delta).
// ---------------------------------------------------------------------------
template <int D, int NW>
struct F32DqSmem {
  alignas(1024) char tile[NW][2][f32_tile_bytes<D>()];  // a wave's K and V, then its dQ partial
  float c[NW][64];
  float dc[NW][32];
};

template <int D, bool FIXED, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1)))
void bwd_dq_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                       const float* __restrict__ V, const float* __restrict__ gate,
                       const float* __restrict__ LSE, const float* __restrict__ dO,
                       const float* __restrict__ delta, float* __restrict__ dQ,
                       float* __restrict__ dcq, int BH, int H, int L, int n_blk, float scale,
                       float scale_log2) {
  constexpr int NL = f32_tile_loads<D>();
  __shared__ F32DqSmem<D, NW> sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, col = lane & 31;
  const uint32_t dma_off = f32_dma_offset<D>(lane);
  const F32Reads<D> kt(sm.tile[wave][0], col, h), vt(sm.tile[wave][1], col, h);
  const lds_byte* c_at = lds_opaque(lds_ptr(&sm.c[wave][4 * h]));
  const long long n_all = (long long)n_blk * BH;

  for (long long blk = blockIdx.x; blk < n_all; blk += gridDim.x) {
    const int bh = (int)(blk % BH);
    const int mb = n_blk - 1 - (int)(blk / BH);
    const size_t head = (size_t)bh * (size_t)L;
    const int q0 = mb * 32;
    const int qi = q0 + col;
    const bool q_valid = qi < L;
    const GateRow<FIXED> gr(gate, bh, H, head);
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(K + head * D, (uint32_t)L * D * 4);
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(V + head * D, (uint32_t)L * D * 4);
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(FIXED ? K : gate + head, (uint32_t)L * 4);

    f32x4 qf[D / 8], gf[D / 8];
    f32_load_row<D>(Q + (head + qi) * D, q_valid, h, qf);
    f32_load_row<D>(dO + (head + qi) * D, q_valid, h, gf);
    const float c_q0 = gr.raw(q0);
    const float cq = q_valid ? gr.diff(qi, q0) : 0.0f;
    const float lq = q_valid ? LSE[head + qi] : INFINITY;
    const float dlt = q_valid ? delta[head + qi] : 0.0f;
    f32x16 acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) acc[db] = f32x16{};
    float dc = 0.0f;

    const int n_tiles = mb + 1;  // the last one holds the diagonal
    auto issue_vc = [&](int j) {
      f32_dma_tile<D>(rv, sm.tile[wave][1], dma_off, 32 * j);
      if constexpr (!FIXED) dma4(rc, &sm.c[wave][0], (uint32_t)(32 * j + lane) * 4);
    };
    auto issue_k = [&](int j) { f32_dma_tile<D>(rk, sm.tile[wave][0], dma_off, 32 * j); };
    if (wave < n_tiles) {
      issue_vc(wave);
      issue_k(wave);
    }
    for (int j = wave; j < n_tiles; j += NW) {
      const bool more = j + NW < n_tiles;
      wait_vmem6<NL>();  // V and c of tile j; its K may still load
      f32x16 dp = {};
      f32_row_product<D>(vt, gf, dp);
      float ck[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 c4 = FIXED ? f32x4{} : *(const lds_f32x4_t*)(c_at + 32 * g);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          ck[4 * g + jj] = gr.diff_raw(32 * j + 8 * g + 4 * h + jj, c4[jj], q0, c_q0);
      }
      wait_lds();     // the prefix values are in registers
      sched_fence();  // every read of the V tile is done
      if (more) {
        issue_vc(j + NW);
        wait_vmem6<NL + (FIXED ? 0 : 1)>();  // K of tile j
      } else {
        wait_vmem6<0>();
      }
      f32x16 s = {};
      f32_row_product<D>(kt, qf, s);
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float p = exp2_fast(s[r] * scale_log2 + ((cq - ck[r]) - lq) * kLog2e);
        if (j >= mb && 32 * j + mfma_row(r, h) > qi) p = 0.0f;
        ds[r] = p * (dp[r] - dlt);
        dc += ds[r];
      }
      f32_tr_product<D>(kt, ds, acc);
      sched_fence();  // every read of the K tile is done
      if (more) issue_k(j + NW);
    }

    f32_put_partial<D>(sm.tile[wave][0], acc, col, h);
    const float dct = wave_sum_pair(dc);
    if (h == 0) sm.dc[wave][col] = dct;
    __syncthreads();
    for (int item = tid; item < 32 * (D / 4); item += 64 * NW) {
      const int q = item / (D / 4), chunk = item % (D / 4);
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
      float dt = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        o += f32_get_partial<D>(sm.tile[w][0], q, chunk);
        dt += sm.dc[w][q];
      }
      if (q0 + q < L) {
        *reinterpret_cast<f32x4*>(dQ + (head + q0 + q) * D + 4 * chunk) = o * scale;
        if (chunk == 0) dcq[head + q0 + q] = dt;
      }
    }
    if (n_all > gridDim.x) __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// dK, dV and dc^k: key-stationary; a wave's tiles hold 32 queries' Q and dO.
// ---------------------------------------------------------------------------
template <int D, int NW>
struct F32KvSmem {
  alignas(1024) char tile[NW][2][f32_tile_bytes<D>()];  // a wave's Q and dO, then dK and dV partials
  float row[NW][3][64];                                  // c_i, LSE_i, Delta_i of the tile's queries
  float dc[NW][32];
};

template <int D, bool FIXED, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1)))
void bwd_dkdv_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                         const float* __restrict__ V, const float* __restrict__ gate,
                         const float* __restrict__ LSE, const float* __restrict__ dO,
                         const float* __restrict__ delta, float* __restrict__ dK,
                         float* __restrict__ dV, float* __restrict__ dck, int BH, int H, int L,
                         int n_blk, float scale, float scale_log2) {
  constexpr int NL = f32_tile_loads<D>();
  __shared__ F32KvSmem<D, NW> sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, col = lane & 31;
  const uint32_t dma_off = f32_dma_offset<D>(lane);
  const F32Reads<D> qt(sm.tile[wave][0], col, h), gt(sm.tile[wave][1], col, h);
  const lds_byte* row_at = lds_opaque(lds_ptr(&sm.row[wave][0][4 * h]));
  const long long n_all = (long long)n_blk * BH;

  for (long long blk = blockIdx.x; blk < n_all; blk += gridDim.x) {
    const int bh = (int)(blk % BH);
    const int kb = (int)(blk / BH);  // key block 0 has the most work: first
    const size_t head = (size_t)bh * (size_t)L;
    const int k0 = kb * 32;
    const int kj = k0 + col;
    const bool k_valid = kj < L;
    const GateRow<FIXED> gr(gate, bh, H, head);
    const __amdgpu_buffer_rsrc_t rq = make_rsrc(Q + head * D, (uint32_t)L * D * 4);
    const __amdgpu_buffer_rsrc_t rg = make_rsrc(dO + head * D, (uint32_t)L * D * 4);
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(FIXED ? Q : gate + head, (uint32_t)L * 4);
    const __amdgpu_buffer_rsrc_t rl = make_rsrc(LSE + head, (uint32_t)L * 4);
    const __amdgpu_buffer_rsrc_t rd = make_rsrc(delta + head, (uint32_t)L * 4);

    f32x4 kf[D / 8], vf[D / 8];
    f32_load_row<D>(K + (head + kj) * D, k_valid, h, kf);
    f32_load_row<D>(V + (head + kj) * D, k_valid, h, vf);
    const float c_k0 = gr.raw(k0);
    const float ck = k_valid ? gr.diff(kj, k0) : 0.0f;
    f32x16 ak[D / 32], av[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) ak[db] = av[db] = f32x16{};
    float dc = 0.0f;

    const int n_tiles = (L + 31) / 32;
    auto issue_q = [&](int j) {
      f32_dma_tile<D>(rq, sm.tile[wave][0], dma_off, 32 * j);
      const uint32_t off = (uint32_t)(32 * j + lane) * 4;
      if constexpr (!FIXED) dma4(rc, &sm.row[wave][0][0], off);
      dma4(rl, &sm.row[wave][1][0], off);
      dma4(rd, &sm.row[wave][2][0], off);
    };
    auto issue_g = [&](int j) { f32_dma_tile<D>(rg, sm.tile[wave][1], dma_off, 32 * j); };
    if (kb + wave < n_tiles) {
      issue_q(kb + wave);
      issue_g(kb + wave);
    }
    for (int j = kb + wave; j < n_tiles; j += NW) {
      const bool more = j + NW < n_tiles;
      wait_vmem6<NL>();  // Q and the row statistics of tile j; its dO may still load
      f32x16 s = {};
      f32_row_product<D>(qt, kf, s);
      wait_vmem6<0>();  // dO of tile j
      f32x16 dp = {};
      f32_row_product<D>(gt, vf, dp);
      float p[16], ds[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 c4 = FIXED ? f32x4{} : *(const lds_f32x4_t*)(row_at + 32 * g);
        const f32x4 l4 = *(const lds_f32x4_t*)(row_at + 256 + 32 * g);
        const f32x4 d4 = *(const lds_f32x4_t*)(row_at + 512 + 32 * g);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int r = 4 * g + jj, qq = 32 * j + 8 * g + 4 * h + jj;
          const float cq = gr.diff_raw(qq, c4[jj], k0, c_k0);
          p[r] = exp2_fast(s[r] * scale_log2 + ((cq - ck) - l4[jj]) * kLog2e);
          p[r] = qq >= kj && qq < L ? p[r] : 0.0f;
          ds[r] = p[r] * (dp[r] - d4[jj]);
          dc -= ds[r];
        }
      }
      f32_tr_product<D>(qt, ds, ak);
      sched_fence();  // every read of the Q tile and of the row statistics is done
      if (more) issue_q(j + NW);
      f32_tr_product<D>(gt, p, av);
      sched_fence();  // every read of the dO tile is done
      if (more) issue_g(j + NW);
    }

    f32_put_partial<D>(sm.tile[wave][0], ak, col, h);
    f32_put_partial<D>(sm.tile[wave][1], av, col, h);
    const float dct = wave_sum_pair(dc);
    if (h == 0) sm.dc[wave][col] = dct;
    __syncthreads();
    for (int item = tid; item < 32 * (D / 4); item += 64 * NW) {
      const int kr = item / (D / 4), chunk = item % (D / 4);
      f32x4 ok = {0.f, 0.f, 0.f, 0.f}, ov = ok;
      float dt = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        ok += f32_get_partial<D>(sm.tile[w][0], kr, chunk);
        ov += f32_get_partial<D>(sm.tile[w][1], kr, chunk);
        dt += sm.dc[w][kr];
      }
      if (k0 + kr < L) {
        *reinterpret_cast<f32x4*>(dK + (head + k0 + kr) * D + 4 * chunk) = ok * scale;
        *reinterpret_cast<f32x4*>(dV + (head + k0 + kr) * D + 4 * chunk) = ov;
        if (chunk == 0) dck[head + k0 + kr] = dt;
      }
    }
    if (n_all > gridDim.x) __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static dim3 f32_grid(int n_blk, int BH) {
  return dim3((unsigned)std::min<long long>((long long)n_blk * BH, kF32MaxGrid));
}

// Waves per workgroup: the most whose tiles fit the LDS (8 at D = 64, 4 at D = 128),
// or half as many with two workgroups per CU.  The finer split halves the longest
// chain, the coarser one rounds a row block's tiles up less and merges half as many
// partials.  With up to two workgroups per CU the chain decides, with more the rest:
// forward / dK/dV / dQ in microseconds, fine against coarse, at B H = 12, L = 1000
// (384 workgroups) 27 / 47 / 36 against 33 / 56 / 44 at D = 64 and 48 / 84 / 66
// against 85 / 154 / 120 at D = 128; at B H = 24, L = 1000 (768) 46 / 80 / 62 against
// 45 / 77 / 59 and 87 / 154 / 121 against 87 / 156 / 122; at B H = 32, L = 2048 (2048)
// 187 / 332 / 258 against 168 / 292 / 227 and 375 / 677 / 527 against 342 / 626 / 485.
// Rows the coarser split already gives one tile per wave gain nothing from the finer.
constexpr long long kF32FineGroups = 512;
template <int D>
constexpr int kF32Nw = D == 64 ? 8 : 4;
template <int D>
static bool f32_fine(int n_blk, int BH) {
  return n_blk > kF32Nw<D> / 2 && (long long)n_blk * BH <= kF32FineGroups;
}

template <int D, bool FIXED, int NW>
static void fwd_f32_t(const float* q, const float* k, const float* v, GateSpec g, float* o,
                      float* lse, int BH, int L, float sl2, hipStream_t s) {
  const int n = (L + 31) / 32;
  if constexpr (NW == kF32Nw<D>)
    if (!f32_fine<D>(n, BH))
      return fwd_f32_t<D, FIXED, NW / 2>(q, k, v, g, o, lse, BH, L, sl2, s);
  hipLaunchKernelGGL((fwd_f32_kernel<D, FIXED, NW>), f32_grid(n, BH), dim3(64 * NW), 0, s, q, k, v,
                     g.ptr, o, lse, BH, g.H, L, n, sl2);
}

hipError_t launch_fwd_f32(const float* q, const float* k, const float* v, GateSpec g, float* o,
                          float* lse, int BH, int L, int d, float scale, hipStream_t s) {
  const float sl2 = scale * kLog2e;
  if (d == 128) {
    if (g.fixed) fwd_f32_t<128, true, 4>(q, k, v, g, o, lse, BH, L, sl2, s);
    else fwd_f32_t<128, false, 4>(q, k, v, g, o, lse, BH, L, sl2, s);
  } else {
    if (g.fixed) fwd_f32_t<64, true, 8>(q, k, v, g, o, lse, BH, L, sl2, s);
    else fwd_f32_t<64, false, 8>(q, k, v, g, o, lse, BH, L, sl2, s);
  }
  return hipGetLastError();
}

template <int D, bool FIXED, int NW>
static void dkdv_f32_t(const float* q, const float* k, const float* v, GateSpec g,
                       const float* lse, const float* d_o, const float* delta, float* dk,
                       float* dv, float* dck, int BH, int L, float scale, hipStream_t s) {
  const int n = (L + 31) / 32;
  if constexpr (NW == kF32Nw<D>)
    if (!f32_fine<D>(n, BH))
      return dkdv_f32_t<D, FIXED, NW / 2>(q, k, v, g, lse, d_o, delta, dk, dv, dck, BH, L, scale,
                                          s);
  hipLaunchKernelGGL((bwd_dkdv_f32_kernel<D, FIXED, NW>), f32_grid(n, BH), dim3(64 * NW), 0, s, q,
                     k, v, g.ptr, lse, d_o, delta, dk, dv, dck, BH, g.H, L, n, scale,
                     scale * kLog2e);
}

hipError_t launch_bwd_dkdv_f32(const float* q, const float* k, const float* v, GateSpec g,
                               const float* lse, const float* d_o, const float* delta, float* dk,
                               float* dv, float* dck, int BH, int L, int d, float scale,
                               hipStream_t s) {
  if (d == 128) {
    if (g.fixed) dkdv_f32_t<128, true, 4>(q, k, v, g, lse, d_o, delta, dk, dv, dck, BH, L, scale, s);
    else dkdv_f32_t<128, false, 4>(q, k, v, g, lse, d_o, delta, dk, dv, dck, BH, L, scale, s);
  } else {
    if (g.fixed) dkdv_f32_t<64, true, 8>(q, k, v, g, lse, d_o, delta, dk, dv, dck, BH, L, scale, s);
    else dkdv_f32_t<64, false, 8>(q, k, v, g, lse, d_o, delta, dk, dv, dck, BH, L, scale, s);
  }
  return hipGetLastError();
}

template <int D, bool FIXED, int NW>
static void dq_f32_t(const float* q, const float* k, const float* v, GateSpec g, const float* lse,
                     const float* d_o, const float* delta, float* dq, float* dcq, int BH, int L,
                     float scale, hipStream_t s) {
  const int n = (L + 31) / 32;
  if constexpr (NW == kF32Nw<D>)
    if (!f32_fine<D>(n, BH))
      return dq_f32_t<D, FIXED, NW / 2>(q, k, v, g, lse, d_o, delta, dq, dcq, BH, L, scale, s);
  hipLaunchKernelGGL((bwd_dq_f32_kernel<D, FIXED, NW>), f32_grid(n, BH), dim3(64 * NW), 0, s, q, k,
                     v, g.ptr, lse, d_o, delta, dq, dcq, BH, g.H, L, n, scale, scale * kLog2e);
}

hipError_t launch_bwd_dq_f32(const float* q, const float* k, const float* v, GateSpec g,
                             const float* lse, const float* d_o, const float* delta, float* dq,
                             float* dcq, int BH, int L, int d, float scale, hipStream_t s) {
  if (d == 128) {
    if (g.fixed) dq_f32_t<128, true, 4>(q, k, v, g, lse, d_o, delta, dq, dcq, BH, L, scale, s);
    else dq_f32_t<128, false, 4>(q, k, v, g, lse, d_o, delta, dq, dcq, BH, L, scale, s);
  } else {
    if (g.fixed) dq_f32_t<64, true, 8>(q, k, v, g, lse, d_o, delta, dq, dcq, BH, L, scale, s);
    else dq_f32_t<64, false, 8>(q, k, v, g, lse, d_o, delta, dq, dcq, BH, L, scale, s);
  }
  return hipGetLastError();
}

}  // namespace fox
