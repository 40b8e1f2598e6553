// One decode step of Forgetting Attention: Eq. fot-weight evaluated for the last
// position T of a sequence whose keys and values sit in a cache.
//
//     c_T   = c_{T-1} + log sigmoid(x_new)           (c_0 = 0)
//     s_j   = s q.k_j + c_T - c_j,   j = 1..T         (key T is the new token)
//     o     = sum_j softmax(s)_j v_j,  lse = log sum_j exp(s_j)
//
// The step streams K and V once from HBM (the bound), so the kernel is built for
// bandwidth: the T keys of each (batch, head) are split across workgroups, a
// group of D/8 (bf16) lanes reads one key's row with 16-byte loads so that a
// wave reads consecutive rows, several keys per lane group are loaded before
// any is used, and every lane group keeps its own running (max, sum, output).
// Workgroups are ordered split-major, most recent keys first, so that work is
// spread over all XCDs also when gate-aware skipping (below) keeps only the
// recent splits of every sequence.
// The lane groups of a workgroup merge through LDS into one partial per split;
// a second kernel merges the splits (log-sum-exp merge) and appends c_T
// to the prefix cache.  Entry T-1 of that cache is never read: every workgroup
// derives c_T itself, so the write cannot race with the readers.
#include <algorithm>
#include <mutex>

#include "fox_device.h"
#include "fox_internal.h"

namespace fox {

constexpr int kDecThreads = 256;
constexpr int kDecUnroll = 4;
// A split is skipped when its scores provably lie this far (base 2) below the
// new token's own score: 150 makes its merge weight exp2(m_split - M) an exact
// fp32 zero, and 10 more absorb the rounding of the bound itself.
constexpr float kSkipMargin = 160.0f;

constexpr int kDirectThreads = 1024;
constexpr int kDirectGroups = 256;

// One launch for the whole step (decode_direct_kernel) pays where the keys of a head are
// one pass of the workgroup's loads (64 KB of keys) and every workgroup has a CU.  Measured (graph replay, us, split and combine / direct):
// bf16 B H = 16, T = 200 7.8 / 6.1 at d = 128 and T = 500 7.5 / 6.2 at d = 64 (51 and 64
// KB), T = 500 8.2 / 10.3 at d = 128 (128 KB, two passes), fp32 T = 500 9.0 / 16.1 (256
// KB); B H = 128, T = 200 10.2 / 8.0; B H = 1024, T = 200 23.5 / 28.7.  One launch less is
// also 3 us less on the host.
static bool decode_direct(int BH, int T, int d, size_t elem) {
  constexpr size_t kPass = (size_t)kDirectThreads * kDecUnroll * 16;
  return BH <= kDirectGroups && (size_t)T * d * elem <= kPass;
}

// Keys per split.  From 256 keys up, the largest split (fewer partials) that still gives
// 2048 workgroups.  Where 256 keys leave fewer than 768 workgroups, the few there are walk
// their keys in a chain of waits for memory, so the split goes on halving down to 32 keys
// (one or two loads in flight per lane group), until 768 workgroups or 256 splits of a
// sequence, beyond which the combine pass costs more than the split gains.  Measured with
// the combine below (bf16, d = 128 unless said; us at 256 / 128 / 64 / 32 keys): B H = 16,
// T = 4097 14.9 / 12.4 / 12.1 / 15.7 (fp32 31.2 / 20.6 / 17.9 / 19.5), T = 500 13.5 / 10.3 /
// 9.0 / 8.0; B H = 2, T = 32768 21.6 / 19.6 / 25.2 / 41.9; above the line, B H = 128,
// T = 2000 27.1 / 30.1 and B H = 12, T = 20000, d = 64 18.3 / 20.4.
//
// A split below one pass of the workgroup's loads (16 KB of keys) leaves some of them
// unused.  That still pays for few heads with prefix gates (above), but not with fixed gates
// (us, 32 keys / one pass: bf16, d = 64, B H = 16, T = 3000 10.1 / 7.1, B H = 64, T = 600
// 8.9 / 7.2, fp32, d = 64, B H = 64, T = 600 8.1 / 7.2; the two are one at fp32, d = 128) nor
// with more heads than the one-launch form takes, whose caches may be as short as a pass
// (bf16, d = 64, B H = 320, T = 100 9.8 / 8.6).
//
// A workspace that holds the partials of 256-key splits always serves: where it is too
// small for the finer ones the split is the finest that fits.  The size a caller is told
// covers the splits of every cache of up to T keys, so a workspace sized for the longest
// gives each step of a growing one its own split.  (A shorter cache can need more than a
// longer one: B H = 16 takes 254 splits at T = 65024 and 128 at 65536, where the split
// doubles.)
constexpr int kSplitKeys = 256, kFineGroups = 768, kFineSplits = 256, kFineKeys = 32;
constexpr int kCoarseGroups = 2048;

static int coarse_keys_per_split(int BH, int T) {
  for (int ks = 1024; ks > kSplitKeys; ks >>= 1)
    if (BH * (((long long)T + ks - 1) / ks) >= kCoarseGroups) return ks;
  return kSplitKeys;
}

static size_t partial_bytes(int BH, long long splits, int d) {
  return (size_t)BH * (size_t)splits * (size_t)(d + 2) * sizeof(float);
}

static int decode_keys_per_split(int BH, int T, int d, size_t elem, bool fixed, size_t ws_bytes) {
  const int pass = (int)((size_t)kDecThreads * kDecUnroll * 16 / (d * elem));
  const int least = fixed || BH > kDirectGroups ? std::max(pass, kFineKeys) : kFineKeys;
  auto splits = [&](int ks) { return ((long long)T + ks - 1) / ks; };
  int ks = coarse_keys_per_split(BH, T);
  if (ks == kSplitKeys)
    while (ks > least && BH * splits(ks) < kFineGroups && splits(ks / 2) <= kFineSplits &&
           partial_bytes(BH, splits(ks / 2), d) <= ws_bytes)
      ks >>= 1;
  return ks;
}

size_t decode_min_workspace_bytes(int BH, int T, int d) {
  const int ks = coarse_keys_per_split(BH, T);
  return partial_bytes(BH, ((long long)T + ks - 1) / ks, d);
}

size_t decode_workspace_bytes(bool bf16_, int BH, int T, int d) {
  const size_t least = decode_min_workspace_bytes(BH, T, d);
  if (decode_direct(BH, T, d, bf16_ ? 2 : 4)) return least;
  // a split is halved below kFineGroups workgroups only, which at most doubles them
  const long long fine = std::min({(long long)kFineSplits, 2LL * ((kFineGroups - 1) / BH),
                                   (T + kFineKeys - 1LL) / kFineKeys});
  // a shorter cache's split of 256 or 512 keys is one whose double would give fewer than
  // kCoarseGroups workgroups, which at most doubles them
  const long long coarse =
      std::min(2LL * ((kCoarseGroups - 1) / BH), (T + kSplitKeys - 1LL) / kSplitKeys);
  return std::max(least, partial_bytes(BH, std::max(fine, coarse), d));
}

template <typename Tt>
struct Vec16;
template <>
struct Vec16<bf16> {
  typedef bf16x8 type;
  static constexpr int N = 8;
};
template <>
struct Vec16<float> {
  typedef f32x4 type;
  static constexpr int N = 4;
};

// A lane group's online softmax over the keys kbeg + g, + KPI, .. below kend: kDecUnroll
// keys' loads in flight before any is used.  gate_row: the prefix cache of this (batch,
// head); unused for fixed gates.
template <typename Tt, int D, bool FIXED, int THREADS>
__device__ __forceinline__ void decode_keys(const Tt* __restrict__ kh, const Tt* __restrict__ vh,
                                            const float* __restrict__ gate_row, int T, float cT,
                                            float lf, int kbeg, int kend, int g,
                                            const float (&qv)[Vec16<Tt>::N], float& m, float& l,
                                            float (&acc)[Vec16<Tt>::N]) {
  typedef typename Vec16<Tt>::type VT;
  constexpr int VEC = Vec16<Tt>::N;
  constexpr int LPK = D / VEC;
  constexpr int KPI = THREADS / LPK;
  for (int base = kbeg; base < kend; base += KPI * kDecUnroll) {
    VT kr[kDecUnroll], vr[kDecUnroll];
    float cj[kDecUnroll];
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      const int key = base + u * KPI + g;
      if (key < kend) {
        kr[u] = __builtin_nontemporal_load(reinterpret_cast<const VT*>(kh + (size_t)key * D));
        vr[u] = __builtin_nontemporal_load(reinterpret_cast<const VT*>(vh + (size_t)key * D));
        if constexpr (FIXED) cj[u] = (float)(key - (T - 1)) * lf * kLog2e;
        else cj[u] = key == T - 1 ? 0.0f : (gate_row[key] - cT) * kLog2e;
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          kr[u][e] = (Tt)0.0f;
          vr[u][e] = (Tt)0.0f;
        }
        cj[u] = INFINITY;
      }
    }
    float sv[kDecUnroll];
    float mu = -INFINITY;
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      float dot = 0.0f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) dot += qv[e] * (float)kr[u][e];
#pragma unroll
      for (int off = 1; off < LPK; off <<= 1) dot += __shfl_xor(dot, off);
      sv[u] = dot - cj[u];
      mu = fmaxf(mu, sv[u]);
    }
    const float m_new = fmaxf(m, mu);
    // A lane group with no key yet keeps m = -inf; a finite reference keeps the
    // exponents below free of (-inf) - (-inf).
    const float m_ref = m_new == -INFINITY ? 0.0f : m_new;
    const float alpha = exp2_fast(m - m_ref);
    // The first key's product is rounded and the old sum scaled within the fma: written out,
    // since the compiler's choice between the two changes with the code around it.
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      const float p = exp2_fast(sv[u] - m_ref);
      l = u == 0 ? fmaf(alpha, l, p) : l + p;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float v = (float)vr[u][e];
        acc[e] = u == 0 ? fmaf(alpha, acc[e], p * v) : fmaf(p, v, acc[e]);
      }
    }
    m = m_new;
  }
}

// FIXED: gate = b [H] (fixed gates, c_T - c_j = (T - 1 - j) log sigmoid(b));
// otherwise gate = the prefix cache [BH, T] and x_new the new token's gate logit.
// SKIP: knorm [BH] bounds the key norms; a split that cannot contribute (its
// merge weight would be an exact zero) writes an empty partial without reading
// its keys, which leaves the result bit for bit as without skipping.
template <typename Tt, int D, bool FIXED, bool SKIP>
__global__ __launch_bounds__(kDecThreads) void decode_split_kernel(
    const Tt* __restrict__ q, const Tt* __restrict__ kc, const Tt* __restrict__ vc,
    const float* __restrict__ gate, const float* __restrict__ x_new,
    const float* __restrict__ knorm, float* __restrict__ part, int H, int T, int keys_per_split,
    int n_split, float scale_log2) {
  typedef typename Vec16<Tt>::type VT;
  constexpr int VEC = Vec16<Tt>::N;
  constexpr int LPK = D / VEC;                // lanes per key
  constexpr int KPI = kDecThreads / LPK;      // keys per workgroup pass
  __shared__ float s_acc[KPI][D];
  __shared__ float s_m[KPI], s_l[KPI];

  const int tid = threadIdx.x;
  const int g = tid / LPK, lp = tid % LPK;
  // split-major, most recent split first: the splits that gate-aware skipping
  // keeps (the recent ones) are spread over all XCDs and dispatched first
  const int n_bh = (int)(gridDim.x / n_split);
  const int bh = blockIdx.x % n_bh, split = n_split - 1 - (int)(blockIdx.x / n_bh);
  const size_t head = (size_t)bh * (size_t)T;
  const int kbeg = split * keys_per_split;
  const int kend = min(T, kbeg + keys_per_split);
  float cT = 0.0f, lf = 0.0f;
  if constexpr (FIXED) {
    lf = log_sigmoid(gate[bh % H]);
  } else {
    cT = (T >= 2 ? gate[head + T - 2] : 0.0f) + log_sigmoid(x_new[bh]);
  }

  float qv[VEC], acc[VEC];
  {
    const VT qq = *reinterpret_cast<const VT*>(q + (size_t)bh * D + lp * VEC);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      qv[e] = (float)qq[e] * scale_log2;
      acc[e] = 0.0f;
    }
  }
  float m = -INFINITY, l = 0.0f;
  const Tt* kh = kc + head * D + lp * VEC;
  const Tt* vh = vc + head * D + lp * VEC;

  if constexpr (SKIP) {
    // Every score of the split is at most ||s log2(e) q|| max||k|| minus the
    // decay to the split's last key (c decreases along the sequence), while the
    // merged maximum is at least the new token's own score.  The butterfly sums
    // below give bitwise the same value in every lane, so the decision is
    // uniform across the workgroup.
    float qq = 0.0f, dot = 0.0f;
    const VT kl = *reinterpret_cast<const VT*>(kh + (size_t)(T - 1) * D);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      qq += qv[e] * qv[e];
      dot += qv[e] * (float)kl[e];
    }
#pragma unroll
    for (int off = 1; off < LPK; off <<= 1) {
      qq += __shfl_xor(qq, off);
      dot += __shfl_xor(dot, off);
    }
    const int jl = kend - 1;  // the split's last (least decayed) key
    float decay = 0.0f;       // (c_jl - c_T) log2(e) >= 0
    if (jl != T - 1) {
      if constexpr (FIXED) decay = (float)(jl - (T - 1)) * lf * kLog2e;
      else decay = (gate[head + jl] - cT) * kLog2e;
    }
    const float bound = sqrtf(qq) * knorm[bh] - decay;
    if (bound < dot - kSkipMargin) {
      float* out = part + ((size_t)bh * n_split + split) * (D + 2);
      for (int dd = tid; dd < D; dd += kDecThreads) out[2 + dd] = 0.0f;
      if (tid == 0) {
        out[0] = -INFINITY;
        out[1] = 0.0f;
      }
      return;
    }
  }

  decode_keys<Tt, D, FIXED, kDecThreads>(kh, vh, FIXED ? gate : gate + head, T, cT, lf, kbeg, kend,
                                         g, qv, m, l, acc);

#pragma unroll
  for (int e = 0; e < VEC; ++e) s_acc[g][lp * VEC + e] = acc[e];
  if (lp == 0) {
    s_m[g] = m;
    s_l[g] = l;
  }
  __syncthreads();
  float M = -INFINITY;
  for (int i = 0; i < KPI; ++i) M = fmaxf(M, s_m[i]);
  float* out = part + ((size_t)bh * n_split + split) * (D + 2);
  for (int dd = tid; dd < D; dd += kDecThreads) {
    float o = 0.0f;
    for (int i = 0; i < KPI; ++i) o += s_acc[i][dd] * exp2_fast(s_m[i] - M);
    out[2 + dd] = o;
  }
  if (tid == 0) {
    float Ls = 0.0f;
    for (int i = 0; i < KPI; ++i) Ls += s_l[i] * exp2_fast(s_m[i] - M);
    out[0] = M;
    out[1] = Ls;
  }
}

// The whole step in one launch for short caches: one workgroup of 1024 threads per
// (batch, head) walks all keys and writes o, lse and c_T itself.  With skipping it reads
// every key all the same: what the bound would drop adds exact zeros.
template <typename Tt, int D, bool FIXED>
__global__ __launch_bounds__(kDirectThreads) void decode_direct_kernel(
    const Tt* __restrict__ q, const Tt* __restrict__ kc, const Tt* __restrict__ vc,
    const float* __restrict__ gate, const float* __restrict__ x_new, float* __restrict__ c_out,
    Tt* __restrict__ o, float* __restrict__ lse, int H, int T, float scale_log2) {
  typedef typename Vec16<Tt>::type VT;
  constexpr int VEC = Vec16<Tt>::N;
  constexpr int LPK = D / VEC;
  constexpr int KPI = kDirectThreads / LPK;
  constexpr int NG = kDirectThreads / D;  // thread groups of the merge, one element each
  __shared__ float s_acc[KPI][D];
  __shared__ float s_m[KPI], s_l[KPI];
  const int tid = threadIdx.x, g = tid / LPK, lp = tid % LPK;
  const int bh = blockIdx.x;
  const size_t head = (size_t)bh * (size_t)T;
  float cT = 0.0f, lf = 0.0f;
  if constexpr (FIXED) {
    lf = log_sigmoid(gate[bh % H]);
  } else {
    cT = (T >= 2 ? gate[head + T - 2] : 0.0f) + log_sigmoid(x_new[bh]);
  }
  float qv[VEC], acc[VEC];
  const VT qq = *reinterpret_cast<const VT*>(q + (size_t)bh * D + lp * VEC);
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    qv[e] = (float)qq[e] * scale_log2;
    acc[e] = 0.0f;
  }
  float m = -INFINITY, l = 0.0f;
  decode_keys<Tt, D, FIXED, kDirectThreads>(kc + head * D + lp * VEC, vc + head * D + lp * VEC,
                                            FIXED ? gate : gate + head, T, cT, lf, 0, T, g, qv, m,
                                            l, acc);
#pragma unroll
  for (int e = 0; e < VEC; ++e) s_acc[g][lp * VEC + e] = acc[e];
  if (lp == 0) {
    s_m[g] = m;
    s_l[g] = l;
  }
  __syncthreads();
  float M = -INFINITY;
#pragma unroll
  for (int i = 0; i < KPI; i += 64) {
    const int k = i + (tid & 63);
    M = fmaxf(M, k < KPI ? s_m[k] : -INFINITY);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  const int mg = tid / D, e = tid % D;
  float ot = 0.0f, lt = 0.0f;
#pragma unroll 4
  for (int i = mg; i < KPI; i += NG) {
    const float w = exp2_fast(s_m[i] - M);
    ot += s_acc[i][e] * w;
    lt += s_l[i] * w;
  }
  __syncthreads();  // every partial has been read
  s_acc[mg][e] = ot;
  if (e == 0) s_l[mg] = lt;
  __syncthreads();
  if (mg > 0) return;
  lt = s_l[0];
#pragma unroll
  for (int k = 1; k < NG; ++k) {
    ot += s_acc[k][e];
    lt += s_l[k];
  }
  o[(size_t)bh * D + e] = (Tt)(ot / lt);
  if (tid == 0) {
    lse[bh] = kLn2 * (M + log2f(lt));
    if constexpr (!FIXED) c_out[head + T - 1] = cT;
  }
}

// The splits' partials of one (batch, head): THREADS / D thread groups take
// every THREADS / D-th split each (all of a thread's loads independent), the
// maximum is found by each wave over the splits in parallel, and the groups meet in LDS.
// One thread per element walking every split twice took most of a long, narrow step:
// B H = 2, T = 32768 72 -> 22 us for the step at the same split.  A single split needs one
// thread per element and no search (THREADS = D; many heads, bf16, d = 64, B H = 512,
// T = 30 8.0 -> 7.5 us for the step).
constexpr int kCombineThreads = 512;
template <typename Tt, int D, int THREADS>
__global__ __launch_bounds__(THREADS) void decode_combine_kernel(
    const float* __restrict__ part, float* __restrict__ cc, const float* __restrict__ x_new,
    Tt* __restrict__ o, float* __restrict__ lse, int T, int n_split) {
  constexpr int NG = THREADS / D;
  const int bh = blockIdx.x, tid = threadIdx.x;
  const int g = tid / D, e = tid % D;
  const float* p = part + (size_t)bh * n_split * (D + 2);
  float M, Ls, acc;
  if constexpr (NG == 1) {  // n_split == 1
    M = p[0];
    Ls = p[1];
    acc = p[2 + e];
  } else {
    __shared__ float s_acc[NG][D];
    __shared__ float s_l[NG];
    M = -INFINITY;
    for (int s = tid & 63; s < n_split; s += 64) M = fmaxf(M, p[(size_t)s * (D + 2)]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    Ls = acc = 0.0f;
#pragma unroll 4
    for (int s = g; s < n_split; s += NG) {
      const float* ps = p + (size_t)s * (D + 2);
      const float w = exp2_fast(ps[0] - M);
      Ls += ps[1] * w;
      acc += ps[2 + e] * w;
    }
    s_acc[g][e] = acc;
    if (e == 0) s_l[g] = Ls;
    __syncthreads();
    if (g > 0) return;
    Ls = s_l[0];
#pragma unroll
    for (int k = 1; k < NG; ++k) {
      acc += s_acc[k][e];
      Ls += s_l[k];
    }
  }
  o[(size_t)bh * D + e] = (Tt)(acc / Ls);
  if (tid == 0) {
    lse[bh] = kLn2 * (M + log2f(Ls));
    if (cc) {  // append c_T to the prefix cache (data-dependent gates)
      const size_t head = (size_t)bh * (size_t)T;
      cc[head + T - 1] = (T >= 2 ? cc[head + T - 2] : 0.0f) + log_sigmoid(x_new[bh]);
    }
  }
}

template <typename Tt, int D, bool FIXED, bool SKIP>
static hipError_t launch_decode_t(const void* q, const void* k_cache, const void* v_cache,
                                  const float* gate, int H, float* c_cache, const float* logit_new,
                                  const float* knorm, void* o, float* lse, void* ws, size_t ws_bytes,
                                  int BH, int T, float scale, hipStream_t s) {
  if (decode_direct(BH, T, D, sizeof(Tt))) {
    hipLaunchKernelGGL((decode_direct_kernel<Tt, D, FIXED>), dim3((unsigned)BH),
                       dim3(kDirectThreads), 0, s, (const Tt*)q, (const Tt*)k_cache,
                       (const Tt*)v_cache, gate, logit_new, c_cache, (Tt*)o, lse, H, T,
                       scale * kLog2e);
    return hipGetLastError();
  }
  const int ks = decode_keys_per_split(BH, T, D, sizeof(Tt), FIXED, ws_bytes);
  const int n_split = (T + ks - 1) / ks;
  float* part = static_cast<float*>(ws);
  hipLaunchKernelGGL((decode_split_kernel<Tt, D, FIXED, SKIP>),
                     dim3((unsigned)n_split * (unsigned)BH), dim3(kDecThreads), 0, s,
                     (const Tt*)q, (const Tt*)k_cache, (const Tt*)v_cache, gate, logit_new, knorm,
                     part, H, T, ks, n_split, scale * kLog2e);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool one = n_split == 1;
  auto combine = one ? decode_combine_kernel<Tt, D, D> : decode_combine_kernel<Tt, D, kCombineThreads>;
  hipLaunchKernelGGL(combine, dim3(BH), dim3(one ? D : kCombineThreads), 0, s, part, c_cache,
                     logit_new, (Tt*)o, lse, T, n_split);
  return hipGetLastError();
}

template <bool FIXED, bool SKIP>
static hipError_t decode_dispatch(bool bf16_, const void* q, const void* k_cache,
                                  const void* v_cache, const float* gate, int H, float* c_cache,
                                  const float* logit_new, const float* knorm, void* o, float* lse,
                                  void* ws, size_t ws_bytes, int BH, int T, int d, float scale,
                                  hipStream_t s) {
  if (bf16_) {
    return d == 128 ? launch_decode_t<bf16, 128, FIXED, SKIP>(q, k_cache, v_cache, gate, H,
                                                              c_cache, logit_new, knorm, o, lse,
                                                              ws, ws_bytes, BH, T, scale, s)
                    : launch_decode_t<bf16, 64, FIXED, SKIP>(q, k_cache, v_cache, gate, H,
                                                             c_cache, logit_new, knorm, o, lse,
                                                             ws, ws_bytes, BH, T, scale, s);
  }
  return d == 128 ? launch_decode_t<float, 128, FIXED, SKIP>(q, k_cache, v_cache, gate, H,
                                                             c_cache, logit_new, knorm, o, lse,
                                                             ws, ws_bytes, BH, T, scale, s)
                  : launch_decode_t<float, 64, FIXED, SKIP>(q, k_cache, v_cache, gate, H,
                                                            c_cache, logit_new, knorm, o, lse,
                                                            ws, ws_bytes, BH, T, scale, s);
}

hipError_t launch_decode(bool bf16_, const void* q, const void* k_cache, const void* v_cache,
                         float* c_cache, const float* logit_new, void* o, float* lse, void* ws,
                         size_t ws_bytes, int BH, int T, int d, float scale, hipStream_t s) {
  return decode_dispatch<false, false>(bf16_, q, k_cache, v_cache, c_cache, 1, c_cache, logit_new,
                                       nullptr, o, lse, ws, ws_bytes, BH, T, d, scale, s);
}

// ---------------------------------------------------------------------------
// The decode step without a caller workspace: the split partials live in a
// file-scope device array, `scratch`, of kDecodeScratchBytes (every device the
// library runs on holds its own copy, loaded with the code object, until the
// process ends).  In host code the name `scratch` is only a host-side stand-in;
// the device address comes from hipGetSymbolAddress, taken once per device with
// that device current and kept in scratch_ptr[].  The partials are fully
// written by the split kernel before the combine kernel reads them (skipped
// splits write empty partials), so nothing needs clearing between calls; calls
// that overlap on one device share the array and race.
// ---------------------------------------------------------------------------
static __device__ __align__(256) float scratch[kDecodeScratchBytes / sizeof(float)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_ptr[kMaxDevices] = {};

hipError_t device_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    scratch_ptr[dev] = p;
  }
  *out = scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

hipError_t launch_decode_noalloc(bool bf16_, const void* q, const void* k_cache,
                                 const void* v_cache, float* c_cache, const float* logit_new,
                                 void* o, float* lse, int BH, int T, int d, float scale,
                                 hipStream_t s) {
  if (decode_min_workspace_bytes(BH, T, d) > kDecodeScratchBytes) return hipErrorInvalidValue;
  const size_t ws_bytes = kDecodeScratchBytes;
  void* ws = nullptr;
  hipError_t e = device_scratch(&ws);
  if (e != hipSuccess) return e;
  return decode_dispatch<false, false>(bf16_, q, k_cache, v_cache, c_cache, 1, c_cache, logit_new,
                                       nullptr, o, lse, ws, ws_bytes, BH, T, d, scale, s);
}

hipError_t launch_decode_skip(bool bf16_, const void* q, const void* k_cache, const void* v_cache,
                              float* c_cache, const float* logit_new, const float* k_norm_max,
                              void* o, float* lse, void* ws, size_t ws_bytes, int BH, int T, int d,
                              float scale, hipStream_t s) {
  return decode_dispatch<false, true>(bf16_, q, k_cache, v_cache, c_cache, 1, c_cache, logit_new,
                                      k_norm_max, o, lse, ws, ws_bytes, BH, T, d, scale, s);
}

hipError_t launch_decode_fixed(bool bf16_, const void* q, const void* k_cache, const void* v_cache,
                               const float* bias, int H, void* o, float* lse, void* ws,
                               size_t ws_bytes, int BH, int T, int d, float scale, hipStream_t s,
                               const float* k_norm_max) {
  if (k_norm_max)
    return decode_dispatch<true, true>(bf16_, q, k_cache, v_cache, bias, H, nullptr, nullptr,
                                       k_norm_max, o, lse, ws, ws_bytes, BH, T, d, scale, s);
  return decode_dispatch<true, false>(bf16_, q, k_cache, v_cache, bias, H, nullptr, nullptr,
                                      nullptr, o, lse, ws, ws_bytes, BH, T, d, scale, s);
}

}  // namespace fox
