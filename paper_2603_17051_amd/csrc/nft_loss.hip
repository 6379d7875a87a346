// Clip-level forward-process RL loss and its gradient w.r.t. the current velocity prediction
// (Sec. 3.1 eq. (1)-(2), Sec. 3.3 reward normalisation, Sec. 3.4 selective KL; Alg. 1 Phase 2),
// fused into one pass over the four velocity-shaped tensors: HBM-bound, every element is read
// once (4 tensors) and its gradient written once (cache-bypassing loads and stores).  Deterministic: per-block partial sums in a
// workspace, summed in a fixed order by one block.  Two launches (main, final sum) up to 1024
// samples, three (prepare, main, final sum) above.
#include <mutex>

#include "kernels.hpp"
#include "mfma_common.hpp"

namespace astro {
namespace {

constexpr int kThreads = 256;  // of the prepare launch
constexpr int kElemsPerBlock = 16384;  // most elements of one sample a workgroup walks

struct NftParams {
  const void *v_theta, *v_old, *v_ref, *target;
  const float* advantage;
  const int32_t* kl_mask;
  float* grad;
  float* loss;      // [3] total, policy, kl
  float* r_tilde;   // workspace [n]
  float* n_masked;  // workspace [1]
  float* partials;  // workspace [n][blocks_per_sample][3]
  int n, blocks_per_sample;
  int64_t E, share;  // elements per sample, and of it per workgroup
  float inv_a_max, beta, lambda_kl;
};

// r~_i = clip(A_i / A_max, -1, 1) / 2 + 0.5 and the number of masked samples
__global__ void __launch_bounds__(kThreads) nft_prepare_kernel(NftParams p) {
  __shared__ int cnt[kThreads];
  int c = 0;
  for (int i = threadIdx.x; i < p.n; i += kThreads) {
    const float a = p.advantage[i] * p.inv_a_max;
    p.r_tilde[i] = fminf(fmaxf(a, -1.f), 1.f) * 0.5f + 0.5f;
    c += p.kl_mask[i] != 0 ? 1 : 0;
  }
  cnt[threadIdx.x] = c;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) cnt[threadIdx.x] += cnt[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *p.n_masked = (float)cnt[0];
}

// Four elements of a tensor.  Also for bf16, where that is an 8-byte load: a lane's gradients are then
// the 16 bytes next to its neighbour's, and a wave's store is 1 KB in one piece (eight elements per lane
// make two stores that each touch every other 16 bytes: 142 us instead of 121 at 192 clips).
constexpr int N = 4;
template <typename Elem>
struct Chunk {
  typedef Elem Vec __attribute__((ext_vector_type(N)));
  // chunks of every tensor in flight per thread, and the most threads of a workgroup.  Measured at 24 /
  // 192 clips of 299520 elements: bf16 20.2 / 122 us (1024 threads: 20.8 / 130, 256: 21.4 / 130, two chunks and 512
  // threads: 20.5 / 126), fp32 29.3 / 196 (512 threads and four chunks: 29.6 / 204, 256 and four: 30.1 / 213)
  static constexpr int kUnroll = sizeof(Elem) == 2 ? 4 : 2;
  static constexpr int kThreads = sizeof(Elem) == 2 ? 512 : 1024;
  Vec v;
  __device__ __forceinline__ void load(const void* base, int64_t i) {
    v = __builtin_nontemporal_load(reinterpret_cast<const Vec*>(static_cast<const Elem*>(base) + i));
  }
  __device__ __forceinline__ float operator[](int j) const { return (float)v[j]; }
};

// Up to this many samples every workgroup derives r~ of its sample and the number of masked
// samples itself (a few KB from L2) and the prepare launch is skipped: at one group of 24 clips the
// three dependent launches took 28 us for 17 us of memory traffic.
constexpr int kMaxSamplesInline = 1024;

// HBM-bound.  A workgroup walks kElemsPerBlock elements of one sample (one triple of partial sums each,
// which is what the workspace holds).  24 clips are 456 workgroups, fewer than two per CU, so a
// workgroup needs many bytes in flight; the first trip's loads are issued before the masked samples are
// counted, so that chain runs under their latency.  With 256 threads and one 16-byte load per tensor at
// a time: 24.9 / 142 us in bf16 at 24 / 192 clips, 32.1 / 221 us in fp32; now 20.2 / 122 and 29.3 / 196.

// grid (blocks_per_sample, n); blockDim.x a multiple of 64 up to Chunk::kThreads
template <typename Elem, bool kInline>
__global__ void __launch_bounds__(Chunk<Elem>::kThreads) nft_loss_kernel(NftParams p) {
  using C = Chunk<Elem>;
  constexpr int kUnroll = C::kUnroll;
  const int threads = blockDim.x, waves = threads / 64, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.y;
  const int64_t lo = (int64_t)blockIdx.x * p.share;
  const int64_t hi = lo + p.share < p.E ? lo + p.share : p.E;
  const int64_t base = (int64_t)i * p.E;
  C vt[kUnroll], vo[kUnroll], vr[kUnroll], tg[kUnroll];
  auto load = [&](int64_t e0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t e = e0 + (int64_t)u * threads * N;
      if (e < hi) {
        vt[u].load(p.v_theta, base + e);
        vo[u].load(p.v_old, base + e);
        vr[u].load(p.v_ref, base + e);
        tg[u].load(p.target, base + e);
      }
    }
  };
  int64_t e0 = lo + (int64_t)threadIdx.x * N;
  load(e0);

  __shared__ float red[3][C::kThreads / 64];
  float r, nm;
  if constexpr (kInline) {
    int c = 0;
    for (int j0 = 0; j0 < p.n; j0 += threads) c += __popcll(__ballot(j0 + (int)threadIdx.x < p.n && p.kl_mask[j0 + threadIdx.x] != 0));
    if (lane == 0) red[0][wave] = (float)c;  // counts up to 1024: exact
    __syncthreads();
    nm = 0.f;
    for (int wv = 0; wv < waves; ++wv) nm += red[0][wv];
    __syncthreads();
    r = fminf(fmaxf(p.advantage[i] * p.inv_a_max, -1.f), 1.f) * 0.5f + 0.5f;
    // the first workgroup leaves both where the final sum reads them
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      p.r_tilde[i] = r;
      if (i == 0) *p.n_masked = nm;
    }
  } else {
    r = p.r_tilde[i];
    nm = *p.n_masked;
  }
  const float c_pol = 2.f * p.beta / (float)p.n;
  const float c_kl = (p.kl_mask[i] != 0 && nm > 0.f) ? 2.f * p.lambda_kl / nm : 0.f;
  float s_pos = 0.f, s_neg = 0.f, s_ref = 0.f;
  for (; e0 < hi;) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t e = e0 + (int64_t)u * threads * N;
      if (e >= hi) continue;
      float g[N];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float bd = p.beta * (vt[u][j] - vo[u][j]);  // v+ = v_old + beta (v_theta - v_old), v- = v_old - beta (...)
        const float e_pos = (vo[u][j] - tg[u][j]) + bd;
        const float e_neg = (vo[u][j] - tg[u][j]) - bd;
        const float d_ref = vt[u][j] - vr[u][j];
        s_pos = fmaf(e_pos, e_pos, s_pos);
        s_neg = fmaf(e_neg, e_neg, s_neg);
        s_ref = fmaf(d_ref, d_ref, s_ref);
        g[j] = c_pol * (r * e_pos - (1.f - r) * e_neg) + c_kl * d_ref;
      }
      float* go = p.grad + base + e;
#pragma unroll
      for (int j = 0; j < N; j += 4)
        __builtin_nontemporal_store(f32x4{g[j], g[j + 1], g[j + 2], g[j + 3]}, reinterpret_cast<f32x4*>(go + j));
    }
    e0 += (int64_t)kUnroll * threads * N;
    load(e0);
  }
  // block reduction of the three sums
  float v[3] = {s_pos, s_neg, s_ref};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    v[k] = sum_quarters(sum_neighbours<16>(v[k]));
    if (lane == 0) red[k][wave] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    float t = 0.f;
    for (int wv = 0; wv < waves; ++wv) t += red[threadIdx.x][wv];
    p.partials[((int64_t)i * p.blocks_per_sample + blockIdx.x) * 3 + threadIdx.x] = t;
  }
}

// Sum over a wave, in every lane of it: within 16 lanes the two 32-bit halves are moved as sum_neighbours() does, across them
// by shuffles.
__device__ __forceinline__ double wave_sum(double x) {
  auto moved = [](double v, auto ctrl) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)u, decltype(ctrl)::value, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), decltype(ctrl)::value, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
  };
  x += moved(x, std::integral_constant<int, 0xB1>{});
  x += moved(x, std::integral_constant<int, 0x4E>{});
  x += moved(x, std::integral_constant<int, 0x141>{});
  x += moved(x, std::integral_constant<int, 0x140>{});
#pragma unroll
  for (int s = 16; s < 64; s <<= 1) x += __shfl_xor(x, s);
  return x;
}

// One workgroup: L_policy = (1/n) sum_i [r~_i S+_i + (1 - r~_i) S-_i], L_KL = (1/|M|) sum_{i in M} Sref_i.
// Both are sums over all triples of partial sums with the weights of their sample, so the threads
// share the triples (one thread per sample walked its triples one after another: 5.5 us at 24 clips
// of 19 triples, most of it latency).  fp64, fixed order.
// What it takes is the chain launch, loads, sum.  Moves between lanes instead of shuffles through the LDS, a division of 32
// bits, the count requested with the triples and no more waves than there are triples for: 2.3 -> 1.8 us at up to 109 triples, where
// one or two waves are left of sixteen, 3.8 as before at 444 and 456.  The main kernel's sums, which take the same moves, gained 0.5 -
// 1.1 us of it at every size; both launches: 4 clips of 30784 elements in bf16 9.3 -> 8.4 us, 109 of 1856 7.4 -> 6.5, 24 of
// 299520 20.1 -> 19.5, 148 of 33240 in fp32 22.4 -> 21.3.
constexpr int kFinalThreads = 1024;
__global__ void __launch_bounds__(kFinalThreads) nft_finalize_kernel(NftParams p) {
  __shared__ double pol[kFinalThreads / 64], kl[kFinalThreads / 64];
  const int64_t n_triples = (int64_t)p.n * p.blocks_per_sample;
  const int threads = blockDim.x, waves = threads / 64;
  const double nm = (double)*p.n_masked;
  double a = 0.0, b = 0.0;
  auto add = [&](int64_t t, int i) __attribute__((always_inline)) {
    const double r = (double)p.r_tilde[i];
    a += r * (double)p.partials[3 * t] + (1.0 - r) * (double)p.partials[3 * t + 1];
    b += p.kl_mask[i] != 0 ? (double)p.partials[3 * t + 2] : 0.0;
  };
  if (n_triples <= INT32_MAX - kFinalThreads)
    for (uint32_t t = threadIdx.x; t < (uint32_t)n_triples; t += threads) add(t, (int)(t / (uint32_t)p.blocks_per_sample));
  else
    for (int64_t t = threadIdx.x; t < n_triples; t += threads) add(t, (int)(t / p.blocks_per_sample));
  a = wave_sum(a);
  b = wave_sum(b);
  if ((threadIdx.x & 63) == 0) {
    pol[threadIdx.x >> 6] = a;
    kl[threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = b = 0.0;
#pragma unroll
    for (int wv = 0; wv < kFinalThreads / 64; ++wv) {
      a += wv < waves ? pol[wv] : 0.0;
      b += wv < waves ? kl[wv] : 0.0;
    }
    const double l_pol = a / (double)p.n;
    const double l_kl = nm > 0.0 ? b / nm : 0.0;
    p.loss[0] = (float)(l_pol + (double)p.lambda_kl * l_kl);
    p.loss[1] = (float)l_pol;
    p.loss[2] = (float)l_kl;
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
int blocks_per_sample(int64_t E) { return (int)((E + kElemsPerBlock - 1) / kElemsPerBlock); }

int workspace_bytes_of(int32_t n_samples, int64_t elems_per_sample, size_t* bytes) {
  if (!bytes || n_samples < 1 || n_samples > 65535 || elems_per_sample < 1 || elems_per_sample > ((int64_t)1 << 40))
    return ASTRO_ERR_INVALID_ARG;
  *bytes = align256((size_t)n_samples * sizeof(float)) + 256 +
           align256((size_t)n_samples * blocks_per_sample(elems_per_sample) * 3 * sizeof(float));
  return ASTRO_OK;
}

// Validation and launches shared by the two entry points; `workspace` is device memory of at
// least the bytes workspace_bytes_of() reports (the caller's, or the static array below).
int run_nft_loss(const void* v_theta, const void* v_old, const void* v_ref, const void* target, const float* advantage,
                 const int32_t* kl_mask, int32_t n_samples, int64_t elems_per_sample, int32_t dtype, float a_max,
                 float beta, float lambda_kl, float* loss, float* grad_v_theta, void* workspace, size_t workspace_bytes,
                 hipStream_t stream, bool timed) {
  size_t need = 0;
  if (workspace_bytes_of(n_samples, elems_per_sample, &need) != ASTRO_OK) return ASTRO_ERR_INVALID_ARG;
  if (!v_theta || !v_old || !v_ref || !target || !advantage || !kl_mask || !loss || !grad_v_theta) return ASTRO_ERR_INVALID_ARG;
  if (dtype != ASTRO_BF16 && dtype != ASTRO_F32) return ASTRO_ERR_INVALID_ARG;
  if (!(a_max > 0.f) || !(beta == beta) || !(lambda_kl == lambda_kl)) return ASTRO_ERR_INVALID_ARG;
  // 16-byte vector accesses: every sample must start on a 16-byte boundary in all tensors
  if (elems_per_sample % (dtype == ASTRO_BF16 ? 8 : 4) != 0) return ASTRO_ERR_UNSUPPORTED;
  for (const void* ptr : {v_theta, v_old, v_ref, target, (const void*)grad_v_theta})
    if ((uintptr_t)ptr & 15) return ASTRO_ERR_INVALID_ARG;
  if (blocks_per_sample(elems_per_sample) > 2147483647 / 3) return ASTRO_ERR_UNSUPPORTED;
  if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255)) return ASTRO_ERR_WORKSPACE;

  NftParams p;
  p.v_theta = v_theta; p.v_old = v_old; p.v_ref = v_ref; p.target = target;
  p.advantage = advantage; p.kl_mask = kl_mask;
  p.grad = grad_v_theta; p.loss = loss;
  char* ws = static_cast<char*>(workspace);
  p.r_tilde = reinterpret_cast<float*>(ws);
  p.n_masked = reinterpret_cast<float*>(ws + align256((size_t)n_samples * sizeof(float)));
  p.partials = reinterpret_cast<float*>(ws + align256((size_t)n_samples * sizeof(float)) + 256);
  p.n = n_samples;
  p.blocks_per_sample = blocks_per_sample(elems_per_sample);
  p.E = elems_per_sample;
  // Even shares where the last of a few workgroups of a sample would have little: as many workgroups of full size with a few
  // elements cost 95 us instead of 69 (1024 samples of 17904 in fp32), 81 instead of 75 (400 of 49312).  A long sample's full
  // shares are two whole trips of the threads (192 of 299520 in fp32 193 us, 199 in even shares).
  const int64_t rest = elems_per_sample % kElemsPerBlock;
  p.share = kElemsPerBlock;
  if (p.blocks_per_sample == 1)
    p.share = elems_per_sample;
  else if (p.blocks_per_sample <= 8 && rest != 0 && rest < kElemsPerBlock / 2)
    p.share = ((elems_per_sample + p.blocks_per_sample - 1) / p.blocks_per_sample + 255) / 256 * 256;
  p.inv_a_max = 1.f / a_max; p.beta = beta; p.lambda_kl = lambda_kl;
  {
    // the entry point that must not allocate never creates timing events, even while profiling is on
    ProfileScope prof("nft_loss", stream, timed);
    const dim3 grid(p.blocks_per_sample, n_samples);
    // as many threads as a workgroup's share has groups of kUnroll chunks, in whole waves
    const bool is_bf16 = dtype == ASTRO_BF16;
    const int per_thread = N * (is_bf16 ? Chunk<__bf16>::kUnroll : Chunk<float>::kUnroll);
    // ... up to the most that pay: with one trip per thread on a small share too few workgroups are on a CU (900 samples
    // of 4816 in bf16 19.4 us with up to 512 threads, 14.7 with 256; 1024 of 6648 in fp32 32.5 with up to 1024, 26.8 with
    // 512).  Above the lines more threads are as fast or faster (3000 of 12056 in fp32 136 us, 145 with 512).
    const int most = is_bf16 ? (p.share < 6144 ? 256 : Chunk<__bf16>::kThreads) : (p.share < 9216 ? 512 : Chunk<float>::kThreads);
    const int64_t want = ((p.share + per_thread - 1) / per_thread + 63) / 64 * 64;
    const int threads = want < most ? (int)want : most;
    if (n_samples <= kMaxSamplesInline) {
      if (is_bf16)
        nft_loss_kernel<__bf16, true><<<grid, threads, 0, stream>>>(p);
      else
        nft_loss_kernel<float, true><<<grid, threads, 0, stream>>>(p);
    } else {
      nft_prepare_kernel<<<1, kThreads, 0, stream>>>(p);
      if (is_bf16)
        nft_loss_kernel<__bf16, false><<<grid, threads, 0, stream>>>(p);
      else
        nft_loss_kernel<float, false><<<grid, threads, 0, stream>>>(p);
    }
    const int64_t n_triples = (int64_t)n_samples * p.blocks_per_sample;
    nft_finalize_kernel<<<1, n_triples < kFinalThreads ? (int)(n_triples + 63) / 64 * 64 : kFinalThreads, 0, stream>>>(p);
  }
  return hipGetLastError() == hipSuccess ? ASTRO_OK : ASTRO_ERR_HIP;
}

// ---- the entry point that allocates nothing -------------------------------------------------
// r~, the masked count and the per-block partial sums live in a file-scope device array instead
// of a caller's workspace.  Every GPU the library runs on holds its own copy of the array at its
// own address for the life of the process; the host-side name of the array is not that address,
// so the address is asked for once per device (with that device current) and kept.
constexpr size_t kStaticScratchBytes = (size_t)1 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return ASTRO_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return ASTRO_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return ASTRO_ERR_HIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return ASTRO_OK;
}

}  // namespace
}  // namespace astro

using namespace astro;

extern "C" {

int astro_nft_loss_workspace_bytes(int32_t n_samples, int64_t elems_per_sample, size_t* bytes) {
  return workspace_bytes_of(n_samples, elems_per_sample, bytes);
}

int astro_nft_loss(const void* v_theta, const void* v_old, const void* v_ref, const void* target, const float* advantage,
                   const int32_t* kl_mask, int32_t n_samples, int64_t elems_per_sample, int32_t dtype, float a_max,
                   float beta, float lambda_kl, float* loss, float* grad_v_theta, void* workspace, size_t workspace_bytes,
                   void* hip_stream) {
  return run_nft_loss(v_theta, v_old, v_ref, target, advantage, kl_mask, n_samples, elems_per_sample, dtype, a_max, beta,
                      lambda_kl, loss, grad_v_theta, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream), true);
}

int astro_nft_loss_static_bytes(size_t* bytes) {
  if (!bytes) return ASTRO_ERR_INVALID_ARG;
  *bytes = kStaticScratchBytes;
  return ASTRO_OK;
}

int astro_nft_loss_static(const void* v_theta, const void* v_old, const void* v_ref, const void* target,
                          const float* advantage, const int32_t* kl_mask, int32_t n_samples, int64_t elems_per_sample,
                          int32_t dtype, float a_max, float beta, float lambda_kl, float* loss, float* grad_v_theta,
                          void* hip_stream) {
  size_t need = 0;
  if (workspace_bytes_of(n_samples, elems_per_sample, &need) != ASTRO_OK) return ASTRO_ERR_INVALID_ARG;
  if (need > kStaticScratchBytes) return ASTRO_ERR_WORKSPACE;  // more partial sums than the static array holds
  void* ws = nullptr;
  const int rc = static_scratch_of_current_device(&ws);
  if (rc != ASTRO_OK) return rc;
  return run_nft_loss(v_theta, v_old, v_ref, target, advantage, kl_mask, n_samples, elems_per_sample, dtype, a_max, beta,
                      lambda_kl, loss, grad_v_theta, ws, kStaticScratchBytes, static_cast<hipStream_t>(hip_stream), false);
}

}  // extern "C"
