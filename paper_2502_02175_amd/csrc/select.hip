// Token selection (Alg. 1 of VLA-Cache) and the layer-adaptive ratio (Sec. 3.4).
//
//   patch_terms_kernel   Eq. (sim): per patch the exact integers dot, |P_t|^2, |P_{t-1}|^2, and
//                        the task-relevance score (mean over layers)
//   select_rank_kernel   threshold (Sim >= tau, cross-multiplied in 128-bit integers),
//                        Top-k by exact rational comparison (Eq. topk), task-relevance
//                        quantile filter (Eq. ptask, Eq. pfinal)
//   select_order_kernel  ascending index list and reuse order
//   layer_ratio_kernel   entropy ratio and Eq. (reuse_ratio), in fp64
//
// All of this is HBM/latency-bound integer work: 2*H*W*3 bytes of pixels per
// stream are read exactly once, with 16-byte loads over the contiguous run of
// image rows that one row of patches covers.
#include <mutex>

#include "common.h"

typedef unsigned __int128 u128;

#define SEL_MAX_LV 4096
struct LayerMask { uint32_t w[16]; };  // bit l set = layer l is averaged over (<= 512 layers)

// The task-relevance score of 256 patches of stream b: the mean over the layers of the mask, fp32,
// layers in ascending order.  Sixteen layers are asked for at a time, those outside the mask too
// (their values are dropped, not added).
__device__ inline void relevance_scores(const float* __restrict__ attn_mean, int n_layers, int B, int b, int L_v,
                                        const LayerMask& mask, int j, float* __restrict__ score) {
  if (j >= L_v) return;
  float s = 0.f;
  if (attn_mean) {
    int n = 0;
    for (int l0 = 0; l0 < n_layers; l0 += 16) {
      float t[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) t[u] = attn_mean[((size_t)min(l0 + u, n_layers - 1) * B + b) * L_v + j];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int l = l0 + u;
        const bool on = l < n_layers && ((mask.w[(l0 >> 5) & 15] >> (l & 31)) & 1u);
        s = on ? s + t[u] : s;
        n += on;
      }
    }
    s = s / (float)(n > 0 ? n : 1);
  }
  score[(size_t)b * L_v + j] = s;
}

struct Frac { uint64_t num, den; };  // Sim^2 as an exact fraction

__device__ inline Frac sim_fraction(uint32_t dot, uint32_t na, uint32_t nb) {
  // two all-zero patches are identical, exactly one all-zero patch is dissimilar
  if (na == 0 && nb == 0) return {1, 1};
  if (na == 0 || nb == 0) return {0, 1};
  return {(uint64_t)dot * dot, (uint64_t)na * nb};
}

// ---------------------------------------------------------------------------
// Eq. (sim) terms.  One workgroup per (patch row, stream); behind them in the grid the workgroups
// that compute the scores, 256 patches each, beside the pixels instead of once per workgroup of
// the ranking kernel (64 times per stream at 1024 patches: 59 us of ranking for 8 such streams then,
// 18 without).
// ---------------------------------------------------------------------------
template <int VEC>
__global__ __launch_bounds__(256) void patch_terms_kernel(const uint8_t* __restrict__ prev,
                                                          const uint8_t* __restrict__ cur, int H,
                                                          int W, int patch, uint64_t tn2, uint64_t td2,
                                                          uint32_t* __restrict__ terms, double* __restrict__ similar,
                                                          const float* __restrict__ attn_mean, int n_layers,
                                                          LayerMask layer_mask, float* __restrict__ score) {
  extern __shared__ uint32_t acc[];  // [gw][3]
  const int gw = W / patch, gh = H / patch;
  const int b = blockIdx.y, pr = blockIdx.x, tid = threadIdx.x;
  if (pr >= gh) {
    relevance_scores(attn_mean, n_layers, gridDim.y, b, gw * gh, layer_mask, (pr - gh) * 256 + tid, score);
    return;
  }
  const size_t base = ((size_t)b * H + (size_t)pr * patch) * W * 3;
  const int rowbytes = W * 3, pbytes = patch * 3, nbytes = patch * rowbytes;
  for (int i = tid; i < gw * 3; i += 256) acc[i] = 0;
  __syncthreads();
  for (int o = tid * VEC; o < nbytes; o += 256 * VEC) {
    uint32_t av[4] = {0, 0, 0, 0}, bv[4] = {0, 0, 0, 0};
    if constexpr (VEC == 16) {
      const uint4 a4 = *(const uint4*)(cur + base + o);
      const uint4 b4 = *(const uint4*)(prev + base + o);
      av[0] = a4.x; av[1] = a4.y; av[2] = a4.z; av[3] = a4.w;
      bv[0] = b4.x; bv[1] = b4.y; bv[2] = b4.z; bv[3] = b4.w;
    } else {
      av[0] = cur[base + o];
      bv[0] = prev[base + o];
    }
    const int c = o % rowbytes;
    int j = c / pbytes, within = c % pbytes;
    uint32_t d = 0, na = 0, nb = 0;
    auto flush = [&]() {
      if (d | na | nb) {
        atomicAdd(&acc[j * 3 + 0], d);
        atomicAdd(&acc[j * 3 + 1], na);
        atomicAdd(&acc[j * 3 + 2], nb);
      }
      d = na = nb = 0;
    };
    auto advance = [&](int n) {
      within += n;
      if (within == pbytes) {
        flush();
        within = 0;
        if (++j == gw) j = 0;
      }
    };
    if constexpr (VEC == 16) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (within + 4 <= pbytes) {  // the whole dword lies in one patch
          d = __builtin_amdgcn_udot4(av[k], bv[k], d, false);
          na = __builtin_amdgcn_udot4(av[k], av[k], na, false);
          nb = __builtin_amdgcn_udot4(bv[k], bv[k], nb, false);
          advance(4);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t x = (av[k] >> (8 * q)) & 255u, y = (bv[k] >> (8 * q)) & 255u;
            d += x * y; na += x * x; nb += y * y;
            advance(1);
          }
        }
      }
    } else {
      d = av[0] * bv[0]; na = av[0] * av[0]; nb = bv[0] * bv[0];
      advance(1);
    }
    flush();
  }
  __syncthreads();
  const int Lv = gw * gh;
  for (int i = tid; i < gw * 3; i += 256)
    terms[((size_t)b * Lv + (size_t)pr * gw) * 3 + i] = acc[i];
  // Sim^2 of every patch once, here, and not in every workgroup of the ranking kernel (64 times per stream at
  // 1024 patches: ranking of 8 such streams 17.6 us, 14.7 now; this kernel 10.7, 10.9); -1: below the threshold
  for (int j = tid; j < gw; j += 256) {
    const Frac f = sim_fraction(acc[j * 3], acc[j * 3 + 1], acc[j * 3 + 2]);
    const bool pass = (u128)f.num * td2 >= (u128)tn2 * f.den;
    similar[(size_t)b * Lv + (size_t)pr * gw + j] = pass ? (double)f.num / (double)f.den : -1.0;
  }
}

void launch_patch_terms(const uint8_t* prev, const uint8_t* cur, int B, int H, int W, int patch, int tau_num,
                        int tau_den, uint32_t* terms, double* similar, const float* attn_mean, int n_layers, const uint8_t* layer_mask_host,
                        float* score, hipStream_t st) {
  const int gw = W / patch, gh = H / patch;
  LayerMask lm;
  for (int i = 0; i < 16; ++i) lm.w[i] = 0;
  for (int l = 0; l < n_layers && l < 512; ++l)
    if (!layer_mask_host || layer_mask_host[l]) lm.w[l >> 5] |= 1u << (l & 31);
  const uint64_t tn2 = (uint64_t)tau_num * (uint64_t)tau_num;
  const uint64_t td2 = (uint64_t)tau_den * (uint64_t)tau_den;
  const size_t shm = (size_t)gw * 3 * sizeof(uint32_t);
  const bool vec = ((size_t)patch * W * 3) % 16 == 0 && ((size_t)H * W * 3) % 16 == 0 &&
                   ((uintptr_t)prev % 16 == 0) && ((uintptr_t)cur % 16 == 0);
  dim3 grid(gh + (gw * gh + 255) / 256, B);
#define VLAC_TERMS(VEC_)                                                                                        \
  hipLaunchKernelGGL(patch_terms_kernel<VEC_>, grid, dim3(256), shm, st, prev, cur, H, W, patch, tn2, td2, terms, \
                     similar, attn_mean, n_layers, lm, score)
  if (vec) VLAC_TERMS(16);
  else VLAC_TERMS(1);
#undef VLAC_TERMS
}

// ---------------------------------------------------------------------------
// Threshold, Top-k, relevance filter.
// ---------------------------------------------------------------------------
// grid (ceil(L_v / 16), B).  flags[b, i] = 1 iff patch i is in P_final.
// A workgroup ranks 256 / SEL_LPT patches, SEL_LPT lanes to a patch: every lane counts, over
// its share of the other patches, those that come before its patch (by similarity for Top-k,
// by score for the relevance quantile), and the counts are added up across the lanes
// (integers: the result does not depend on how the patches are dealt).  Every workgroup
// first copies the stream's similarities and scores to LDS, so many lanes per patch pay
// while the launch is small (16 lanes: 8 us instead of 46 us at one stream of 256 patches)
// and one lane per patch is right once the streams alone fill the chip.
template <int SEL_LPT>
__global__ __launch_bounds__(256) void select_rank_kernel(
    const uint32_t* __restrict__ terms, const double* __restrict__ similar, int L_v, int top_k,
    const float* __restrict__ relevance, int n_rel, uint8_t* __restrict__ flags) {
  __shared__ double approx[SEL_MAX_LV];
  __shared__ float score[SEL_MAX_LV];
  const int b = blockIdx.y, tid = threadIdx.x;
  const uint32_t* t = terms + (size_t)b * L_v * 3;
  for (int j = tid; j < L_v; j += 256) {
    approx[j] = similar[(size_t)b * L_v + j];
    score[j] = relevance[(size_t)b * L_v + j];
  }
  __syncthreads();
  constexpr int SEL_PPW = 256 / SEL_LPT;
  const int sub = tid % SEL_LPT;
  const int i = blockIdx.x * SEL_PPW + tid / SEL_LPT;
  const bool live = i < L_v;           // (a patch's 16 lanes lie in one wave and leave together)
  const int ii = live ? i : 0;
  const bool passed = approx[ii] >= 0 && top_k > 0;
  int rank = 0, rr = 0;
  if (passed) {
    // rank among the passers: higher similarity first, ties -> lower index
    const double ai = approx[ii];
    const Frac fi = sim_fraction(t[ii * 3], t[ii * 3 + 1], t[ii * 3 + 2]);
    for (int j = sub; j < L_v; j += SEL_LPT) {
      const double aj = approx[j];
      if (aj < 0 || j == ii) continue;
      const double dlt = aj - ai;
      bool beats;
      if (dlt > 1e-12) beats = true;
      else if (dlt < -1e-12) beats = false;
      else {  // too close for fp64: exact cross-multiplication
        const Frac fj = sim_fraction(t[j * 3], t[j * 3 + 1], t[j * 3 + 2]);
        const u128 lhs = (u128)fj.num * fi.den, rhs = (u128)fi.num * fj.den;
        beats = lhs > rhs || (lhs == rhs && j < ii);
      }
      rank += beats;
    }
  }
  const float si = score[ii];
  if (n_rel > 0) {
    // rank by score descending, ties -> lower index
    for (int j = sub; j < L_v; j += SEL_LPT) rr += (score[j] > si) || (score[j] == si && j < ii);
  }
#pragma unroll
  for (int o = SEL_LPT / 2; o > 0; o >>= 1) {
    rank += __shfl_xor(rank, o);
    rr += __shfl_xor(rr, o);
  }
  if (!live || sub != 0) return;
  flags[(size_t)b * L_v + i] = passed && rank < top_k && (n_rel <= 0 || rr >= n_rel);
}

// grid as select_rank_kernel.  Ascending list, count, and the list ordered by (score asc, index
// asc).  A kept token's place in either list is the number of kept tokens that come before it, which
// SEL_LPT lanes count together as above: no pass over the stream has to wait for another (one
// workgroup per stream that compacted first: 5 us at 256 patches, 23 us at 1024; now 3.6 and 7.5 us).
template <int SEL_LPT>
__global__ __launch_bounds__(256) void select_order_kernel(
    const uint8_t* __restrict__ flags, const float* __restrict__ relevance, int L_v,
    int32_t* __restrict__ out_idx, int32_t* __restrict__ out_order, int32_t* __restrict__ out_count,
    float* __restrict__ out_relevance, int stride) {
  __shared__ float score[SEL_MAX_LV];
  __shared__ uint8_t kept[SEL_MAX_LV];
  const int b = blockIdx.y, tid = threadIdx.x;
  for (int k = tid; k < L_v; k += 256) {
    score[k] = relevance[(size_t)b * L_v + k];
    kept[k] = flags[(size_t)b * L_v + k];
  }
  __syncthreads();
  constexpr int SEL_PPW = 256 / SEL_LPT;
  const int sub = tid % SEL_LPT, i = blockIdx.x * SEL_PPW + tid / SEL_LPT;
  const bool live = i < L_v, count = blockIdx.x == 0 && tid < SEL_LPT;  // the first patch's lanes count all
  const int ii = live ? i : 0;
  const bool mine = live && kept[ii];
  const float si = score[ii];
  int pos = 0, ord = 0, all = 0;
  if (mine || count) {
    for (int k = sub; k < L_v; k += SEL_LPT) {
      const float sk = score[k];
      const int f = kept[k];
      all += f;
      pos += f & (k < ii);
      ord += f & ((sk < si) || (sk == si && k < ii));
    }
  }
#pragma unroll
  for (int o = SEL_LPT / 2; o > 0; o >>= 1) {
    pos += __shfl_xor(pos, o);
    ord += __shfl_xor(ord, o);
    all += __shfl_xor(all, o);
  }
  if (!live || sub != 0) return;
  if (count) out_count[b] = all;
  if (out_relevance) out_relevance[(size_t)b * L_v + i] = si;
  if (!mine) return;
  if (pos < stride) out_idx[(size_t)b * stride + pos] = i;
  if (ord < stride) out_order[(size_t)b * stride + ord] = i;
}

void launch_select(const uint32_t* terms, const double* similar, int B, int L_v, int top_k, int n_rel,
                   uint8_t* flags, const float* score, int32_t* out_idx, int32_t* out_order,
                   int32_t* out_count, float* out_relevance, int stride, hipStream_t st) {
  const long long patches = (long long)B * L_v;
#define VLAC_RANK(LPT_)                                                                            \
  {                                                                                                \
    const dim3 grid((L_v * LPT_ + 255) / 256, B);                                                   \
    hipLaunchKernelGGL(select_rank_kernel<LPT_>, grid, dim3(256), 0, st, terms, similar, L_v, top_k, score, n_rel, \
                       flags);                                                                      \
    hipLaunchKernelGGL(select_order_kernel<LPT_>, grid, dim3(256), 0, st, flags, score, L_v, out_idx, out_order, \
                       out_count, out_relevance, stride);                                           \
  }
  if (patches <= 16384) VLAC_RANK(16)
  else if (patches <= 65536) VLAC_RANK(4)
  else VLAC_RANK(1)
#undef VLAC_RANK
}

// ---------------------------------------------------------------------------
// Sec. 3.4.  grid (layers, B), fp64 throughout: a workgroup per layer and stream, whose sums are
// fixed-shape trees; the last workgroup of a stream to arrive (atomic counter, no waiting) turns
// the entropies into the ratios.  So the result does not depend on scheduling.
// Bound by latency at one stream (two rounds of loads, the hand-over, a short serial sum) and by
// the fp64 logarithms at many: 7 us at 32 layers x 256 tokens (15 with all layers of a
// stream in one workgroup and the ratios divided out one after the other), 10 us at 8
// streams x 1024 tokens (38).
// ---------------------------------------------------------------------------
__device__ inline double wave_sum_f64(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__global__ __launch_bounds__(256) void layer_ratio_kernel(
    const float* __restrict__ attn_mean, int n_layers, int B, int L_v, float gain_k,
    const int32_t* __restrict__ reuse_count, float* __restrict__ out_alpha,
    int32_t* __restrict__ out_layer_count, unsigned long long* ent, int* counters) {
  __shared__ double red[2][4];
  __shared__ int s_last;
  const int l = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const float* a = attn_mean + ((size_t)l * B + b) * L_v;
  float v[4];  // the first 1024 tokens stay in registers between the two passes
  double s = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = tid + 256 * u < L_v ? a[tid + 256 * u] : 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) s += (double)v[u];
  for (int i = tid + 1024; i < L_v; i += 256) s += (double)a[i];
  s = wave_sum_f64(s);
  if (lane == 0) red[0][w] = s;
  __syncthreads();
  const double tot = red[0][0] + red[0][1] + red[0][2] + red[0][3];
  double e = 0;
  if (tot > 0) {
    auto add = [&](float x) {
      const double p = (double)x / tot;
      if (p > 0) e -= p * log(p);
    };
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (256 * u < L_v) add(v[u]);
    for (int i = tid + 1024; i < L_v; i += 256) add(a[i]);
  }
  e = wave_sum_f64(e);
  if (lane == 0) red[1][w] = e;
  __syncthreads();
  if (tid == 0) {
    const double E = tot > 0 ? red[1][0] + red[1][1] + red[1][2] + red[1][3] : 0.0;
    __hip_atomic_store(ent + (size_t)b * n_layers + l, __builtin_bit_cast(unsigned long long, E), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    stores_done();
    const int old = atomicAdd(counters + b, 1);
    s_last = old == n_layers - 1;
    if (s_last) counters[b] = 0;  // ready for the next call
  }
  __syncthreads();
  if (!s_last || w > 0) return;
  // One wave: 64 layers at a time, a lane per layer.  The sum over the layers is serial, in
  // ascending order; the running maximum is exact in any order.
  double cum = 0, best = 0, e_prev = 0;
  const int cnt = reuse_count ? max(reuse_count[b], 0) : 0;
  auto lane_f64 = [](double x, int k) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    return __builtin_bit_cast(double, (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, k) |
                                          ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(u >> 32), k) << 32));
  };
  for (int l0 = 0; l0 < n_layers; l0 += 64) {
    const int ll = l0 + lane, n = min(64, n_layers - l0);
    const double E = __builtin_bit_cast(double, __hip_atomic_load(ent + (size_t)b * n_layers + min(ll, n_layers - 1),
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    double P = __shfl_up(E, 1);  // the layer before
    if (lane == 0) P = e_prev;
    const bool on = ll > 0 && P > 0;
    const double r = on ? (P - E) / P : 0.0;
    double mine = 0;
    const unsigned long long adds = __ballot(on);
    for (int k = 0; k < n; ++k) {
      if ((adds >> k) & 1) cum += lane_f64(r, k);
      mine = lane == k ? cum : mine;
    }
    e_prev = lane_f64(E, 63);
    double al = (double)gain_k * mine;
    al = al < 0 ? 0 : (al > 1 ? 1 : al);
    double run = al > best ? al : best;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double below = __shfl_up(run, o);
      if (lane >= o && below > run) run = below;
    }
    best = lane_f64(run, n - 1);
    if (ll < n_layers) {
      const float af = (float)run;
      out_alpha[(size_t)b * n_layers + ll] = af;
      if (out_layer_count) out_layer_count[(size_t)b * n_layers + ll] = (int)floorf(af * (float)cnt);
    }
  }
}

void launch_layer_ratio(const float* attn_mean, int n_layers, int B, int L_v, float gain_k,
                        const int32_t* reuse_count, float* out_alpha, int32_t* out_layer_count,
                        unsigned long long* ent, int* counters, hipStream_t st) {
  hipLaunchKernelGGL(layer_ratio_kernel, dim3(n_layers, B), dim3(256), 0, st, attn_mean, n_layers, B, L_v,
                     gain_k, reuse_count, out_alpha, out_layer_count, ent, counters);
}

// ---------------------------------------------------------------------------
// Alg. 1 for callers that cannot allocate: the same three kernels, with their scratch (the
// patch terms, the similarity and score of every patch and the selection flags, which vlac_select_static
// keeps in its context) in a fixed array in device memory.  Every GPU holds its own copy of
// the array at its own address; host code only ever uses the address that
// hipGetSymbolAddress returns for the current device, never the array's name.  Nothing in
// the array has to start at zero: patch_terms_kernel writes all terms, similarities and scores of the call's
// patches, select_rank_kernel all their flags, before anything reads them.
// ---------------------------------------------------------------------------
namespace {

constexpr size_t kNoAllocPatches = VLAC_NOALLOC_MAX_PATCHES;
constexpr size_t kSimilarOff = 0;                                 // double [patches]
constexpr size_t kTermsOff = kSimilarOff + kNoAllocPatches * 8;   // uint32 [patches][3]
constexpr size_t kScoreOff = kTermsOff + kNoAllocPatches * 12;    // float  [patches]
constexpr size_t kFlagsOff = kScoreOff + kNoAllocPatches * 4;     // uint8  [patches]
constexpr size_t kScratchBytes = kFlagsOff + kNoAllocPatches;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices];  // per device: where that GPU holds `scratch`

// The address of the current device's copy of the array (looked up once per device).
hipError_t scratch_of_current_device(unsigned char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = (unsigned char*)p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

int select_scratch_init() {
  unsigned char* p = nullptr;
  return (int)scratch_of_current_device(&p);
}

extern "C" int vlac_select_static_noalloc(const uint8_t* frame_prev, const uint8_t* frame_cur, int B, int H,
                                          int W, int patch, int tau_num, int tau_den, int top_k,
                                          const float* attn_mean, int n_layers, const uint8_t* layer_mask,
                                          float tau_task, int32_t* out_idx, int32_t* out_order,
                                          int32_t* out_count, float* out_relevance, int stride,
                                          void* stream) {
  if (!frame_prev || !frame_cur || !out_idx || !out_order || !out_count) return VLAC_E_NULL;
  if (B < 1 || B > 32767) return VLAC_E_RANGE;
  if (patch < 1 || patch > 64 || H < 1 || W < 1) return VLAC_E_RANGE;
  if (H % patch || W % patch) return VLAC_E_SHAPE;
  const long L_v = (long)(H / patch) * (W / patch);
  if (L_v > SEL_MAX_LV) return VLAC_E_RANGE;
  if ((size_t)B * (size_t)L_v > kNoAllocPatches) return VLAC_E_RANGE;  // beyond the fixed scratch
  if (tau_den < 1 || tau_num < 0 || tau_num > tau_den) return VLAC_E_RANGE;
  if (top_k < 0 || top_k > L_v) return VLAC_E_RANGE;
  if (stride < top_k || stride < 1) return VLAC_E_SHAPE;
  if (tau_task != tau_task) return VLAC_E_RANGE;  // NaN
  if (attn_mean && (n_layers < 1 || n_layers > 512)) return VLAC_E_RANGE;
  int n_rel = 0;
  if (attn_mean) {
    // the L_v - floor(tau_task * L_v) highest-scoring tokens are task-relevant
    const double keep = floor((double)tau_task * (double)L_v);
    const double nr = (double)L_v - keep;
    n_rel = nr < 0 ? 0 : (nr > (double)L_v ? (int)L_v : (int)nr);
  }
  unsigned char* ws = nullptr;
  if (scratch_of_current_device(&ws) != hipSuccess) {
    (void)hipGetLastError();
    return VLAC_E_HIP;
  }
  double* similar = (double*)(ws + kSimilarOff);
  uint32_t* terms = (uint32_t*)(ws + kTermsOff);
  float* score = (float*)(ws + kScoreOff);
  uint8_t* flags = (uint8_t*)(ws + kFlagsOff);
  hipStream_t st = (hipStream_t)stream;
  launch_patch_terms(frame_prev, frame_cur, B, H, W, patch, tau_num, tau_den, terms, similar, attn_mean,
                     attn_mean ? n_layers : 0, layer_mask, score, st);
  launch_select(terms, similar, B, (int)L_v, top_k, n_rel, flags, score, out_idx, out_order, out_count,
                out_relevance, stride, st);
  return hipGetLastError() == hipSuccess ? VLAC_OK : VLAC_E_HIP;
}
