// Refinement importance of the active regions (the Patch Gate's own signal):
// R_i = |A_i|^-2 sum_{u,v in A_i} SA_uv with SA one block's self-attention
// averaged over its heads, recomputed for the pairs inside each active region
// from that block's queries, key cache and per-query softmax normalisers (base-2
// log-sum-exp of the scaled scores, written by the attention kernel); then
// Delta_i = |R_i - Rbar_i| and Rbar_i = R_i.  The full attention matrix is never
// formed: only |A_i|^2 scores per region and head.
#include <type_traits>

#include "fd_common.h"

namespace {

constexpr int kImpMaxWaves = 8;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// pos[idx[i]] = i for i < M: the active row of every active token.  The entry and M
// are loaded together (idx holds n entries, those past M unused).
__global__ __launch_bounds__(256) void row_of_token_kernel(const int32_t* __restrict__ idx,
                                                           const int32_t* __restrict__ m_dev, int n,
                                                           int32_t* __restrict__ pos) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int u = i < n ? idx[i] : 0;
  if (i < min(*m_dev, n)) pos[u] = i;
}

// LDS place of 16-byte chunk c of key row k of the region: 16 lanes reading one chunk of
// 16 consecutive rows hit 16 different bank groups.
template <int DH>
FD_DEVICE int key_chunk(int k, int c) {
  constexpr int KCH = DH / 8;
  return k * KCH + (c ^ (KCH >= 16 ? k & 15 : KCH == 8 ? (k >> 1) & 7 : (k >> 3) & (KCH - 1)));
}

// part[r][h] = sum_{u in A_r} sum_{v in A_r} exp2(scale_log2 * q_u,h . k_v,h - lse_u,h)
// for active regions r; one workgroup per (region, head), a wave per tile of 32 query
// rows.  The scores come from v_mfma_f32_32x32x16_bf16 with the keys as the first
// operand, so a lane holds 16 keys of one query and needs that query's normaliser only.
// The region's key rows of the head are brought into LDS once, in whole rows; the chain
// token -> row -> query rows of a wave's first tile runs beside those loads.  A ragged
// last key tile re-reads the region's last row, and is masked.  Sums in fp32 (four
// chains per lane, the workgroup's in wave order).  Video step (42 regions of 234
// tokens, 12 heads x 128): 285 us with one query row per lane and v_dot2 products, 24
// now, where 60 MB of scattered query and key rows take 10 and the empty workgroups of
// skipped regions 3; 32 us with two query tiles per wave, 36 with four waves.
template <int DH>
__global__ __launch_bounds__(kImpMaxWaves * 64) void importance_partial_kernel(
    const int32_t* __restrict__ region_ptr, const int32_t* __restrict__ region_tokens,
    const uint8_t* __restrict__ active, const int32_t* __restrict__ pos, const uint16_t* __restrict__ q,
    const uint16_t* __restrict__ kc, const float* __restrict__ lse, int D, int H, float scale_log2,
    float* __restrict__ part) {
  constexpr int KS = DH / 16, KCH = DH / 8, U = 8;   // k16 steps and chunks of the head dim; loads in flight
  extern __shared__ u32x4_t s_key[];   // [n][KCH]
  __shared__ float wsum[kImpMaxWaves];
  const int r = blockIdx.x, h = blockIdx.y;
  const int t0 = region_ptr[r], n = region_ptr[r + 1] - t0;
  if (!active[r]) return;   // whole workgroup
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int l32 = lane & 31, lg = lane >> 5;
  const int32_t* toks = region_tokens + t0;
  const int total = n * KCH, tiles = (n + 31) / 32, step = static_cast<int>(blockDim.x);
  u32x4_t qf[KS];
  float li = 0.f;
  auto load_queries = [&](int row) {
    const u32x4_t* qr = reinterpret_cast<const u32x4_t*>(q + static_cast<size_t>(row) * D + h * DH + 8 * lg);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = qr[2 * ks];
    li = lse[static_cast<size_t>(row) * H + h];
  };
  auto key_row = [&](int tok) { return reinterpret_cast<const u32x4_t*>(kc + static_cast<size_t>(tok) * D + h * DH); };
  // the chain token -> row -> query rows of the first tile runs beside the key loads
  const int tok_q = toks[min(wave * 32 + l32, n - 1)];
  int tok_k[U];
#pragma unroll
  for (int u = 0; u < U; ++u) tok_k[u] = toks[min(static_cast<int>(threadIdx.x) + u * step, total - 1) / KCH];
  const int row_q = pos[tok_q];
  u32x4_t v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = key_row(tok_k[u])[min(static_cast<int>(threadIdx.x) + u * step, total - 1) % KCH];
  load_queries(row_q);
  for (int e0 = threadIdx.x;;) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * step;
      if (e < total) s_key[key_chunk<DH>(e / KCH, e % KCH)] = v[u];
    }
    e0 += U * step;
    if (e0 - static_cast<int>(threadIdx.x) >= total) break;   // the same for every thread
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = min(e0 + u * step, total - 1);
      v[u] = key_row(toks[e / KCH])[e % KCH];
    }
  }
  __syncthreads();
  float sum = 0.f;
  for (int qt = wave; qt < tiles; qt += waves) {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    auto key_tile = [&](int kt, auto ragged) {
      const int k = ragged.value ? min(kt * 32 + l32, n - 1) : kt * 32 + l32;
      f32x16_t s = {};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, s_key[key_chunk<DH>(k, 2 * ks + lg)]),
                                                    __builtin_bit_cast(bf16x8_t, qf[ks]), s, 0, 0, 0);
      const int left = n - kt * 32 - 4 * lg;   // this lane's keys 8 (e / 4) + e % 4 below it are in the region
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float p = __builtin_amdgcn_exp2f(s[e] * scale_log2 - li);
        acc[e & 3] += !ragged.value || 8 * (e >> 2) + (e & 3) < left ? p : 0.f;
      }
    };
    for (int kt = 0; kt < n / 32; ++kt) key_tile(kt, std::false_type{});
    if (n % 32) key_tile(n / 32, std::true_type{});
    sum += qt * 32 + l32 < n ? (acc[0] + acc[1]) + (acc[2] + acc[3]) : 0.f;
    if (qt + waves < tiles) load_queries(pos[toks[min((qt + waves) * 32 + l32, n - 1)]]);
  }
  sum = fd::wave_sum(sum);
  if (lane == 0) wsum[wave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
    for (int w = 0; w < waves; ++w) t += wsum[w];
    part[static_cast<size_t>(r) * H + h] = t;
  }
}

// Active regions: R = (sum_h part[r][h]) / (H |A_r|^2), Delta = |R - Rbar|, Rbar = R;
// skipped regions keep both.  importance[r] = R (NaN for skipped ones) when given.
__global__ __launch_bounds__(64) void importance_update_kernel(const int32_t* __restrict__ region_ptr,
                                                                const uint8_t* __restrict__ active,
                                                                const float* __restrict__ part, int R, int H,
                                                                double* __restrict__ r_bar,
                                                                double* __restrict__ delta,
                                                                double* __restrict__ importance) {
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < R; r += gridDim.x * blockDim.x) {
    if (active[r]) {
      double sum = 0.0;
#pragma unroll 8
      for (int h = 0; h < H; ++h) sum += static_cast<double>(part[static_cast<size_t>(r) * H + h]);
      const double n = static_cast<double>(region_ptr[r + 1] - region_ptr[r]);
      const double imp = sum / (static_cast<double>(H) * n * n);
      delta[r] = fabs(imp - r_bar[r]);
      r_bar[r] = imp;
      if (importance) importance[r] = imp;
    } else if (importance) {
      importance[r] = __builtin_nan("");
    }
  }
}

}  // namespace

namespace fdh {

size_t importance_lds_bytes(int dh, int max_region_tokens) {
  return static_cast<size_t>(max_region_tokens) * (dh / 2) * sizeof(uint32_t);
}

hipError_t launch_importance(const fd_plan* p, int D, int H, int dh, const int32_t* idx, const int32_t* m,
                             const uint8_t* active, const uint16_t* q, const uint16_t* kc, const float* lse,
                             int32_t* pos, float* part, double* r_bar, double* delta, double* importance,
                             hipStream_t s) {
  row_of_token_kernel<<<(p->n_tokens + 255) / 256, 256, 0, s>>>(idx, m, p->n_tokens, pos);
  const float scale_log2 = 1.4426950408889634f / sqrtf(static_cast<float>(dh));
  const size_t lds = importance_lds_bytes(dh, p->max_region_tokens);
  const int tiles = (p->max_region_tokens + 31) / 32;
  const int threads = 64 * (tiles < kImpMaxWaves ? tiles : kImpMaxWaves);
  const dim3 grid(p->n_regions, H);
#define FD_IMP(DHV)                                                                                                   \
  importance_partial_kernel<DHV><<<grid, threads, lds, s>>>(p->region_ptr, p->region_tokens, active, pos, q, kc, lse, \
                                                            D, H, scale_log2, part)
  switch (dh) {
    case 16: FD_IMP(16); break;
    case 64: FD_IMP(64); break;
    case 128: FD_IMP(128); break;
    default:
      return hipErrorInvalidValue;
  }
#undef FD_IMP
  const int ugrid = (p->n_regions + 63) / 64;
  importance_update_kernel<<<ugrid, 64, 0, s>>>(p->region_ptr, active, part, p->n_regions, H, r_bar, delta,
                                                 importance);
  return hipGetLastError();
}

}  // namespace fdh
