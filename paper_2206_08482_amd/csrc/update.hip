// Trainer role (Section 3 of the paper, "DRL Trainer"; stage (ii) of Section 5.1): clipped-surrogate
// loss, exact backward through both MLPs, Adam on the fp32 master parameters, shadow refresh.
#include <math.h>
#include <algorithm>

#include "internal.h"

namespace {

__device__ __forceinline__ uint16_t f_to_bf16_u(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ void store_elem(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_elem(uint16_t* p, float v) { *p = f_to_bf16_u(v); }

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// One thread per sample (grid-stride).  Per workgroup partial sums go to
//   stat_part[blk][0..4] = sum policy term, sum value term, entropy (workgroup 0 only), sum kl, sum clipped
//   stat_part[blk][kStatStride + j] = partial dL/dlog_std_j (without the entropy term)
// and, if want_grad, dL/dmu and dL/dv rows are written for the backward products.
template <typename T>
__global__ __launch_bounds__(256) void loss_kernel(int rows, int A, const float* __restrict__ mu,
                                                   const float* __restrict__ val, const float* __restrict__ act,
                                                   const float* __restrict__ logp_old, const float* __restrict__ adv,
                                                   const float* __restrict__ ret, const float* __restrict__ log_std,
                                                   float clip, float c_v, int want_grad, T* __restrict__ dmu,
                                                   int ld_dmu, T* __restrict__ dv, int ld_dv,
                                                   float* __restrict__ stat_part) {
  extern __shared__ float sh[];            // [4][A] log_std partials, then [4][4] stats
  float* s_dls = sh;
  float* s_st = sh + 4 * A;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < 4 * A + 16; i += 256) sh[i] = 0.f;
  __syncthreads();
  const float inv_m = 1.0f / (float)rows;
  float s_pl = 0.f, s_vl = 0.f, s_kl = 0.f, s_cf = 0.f;
  const int n_iter = (rows + gridDim.x * 256 - 1) / (gridDim.x * 256);
  for (int it = 0; it < n_iter; ++it) {
    const int r = (it * gridDim.x + blockIdx.x) * 256 + tid;
    const bool ok = r < rows;
    float lp = 0.f;
    if (ok) {
      for (int j = 0; j < A; ++j) {
        const float ls = log_std[j];
        const float z = (act[(int64_t)r * A + j] - mu[(int64_t)r * A + j]) * expf(-ls);
        lp += -0.5f * z * z - ls - 0.918938533204672742f;
      }
    }
    float g_lp = 0.f;
    if (ok) {
      const float lo = logp_old[r], a = adv[r];
      const float ratio = expf(lp - lo);
      const float s1 = ratio * a;
      const float s2 = fminf(fmaxf(ratio, 1.0f - clip), 1.0f + clip) * a;
      s_pl += -fminf(s1, s2);
      s_kl += lo - lp;
      s_cf += fabsf(ratio - 1.0f) > clip ? 1.f : 0.f;
      g_lp = (s1 <= s2) ? -(a * ratio) * inv_m : 0.f;
      const float dvv = val[r] - ret[r];
      s_vl += dvv * dvv;
      if (want_grad) store_elem(dv + (int64_t)r * ld_dv, 2.0f * c_v * dvv * inv_m);
    }
    // dL/dmu_j = g_lp * z_j / sigma_j ;  dL/dlog_std_j += g_lp * (z_j^2 - 1)   (wave reduction per j)
    for (int j = 0; j < A; ++j) {
      float c = 0.f;
      if (ok) {
        const float inv_sigma = expf(-log_std[j]);
        const float z = (act[(int64_t)r * A + j] - mu[(int64_t)r * A + j]) * inv_sigma;
        if (want_grad) store_elem(dmu + (int64_t)r * ld_dmu + j, g_lp * z * inv_sigma);
        c = g_lp * (z * z - 1.0f);
      }
      c = wave_sum_f(c);
      if (lane == 0) s_dls[wave * A + j] += c;
    }
  }
  s_pl = wave_sum_f(s_pl); s_vl = wave_sum_f(s_vl); s_kl = wave_sum_f(s_kl); s_cf = wave_sum_f(s_cf);
  if (lane == 0) { s_st[wave * 4 + 0] = s_pl; s_st[wave * 4 + 1] = s_vl; s_st[wave * 4 + 2] = s_kl; s_st[wave * 4 + 3] = s_cf; }
  __syncthreads();
  float* out = stat_part + (int64_t)blockIdx.x * (gmi::kStatStride + A);
  if (tid < 4) {
    const float v = s_st[tid] + s_st[4 + tid] + s_st[8 + tid] + s_st[12 + tid];
    const int slot = tid == 0 ? 0 : (tid == 1 ? 1 : (tid == 2 ? 3 : 4));
    out[slot] = v;
  }
  if (tid == 4) {
    float ent = 0.f;
    if (blockIdx.x == 0)
      for (int j = 0; j < A; ++j) ent += log_std[j] + 1.418938533204672742f;
    out[2] = ent;
  }
  for (int j = tid; j < A; j += 256)
    out[gmi::kStatStride + j] = s_dls[j] + s_dls[A + j] + s_dls[2 * A + j] + s_dls[3 * A + j];
}

struct AdamScalars {
  float lr, b1, b2, eps, c1, c2;   // c1 = 1 - b1^k, c2 = 1 - b2^k
};

// Adam step of one parameter given its gradient (Adam as in the PPO trainer of Section 2: bias-corrected
// moments, epsilon outside the square root).
__device__ __forceinline__ float adam_one(float g, float* __restrict__ params, float* __restrict__ am,
                                          float* __restrict__ av, int64_t p, const AdamScalars& hs) {
  const float m = hs.b1 * am[p] + (1.0f - hs.b1) * g;
  const float v = hs.b2 * av[p] + (1.0f - hs.b2) * g * g;
  am[p] = m;
  av[p] = v;
  const float w = params[p] - hs.lr * (m / hs.c1) / (sqrtf(v / hs.c2) + hs.eps);
  params[p] = w;
  return w;
}

// The same expressions on values held in registers: m, v and w are updated.
__device__ __forceinline__ void adam_step(float g, float& m, float& v, float& w, const AdamScalars& hs) {
  m = hs.b1 * m + (1.0f - hs.b1) * g;
  v = hs.b2 * v + (1.0f - hs.b2) * g * g;
  w = w - hs.lr * (m / hs.c1) / (sqrtf(v / hs.c2) + hs.eps);
}

// Gradient partials of the trainer instances whose replicas are reduced into one update (one entry for an
// ordinary single-instance update): per instance [n_split, part_stride] weight partials (of tiled ones as many rows as the layer
// has splits) and the loss kernel's [n_stat, kStatStride + A] statistics partials.  The counts are the replica's own: they follow from the path
// its instance takes (gmi_set_fusion, compute units).
constexpr int kMaxGroup = 16;
struct Partials {
  const float *part, *stat;      // stat NULL: a caller-supplied gradient
  int n_split, n_stat;           // n_split: partials in flat order
};
struct PartSet {
  int n;
  Partials r[kMaxGroup];
  gmi::WgradSplits split[kMaxGroup];      // partials in tiled order
};
// Partials are read once: streaming loads leave no copy in this die's cache, which the next minibatch's workgroups, on other dies, would
// have to wait for when they write the same lines.  (us per iteration without / with: 45:128:128:12 657 / 620, 108:400:200:100:21 3240 / 3108;
// a workgroup of the former spent 14 thousand cycles storing its partial gradient, 3 thousand into lines that nobody had read.)
typedef float floatx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 stream_load4(const float* p) {
  const floatx4 t = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(p));
  return make_float4(t.x, t.y, t.z, t.w);
}
// (by words: the argument segment has no scalar byte loads)
__device__ __forceinline__ int layer_splits(const PartSet& ps, int replica, int li) {
  return reinterpret_cast<const uint32_t*>(ps.split[replica].n)[li >> 2] >> (8 * (li & 3)) & 255;
}

// Sum over the replicas and splits of the partials at p, splits grp, grp + G, grp + 2 G, ...: fixed order of additions,
// 16 (then 4) loads in flight.
template <int G>
__device__ __forceinline__ float sum_partials(const PartSet& ps, int64_t p, int64_t part_stride, int grp) {
  float g = 0.f;
  Partials r = ps.r[0];      // the first entry comes with the other arguments, ahead of the loop
  for (int i = 1;; ++i) {
    const float* q = r.part + p;
    const int n_split = r.n_split;
    int s = grp;
    for (; s + 15 * G < n_split; s += 16 * G) {
      float t[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) t[u] = q[(int64_t)(s + u * G) * part_stride];
#pragma unroll
      for (int u = 0; u < 16; ++u) g += t[u];
    }
    for (; s + 3 * G < n_split; s += 4 * G) {
      float t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = q[(int64_t)(s + u * G) * part_stride];
#pragma unroll
      for (int u = 0; u < 4; ++u) g += t[u];
    }
    for (; s < n_split; s += G) g += q[(int64_t)s * part_stride];
    if (i >= ps.n) break;
    r = ps.r[i];
  }
  return g;
}

// Finalises the minibatch statistics and owns log_std, whose gradient is the sum of the loss partials minus the entropy
// coefficient: one workgroup of NT threads reduces the [n_stat, kStatStride + A] partials cooperatively (a serial
// walk by one thread per column costs one memory round trip per loss workgroup).
template <int NT>
__device__ __forceinline__ void finish_stats(const gmi::ShadowTable& tab, float* __restrict__ params, float* __restrict__ am,
                                             float* __restrict__ av, const PartSet& ps, int64_t part_stride,
                                             int A, float c_e, float inv_rows, const AdamScalars& hs,
                                             float* __restrict__ log_std_shadow, float* __restrict__ stats_out,
                                             float* __restrict__ grad_out, int do_update, float* s_col) {
  const int C = gmi::kStatStride + A;              // columns of a statistics row
  const int tid = threadIdx.x;
  // up to NT columns per pass; narrow rows are walked by NT / C row groups in parallel
  const int width = C < NT ? C : NT;
  const int groups = NT / width;
  const bool have_stat = ps.r[0].stat != nullptr;
  const float inv_n = 1.0f / (float)ps.n;
  for (int cbase = 0; cbase < C; cbase += NT) {
    const int col = cbase + tid % width, grp = tid / width;
    float s = 0.f;
    if (have_stat && grp < groups && col < C)
      for (int i = 0; i < ps.n; ++i) {
        // rows grp, grp + groups, ...: 16 loads in flight, fixed order of additions
        const float* q = ps.r[i].stat + col;
        const int n_stat = ps.r[i].n_stat;
        int b = grp;
        for (; b + 15 * groups < n_stat; b += 16 * groups) {
          float t[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) t[u] = q[(int64_t)(b + u * groups) * C];
#pragma unroll
          for (int w = 8; w > 0; w >>= 1)
#pragma unroll
            for (int u = 0; u < w; ++u) t[u] += t[u + w];
          s += t[0];
        }
        for (; b + 7 * groups < n_stat; b += 8 * groups) {
          float t[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) t[u] = q[(int64_t)(b + u * groups) * C];
          s += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        }
        for (; b < n_stat; b += groups) s += q[(int64_t)b * C];
      }
    s_col[tid] = s;
    __syncthreads();
    const int c = cbase + tid;
    if (tid < width && c < C) {
      float t = 0.f;
      for (int q = 0; q < groups; ++q) t += s_col[q * width + tid];
      t *= inv_n;                                   // mean over the replicas (exact for one)
      if (have_stat && stats_out && c < 5) stats_out[c] = c == 2 ? t : t * inv_rows;
      if (c >= gmi::kStatStride) {
        const int j = c - gmi::kStatStride;
        const int64_t p = tab.logstd_off + j;
        // without loss partials (a caller-supplied gradient) log_std takes the split sums like any weight
        float g = 0.f;
        if (have_stat) g = t - c_e;
        else for (int q = 0; q < ps.r[0].n_split; ++q) g += ps.r[0].part[(int64_t)q * part_stride + p];
        if (grad_out) grad_out[p] = g;
        if (do_update) {
          const float w = adam_one(g, params, am, av, p, hs);
          if (log_std_shadow) log_std_shadow[j] = w;
        }
      }
    }
    __syncthreads();
  }
}

// fp32 models and caller-supplied gradients (partials in flat parameter order): a workgroup of 64 G waves'
// worth of threads owns 256 consecutive parameters, G threads per parameter each summing every G-th partial row.
// grad(p) = (1/n) sum_i sum_s part_i[s * part_stride + p]: the in-memory mean over the n replicas (Section 4.1's gradient
// reduction for instances that share one address space), fixed summation order.  The first workgroup finalises the
// statistics and log_std: its walk over the statistics rows is the longest way of all.
template <int G>
__global__ __launch_bounds__(256 * G) void adam_kernel(gmi::ShadowTable tab, float* __restrict__ params,
                                                       float* __restrict__ am, float* __restrict__ av, PartSet ps,
                                                       int64_t part_stride, int A, float c_e, float inv_rows, AdamScalars hs,
                                                       float* __restrict__ stats_out, float* __restrict__ grad_out,
                                                       int do_update) {
  __shared__ float s_sum[256 * G];
  if (blockIdx.x == 0) {
    finish_stats<256 * G>(tab, params, am, av, ps, part_stride, A, c_e, inv_rows, hs, nullptr,
                          stats_out, grad_out, do_update, s_sum);
    return;
  }
  const int t = threadIdx.x & 255, grp = threadIdx.x >> 8;
  const int64_t p = (int64_t)(blockIdx.x - 1) * 256 + t;
  const bool ok = p < tab.logstd_off;
  // the moments and the parameter are fetched ahead of the partials (their latency would otherwise follow the sum's)
  float m0 = 0.f, v0 = 0.f, w0 = 0.f;
  if (do_update && ok && grp == 0) { m0 = am[p]; v0 = av[p]; w0 = params[p]; }
  float g = ok ? sum_partials<G>(ps, p, part_stride, grp) : 0.f;
  if constexpr (G > 1) {
    s_sum[threadIdx.x] = g;
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int q = 1; q < G; ++q) g += s_sum[q * 256 + t];
  }
  if (!ok) return;
  g *= 1.0f / (float)ps.n;
  if (grad_out) grad_out[p] = g;
  if (!do_update) return;
  adam_step(g, m0, v0, w0, hs);
  am[p] = m0;
  av[p] = v0;
  params[p] = w0;
}

// Index of block (feature tile ft, k step ks) inside a chain-stream segment of nft tiles and nks k steps whose
// tiles are grouped gm, .., gm, (2), (1): groups one after the other, a group's blocks k step major.
__device__ __forceinline__ int chain_block_index(int nft, int nks, int gm, int ft, int ks) {
  const int full = nft / gm;
  int base, gs, t;
  if (ft < gm * full) {
    const int gi = ft / gm;
    base = gi * gm * nks; gs = gm; t = ft - gi * gm;
  } else {
    base = full * gm * nks;
    const int r = ft - gm * full;
    if ((nft % gm) >= 2) {
      if (r < 2) { gs = 2; t = r; }
      else { base += 2 * nks; gs = 1; t = 0; }
    } else {
      gs = 1; t = 0;
    }
  }
  return base + ks * gs + t;
}

// BF16 models: the sum of the partials, Adam and every bf16 copy of the weights in one pass (a second kernel that rebuilt
// the transposed copies from the first one's output cost 5-6 us per minibatch, most of it launch and round trips).  A
// workgroup owns one quad of one 32 x 32 tile of the partials (ModelLayout::part_floats) = 8 outputs x 32 inputs, i.e. 1 KiB
// of every partial row, and just what the copies' 16-byte pieces need: 8 consecutive inputs of an output (row-major and
// fragment-major W), 8 consecutive outputs of an input (W^T, its fragment-major copy), the chain streams' permuted k
// orders; in the first input tile also the 8 biases.  Wave w sums the partial rows w, w + 4, ...  grad_out: the gradient
// into the flat parameter order instead, updating nothing.
struct AdamTiles {
  int n;
  int start[gmi::kMaxWgradProblems + 1];
};
template <int U>
__global__ __launch_bounds__(256) void adam_shadow_kernel(gmi::ShadowTable tab, AdamTiles tt, gmi::ChainEmit ce,
                                                          float* __restrict__ params, float* __restrict__ am,
                                                          float* __restrict__ av, PartSet ps, int64_t part_stride,
                                                          int A, float c_e, float inv_rows, AdamScalars hs, char* __restrict__ shadow,
                                                          float* __restrict__ stats_out, float* __restrict__ grad_out,
                                                          int do_update) {
  __shared__ __attribute__((aligned(16))) float s_sum[4][256];
  __shared__ float s_bsum[4][8];
  __shared__ __attribute__((aligned(16))) uint16_t s_t[8][40];
  const int n_tiles = gridDim.x - 1;
  // first: its walk over the statistics rows is the longest way of all (last and with half the loads in flight, us:
  // 108:400:200:100:21 with 512 rows of them 13.5, now 11.0; 211:512:512:256:128:20 with 256 26.6, now 24.0)
  if (blockIdx.x == 0) {
    finish_stats<256>(tab, params, am, av, ps, part_stride, A, c_e, inv_rows, hs,
                      do_update ? reinterpret_cast<float*>(shadow + tab.sh_logstd) : nullptr, stats_out, grad_out, do_update, &s_sum[0][0]);
    return;
  }
  // neighbouring tiles, which share memory lines of the parameters and moments, on the same die (ids go round-robin over 8)
  const int per = n_tiles >> 3, whole = per << 3;
  const int id = (int)blockIdx.x - 1, tile = id < whole ? (id & 7) * per + (id >> 3) : id;
  int li = 0;      // the layer whose tiles hold this one (entries past the last layer hold no tile: all loads at once)
#pragma unroll
  for (int k = 1; k < gmi::kMaxWgradProblems; ++k) li += tile >= tt.start[k] ? 1 : 0;
  const gmi::ShadowLayer& L = tab.l[li];
  const int local = tile - tt.start[li], n_ti = (L.in + 31) >> 5;
  const int o0 = (local / n_ti) * 8, it = local % n_ti, i0 = it * 32;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int o = o0 + (t >> 5), i = i0 + (t & 31);
  const bool ok = o < L.out && i < L.in;
  const bool okb = i0 == 0 && t < 8 && o0 + t < L.out;
  const int64_t p = ok ? L.w_off + (int64_t)o * L.in + i : L.w_off, pb = okb ? L.b_off + o0 + t : L.b_off;
  float m0 = 0.f, v0 = 0.f, w0 = 0.f, mb = 0.f, vb = 0.f, wb = 0.f;
  if (do_update) {
    m0 = am[p]; v0 = av[p]; w0 = params[p];
    if (okb) { mb = am[pb]; vb = av[pb]; wb = params[pb]; }
  }
  const int64_t src = L.part_w + (((int64_t)(o0 >> 5) * (L.in_pad >> 5) + it) * 4 + ((o0 >> 3) & 3)) * 256 +
                      4 * (i0 + (lane & 31) < L.in ? lane : lane & 32);      // padding inputs read a neighbour
  const int64_t srcb = L.part_b + o0 + (lane & 7);
  float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
  float gb = 0.f;
  Partials r = ps.r[0];      // the first entry comes with the other arguments, ahead of the loop
  int n_split = layer_splits(ps, 0, li);
  for (int k = 1;; ++k) {
    const float* q = r.part + src;
    const float* qb = r.part + srcb;
    for (int s = wave; s < n_split; s += 4 * U) {      // rows s, s + 4, ...: all loads before the first addition, fixed order
      float4 x[U];
      float y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = stream_load4(q + (int64_t)min(s + 4 * u, n_split - 1) * part_stride);
      if (i0 == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) y[u] = qb[(int64_t)min(s + 4 * u, n_split - 1) * part_stride];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + 4 * u < n_split) {
          g.x += x[u].x; g.y += x[u].y; g.z += x[u].z; g.w += x[u].w;
          if (i0 == 0) gb += y[u];
        }
    }
    if (k >= ps.n) break;
    r = ps.r[k];
    n_split = layer_splits(ps, k, li);
  }
  *reinterpret_cast<float4*>(&s_sum[wave][lane * 4]) = g;
  if (lane < 8) s_bsum[wave][lane] = gb;
  __syncthreads();
  const float inv_n = 1.0f / (float)ps.n;
  // element of (o, i): 4 (32 h + i) + e with o - o0 = 4 h + e
  const int el = 4 * (32 * (t >> 7) + (t & 31)) + ((t >> 5) & 3);
  const float gs = (((s_sum[0][el] + s_sum[1][el]) + s_sum[2][el]) + s_sum[3][el]) * inv_n;
  const float gbs = t < 8 ? (((s_bsum[0][t] + s_bsum[1][t]) + s_bsum[2][t]) + s_bsum[3][t]) * inv_n : 0.f;
  if (grad_out) {
    if (ok) grad_out[p] = gs;
    if (okb) grad_out[pb] = gbs;
  }
  if (!do_update) return;
  adam_step(gs, m0, v0, w0, hs);
  if (ok) { am[p] = m0; av[p] = v0; params[p] = w0; }
  s_t[t >> 5][t & 31] = ok ? f_to_bf16_u(w0) : 0;
  if (okb) {
    adam_step(gbs, mb, vb, wb, hs);
    am[pb] = mb; av[pb] = vb; params[pb] = wb;
    reinterpret_cast<float*>(shadow + L.sh_b)[o0 + t] = wb;
  }
  __syncthreads();
  auto column = [&](int c) {      // the 8 outputs of input c
    uint4 v;
    v.x = s_t[0][c] | ((uint32_t)s_t[1][c] << 16); v.y = s_t[2][c] | ((uint32_t)s_t[3][c] << 16);
    v.z = s_t[4][c] | ((uint32_t)s_t[5][c] << 16); v.w = s_t[6][c] | ((uint32_t)s_t[7][c] << 16);
    return v;
  };
  const int e = t & 31;
  if (t < 32) {                    // W, row-major
    const int r = e >> 2, c = (e & 3) * 8;
    *reinterpret_cast<uint4*>(shadow + L.sh_w + 2 * ((int64_t)(o0 + r) * L.in_pad + i0 + c)) = *reinterpret_cast<const uint4*>(&s_t[r][c]);
  } else if (t < 64) {             // W, fragment-major
    const int r = e & 7, c = (e >> 3) * 8;
    *reinterpret_cast<uint4*>(shadow + L.sh_wf + 2 * gmi::wfrag_index(o0 + r, i0 + c, L.in_pad)) = *reinterpret_cast<const uint4*>(&s_t[r][c]);
  } else if (t < 96) {             // W^T, row-major
    *reinterpret_cast<uint4*>(shadow + L.sh_wt + 2 * ((int64_t)(i0 + e) * L.out_pad + o0)) = column(e);
  } else if (t < 128) {            // W^T, fragment-major
    if (L.sh_wtf >= 0) *reinterpret_cast<uint4*>(shadow + L.sh_wtf + 2 * gmi::wfrag_index(i0 + e, o0, L.out_pad)) = column(e);
  } else if (ce.gmax > 0) {
    // the chain streams of the one-launch trainer kernels: lane (s, h) of a block holds, for its row, the k indices
    // 16 ks + 8 (j / 4) + 4 h + j % 4, j = 0..7 (natural order 8 h + j in the first forward layer)
    char* cs = shadow + ce.out[li / ce.n_layers];
    const gmi::ChainEmitLayer& E = ce.l[li];
    if (t < 160) {                 // forward segment: rows = output features, k = input features
      const int r = e & 7, ks = e >> 4, h = (e >> 3) & 1, il = 16 * ks;
      uint4 v;
      if (E.natural) {
        v = *reinterpret_cast<const uint4*>(&s_t[r][il + 8 * h]);
      } else {
        const uint2 a = *reinterpret_cast<const uint2*>(&s_t[r][il + 4 * h]);
        const uint2 b = *reinterpret_cast<const uint2*>(&s_t[r][il + 8 + 4 * h]);
        v = make_uint4(a.x, a.y, b.x, b.y);
      }
      const int dst = E.fwd_blk + chain_block_index(L.out_pad >> 5, L.in_pad >> 4, ce.gmax, (o0 + r) >> 5, (i0 + il) >> 4);
      *reinterpret_cast<uint4*>(cs + ((int64_t)dst * 64 + ((o0 + r) & 31) + 32 * h) * 16) = v;
    } else if (t >= 192 && E.bwd_blk >= 0) {      // input-gradient segment: rows = input features, k = output features
      const int h = (t >> 5) & 1, q = 4 * h;      // this tile's 8 outputs are half (o0 / 8) % 2 of a k step
      const uint2 v = make_uint2(s_t[q][e] | ((uint32_t)s_t[q + 1][e] << 16), s_t[q + 2][e] | ((uint32_t)s_t[q + 3][e] << 16));
      const int dst = E.bwd_blk + chain_block_index(L.in_pad >> 5, L.out_pad >> 4, ce.gmax, i0 >> 5, o0 >> 4);
      *reinterpret_cast<uint2*>(cs + ((int64_t)dst * 64 + e + 32 * h) * 16 + 8 * ((o0 >> 3) & 1)) = v;
    }
  }
}

AdamScalars adam_scalars(const gmi_ppo_hparams* hp, uint32_t k) {
  AdamScalars s;
  s.lr = hp->lr; s.b1 = hp->beta1; s.b2 = hp->beta2; s.eps = hp->adam_eps;
  s.c1 = (float)(1.0 - pow((double)hp->beta1, (double)k));
  s.c2 = (float)(1.0 - pow((double)hp->beta2, (double)k));
  return s;
}

int check_hp(const char* fn, const gmi_ppo_hparams* hp) {
  if (!hp) GMI_FAIL(GMI_ERR_INVALID_ARG, "%s: hparams is NULL", fn);
  if (!(hp->clip >= 0.f) || !(hp->beta1 >= 0.f && hp->beta1 < 1.f) || !(hp->beta2 >= 0.f && hp->beta2 < 1.f))
    GMI_FAIL(GMI_ERR_INVALID_ARG, "%s: need clip >= 0 and betas in [0,1)", fn);
  return GMI_OK;
}

int check_model_buffer(const char* fn, gmi_model_t m, gmi_buffer_t b) {
  if (m->L.obs_dim != b->d.obs_dim || m->L.act_dim != b->d.act_dim)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "%s: model (obs %d, act %d) and buffer (obs %d, act %d) disagree", fn, m->L.obs_dim,
             m->L.act_dim, b->d.obs_dim, b->d.act_dim);
  return GMI_OK;
}

// The per-layer form of a minibatch pass: gather, forward of every layer, loss, and (want_grad) the input-gradient
// products, one launch each.  Leaves h, dz and one statistics row per loss workgroup (*n_loss_blocks_out rows).
int layers_pass(gmi_instance* g, gmi_model* m, gmi_buffer* b, const gmi_ppo_hparams* hp, const int32_t* idx, int rows,
                bool want_grad, int* n_loss_blocks_out) {
  const ModelLayout& L = m->L;
  const bool bf = L.dtype == GMI_DTYPE_BF16;
  const int A = L.act_dim;
  int rc = gmi::launch_gather(g, m, b->d.obs, b->d.n_envs, b->d.ld_envs, idx, rows, &b->d);
  if (rc != GMI_OK) return rc;
  rc = gmi::forward_nets(g, m, rows, true, true, m->mu, m->val);
  if (rc != GMI_OK) return rc;
  int nlb = (rows + 255) / 256;
  if (nlb > gmi::kLossBlocksMax) nlb = gmi::kLossBlocksMax;
  *n_loss_blocks_out = nlb;
  const float* log_std = bf ? reinterpret_cast<const float*>(m->shadow + L.sh_logstd) : m->params + L.logstd_off;
  const int head = L.n_layers - 1;
  const size_t lds = sizeof(float) * (4 * A + 16);
  {
    gmi::ProfScope ps(g, gmi::kClsLoss);
    if (bf)
      ps.launch(loss_kernel<uint16_t>, dim3(nlb), dim3(256), lds, rows, A, m->mu, m->val, m->mb_act, m->mb_logp, m->mb_adv, m->mb_ret,
                                                log_std, hp->clip, hp->c_v, want_grad ? 1 : 0,
                                                (uint16_t*)m->dz[0][head], L.net[0][head].out_pad,
                                                (uint16_t*)m->dz[1][head], L.net[1][head].out_pad, m->stat_part);
    else
      ps.launch(loss_kernel<float>, dim3(nlb), dim3(256), lds, rows, A, m->mu, m->val, m->mb_act, m->mb_logp, m->mb_adv, m->mb_ret,
                                             log_std, hp->clip, hp->c_v, want_grad ? 1 : 0, (float*)m->dz[0][head],
                                             L.net[0][head].out_pad, (float*)m->dz[1][head], L.net[1][head].out_pad,
                                             m->stat_part);
  }
  GMI_LAUNCH_CHECK();
  if (!want_grad) return GMI_OK;

  // input gradients, head to first hidden layer: dz[l-1] = (dz[l] W_l) * ELU'(h[l])
  for (int l = L.n_layers - 1; l >= 1; --l) {
    gmi::LinearBatch lb;
    lb.n = 2;
    for (int net = 0; net < 2; ++net) {
      const LayerInfo& li = L.net[net][l];
      gmi::LinearProblem& p = lb.p[net];
      p.x = m->dz[net][l]; p.ldx = li.out_pad;
      if (bf) {
        p.w = m->shadow + li.sh_wt; p.ldw = li.out_pad; p.wsf = li.out_pad; p.wsk = 1;
        p.K = li.out_pad; p.F = li.in_pad;
      } else {
        p.w = m->params + li.w_off; p.ldw = li.in; p.wsf = 1; p.wsk = li.in;
        p.K = li.out; p.F = li.in;
      }
      p.bias = nullptr;
      p.h = m->h[net][l]; p.ldh = li.in_pad;
      p.y = m->dz[net][l - 1]; p.ldy = li.in_pad;
      p.F_store = p.F;
      p.K_log = li.out; p.F_log = li.in;
    }
    rc = gmi::launch_linear(g, L.dtype, gmi::kEpiEluGrad, rows, lb);
    if (rc != GMI_OK) return rc;
  }
  return GMI_OK;
}

// Rows of gradient partials a minibatch leaves: in flat parameter order (fp32), in tiled order per layer (bf16).
struct PartRows {
  int flat;
  gmi::WgradSplits split;
};

// Forward + loss (+ backward products) of the `rows` samples idx[0..rows) of the buffer.
// Leaves gradient partials in m->grad_part / m->stat_part; their numbers of rows follow from the path, and with that from
// the instance's switch and compute units.
int minibatch_pass(gmi_instance* g, gmi_model* m, gmi_buffer* b, const gmi_ppo_hparams* hp, const int32_t* idx,
                   int rows, int cus, bool want_grad, PartRows* parts, int* n_loss_blocks_out, bool obs16_ready = false, int replicas = 1) {
  const ModelLayout& L = m->L;
  const bool bf = L.dtype == GMI_DTYPE_BF16;
  int rc = GMI_ERR_UNSUPPORTED;
  bool blocks = false;
  if (g->fusion >= 1 && want_grad && !bf) {
    // fp32: everything up to the gradient partials in one launch
    rc = gmi::launch_train_f32(g, m, b, hp, idx, rows, cus, &parts->flat);
    if (rc == GMI_OK) { *n_loss_blocks_out = parts->flat; return GMI_OK; }
    if (rc != GMI_ERR_UNSUPPORTED) return rc;
  }
  if (g->fusion >= 1 && want_grad && bf && gmi::use_resident(L, rows, cus)) {
    // the tile's activations resident in LDS; small nets' weight gradients in the same launch
    int n = 0;
    rc = gmi::launch_train_resident(g, m, b, hp, idx, rows, cus, &n, n_loss_blocks_out);
    for (int i = 0; i < gmi::kMaxWgradProblems; ++i) parts->split.n[i] = (uint8_t)n;
    if (rc == GMI_OK && n > 0) return GMI_OK;
  }
  if (rc == GMI_ERR_UNSUPPORTED && g->fusion >= 1 && want_grad && bf) {
    // row-tile kernel (gather + forward + loss + input gradients in one launch) where this shape has one; it leaves the hidden
    // activations and the gradients in its block layout
    rc = gmi::launch_train_chain(g, m, b, hp, idx, rows, n_loss_blocks_out, obs16_ready);
    blocks = rc == GMI_OK;
  }
  if (rc == GMI_ERR_UNSUPPORTED) rc = layers_pass(g, m, b, hp, idx, rows, want_grad, n_loss_blocks_out);
  if (rc != GMI_OK || !want_grad) return rc;
  // weight / bias gradients of every layer of both nets in one launch
  int n_split = (rows + 63) / 64;
  if (n_split > m->n_split_max) n_split = m->n_split_max;
  if (n_split < 1) n_split = 1;
  int chunk = (rows + n_split - 1) / n_split;
  chunk = (chunk + 63) / 64 * 64;
  parts->flat = n_split;
  gmi::WgradBatch wb;
  wb.n = 0;
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      gmi::WgradProblem& p = wb.p[wb.n++];
      p.dz = m->dz[net][l]; p.lddz = li.out_pad;
      p.x = m->h[net][l]; p.ldx = li.in_pad;
      p.out = li.out; p.in = li.in; p.out_pad = li.out_pad; p.in_pad = li.in_pad;
      p.w_off = li.part_w; p.b_off = li.part_b;
      int most = std::min<int>(m->split.n[wb.n - 1], (rows + 63) / 64);      // at least 64 rows each
      // one Adam launch reads the partials of all replicas, which takes longer than the splits save.  (Four of 60:256:128:64:8 with 8192 rows
      // each, us of Adam with the splits per layer / no more than even ones: on 64 compute units each 27.0 / 20.0, unmasked 16.0 / 13.1.)
      if (replicas > 1) most = std::min(most, m->n_split_even);
      p.chunk = ((rows + most - 1) / most + 31) / 32 * 32;
      p.n_split = (rows + p.chunk - 1) / p.chunk;
      parts->split.n[wb.n - 1] = (uint8_t)p.n_split;
      // the row-tile kernel leaves every activation and every gradient in its block layout
      if (blocks && l == 0) p.x = m->x0b;
      p.x_blocks = blocks ? (l == 0 ? 2 : 1) : 0;
      p.dz_blocks = blocks ? 1 : 0;
    }
  return gmi::launch_wgrad(g, L.dtype, rows, n_split, chunk, wb, m->grad_part, L.part_floats,
                           gmi::beyond_cache(L, rows));
}

// Reduces the partials of the n bindings ms[0..n) (replicas of one model: same parameter arrays, own
// workspaces; parts[i] and n_stat[i] rows of them) and applies one Adam step through ms[0]; launched on instance g.
int launch_adam(gmi_instance* g, gmi_model* const* ms, int n, const PartRows* parts, const int* n_stat,
                const gmi_ppo_hparams* hp, int rows, uint32_t k, float* stats_out, float* grad_out, bool do_update) {
  gmi_model* m = ms[0];
  const gmi::ShadowTable tab = gmi::make_shadow_table(m->L);
  gmi::ProfScope ps(g, gmi::kClsAdam);
  PartSet set = {};
  set.n = n;
  int most = 0;
  for (int i = 0; i < n; ++i) {
    set.r[i] = Partials{ms[i]->grad_part, ms[i]->stat_part, parts[i].flat, n_stat[i]};
    set.split[i] = parts[i].split;
    most = std::max(most, parts[i].flat);
  }
  if (m->L.dtype == GMI_DTYPE_BF16) {
    AdamTiles tt;
    tt.n = tab.n;
    int total = 0;
    for (int i = 0; i < tab.n; ++i) {
      tt.start[i] = total;
      if (do_update || grad_out) total += ((tab.l[i].out + 7) / 8) * ((tab.l[i].in + 31) / 32);
    }
    for (int i = tab.n; i <= gmi::kMaxWgradProblems; ++i) tt.start[i] = INT32_MAX;
    gmi::ChainEmit ce;
    gmi::fill_chain_emit(m->L, &ce);
    // loads in flight per thread: all of a layer's partial rows in one round trip (up to 96 rows)
    auto go = [&](auto kernel) {
      ps.launch(kernel, dim3(total + 1), dim3(256), 0, tab, tt, ce, m->params, m->adam_m, m->adam_v, set, m->L.part_floats,
                m->L.act_dim, hp->c_e, 1.0f / (float)rows, adam_scalars(hp, k), m->shadow, stats_out, grad_out, do_update ? 1 : 0);
    };
    int deep = 0;
    for (int i = 0; i < n; ++i)
      for (int l = 0; l < tab.n; ++l) deep = std::max<int>(deep, parts[i].split.n[l]);
    if (deep <= 16) go(adam_shadow_kernel<4>);
    else if (deep <= 32) go(adam_shadow_kernel<8>);
    else if (deep <= 48) go(adam_shadow_kernel<12>);
    else if (deep <= 96) go(adam_shadow_kernel<24>);
    else go(adam_shadow_kernel<16>);      // two round trips
    GMI_LAUNCH_CHECK();
    return GMI_OK;
  }
  // four threads per parameter where one per parameter would leave the device short of loads in flight (fewer than
  // about 1024 workgroups of 256) or make each thread walk a long column
  const bool split4 = most >= 4 && (most >= 64 || m->L.logstd_off < 256 * 1024);
  const unsigned grid = (unsigned)((m->L.logstd_off + 255) / 256) + 1;
  auto go = [&](auto kernel, int threads) {
    ps.launch(kernel, dim3(grid), dim3(threads), 0, tab, m->params, m->adam_m, m->adam_v, set, m->L.part_floats,
              m->L.act_dim, hp->c_e, 1.0f / (float)rows, adam_scalars(hp, k), stats_out, grad_out, do_update ? 1 : 0);
  };
  if (split4) go(adam_kernel<4>, 1024); else go(adam_kernel<1>, 256);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

}  // namespace

extern "C" int ppo_update(gmi_t g, gmi_model_t m, gmi_buffer_t b, const gmi_ppo_hparams* hp, float* stats_out) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "ppo_update: bad instance");
  if (!valid(m)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "ppo_update: bad model");
  if (!valid(b)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "ppo_update: bad buffer");
  int rc = check_hp("ppo_update", hp);
  if (rc != GMI_OK) return rc;
  rc = check_model_buffer("ppo_update", m, b);
  if (rc != GMI_OK) return rc;
  if (!m->adam_m) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update: the model binding has no Adam state");
  const int64_t B = (int64_t)b->d.horizon * b->d.n_envs;
  if (hp->epochs < 0 || hp->minibatch < 1) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update: epochs >= 0 and minibatch >= 1");
  if (B == 0 || hp->epochs == 0) return GMI_OK;
  if (B % hp->minibatch != 0)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "ppo_update: minibatch %d does not divide T*N = %lld", hp->minibatch, (long long)B);
  if (hp->minibatch > m->max_rows)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "ppo_update: minibatch %d exceeds the binding's max_rows %d", hp->minibatch, m->max_rows);
  const int nmb = (int)(B / hp->minibatch);
  uint32_t k = hp->adam_step0;
  bool obs16 = false;
  const int cus = gmi::trainer_cus(g, 1);
  rc = gmi::prepare_obs16(g, m, b, hp->minibatch, cus, &obs16);
  if (rc != GMI_OK) return rc;
  for (int e = 0; e < hp->epochs; ++e) {
    // the shuffles of up to kPermEpochs epochs in one launch (each launch of this small kernel is mostly latency)
    const int32_t* perm = b->perm + (int64_t)(e % gmi::kPermEpochs) * B;
    if (e % gmi::kPermEpochs == 0) {
      const int ne = hp->epochs - e < gmi::kPermEpochs ? hp->epochs - e : gmi::kPermEpochs;
      rc = gmi::launch_permutation(g, (int)B, hp->seed, hp->iteration, (uint32_t)e, ne, b->perm);
      if (rc != GMI_OK) return rc;
    }
    for (int j = 0; j < nmb; ++j) {
      PartRows parts = {};
      int nlb = 1;
      rc = minibatch_pass(g, m, b, hp, perm + (int64_t)j * hp->minibatch, hp->minibatch, cus, true, &parts, &nlb,
                          obs16);
      if (rc != GMI_OK) return rc;
      ++k;
      rc = launch_adam(g, &m, 1, &parts, &nlb, hp, hp->minibatch, k,
                       stats_out ? stats_out + 5 * ((int64_t)e * nmb + j) : nullptr, nullptr, true);
      if (rc != GMI_OK) return rc;
    }
  }
  return GMI_OK;
}

extern "C" int ppo_update_group(const gmi_t* gs, const gmi_model_t* ms, const gmi_buffer_t* bs, int32_t n,
                                const gmi_ppo_hparams* hp, float* stats_out) {
  if (n < 1 || n > kMaxGroup) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update_group: 1 <= n <= %d instances", kMaxGroup);
  if (!gs || !ms || !bs) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update_group: NULL handle array");
  int rc = check_hp("ppo_update_group", hp);
  if (rc != GMI_OK) return rc;
  for (int i = 0; i < n; ++i) {
    if (!valid(gs[i])) GMI_FAIL(GMI_ERR_BAD_HANDLE, "ppo_update_group: bad instance %d", i);
    if (!valid(ms[i])) GMI_FAIL(GMI_ERR_BAD_HANDLE, "ppo_update_group: bad model %d", i);
    if (!valid(bs[i])) GMI_FAIL(GMI_ERR_BAD_HANDLE, "ppo_update_group: bad buffer %d", i);
    rc = check_model_buffer("ppo_update_group", ms[i], bs[i]);
    if (rc != GMI_OK) return rc;
    for (int j = 0; j < i; ++j)
      if (gs[j] == gs[i] || ms[j] == ms[i] || bs[j] == bs[i])
        GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update_group: entries %d and %d share a handle", j, i);
    // replicas of one model: same arrays, own workspaces
    if (ms[i]->params != ms[0]->params || ms[i]->adam_m != ms[0]->adam_m || ms[i]->adam_v != ms[0]->adam_v ||
        ms[i]->shadow != ms[0]->shadow || ms[i]->L.n_params != ms[0]->L.n_params || ms[i]->L.dtype != ms[0]->L.dtype ||
        ms[i]->n_split_max != ms[0]->n_split_max)
      GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update_group: model %d is not a binding of model 0's parameter arrays", i);
    if (bs[i]->d.horizon != bs[0]->d.horizon || bs[i]->d.n_envs != bs[0]->d.n_envs)
      GMI_FAIL(GMI_ERR_BAD_SHAPE, "ppo_update_group: buffer %d has another size than buffer 0", i);
    if (gs[i]->device != gs[0]->device) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update_group: instances on different devices");
  }
  if (!ms[0]->adam_m) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update_group: the model bindings have no Adam state");
  const int64_t B = (int64_t)bs[0]->d.horizon * bs[0]->d.n_envs;
  if (hp->epochs < 0 || hp->minibatch < 1) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_update_group: epochs >= 0 and minibatch >= 1");
  if (B == 0 || hp->epochs == 0) return GMI_OK;
  if (B % hp->minibatch != 0)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "ppo_update_group: minibatch %d does not divide T*N = %lld", hp->minibatch, (long long)B);
  for (int i = 0; i < n; ++i)
    if (hp->minibatch > ms[i]->max_rows)
      GMI_FAIL(GMI_ERR_BAD_SHAPE, "ppo_update_group: minibatch %d exceeds binding %d's max_rows %d", hp->minibatch, i,
               ms[i]->max_rows);
  const int nmb = (int)(B / hp->minibatch);
  uint32_t k = hp->adam_step0;
  gmi_instance* g0 = gs[0];
  gmi_model* models[kMaxGroup];
  for (int i = 0; i < n; ++i) models[i] = ms[i];
  // instance 0's stream also reads what the other instances' earlier calls left (e.g. their buffers are
  // theirs alone, but the shared parameters were last written on stream 0): nothing to order before the loop.
  bool obs16[kMaxGroup];
  for (int i = 0; i < n; ++i) {
    rc = gmi::prepare_obs16(gs[i], ms[i], bs[i], hp->minibatch, gmi::trainer_cus(gs[i], n), &obs16[i]);
    if (rc != GMI_OK) return rc;
  }
  for (int e = 0; e < hp->epochs; ++e) {
    if (e % gmi::kPermEpochs == 0) {
      const int ne = hp->epochs - e < gmi::kPermEpochs ? hp->epochs - e : gmi::kPermEpochs;
      for (int i = 0; i < n; ++i) {
        rc = gmi::launch_permutation(gs[i], (int)B, hp->seed + (uint64_t)i, hp->iteration, (uint32_t)e, ne, bs[i]->perm);
        if (rc != GMI_OK) return rc;
      }
    }
    const int64_t perm_off = (int64_t)(e % gmi::kPermEpochs) * B;
    for (int j = 0; j < nmb; ++j) {
      PartRows parts[kMaxGroup] = {};
      int nlb[kMaxGroup];
      for (int i = 0; i < n; ++i) {
        rc = minibatch_pass(gs[i], ms[i], bs[i], hp, bs[i]->perm + perm_off + (int64_t)j * hp->minibatch, hp->minibatch,
                            gmi::trainer_cus(gs[i], n), true, &parts[i], &nlb[i], obs16[i], n);
        if (rc != GMI_OK) return rc;
        // replica i's partials are complete: let instance 0 see them
        if (i > 0) {
          GMI_HIP(hipEventRecord(gs[i]->event, gs[i]->stream));
          GMI_HIP(hipStreamWaitEvent(g0->stream, gs[i]->event, 0));
        }
      }
      ++k;
      rc = launch_adam(g0, models, n, parts, nlb, hp, hp->minibatch, k,
                       stats_out ? stats_out + 5 * ((int64_t)e * nmb + j) : nullptr, nullptr, true);
      if (rc != GMI_OK) return rc;
      // the updated parameters are complete: the other instances may start their next forward pass
      if (n > 1) {
        GMI_HIP(hipEventRecord(g0->event, g0->stream));
        for (int i = 1; i < n; ++i) GMI_HIP(hipStreamWaitEvent(gs[i]->stream, g0->event, 0));
      }
    }
  }
  return GMI_OK;
}

static int check_idx_call(const char* fn, gmi_t g, gmi_model_t m, gmi_buffer_t b, const gmi_ppo_hparams* hp,
                          const int32_t* idx, int32_t n) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "%s: bad instance", fn);
  if (!valid(m)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "%s: bad model", fn);
  if (!valid(b)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "%s: bad buffer", fn);
  int rc = check_hp(fn, hp);
  if (rc != GMI_OK) return rc;
  rc = check_model_buffer(fn, m, b);
  if (rc != GMI_OK) return rc;
  if (n < 1 || n > m->max_rows) GMI_FAIL(GMI_ERR_BAD_SHAPE, "%s: n=%d outside [1, max_rows=%d]", fn, n, m->max_rows);
  if (!idx) GMI_FAIL(GMI_ERR_INVALID_ARG, "%s: idx is NULL", fn);
  return GMI_OK;
}

extern "C" int ppo_evaluate(gmi_t g, gmi_model_t m, gmi_buffer_t b, const gmi_ppo_hparams* hp, const int32_t* idx,
                            int32_t n, float* stats_out) {
  int rc = check_idx_call("ppo_evaluate", g, m, b, hp, idx, n);
  if (rc != GMI_OK) return rc;
  if (!stats_out) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_evaluate: stats_out is NULL");
  PartRows parts = {};
  int nlb = 1;
  rc = minibatch_pass(g, m, b, hp, idx, n, gmi::trainer_cus(g, 1), false, &parts, &nlb);
  if (rc != GMI_OK) return rc;
  return launch_adam(g, &m, 1, &parts, &nlb, hp, n, 1, stats_out, nullptr, false);
}

extern "C" int ppo_gradient(gmi_t g, gmi_model_t m, gmi_buffer_t b, const gmi_ppo_hparams* hp, const int32_t* idx,
                            int32_t n, float* grad_out, float* stats_out) {
  int rc = check_idx_call("ppo_gradient", g, m, b, hp, idx, n);
  if (rc != GMI_OK) return rc;
  if (!grad_out) GMI_FAIL(GMI_ERR_INVALID_ARG, "ppo_gradient: grad_out is NULL");
  PartRows parts = {};
  int nlb = 1;
  rc = minibatch_pass(g, m, b, hp, idx, n, gmi::trainer_cus(g, 1), true, &parts, &nlb);
  if (rc != GMI_OK) return rc;
  return launch_adam(g, &m, 1, &parts, &nlb, hp, n, 1, stats_out, grad_out, false);
}

extern "C" int adam_update(gmi_t g, float* params, float* adam_m, float* adam_v, const float* grad, int64_t n,
                           const gmi_ppo_hparams* hp, uint32_t step) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "adam_update: bad instance");
  int rc = check_hp("adam_update", hp);
  if (rc != GMI_OK) return rc;
  if (n < 0) GMI_FAIL(GMI_ERR_BAD_SHAPE, "adam_update: negative n");
  if (n == 0) return GMI_OK;
  if (step < 1) GMI_FAIL(GMI_ERR_INVALID_ARG, "adam_update: step is 1-based");
  if (!params || !adam_m || !adam_v || !grad) GMI_FAIL(GMI_ERR_INVALID_ARG, "adam_update: NULL pointer");
  gmi::ShadowTable tab;
  tab.n = 0;
  tab.logstd_off = n;
  tab.sh_logstd = 0;
  tab.act_dim = 0;
  tab.n_params = n;
  gmi::ProfScope ps(g, gmi::kClsAdam);
  PartSet set = {};
  set.n = 1;
  set.r[0] = Partials{grad, nullptr, 1, 0};
  ps.launch(adam_kernel<1>, dim3((unsigned)((n + 255) / 256) + 1), dim3(256), 0, tab, params, adam_m, adam_v, set, n,
            0, 0.f, 1.f, adam_scalars(hp, step), nullptr, nullptr, 1);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}
