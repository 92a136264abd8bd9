// Inference-only agents in 8-bit floating point (the agent role of Section 3 of the paper needs the forward pass
// alone): weights of every layer as E4M3 with one power-of-two scale per layer, the observation and the hidden
// activations as unscaled E4M3 (saturating), products on the 64-deep fp8 matrix instruction with fp32 accumulation,
// scale, bias and ELU in fp32, the heads' outputs in fp32.  The action is then drawn exactly as agent_act draws it.
//
// The kernel is agent_kernel (agent_kernel.h), instantiated for fp8.  Weights lie packed in operand order: for feature tile
// ft and k-step ks (64 deep), lane (f = lane % 32, kh = lane / 32) holds the 32 bytes k = 64 ks + 32 kh + 0..31 of feature
// 32 ft + f, stored as two 16-byte halves [block][half][lane] so that each load instruction reads 1 KiB contiguously.
// Activations are read with the same (kh, byte) -> k rule, which is all the dot product needs: how the instruction orders k
// inside a lane pair does not matter as long as both operands use one rule.  Layer widths are padded to 64 (heads to 32)
// with zero weights.
//
// The fp8 matrix instructions do not add their products exactly: a product more than 2^13 times smaller than the
// largest one of the instruction is dropped (measured on the 16-deep form: 1*1 + 2^-13 is exact, 1*1 + 2^-14 gives
// 1).  Results therefore follow an exact-sum model of the same roundings to ~1e-4 per activation, not to fp32
// rounding.
#include "agent_kernel.h"
#include "tile_kernel.h"

#include <vector>

struct gmi_fp8 {
  uint32_t magic;
  int device;
  ModelLayout L;
  int max_rows;
  char* base;                              // everything below, one allocation
  size_t bytes;
  std::vector<int64_t> w_off[2];           // packed E4M3 weights of (net, layer), byte offsets
  std::vector<int64_t> b_off[2];           // fp32 bias [F], zero padded; a net's layers one after the other
  int64_t scale_off, max_off, logstd_off, mu_off;   // fp32 [2 * n_layers], u32 [2 * n_layers], fp32 [A], fp32 [max_rows, A]
};

namespace {
constexpr uint32_t kMagicFp8 = 0x474d4938;   // "GMI8"
bool valid(gmi_fp8_t w) { return w && w->magic == kMagicFp8; }
int pad64(int x) { return (x + 63) & ~63; }
using namespace gmi_agent;

struct Fp8Layer {
  const float* w;          // fp32 [out, in] of the parameter vector
  const float* b;          // fp32 [out]
  uint32_t* packed;        // E4M3 bytes in operand order, as words
  float* bias;             // fp32 [F]
  int in, out, K, F;       // K = in padded to 64; F = out padded to 64 (hidden) or 32 (head)
};
struct Fp8Table {
  Fp8Layer l[2 * kMaxLayers];
  int n;                   // layers of both nets
  uint32_t* maxbits;       // [n] bit patterns of max|w| (non-negative floats order like their bit patterns)
  float* scale;            // [n]
  const float* log_std;
  float* log_std_out;
  int act_dim;
};

__global__ void fp8_clear_kernel(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

__global__ void fp8_absmax_kernel(Fp8Table t) {
  const Fp8Layer& L = t.l[blockIdx.y];
  const int64_t n = (int64_t)L.in * L.out;
  float m = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    m = fmaxf(m, fabsf(L.w[i]));
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0 && m > 0.f) atomicMax(t.maxbits + blockIdx.y, __float_as_uint(m));
}

// The smallest power of two s with m <= 448 s, from m's exponent and mantissa: m = f 2^e with 0.5 <= f < 1 and
// 448 = 0.875 * 2^9, so s = 2^(e - 9) if f <= 0.875, else 2^(e - 8).  1 for m = 0.
__device__ float scale_for(uint32_t maxbits) {
  if (maxbits == 0u) return 1.0f;
  int e;
  const float f = frexpf(__uint_as_float(maxbits), &e);
  return ldexpf(1.0f, f <= 0.875f ? e - 9 : e - 8);
}

// One thread per packed word (4 consecutive k of one feature); also the scales, the padded biases and log_std.
__global__ void fp8_pack_kernel(Fp8Table t) {
  const Fp8Layer& L = t.l[blockIdx.y];
  const float s = scale_for(t.maxbits[blockIdx.y]);
  const float inv = 1.0f / s;                 // a power of two: exact
  const int nks = L.K / 64;
  const int64_t words = (int64_t)L.F * L.K / 4;
  for (int64_t wd = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; wd < words; wd += (int64_t)gridDim.x * blockDim.x) {
    const int q = (int)(wd & 3);              // word within the 16-byte piece
    const int lane = (int)((wd >> 2) & 63);
    const int half = (int)((wd >> 8) & 1);
    const int64_t blk = wd >> 9;              // ft * nks + ks
    const int ks = (int)(blk % nks), ft = (int)(blk / nks);
    const int f = 32 * ft + (lane & 31);
    const int k = 64 * ks + 32 * (lane >> 5) + 16 * half + 4 * q;
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (f < L.out && k + j < L.in) ? L.w[(int64_t)f * L.in + k + j] * inv : 0.f;
    L.packed[wd] = to_e4m3x4(v[0], v[1], v[2], v[3]);
  }
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < L.F; i += blockDim.x) L.bias[i] = i < L.out ? L.b[i] : 0.f;
    if (threadIdx.x == 0) t.scale[blockIdx.y] = s;
    if (blockIdx.y == 0)
      for (int i = threadIdx.x; i < t.act_dim; i += blockDim.x) t.log_std_out[i] = t.log_std[i];
  }
}

int table_of(gmi_fp8* w, const float* params, Fp8Table* t) {
  const ModelLayout& L = w->L;
  t->n = 2 * L.n_layers;
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      Fp8Layer& o = t->l[net * L.n_layers + l];
      o.w = params + li.w_off;
      o.b = params + li.b_off;
      o.packed = reinterpret_cast<uint32_t*>(w->base + w->w_off[net][l]);
      o.bias = reinterpret_cast<float*>(w->base + w->b_off[net][l]);
      o.in = li.in; o.out = li.out; o.K = pad64(li.in); o.F = li.head ? li.out_pad : pad64(li.out);
    }
  t->maxbits = reinterpret_cast<uint32_t*>(w->base + w->max_off);
  t->scale = reinterpret_cast<float*>(w->base + w->scale_off);
  t->log_std = params + L.logstd_off;
  t->log_std_out = reinterpret_cast<float*>(w->base + w->logstd_off);
  t->act_dim = L.act_dim;
  return GMI_OK;
}

typedef int (*fp8_part_fn)(gmi_instance*, const ModelLayout&, const gmi_chain::ChainArgs&, int);
const fp8_part_fn kTileParts[gmi::kTileFp8Parts] = {gmi::launch_tile_fp8_part0, gmi::launch_tile_fp8_part1, gmi::launch_tile_fp8_part2,
                                                    gmi::launch_tile_fp8_part3, gmi::launch_tile_fp8_part4};

// The row-tile kernel computes in agent_kernel's order, so either may serve a call.  agent_kernel / this one, us:
//   60:256:128:64:8 8.4 / 7.2 for 64 rows, 8.7 / 7.6 for 4096, 10.2 / 7.8 for 8192, 32 / 24 for 65536, 111 / 83 for 262144, on 64 compute
//     units 8.5 / 7.2 for 256;
//   108:400:200:100:21 10.8 / 13.9 for 512 rows, 13.0 / 14.1 for 5000, 14.0 / 14.6 for 8192, 17.6 / 15.2 for 12000, 67 / 58 for 65536, on
//     64 compute units 12.4 / 13.9 for 2048, 16.6 / 14.3 for 4096;
//   211:512:512:256:128:20 14 / 19 for 512 rows, 19.4 / 19.8 for 5000, 21.2 / 21.0 for 8192, 28 / 23 for 12000, 126 / 103 for 65536, on 64
//     compute units 18.2 / 19.3 for 2048, 28.5 / 20.4 for 4096.
// Layers of more than 8 feature tiles, which its 4 waves take 4 at a time, beyond 32 rows per compute unit; narrower models always.
bool use_tile(const gmi_instance* g, const ModelLayout& L, int rows) {
  return L.obs_dim >= 4 && (pad64(L.max_width_pad) <= 256 || rows > 32 * (int64_t)g->cu_count);
}

// The decision through the row-tile kernel (tile_kernel.h): GMI_ERR_UNSUPPORTED if none is compiled for the shape.
int launch_tile(gmi_instance* g, const gmi_fp8* w, const AgentArgs& in) {
  const ModelLayout& L = w->L;
  gmi_chain::ChainArgs a = {};
  for (int net = 0; net < 2; ++net) {
    a.wstream[net] = w->base;
    for (int l = 0; l < L.n_layers; ++l) {
      a.bias[net][l] = in.l[net][l].bias;
      a.wf_off[net][l] = (int)w->w_off[net][l];
    }
  }
  a.scale = in.l[0][0].scale;
  a.log_std = in.log_std;
  a.b_obs = in.obs; a.obs_dim = in.O; a.act_dim = in.A;
  a.T = 1;
  a.x0_ready = 3;
  a.rows = in.n;
  a.mu_out = in.mu_out; a.val_out = in.value; a.act_out = in.act; a.logp_out = in.logp;
  a.k0 = in.k0; a.k1 = in.k1; a.step = in.step; a.env_offset = in.env_offset;
  int rc = GMI_ERR_UNSUPPORTED;
  for (int p = 0; p < gmi::kTileFp8Parts && rc == GMI_ERR_UNSUPPORTED; ++p) rc = kTileParts[p](g, L, a, in.n);
  return rc;
}

}  // namespace

extern "C" int gmi_fp8_bind(gmi_t g, const gmi_model_desc* d, gmi_fp8_t* out) {
  if (!out) GMI_FAIL(GMI_ERR_INVALID_ARG, "gmi_fp8_bind: out is NULL");
  *out = nullptr;
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "gmi_fp8_bind: bad instance");
  if (!d) GMI_FAIL(GMI_ERR_INVALID_ARG, "gmi_fp8_bind: desc is NULL");
  if (d->max_rows < 1) GMI_FAIL(GMI_ERR_BAD_SHAPE, "gmi_fp8_bind: max_rows < 1");
  gmi_fp8* w = new gmi_fp8();
  gmi_model_desc dd = *d;
  dd.dtype = GMI_DTYPE_BF16;      // the layout's padded sizes (multiples of 32) are those of the matrix-core paths
  const int rc = build_layout(&dd, &w->L);
  if (rc != GMI_OK) { delete w; return rc; }
  if (pad64(w->L.max_width_pad) > 512) {
    delete w;
    GMI_FAIL(GMI_ERR_UNSUPPORTED, "gmi_fp8_bind: the activation buffers of layers this wide (%d) do not fit in LDS",
             w->L.max_width_pad);
  }
  w->device = g->device;
  w->max_rows = d->max_rows;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~(size_t)255; return (int64_t)o; };
  int64_t bias_floats = 0;      // of the policy net, whose head is the wider one: both nets get room for as many
  for (const LayerInfo& li : w->L.net[0]) bias_floats += li.head ? li.out_pad : pad64(li.out);
  for (int net = 0; net < 2; ++net) {
    int64_t b = take((size_t)bias_floats * 4);
    for (const LayerInfo& li : w->L.net[net]) {
      const int K = pad64(li.in), F = li.head ? li.out_pad : pad64(li.out);
      w->w_off[net].push_back(take((size_t)F * K));
      w->b_off[net].push_back(b);
      b += (int64_t)F * 4;
    }
  }
  w->scale_off = take(2 * kMaxLayers * 4);
  w->max_off = take(2 * kMaxLayers * 4);
  w->logstd_off = take((size_t)w->L.act_dim * 4);
  w->mu_off = take((size_t)d->max_rows * w->L.act_dim * 4);
  w->bytes = off;
  hipError_t e = hipMalloc((void**)&w->base, w->bytes);
  if (e != hipSuccess) {
    delete w;
    GMI_FAIL(GMI_ERR_HIP, "gmi_fp8_bind: hipMalloc(%zu) failed: %s", off, hipGetErrorString(e));
  }
  w->magic = kMagicFp8;
  *out = w;
  return GMI_OK;
}

extern "C" int gmi_fp8_destroy(gmi_fp8_t w) {
  if (!valid(w)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "gmi_fp8_destroy: bad handle");
  (void)hipFree(w->base);
  w->magic = 0;
  delete w;
  return GMI_OK;
}

extern "C" int gmi_fp8_refresh(gmi_t g, gmi_fp8_t w, const float* params) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "gmi_fp8_refresh: bad instance");
  if (!valid(w)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "gmi_fp8_refresh: bad weights");
  if (!params) GMI_FAIL(GMI_ERR_INVALID_ARG, "gmi_fp8_refresh: params is NULL");
  if (g->device != w->device) GMI_FAIL(GMI_ERR_INVALID_ARG, "gmi_fp8_refresh: instance and weights live on different devices");
  Fp8Table t;
  table_of(w, params, &t);
  fp8_clear_kernel<<<1, 64, 0, g->stream>>>(t.maxbits, t.n);
  fp8_absmax_kernel<<<dim3(32, (unsigned)t.n), 256, 0, g->stream>>>(t);
  fp8_pack_kernel<<<dim3(64, (unsigned)t.n), 256, 0, g->stream>>>(t);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

extern "C" int agent_act_fp8(gmi_t g, gmi_fp8_t w, const float* obs, int32_t n_rows, uint64_t seed, uint32_t step,
                             uint32_t env_offset, float* act, float* logp, float* value, float* mu) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "agent_act_fp8: bad instance");
  if (!valid(w)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "agent_act_fp8: bad weights");
  if (n_rows < 0 || n_rows > w->max_rows)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "agent_act_fp8: n_rows=%d outside 0..max_rows=%d", n_rows, w->max_rows);
  if (n_rows == 0) return GMI_OK;
  if (!obs || !act || !logp || !value) GMI_FAIL(GMI_ERR_INVALID_ARG, "agent_act_fp8: NULL pointer");
  if (g->device != w->device) GMI_FAIL(GMI_ERR_INVALID_ARG, "agent_act_fp8: instance and weights live on different devices");
  const ModelLayout& L = w->L;
  AgentArgs a = {};
  float* mu_ws = reinterpret_cast<float*>(w->base + w->mu_off);
  const float* scale = reinterpret_cast<const float*>(w->base + w->scale_off);
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      a.l[net][l] = {reinterpret_cast<const uint4*>(w->base + w->w_off[net][l]), reinterpret_cast<const float*>(w->base + w->b_off[net][l]),
                     scale + net * L.n_layers + l, pad64(li.in), li.head ? li.out_pad : pad64(li.out)};
    }
  a.nl = L.n_layers; a.net0 = 0;
  a.n = n_rows; a.O = L.obs_dim; a.A = L.act_dim;
  a.vec_obs = ((uintptr_t)obs & 15) == 0 ? 1 : 0;
  a.lp_blocks = 0;
  a.k0 = (uint32_t)seed; a.k1 = (uint32_t)(seed >> 32); a.step = step; a.env_offset = env_offset;
  a.log_std = reinterpret_cast<const float*>(w->base + w->logstd_off);
  a.obs = obs; a.act = act; a.logp = logp; a.value = value; a.mu_out = mu;
  if (use_tile(g, L, n_rows)) {
    const int rc = launch_tile(g, w, a);
    if (rc != GMI_ERR_UNSUPPORTED) return rc;
  }
  // draws and densities in the same launch unless the action is so wide that they do not fit beside a 32-row tile
  const bool sample = agent_lds<Fp8>(a, 1, true) <= kLdsMax;
  if (!sample) { a.act = nullptr; a.mu_out = mu_ws; }
  // Rows per workgroup, us for 32 / 64 / 128 rows:
  //   32 while all workgroups are resident at once (two per compute unit): 8192 rows of 108:400:200:100:21 14 / 16 / 22;
  //   128 where two such tiles fit a compute unit and there are enough of them: 32768 rows of 60:256:128:64:8 31 / 24 / 19
  //   (16384 rows: 18 / 14 / 14), 262144: 220 / 156 / 112;
  //   64 where two of those fit: 65536 rows of 108:400:200:100:21 87 / 72 / 81;
  //   128 on 16 waves where one tile fills a compute unit: 65536 rows of 211:512:512:256:128:20 154 / 167 / 134 (on 8 waves
  //   with twice the registers 141), 16384 rows 44 / 48 / 37.
  const int64_t slots = 2 * (int64_t)g->cu_count;
  auto groups = [&](int rt) { return (int64_t)((n_rows + 32 * rt - 1) / (32 * rt)) * 2; };
  auto per_cu = [&](int rt) { return (int)(kLdsMax / agent_lds<Fp8>(a, rt, sample)); };
  int rc;
  if (groups(1) > slots && per_cu(4) >= 2 && groups(4) >= slots) rc = launch<Fp8, 4, 2, 2, 4>(g, a, 2, sample);
  else if (groups(1) > slots && per_cu(2) >= 2) rc = launch<Fp8, 2, 2, 2, 4>(g, a, 2, sample);
  else if (per_cu(4) >= 1 && 2 * groups(4) >= slots) rc = launch<Fp8, 4, 2, 2, 4, 16>(g, a, 2, sample);
  else rc = launch<Fp8, 1, 4, 1, 4>(g, a, 2, sample);
  if (rc != GMI_OK || sample) return rc;
  return gmi::launch_sample(g, mu_ws, a.log_std, n_rows, L.act_dim, seed, step, env_offset, act, logp, mu);
}
