// Full-precision (fp32) networks, a row tile per workgroup: the agent's action decision, the experience collection of a
// whole horizon, and a minibatch's forward pass, loss, backward pass and weight gradients -- one launch each (Section 3
// of the paper, "DRL Agent" and "DRL Trainer").
//
// Products run on the fp32 matrix instruction (16x16x4: exact fp32 operands and sums, twice the vector unit's rate
// without packed arithmetic).  A workgroup of 8 waves keeps its rows' activations in LDS, [row][feature] with
// 16 m + 4 floats per row: a lane takes 4 consecutive features as one 16-byte read, and the four products of a 16-wide
// k chunk use element j of every lane, i.e. k = 16 c + 4 g + j for lane group g (any order of k will do as long as both
// operands share it); the rows' stride, an odd multiple of 4 floats, spreads the 8 lanes of a read phase over all banks.
// Weights come straight from the parameter vector (row-major [out, in] at any alignment: a 16-byte load needs 4-byte
// alignment only), four chunks ahead; the collection, which passes over them every step, keeps a zero-padded LDS copy where it
// fits (WL).
//
// Bound: small models by the instructions of one pass -- a wave fetches straight-line code at about a byte per cycle, so that
// every 8-byte instruction costs 8 cycles whatever it does -- and by the latencies between them; large batches by the fp32
// matrix instruction (157 TFLOP/s).  Requesting a layer's weights during the epilogue before it, or staging them into LDS,
// takes more instructions than the waits it saves (agent_act of 60:256:128:64:8 with 2048 rows 35 and 19 us instead of 15).
// The one-thread-per-output kernels (mlp.hip) remain for gmi_set_fusion(.., 0) and for models whose 16-row tile does not fit
// LDS; against them agent_act of 60:256:128:64:8 with 2048 rows takes 15 us instead of 468.
#include <algorithm>

#include "rollout.h"

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
struct __attribute__((packed, aligned(4))) Float4U { float x, y, z, w; };      // 16-byte load at 4-byte alignment

constexpr int kNT = 512, kNW = kNT / 64;
constexpr size_t kLdsMax = 160 * 1024;
constexpr int kMaxLayers = GMI_MAX_HIDDEN + 1;

__host__ __device__ __forceinline__ constexpr int pad16(int x) { return (x + 15) & ~15; }
__host__ __device__ __forceinline__ constexpr int rstride(int width) { return pad16(width) + 4; }      // floats of an LDS row

struct F32Layer {
  int in, out;
  int w_off, b_off;          // floats from the start of the parameter vector: W [out, in], b [out]
  uint32_t piece_magic;      // of the 16-byte pieces of a padded row of W
  uint32_t fill[3];
};
struct F32Net {
  F32Layer l[kMaxLayers];
};
// A net's layers, layer l in lane l: fetched at the kernel's start, once.  (Out of the kernel's arguments by a layer index that
// only the wave knows, every field is a scalar load of its own, 300 to 700 cycles in front of every layer's products.)
struct Layers {
  F32Layer mine;
  __device__ __forceinline__ explicit Layers(const F32Net& N) : mine(N.l[min((int)(threadIdx.x & 63), kMaxLayers - 1)]) {}
  __device__ __forceinline__ F32Layer operator[](int l) const {
    F32Layer r;
    r.in = __builtin_amdgcn_readlane(mine.in, l);
    r.out = __builtin_amdgcn_readlane(mine.out, l);
    r.w_off = __builtin_amdgcn_readlane(mine.w_off, l);
    r.b_off = __builtin_amdgcn_readlane(mine.b_off, l);
    r.piece_magic = (uint32_t)__builtin_amdgcn_readlane((int)mine.piece_magic, l);
    return r;
  }
};

// n / d for n * d < 2^32 through one multiply: m = magic(d).
__host__ __device__ __forceinline__ uint32_t magic(uint32_t d) { return d == 1 ? 0u : 0xFFFFFFFFu / d + 1u; }
__device__ __forceinline__ int div_magic(int n, uint32_t m) { return m ? (int)__umulhi((uint32_t)n, m) : n; }

// Floats 4 c .. 4 c + 3 of a row of `width` floats, zero beyond it: one 16-byte load that ends with the row.
__device__ __forceinline__ float4 load_piece(const float* row, int c, int width) {
  float4 v;
  if (width >= 4) {
    const int st = min(4 * c, width - 4), d = 4 * c - st;
    const Float4U t = *reinterpret_cast<const Float4U*>(row + st);
    v.x = d == 0 ? t.x : d == 1 ? t.y : d == 2 ? t.z : t.w;
    v.y = d == 0 ? t.y : d == 1 ? t.z : t.w;
    v.z = d == 0 ? t.z : t.w;
    v.w = t.w;
  } else {
    v = make_float4(row[0], row[min(1, width - 1)], row[min(2, width - 1)], 0.f);
  }
  v.x = 4 * c + 0 < width ? v.x : 0.f; v.y = 4 * c + 1 < width ? v.y : 0.f;
  v.z = 4 * c + 2 < width ? v.z : 0.f; v.w = 4 * c + 3 < width ? v.w : 0.f;
  return v;
}

// A net's weights on their way into its zero-padded LDS copy (layer after layer, [pad16(out)][rstride(in)]): 16-byte pieces,
// the threads' nt at a time, U rounds of loads before the first of them is stored.  (Element by element the copy of 9 KB
// took longer than it saved; these loads are issued ahead of everything the workgroup waits for first.)
template <int U>
struct WeightStage {
  int l = 0, p0 = 0, off = 0;      // next round: pieces p0 + tid of layer l, whose copy starts at off
  float4 v[U];
  __device__ __forceinline__ void advance(const F32Layer& L, int nt) {
    p0 += nt;
    if (p0 >= pad16(L.out) * (pad16(L.in) >> 2)) {
      off += pad16(L.out) * rstride(L.in);
      p0 = 0;
      ++l;
    }
  }
  __device__ __forceinline__ void request(const float* params, const Layers& N, int nl, int tid, int nt) {      // does not move on
    WeightStage<U> w = *this;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (w.l >= nl) break;
      const F32Layer L = N[w.l];
      const int nc = pad16(L.in) >> 2, p = w.p0 + tid, r = div_magic(p, L.piece_magic), c = p - r * nc;
      v[u] = load_piece(params + L.w_off + (int64_t)min(r, L.out - 1) * L.in, c, L.in);
      if (r >= L.out) v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      w.advance(L, nt);
    }
  }
  __device__ __forceinline__ void store(const Layers& N, int nl, float* s_w, int tid, int nt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (l >= nl) break;
      const F32Layer L = N[l];
      const int nc = pad16(L.in) >> 2, p = p0 + tid, r = div_magic(p, L.piece_magic), c = p - r * nc;
      if (r < pad16(L.out)) *reinterpret_cast<float4*>(s_w + off + r * rstride(L.in) + 4 * c) = v[u];
      advance(L, nt);
    }
  }
};
// Bias e of all layers' biases, layer after layer, each zero-padded to pad16(out).
__device__ __forceinline__ float bias_elem(const float* params, const Layers& N, int nl, int e) {
  int off = -1;
  for (int l = 0; l < nl; ++l) {
    const F32Layer L = N[l];
    if (e >= 0 && e < L.out) off = L.b_off + e;
    e -= pad16(L.out);
  }
  const float v = params[max(off, 0)];
  return off >= 0 ? v : 0.f;
}
// Rows of `width` floats, row(r) -> their address, into LDS rows of stride rstride(width), zero padded; magic of pad16(width) / 4.
template <int R, class Row>
__device__ __forceinline__ void stage_rows(int width, uint32_t pmagic, Row row, float* dst, int tid) {
  const int nc = pad16(width) >> 2, n = R * nc, ld = rstride(width);
  for (int e0 = tid; e0 < n; e0 += 2 * kNT) {
    float4 v[2];
    int d[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = min(e0 + u * kNT, n - 1), r = div_magic(e, pmagic), c = e - r * nc;
      v[u] = load_piece(row(r), c, width);
      d[u] = r * ld + 4 * c;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) *reinterpret_cast<float4*>(dst + d[u]) = v[u];      // past the end: the last piece again
  }
}

// acc[i] += sum over nchunk 16-wide k chunks of A (load(c): this lane's 4 values of chunk c) and of the NR row tiles at
// xp, xp + xts (this lane's row and lane group: xp points at k = 4 g).  The operands of D chunks are in flight.
template <int NR, int D, class LoadA>
__device__ __forceinline__ void products(floatx4 (&acc)[NR], int nchunk, LoadA load, const float* xp, int xts) {
  if (nchunk <= 0) return;
  float4 a[D], x[D][NR];
  auto fetch = [&](int u, int c) {
    a[u] = load(c);
#pragma unroll
    for (int i = 0; i < NR; ++i) x[u][i] = *reinterpret_cast<const float4*>(xp + i * xts + 16 * c);
  };
  auto step = [&](int u) {
#pragma unroll
    for (int i = 0; i < NR; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u].x, x[u][i].x, acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NR; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u].y, x[u][i].y, acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NR; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u].z, x[u][i].z, acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NR; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u].w, x[u][i].w, acc[i], 0, 0, 0);
  };
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (u < nchunk) fetch(u, u);
  int c = 0;
  for (; c + D < nchunk; c += D)
#pragma unroll
    for (int u = 0; u < D; ++u) {
      step(u);
      if (c + D + u < nchunk) fetch(u, c + D + u);
    }
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (c + u < nchunk) step(u);
}

// e^z - 1 for z <= 0 as 2^n (e^r - 1) + (2^n - 1), z = n ln 2 + r, |r| <= ln 2 / 2 (ln 2 in two words): e^r - 1 = r + r^2 q(r), q
// of degree 5 fitted to the least relative error.  Within 0.86 ulp of expm1 over [-20, 0] (checked against 64 bits); 18
// instructions.  z < -30 gives -1, as the nearest float does from -17.4 on.
__device__ __forceinline__ float elu32(float z) {
  const float c = z < -30.f ? -30.f : z;
  const float n = __builtin_rintf(c * 0x1.715476p+0f);
  const float r = fmaf(n, -0x1.7f7d1cp-20f, fmaf(n, -0x1.62e4p-1f, c));
  float q = 0x1.a032c4p-13f;
  q = fmaf(q, r, 0x1.6d723ep-10f);
  q = fmaf(q, r, 0x1.11118ap-7f);
  q = fmaf(q, r, 0x1.5554bp-5f);
  q = fmaf(q, r, 0x1.555554p-3f);
  q = fmaf(q, r, 0.5f);
  const float p = fmaf(r * r, q, r);
  const float s = __builtin_amdgcn_ldexpf(1.0f, (int)n);
  return z > 0.f ? z : fmaf(s, p, s - 1.0f);
}
__device__ __forceinline__ float elu_grad32(float h) { return h > 0.f ? 1.0f : h + 1.0f; }

// Sum over the 8 lanes 8 i .. 8 i + 7, in all of them.
__device__ __forceinline__ float sum8(float v) {
  auto add = [&](auto ctrl) { v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true)); };
  add(std::integral_constant<int, 0xB1>{});       // lane ^ 1
  add(std::integral_constant<int, 0x4E>{});       // lane ^ 2
  add(std::integral_constant<int, 0x141>{});      // mirrored among 8: the other four
  return v;
}

enum { kHidden = 0, kHead = 1, kGrad = 2 };

// One tile of a layer for NR row tiles: 16 features from f0 of rows from row tile rt0.
//   kHidden / kHead: y[r][f] = ELU(x W^T + b) / x W^T + b        kGrad: y[r][i] = (x W)[r][i] ELU'(h[r][i])
// s_w: the layer's LDS copy (WL).  Padding features of y come out as zero.
template <bool WL, int NR, int KIND>
__device__ __forceinline__ void tile_product(const float* params, const F32Layer& L, const float* s_w, const float* s_bias, const float* s_x,
                                             int sx, const float* s_h, float* s_y, int sy, int f0, int rt0, int lane) {
  const int j = lane & 15, g = lane >> 4;
  const int ld = rstride(L.in);
  floatx4 acc[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  const float* xp = s_x + (rt0 * 16 + j) * sx + 4 * g;
  const int F = KIND == kGrad ? L.in : L.out;            // features of y
  const int f = f0 + j;                                   // operand A's feature of this lane
  const int fr = f0 + 4 * g;                              // this lane's results: features fr + 0..3 of row j of each row tile
  float4 bv = make_float4(0.f, 0.f, 0.f, 0.f), hv[NR];
  if constexpr (KIND != kGrad) bv = *reinterpret_cast<const float4*>(s_bias + fr);
  else
#pragma unroll
    for (int i = 0; i < NR; ++i) hv[i] = *reinterpret_cast<const float4*>(s_h + ((rt0 + i) * 16 + j) * sy + fr);
  if constexpr (KIND != kGrad) {
    if constexpr (WL) {
      const float* wp = s_w + f * ld + 4 * g;
      products<NR, 4>(acc, pad16(L.in) >> 4, [&](int c) { return *reinterpret_cast<const float4*>(wp + 16 * c); }, xp, 16 * sx);
    } else {
      const float* wp = params + L.w_off + (int64_t)(f < F ? f : F - 1) * L.in;
      const int nfull = L.in >> 4;
      products<NR, 4>(acc, nfull, [&](int c) {
        const Float4U v = *reinterpret_cast<const Float4U*>(wp + 16 * c + 4 * g);
        return make_float4(v.x, v.y, v.z, v.w);
      }, xp, 16 * sx);
      if (L.in & 15) {                                    // the ragged chunk: x is zero beyond `in`
        products<NR, 1>(acc, 1, [&](int) {
          const int k = 16 * nfull + 4 * g;
          return make_float4(wp[min(k, L.in - 1)], wp[min(k + 1, L.in - 1)], wp[min(k + 2, L.in - 1)], wp[min(k + 3, L.in - 1)]);
        }, xp + 16 * nfull, 16 * sx);
      }
    }
  } else {                                                // A = W^T: lane's feature = input i, k = output o
    if constexpr (WL) {
      const float* wp = s_w + f;
      products<NR, 4>(acc, pad16(L.out) >> 4, [&](int c) {
        const float* p = wp + (16 * c + 4 * g) * ld;
        return make_float4(p[0], p[ld], p[2 * ld], p[3 * ld]);
      }, xp, 16 * sx);
    } else {
      const float* wp = params + L.w_off + (f < F ? f : F - 1);
      products<NR, 4>(acc, pad16(L.out) >> 4, [&](int c) {   // x is zero beyond `out`
        const int o = 16 * c + 4 * g, m = L.out - 1;
        return make_float4(wp[(int64_t)min(o, m) * L.in], wp[(int64_t)min(o + 1, m) * L.in], wp[(int64_t)min(o + 2, m) * L.in],
                           wp[(int64_t)min(o + 3, m) * L.in]);
      }, xp, 16 * sx);
    }
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int r = (rt0 + i) * 16 + j;
    float o[4] = {acc[i][0] + bv.x, acc[i][1] + bv.y, acc[i][2] + bv.z, acc[i][3] + bv.w};
    if constexpr (KIND == kHidden) {
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v] = elu32(o[v]);
    } else if constexpr (KIND == kGrad) {
      const float4& h = hv[i];
      o[0] *= elu_grad32(h.x); o[1] *= elu_grad32(h.y); o[2] *= elu_grad32(h.z); o[3] *= elu_grad32(h.w);
    }
    if (f0 + 16 > F)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v] = fr + v < F ? o[v] : 0.f;
    *reinterpret_cast<float4*>(s_y + r * sy + fr) = make_float4(o[0], o[1], o[2], o[3]);
  }
}

// Tile items of a layer: feature tiles x groups of row tiles (pairs where there are enough tiles for every wave: a
// weight operand then serves two products).
__device__ __forceinline__ int pair_rows(int n_ft, int RT, int nw) { return RT >= 2 && n_ft * (RT / 2) >= nw ? 2 : 1; }

template <bool WL, int KIND>
__device__ __forceinline__ void layer(const float* params, const F32Layer& L, const float* s_w, const float* s_bias, const float* s_x, int sx,
                                      const float* s_h, float* s_y, int sy, int RT, int wave, int nw, int lane) {
  const int n_ft = pad16(KIND == kGrad ? L.in : L.out) >> 4;
  const int pr = pair_rows(n_ft, RT, nw);
  int ft = wave, rg = 0;
  for (;; ft += nw) {
    while (ft >= n_ft) { ft -= n_ft; ++rg; }
    if (rg >= RT / pr) break;
    if (pr == 2) tile_product<WL, 2, KIND>(params, L, s_w, s_bias, s_x, sx, s_h, s_y, sy, ft * 16, rg * 2, lane);
    else tile_product<WL, 1, KIND>(params, L, s_w, s_bias, s_x, sx, s_h, s_y, sy, ft * 16, rg, lane);
  }
}

// All layers of a net on the tile in s_x0; hidden activations ping-pong between s_a and s_b (stride sh); the head goes to
// s_out (stride so).  `run`: whether these waves take part (every thread reaches every barrier).  beside(): called with the head.
template <bool WL, class Beside>
__device__ __forceinline__ void net_forward(const float* params, const Layers& N, int nl, const float* s_w, const float* s_bias, const float* s_x0,
                                            int sx0, float* s_a, float* s_b, int sh, float* s_out, int so, int RT, bool run,
                                            int wave, int nw, int lane, Beside beside) {
  const float* x = s_x0;
  int sx = sx0;
  float* y = s_a;
  for (int l = 0; l < nl; ++l) {
    const F32Layer L = N[l];
    if (run) {
      if (l < nl - 1) layer<WL, kHidden>(params, L, s_w, s_bias, x, sx, nullptr, y, sh, RT, wave, nw, lane);
      else layer<WL, kHead>(params, L, s_w, s_bias, x, sx, nullptr, s_out, so, RT, wave, nw, lane);
    }
    if (l == nl - 1) beside();
    __syncthreads();
    if constexpr (WL) s_w += pad16(L.out) * rstride(L.in);
    s_bias += pad16(L.out);
    x = y;
    sx = sh;
    y = y == s_a ? s_b : s_a;
  }
}

// The same for 16 rows and layers of at most four feature tiles, for a kernel that passes over the net many times: the wave's tile of
// every layer stays in its registers, that of the first (W0 = false: an input of more than 64 features) in LDS.
constexpr int kPlanLayers = 4;
template <int NL, bool W0>
struct NetRegs {
  float4 w[NL][4];      // this lane's pieces of row f of W
  int nc[NL];           // k chunks; 0: the wave has no tile
  __device__ __forceinline__ void load(const float* params, const Layers& N, int wave, int lane, float* s_w0) {
    const int j = lane & 15, g = lane >> 4, f = 16 * wave + j;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const F32Layer L = N[l];
      nc[l] = 16 * wave < L.out ? pad16(L.in) >> 4 : 0;
      const float* row = params + L.w_off + (int64_t)min(f, L.out - 1) * L.in;
      auto piece = [&](int c) {      // (load_piece reads inside the row wherever the piece lies)
        float4 v = load_piece(row, 4 * c + g, L.in);
        if (f >= L.out) v = make_float4(0.f, 0.f, 0.f, 0.f);
        return v;
      };
      if (l == 0 && !W0) {
        for (int c = 0; c < nc[0]; ++c) *reinterpret_cast<float4*>(s_w0 + f * rstride(L.in) + 16 * c + 4 * g) = piece(c);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < nc[l]) w[l][c] = piece(c);
      }
    }
  }
};
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}
// x W^T of the wave's tile (padding features: zero) for inputs of nc chunks; xp: this lane's row and lane group of the input.
__device__ __forceinline__ floatx4 tile_of_regs(const float4 (&w)[4], int nc, const float* xp) {
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  float4 x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (u < nc) x[u] = *reinterpret_cast<const float4*>(xp + 16 * u);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (u >= nc) break;
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u].x, x[u].x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u].y, x[u].y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u].z, x[u].z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u].w, x[u].w, acc, 0, 0, 0);
  }
  return acc;
}

// ------------------------------------------------------------------------------------------------
// Action decision: grid (row tiles, nets).
struct AgentF32Args {
  const float* obs;
  int nl, n, obs_dim, act_dim, net0, sh, b_floats, b_net[2];
  uint32_t o_magic;
  F32Net net[2];
  const float* params;
  const float* log_std;
  uint32_t k0, k1, step, env_offset;
  float* act; float* logp; float* value; float* mu_out;
};

template <int RT>
__global__ __launch_bounds__(kNT) void agent_f32_kernel(AgentF32Args a) {
  constexpr int R = 16 * RT;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int net = blockIdx.y + a.net0;
  const Layers N(a.net[net]);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int O = a.obs_dim, A = a.act_dim, sx0 = rstride(O), so = rstride(A), nba = (A + 3) >> 2;
  float* s_bias = smem;
  float* s_x0 = s_bias + a.b_floats;
  float* s_a = s_x0 + R * sx0;
  float* s_b = s_a + R * a.sh;
  float* s_out = s_b + R * a.sh;
  float* s_lp = s_out + R * so;
  const int r0 = blockIdx.x * R;
  stage_rows<R>(O, a.o_magic, [&](int r) { return a.obs + (int64_t)min(r0 + r, a.n - 1) * O; }, s_x0, tid);
  for (int e = tid; e < a.b_net[net]; e += kNT) s_bias[e] = bias_elem(a.params, N, a.nl, e);
  __syncthreads();
  net_forward<false>(a.params, N, a.nl, smem, s_bias, s_x0, sx0, s_a, s_b, a.sh, s_out, so, RT, true, wave, kNW, lane, []() {});
  if (net == 1) {
    for (int r = tid; r < R; r += kNT)
      if (r0 + r < a.n) a.value[r0 + r] = s_out[r * so];
    return;
  }
  // act = mu + exp(log_std) * eps; log-prob partial per block of 4 action elements
  for (int item = tid; item < R * nba; item += kNT) {
    const int r = item / nba, b = item - r * nba;
    const int e = r0 + r;
    float lp = 0.f;
    if (e < a.n) {
      float z[4];
      gmi::normal_block(a.env_offset + (uint32_t)e, a.step, gmi::kStreamAction, (uint32_t)b, a.k0, a.k1, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = 4 * b + i;
        if (j < A) {
          const float ls = a.log_std[j];
          const float m = s_out[r * so + j];
          a.act[(int64_t)e * A + j] = fmaf(expf(ls), z[i], m);
          if (a.mu_out) a.mu_out[(int64_t)e * A + j] = m;
          lp += -0.5f * z[i] * z[i] - ls - 0.918938533204672742f;
        }
      }
    }
    s_lp[r * nba + b] = lp;
  }
  __syncthreads();
  for (int r = tid; r < R; r += kNT) {
    if (r0 + r >= a.n) continue;
    float lp = 0.f;
    for (int b = 0; b < nba; ++b) lp += s_lp[r * nba + b];
    a.logp[r0 + r] = lp;
  }
}

// ------------------------------------------------------------------------------------------------
// Minibatch: grid (row-tile groups, nets).  A workgroup takes the row tiles blockIdx.x, + gridDim.x, ...; its weight
// gradients go to row blockIdx.x of the partials (written for its first tile, accumulated in place for later ones) and
// its statistics to row blockIdx.x of the statistics partials.  The last tile's gradients are written through: left in the die's cache they
// have to be written back before the next kernel may start (us per iteration, 17:64:64:6 478 / 448, 37:128:64:12 862 / 807).
struct TrainF32Args {
  F32Net net[2];
  const float* params;
  const float* log_std;
  const int32_t* idx;
  const float *b_obs, *b_act, *b_logp, *b_adv, *b_ret;
  int n_envs, ld_envs, obs_dim, act_dim, nl, rows, n_tiles, sdz, b_floats;
  int b_net[2];                // floats of each net's biases (b_floats: of the larger)
  int h_off[kMaxLayers];       // floats from the start of the activation area
  int h_floats;
  uint32_t o_magic, a_magic;
  float clip, c_v;
  float* part; int64_t part_stride;
  float* stat_part;
};

// What the kernel waits for first -- sample indices, then the rows they name -- is requested first; the biases travel meanwhile.
// The weights are read from L2: an LDS copy of them made by every workgroup costs more instructions than its reads save.  Loss: 8
// lanes per sample share its actions.  Backward, a layer: input-gradient tiles, weight-gradient tiles and, with the head's, the sums
// over the tile's samples (statistics, log_std) are items of one list, dealt to the waves.
template <int RT>
__global__ __launch_bounds__(kNT) void train_f32_kernel(TrainF32Args a) {
  constexpr int R = 16 * RT;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int net = blockIdx.y;
  const Layers N(a.net[net]);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int O = a.obs_dim, A = a.act_dim, so = rstride(A), nl = a.nl;
  float* s_bias = smem;
  float* s_h = s_bias + a.b_floats;
  float* s_dz0 = s_h + a.h_floats;
  float* s_dz1 = s_dz0 + R * a.sdz;
  float* s_out = s_dz1 + R * a.sdz;               // head outputs, then per-sample log_std gradient terms
  float* s_act = s_out + R * so;                  // [R][A]
  float* s_scal = s_act + ((R * A + 3) & ~3);     // [3][R] old log-prob, advantage, return
  int64_t* s_slot = reinterpret_cast<int64_t*>(s_scal + 3 * R);      // [R]
  float* s_stat = s_scal + 5 * R;                 // [4][R] policy term, value term, kl, clipped of each sample
  float* s_ls = s_stat + 4 * R;                   // [A] log_std, [A] exp(-log_std)
  float* s_sum = s_ls + 2 * A;                    // [4] statistics, [A] log_std gradient, over all tiles
  const float inv_m = 1.0f / (float)a.rows;
  float* part = a.part + (int64_t)blockIdx.x * a.part_stride;

  // sample of row tid of the present tile (rows past the batch repeat its last sample, their gradient is zero)
  int sample = tid < R ? a.idx[min((int)blockIdx.x * R + tid, a.rows - 1)] : 0;
  for (int e = tid; e < a.b_net[net]; e += kNT) s_bias[e] = bias_elem(a.params, N, nl, e);
  for (int j = tid; j < A; j += kNT) {
    const float ls = a.log_std[j];
    s_ls[j] = ls;
    s_ls[A + j] = expf(-ls);
  }
  for (int j = tid; j < 4 + A; j += kNT) s_sum[j] = 0.f;

  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    const int r0 = tile * R;
    const bool first = tile == (int)blockIdx.x, last = tile + (int)gridDim.x >= a.n_tiles;
    if (tid < R) s_slot[tid] = (int64_t)(sample / a.n_envs) * a.ld_envs + (sample % a.n_envs);
    __syncthreads();
    {   // the gather: everything is requested before the first result is stored
      float sc0 = 0.f, sc1 = 0.f, av = 0.f;
      if (tid < R) {
        const int64_t slot = s_slot[tid];
        sc0 = net == 0 ? a.b_logp[slot] : a.b_ret[slot];
        sc1 = a.b_adv[slot];
        sample = a.idx[min((tile + (int)gridDim.x) * R + tid, a.rows - 1)];      // the next tile's
      }
      const int e0 = min(tid, R * A - 1), ar = div_magic(e0, a.a_magic);
      if (net == 0) av = a.b_act[s_slot[ar] * A + e0 - ar * A];
      stage_rows<R>(O, a.o_magic, [&](int r) { return a.b_obs + s_slot[r] * O; }, s_h, tid);
      if (tid < R) { s_scal[net == 0 ? tid : 2 * R + tid] = sc0; s_scal[R + tid] = sc1; }
      if (net == 0) {
        if (tid < R * A) s_act[tid] = av;
        for (int e = tid + kNT; e < R * A; e += kNT) {
          const int r = div_magic(e, a.a_magic);
          s_act[e] = a.b_act[s_slot[r] * A + e - r * A];
        }
      }
    }
    __syncthreads();
    {   // forward
      const float* bias = s_bias;
      for (int l = 0; l < nl; ++l) {
        const F32Layer L = N[l];
        const float* x = s_h + a.h_off[l];
        if (l < nl - 1)
          layer<false, kHidden>(a.params, L, nullptr, bias, x, rstride(L.in), nullptr, s_h + a.h_off[l + 1], rstride(L.out), RT, wave,
                                kNW, lane);
        else
          layer<false, kHead>(a.params, L, nullptr, bias, x, rstride(L.in), nullptr, s_out, so, RT, wave, kNW, lane);
        __syncthreads();
        bias += pad16(L.out);
      }
    }
    // loss: lanes 8 r .. 8 r + 7 have sample r; the head's gradient rows into s_dz0, stride rstride(head width)
    const int sd = rstride(net == 0 ? A : 1), wd = pad16(net == 0 ? A : 1);
    if (tid < 8 * R) {
      const int r = tid >> 3, j0 = tid & 7;
      const bool ok = r0 + r < a.rows;
      if (net == 0) {
        float lp = 0.f;
        for (int j = j0; j < A; j += 8) {
          const float z = (s_act[r * A + j] - s_out[r * so + j]) * s_ls[A + j];
          lp += -0.5f * z * z - s_ls[j] - 0.918938533204672742f;
        }
        lp = sum8(lp);
        float g_lp = 0.f, pl = 0.f, kl = 0.f, cf = 0.f;
        if (ok) {
          const float lo = s_scal[r], ad = s_scal[R + r];
          const float ratio = expf(lp - lo);
          const float u1 = ratio * ad;
          const float u2 = fminf(fmaxf(ratio, 1.0f - a.clip), 1.0f + a.clip) * ad;
          pl = -fminf(u1, u2);
          kl = lo - lp;
          cf = fabsf(ratio - 1.0f) > a.clip ? 1.f : 0.f;
          g_lp = (u1 <= u2) ? -(ad * ratio) * inv_m : 0.f;
        }
        if (j0 == 0) { s_stat[r] = pl; s_stat[2 * R + r] = kl; s_stat[3 * R + r] = cf; }
        for (int j = j0; j < wd; j += 8) {
          float dz = 0.f;
          if (j < A) {
            const float z = (s_act[r * A + j] - s_out[r * so + j]) * s_ls[A + j];
            dz = g_lp * z * s_ls[A + j];
            s_out[r * so + j] = g_lp * (z * z - 1.0f);
          }
          s_dz0[r * sd + j] = dz;
        }
      } else {
        const float dv = ok ? s_out[r * so] - s_scal[2 * R + r] : 0.f;
        if (j0 == 0) s_stat[R + r] = dv * dv;
        for (int j = j0; j < wd; j += 8) s_dz0[r * sd + j] = j == 0 ? 2.0f * a.c_v * dv * inv_m : 0.f;
      }
    }
    __syncthreads();
    // backward, head to first layer
    const float* dz = s_dz0;
    float* dn = s_dz1;
    for (int l = nl - 1; l >= 0; --l) {
      const F32Layer L = N[l];
      const int sz = rstride(L.out), shl = rstride(L.in);
      const float* h = s_h + a.h_off[l];
      const int n_it = pad16(L.in) >> 4, n_ot = pad16(L.out) >> 4;
      const int pr = pair_rows(n_it, RT, kNW);
      const int n_grad = l > 0 ? RT / pr : 0;      // rows of n_it items: input gradients, then weight gradients
      const int j = lane & 15, g = lane >> 4;
      int it = wave, row = 0;
      for (;; it += kNW) {
        while (it >= n_it) { it -= n_it; ++row; }
        if (row >= n_grad + n_ot) break;
        if (row < n_grad) {
          if (pr == 2) tile_product<false, 2, kGrad>(a.params, L, nullptr, nullptr, dz, sz, h, dn, shl, it * 16, row * 2, lane);
          else tile_product<false, 1, kGrad>(a.params, L, nullptr, nullptr, dz, sz, h, dn, shl, it * 16, row, lane);
        } else {
          // dW[o][i] = sum_r dz[r][o] h[r][i]: operands straight from the rows (lane = feature, lane group = row)
          const int ot = row - n_grad;
          const float* zp = dz + g * sz + ot * 16 + j;
          const float* hp = h + g * shl + it * 16 + j;
          const int i = it * 16 + j, o = ot * 16 + 4 * g;
          float* dst = part + L.w_off + (int64_t)o * L.in + i;
          float* db = part + L.b_off + ot * 16 + j;
          floatx4 acc = {0.f, 0.f, 0.f, 0.f};
          float x[R / 4], y[R / 4], b = 0.f, bold = 0.f;
#pragma unroll
          for (int q = 0; q < R / 4; ++q) { x[q] = zp[4 * q * sz]; y[q] = hp[4 * q * shl]; }
          if (!first) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (o + v < L.out && i < L.in) acc[v] = dst[(int64_t)v * L.in];
            if (it == 0 && ot * 16 + j < L.out) bold = *db;
          }
#pragma unroll
          for (int q = 0; q < R / 4; ++q) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], y[q], acc, 0, 0, 0);
            b += x[q];
          }
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (o + v < L.out && i < L.in) {
              if (last) gmi::store_through(dst + (int64_t)v * L.in, acc[v]);
              else dst[(int64_t)v * L.in] = acc[v];
            }
          if (it == 0) {
            b += __shfl_xor(b, 16, 64);
            b += __shfl_xor(b, 32, 64);
            if (g == 0 && ot * 16 + j < L.out) *db = bold + b;
          }
        }
      }
      // the sums over the tile's samples, with the head's items, by the last two waves
      if (l == nl - 1 && wave == kNW - 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if ((q == 1) != (net == 1)) continue;
          float v = lane < R ? s_stat[q * R + lane] : 0.f;
#pragma unroll
          for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
          if (lane == 0) s_sum[q] += v;
        }
      } else if (l == nl - 1 && wave == kNW - 2 && net == 0) {
        for (int k = lane; k < A; k += 64) {
          float v = 0.f;
#pragma unroll 16
          for (int r = 0; r < R; ++r) v += s_out[r * so + k];
          s_sum[4 + k] += v;
        }
      }
      __syncthreads();
      float* t = const_cast<float*>(dz);
      dz = dn;
      dn = t;
    }
  }
  // this workgroup's statistics (the slots of the other net belong to the other net's workgroup)
  float* out = a.stat_part + (int64_t)blockIdx.x * (gmi::kStatStride + A);
  if (net == 0) {
    if (tid == 0) { out[0] = s_sum[0]; out[3] = s_sum[2]; out[4] = s_sum[3]; }
    if (tid == 1) {
      float ent = 0.f;
      if (blockIdx.x == 0)
        for (int j = 0; j < A; ++j) ent += s_ls[j] + 1.418938533204672742f;
      out[2] = ent;
      out[5] = out[6] = out[7] = 0.f;
    }
    for (int j = tid; j < A; j += kNT) out[gmi::kStatStride + j] = s_sum[4 + j];
  } else if (tid == 0) {
    out[1] = s_sum[1];
  }
}

// ------------------------------------------------------------------------------------------------
// Experience collection of a whole horizon (see rollout_fused_kernel, fused.hip, whose phases this kernel has with fp32
// networks): waves 0-3 run the policy net, waves 4-7 the value net.
struct RolloutF32Args : RolloutEnv {
  F32Net net[2];
  const float* params;
  int nl, sh, w_floats[2], b_floats[2], mr_lds;
  int ahead;               // 1: a step's draws are made beside the step before it (two buffers), 0: ahead of it, in the idle hidden space
  int hid_floats;          // of all hidden activations
};

__host__ __device__ __forceinline__ int in_stride(int O, int A) { return (O + A + 3) & ~3; }

template <bool WL>
__global__ __launch_bounds__(kNT) void rollout_f32_kernel(RolloutF32Args a) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int half = __builtin_amdgcn_readfirstlane(tid >> 8), wave4 = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int R = a.rows_per_wg, O = a.obs_dim, A = a.act_dim, OS = in_stride(O, A), nbo = a.o4 >> 2, nba = (A + 3) >> 2;
  const int npr = nba + nbo + 1, sx0 = rstride(O), so = rstride(A);
  float* s_w = smem;
  float* s_bias = s_w + (WL ? a.w_floats[0] + a.w_floats[1] : 0);
  float* s_x0 = s_bias + a.b_floats[0] + a.b_floats[1];
  float* s_hid = s_x0 + R * sx0;                                   // [2 nets][2][R][sh]
  float* s_mu = s_hid + a.hid_floats;                              // [R][so]
  float* s_val = s_mu + R * so;                                    // [R][rstride(1)]
  float* s_in2 = s_val + R * rstride(1);                           // [2][R][OS] state | action, of this and the next step
  float* s_end = s_in2 + 2 * R * OS;
  float4* s_noise2 = reinterpret_cast<float4*>(a.ahead ? s_end : s_hid);      // [ahead + 1][R][npr]
  float* s_lp = a.ahead ? s_end + 8 * R * npr : s_end;             // [R][nba]
  float* s_part = s_lp + R * nba;                                  // [R][nbo]
  int* s_done = reinterpret_cast<int*>(s_part + R * nbo);          // [R]
  float* s_ls = reinterpret_cast<float*>(s_done + R);              // [A] log_std, [A] exp(log_std)
  float* s_m = s_ls + ((2 * A + 3) & ~3);                          // [o4][ms] when mr_lds
  const Layers N(a.net[half]);
  const float* s_wn = s_w + (half ? a.w_floats[0] : 0);
  const float* s_bn = s_bias + (half ? a.b_floats[0] : 0);
  float* s_a = s_hid + half * 2 * R * a.sh;
  float* s_b = s_a + R * a.sh;

  for (int j = tid; j < A; j += kNT) { s_ls[j] = a.log_std[j]; s_ls[A + j] = expf(a.log_std[j]); }
  if constexpr (WL) {
    WeightStage<8> ws;
    while (ws.l < a.nl) {
      ws.request(a.params, N, a.nl, tid & 255, 256);
      ws.store(N, a.nl, s_w + (half ? a.w_floats[0] : 0), tid & 255, 256);
    }
  }
  for (int e = tid & 255; e < a.b_floats[half]; e += 256) s_bias[(half ? a.b_floats[0] : 0) + e] = bias_elem(a.params, N, a.nl, e);
  if (a.mr_lds)
    for (int i = tid; i < a.o4 * (a.ms >> 2); i += kNT) reinterpret_cast<float4*>(s_m)[i] = reinterpret_cast<const float4*>(a.m_r)[i];
  for (int i = tid; i < R * sx0; i += kNT) s_x0[i] = 0.f;
  for (int i = tid; i < R * OS; i += kNT) s_in2[R * OS + i] = 0.f;
  const SimLane sl = sim_lane(a, wave8, OS, lane);
  const int draw_top = draw_thread(a, npr);
  __syncthreads();

  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    const int r0 = tile * R;
    load_states(a, r0, s_in2, OS, tid);
    const int et = tid - (kNT - 64);          // the last wave carries the episode counters, makes the done flags and writes the sums
    const bool env_thread = et >= 0 && et < R, env_ok = env_thread && r0 + et < a.n;
    uint32_t ep = 0;
    if (env_ok) ep = a.episode_step[r0 + et];
    if (a.ahead) draw_all(a, s_noise2, a.step0, r0, npr, nba, tid);
    __syncthreads();
    {
      const int r = tid >> a.row_shift, c = tid & ((1 << a.row_shift) - 1), nc = 1 << a.row_shift;
      for (int k = c; k < O; k += nc) s_x0[r * sx0 + k] = s_in2[r * OS + k];
    }
    __syncthreads();
    int64_t slot0 = r0;
    auto reward = [&]() {      // of the step before
      if (env_ok) a.b_rew[slot0 - a.ld_envs + et] = -a.reward_scale * block_sum(s_part + et * nbo, nbo);
    };
    for (int t = 0; t <= a.T; ++t, slot0 += a.ld_envs) {
      float* s_in = s_in2 + (t & 1) * R * OS;
      float4* s_noise = s_noise2 + (a.ahead ? (t & 1) * R * npr : 0);
      const uint32_t step = a.step0 + (uint32_t)t;
      // beside the heads, whose tiles leave the last wave idle: the reward of the step before and, where the draws are there,
      // this step's done flags
      auto beside = [&]() {
        if (!env_thread) return;
        if (t > 0) reward();
        if (a.ahead && t < a.T) finish_env(a, r0, slot0, et, s_noise, npr, ep, s_done);
      };
      net_forward<WL>(a.params, N, a.nl, s_wn, s_bn, s_x0, sx0, s_a, s_b, a.sh, half ? s_val : s_mu, half ? rstride(1) : so, R / 16,
                      half == 1 || t < a.T, wave4, 4, lane, beside);
      if (t == a.T) {
        if (env_ok) a.last_value[r0 + et] = s_val[et * rstride(1)];
        break;
      }
      if (!a.ahead) {
        draw_all(a, s_noise, step, r0, npr, nba, tid);
        __syncthreads();
        if (env_thread) finish_env(a, r0, slot0, et, s_noise, npr, ep, s_done);
      }
      sample_and_store(a, r0, slot0, s_in, OS, s_mu, so, s_noise, npr, nba, s_ls, s_lp, tid);
      __syncthreads();
      float* s_nxt = s_in2 + ((t + 1) & 1) * R * OS;
      auto put = [&](int r, int o, const float (&v)[4]) {      // (what lies beyond the state belongs to the next step's actions)
        *reinterpret_cast<float4*>(s_nxt + r * OS + o) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(s_x0 + r * sx0 + o) =
            make_float4(v[0], o + 1 < O ? v[1] : 0.f, o + 2 < O ? v[2] : 0.f, o + 3 < O ? v[3] : 0.f);
      };
      if (a.mr_lds) sim_items(a, r0, step, sl, s_in, OS, s_m, s_part, s_done, s_noise, npr, nba, wave8, lane, put);
      else sim_items(a, r0, step, sl, s_in, OS, a.m_r, s_part, s_done, s_noise, npr, nba, wave8, lane, put);
      if (env_ok) {
        a.b_logp[slot0 + et] = block_sum(s_lp + et * nba, nba);
        a.b_val[slot0 + et] = s_val[et * rstride(1)];
      }
      if (a.ahead && t + 1 < a.T) draw_rest(a, s_noise2 + ((t + 1) & 1) * R * npr, step + 1u, r0, npr, nba, tid, draw_top);
      __syncthreads();
    }
    {
      const float* s_in = s_in2 + (a.T & 1) * R * OS;
      const int r = tid >> a.row_shift, c = tid & ((1 << a.row_shift) - 1), nc = 1 << a.row_shift;
      if (r0 + r < a.n)
        for (int k = c; k < O; k += nc) a.obs_state[(int64_t)(r0 + r) * O + k] = s_in[r * OS + k];
    }
    if (env_ok) a.episode_step[r0 + et] = ep;
    __syncthreads();
  }
}

// The same for small nets, 16 envs per workgroup, with the roles on waves of their own (rollout.h): waves 0-3 have the policy net, waves
// 4-7 the value net in their registers.  LDS, in floats: what split_lds lays out.
struct SplitLds { int x0, hid, in2, noise, lp, part, done, val, bias, ls, w0, m, floats; };
__host__ __device__ __forceinline__ SplitLds split_lds(int O, int A, int sh, int w0_rows, int m_floats) {
  const int OS = split_stride(O, A), nbo = (O + 3) >> 2, nba = (A + 3) >> 2, npr = nba + nbo + 1;
  SplitLds s;
  s.x0 = 0;                                   // [16][rstride(O)]
  s.hid = s.x0 + 16 * rstride(O);             // [2 nets][2][16][sh]
  s.in2 = s.hid + 64 * sh;                    // [2][16][OS]
  s.noise = s.in2 + 32 * OS;                  // [2][16][npr] float4
  s.lp = s.noise + 128 * npr;                 // [16][nba]
  s.part = s.lp + 16 * nba;                   // [16][nbo]
  s.done = s.part + 16 * nbo;                 // [16]
  s.val = s.done + 16;                        // [16]
  s.bias = s.val + 16;                        // [2 nets][kPlanLayers][64]
  s.ls = s.bias + 128 * kPlanLayers;          // [A]
  s.w0 = s.ls + ((A + 3) & ~3);               // [2 nets][w0_rows][rstride(O)] where the first layer is not in registers
  s.m = s.w0 + 2 * w0_rows * rstride(O);      // [o4][ms] when it fits
  s.floats = s.m + m_floats;
  return s;
}

// NL: layers of a net.
template <int NL, bool W0, bool MR>
__global__ __launch_bounds__(kSplitThreads) void rollout_split_kernel(RolloutF32Args) {
  // The kinds of waves part early, for all tiles, and each reads the arguments for itself: what one keeps in registers is nothing to
  // the others.
  typedef const __attribute__((address_space(4))) RolloutF32Args KernelArgs;
  auto arguments = []() -> const RolloutF32Args& {
    KernelArgs* p = (KernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const RolloutF32Args*)p;
  };
  auto layout = [](const RolloutF32Args& a) { return split_lds(a.obs_dim, a.act_dim, a.sh, W0 ? 0 : pad16(a.net[0].l[0].out), 0); };
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  {
    const RolloutF32Args& a = arguments();
    const SplitLds s = layout(a);
    for (int j = tid; j < a.act_dim; j += kSplitThreads) smem[s.ls + j] = a.log_std[j];
    if constexpr (MR)
      for (int i = tid; i < a.o4 * (a.ms >> 2); i += kSplitThreads)
        reinterpret_cast<float4*>(smem + s.m)[i] = reinterpret_cast<const float4*>(a.m_r)[i];
    for (int i = tid; i < s.hid - s.x0; i += kSplitThreads) smem[s.x0 + i] = 0.f;
    for (int i = tid; i < s.noise - s.in2; i += kSplitThreads) smem[s.in2 + i] = 0.f;
  }
  if (wave < kNetWaves) {
    const RolloutF32Args& a = arguments();
    const SplitLds s = layout(a);
    const int half = wave >> 2, wave4 = (wave + 2 * half) & 3;      // (a net of two tiles: SIMDs 0, 1 and 2, 3)
    const int O = a.obs_dim, A = a.act_dim, OS = split_stride(O, A), nba = (A + 3) >> 2, npr = nba + ((O + 3) >> 2) + 1, sx0 = rstride(O);
    const int j = lane & 15, g = lane >> 4, b = 4 * wave4 + g;
    const Layers N(a.net[half]);
    NetRegs<NL, W0> net;
    float* s_w0 = smem + s.w0 + half * (W0 ? 0 : pad16(a.net[0].l[0].out)) * sx0;
    net.load(a.params, N, wave4, lane, s_w0);
    float* s_bias = smem + s.bias + half * 64 * kPlanLayers;
    if (wave4 < NL) {      // of layer wave4, feature `lane`
      const F32Layer L = N[wave4];
      const float v = a.params[L.b_off + min(lane, L.out - 1)];
      s_bias[64 * wave4 + lane] = lane < L.out ? v : 0.f;
    }
    // exp(log_std) of the actions that this lane decides
    auto std_of = [&](int i) { return expf(a.log_std[min(4 * b + i, A - 1)]); };
    const float4 std = make_float4(std_of(0), std_of(1), std_of(2), std_of(3));
    float* s_a = smem + s.hid + half * 32 * a.sh + j * a.sh + 4 * g;      // this lane's row and lane group
    float* s_b = s_a + 16 * a.sh;
    const float* x0 = smem + s.x0 + j * sx0 + 4 * g;
    const float* wp = s_w0 + (16 * wave4 + j) * sx0 + 4 * g;
    const float* bias = s_bias + 4 * b;
    auto layer = [&](auto l_, float (&o)[4]) {      // of the wave's tile: x W^T + b
      constexpr int l = decltype(l_)::value;
      const float4 bv = *reinterpret_cast<const float4*>(bias + 64 * l);
      floatx4 acc[1] = {{0.f, 0.f, 0.f, 0.f}};
      if constexpr (l == 0 && !W0)
        products<1, 4>(acc, net.nc[0], [&](int c) { return *reinterpret_cast<const float4*>(wp + 16 * c); }, x0, 0);
      else
        acc[0] = tile_of_regs(net.w[l], net.nc[l], l == 0 ? x0 : l & 1 ? s_a : s_b);
      o[0] = acc[0][0] + bv.x; o[1] = acc[0][1] + bv.y; o[2] = acc[0][2] + bv.z; o[3] = acc[0][3] + bv.w;
      if constexpr (l < NL - 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = elu32(o[v]);
        *reinterpret_cast<float4*>((l & 1 ? s_b : s_a) + 16 * wave4) = make_float4(o[0], o[1], o[2], o[3]);
      }
    };
    float4* s_noise2 = reinterpret_cast<float4*>(smem + s.noise);
    __syncthreads();
#pragma unroll 1
    for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
      first_draws(a, s_noise2, tile * 16, npr, nba, wave, lane);
      if (half == 0) {
        __builtin_amdgcn_s_setprio(2);
#pragma unroll 1
        for (int t = 0; t <= a.T; ++t) {
          const bool step = t < a.T;
          static_for<NL>([&](auto l) {
            if (net.nc[l.value] > 0 && step) {
              float o[4];
              if constexpr (l.value == NL - 1) {
                const float4 z = s_noise2[(t & 1) * 16 * npr + j * npr + min(b, nba - 1)];
                layer(l, o);
                if (b < nba) decide_actions(smem + s.in2 + (t & 1) * 16 * OS, OS, O, z, std, j, b, o);
              } else {
                layer(l, o);
              }
            }
            __syncthreads();
          });
          __syncthreads();                    // the simulator's
        }
        __builtin_amdgcn_s_setprio(0);
      } else {
#pragma unroll 1
        for (int t = 0; t <= a.T; ++t) {
          static_for<NL>([&](auto l) {
            __syncthreads();                  // an interval behind the policy
            if (net.nc[l.value] > 0) {
              float o[4];
              layer(l, o);
              if constexpr (l.value == NL - 1)
                if (g == 0) smem[s.val + j] = o[0];
            }
          });
          __syncthreads();
        }
      }
      __syncthreads();                        // the final states are out
    }
    return;
  }
  auto tiles = [&](const RolloutF32Args& a, auto steps) {
    const SplitLds s = layout(a);
    const int O = a.obs_dim, A = a.act_dim, OS = split_stride(O, A), nba = (A + 3) >> 2, npr = nba + ((O + 3) >> 2) + 1, sx0 = rstride(O);
    const SplitArrays arr{smem + s.in2, reinterpret_cast<float4*>(smem + s.noise), smem + s.lp, smem + s.part,
                          reinterpret_cast<int*>(smem + s.done), smem + s.val, smem + s.ls};
    const int at = tid - 64 * kNetWaves, r = at >> 5, c = at & 31;      // 32 threads per env
    __syncthreads();
#pragma unroll 1
    for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
      const int r0 = tile * 16;
      float* state = a.obs_state + (int64_t)min(r0 + r, a.n - 1) * O;
      for (int k = c; k < O; k += 32) {
        const float v = r0 + r < a.n ? state[k] : 0.f;
        arr.in2[r * OS + k] = v;
        smem[s.x0 + r * sx0 + k] = v;
      }
      first_draws(a, arr.noise2, r0, npr, nba, wave, lane);
      steps(s, arr, r0);
      if (r0 + r < a.n)
        for (int k = c; k < O; k += 32) state[k] = arr.in2[(a.T & 1) * 16 * OS + r * OS + k];
      __syncthreads();
    }
  };
  if (wave < kNetWaves + kSimWaves) {
    const RolloutF32Args& a = arguments();
    tiles(a, [&](const SplitLds& s, const SplitArrays& arr, int r0) {
      sim_wave_steps<NL>(a, arr, MR ? smem + s.m : a.m_r, r0, (wave + 1) & 3, lane, [&](int t, int r, int o, const float (&v)[4]) {
        const int O = fresh(a.obs_dim), OS = split_stride(O, a.act_dim);
        // (what lies beyond the state belongs to the next step's actions)
        *reinterpret_cast<float4*>(arr.in2 + (~t & 1) * 16 * OS + r * OS + o) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(smem + s.x0 + r * rstride(O) + o) =
            make_float4(v[0], o + 1 < O ? v[1] : 0.f, o + 2 < O ? v[2] : 0.f, o + 3 < O ? v[3] : 0.f);
      });
    });
  } else {
    const RolloutF32Args& a = arguments();
    tiles(a, [&](const SplitLds& s, const SplitArrays& arr, int r0) {
      const int m = wave - kNetWaves - kSimWaves;
      const bool env_ok = m == 0 && lane < 16 && r0 + lane < a.n;
      uint32_t ep = env_ok ? a.episode_step[r0 + lane] : 0u;
      draw_wave_steps<NL>(a, arr, r0, m, lane, ep);
      if (env_ok) {
        a.last_value[r0 + lane] = smem[s.val + lane];
        a.episode_step[r0 + lane] = ep;
      }
    });
  }
}

// ------------------------------------------------------------------------------------------------
void fill_net(const gmi_model* m, int net, F32Net* N, int* w_floats, int* b_floats) {
  *w_floats = *b_floats = 0;
  for (int l = 0; l < m->L.n_layers; ++l) {
    const LayerInfo& li = m->L.net[net][l];
    N->l[l] = F32Layer{li.in, li.out, (int)li.w_off, (int)li.b_off, magic(pad16(li.in) / 4), {0, 0, 0}};
    *w_floats += pad16(li.out) * rstride(li.in);
    *b_floats += pad16(li.out);
  }
}
int max_hidden(const ModelLayout& L) {
  int w = 0;
  for (int l = 0; l < L.n_hidden; ++l) w = std::max(w, L.net[0][l].out);
  return w;
}

size_t train_lds(const ModelLayout& L, int R, int b_floats) {
  size_t n = b_floats;
  int sdz = 0;
  for (int l = 0; l < L.n_layers; ++l) {
    n += (size_t)R * rstride(L.net[0][l].in);
    sdz = std::max(sdz, rstride(L.net[0][l].out));
  }
  const int A = L.act_dim;
  n += (size_t)R * (2 * sdz + rstride(A)) + ((R * A + 3) & ~3) + 9 * R + 2 * A + 4 + A;
  return 4 * n;
}

}  // namespace

namespace gmi {

// Rows of gradient partials that the fp32 trainer kernel may fill: at most one per workgroup of a net, and no more than
// about 64 MB of them.
int f32_part_rows(const ModelLayout& L) {
  const int64_t n = ((int64_t)64 << 20) / (4 * L.n_params);
  return (int)std::min<int64_t>(trainer_groups(INT32_MAX), std::max<int64_t>(n, 1));
}

int launch_agent_f32(gmi_instance* g, gmi_model* m, const float* obs, int n, uint64_t seed, uint32_t step,
                     uint32_t env_offset, float* act, float* logp, float* value, float* mu_out, bool do_policy) {
  const ModelLayout& L = m->L;
  if (L.dtype != GMI_DTYPE_F32) return GMI_ERR_UNSUPPORTED;
  AgentF32Args a;
  int wf[2], bf[2];
  for (int net = 0; net < 2; ++net) fill_net(m, net, &a.net[net], &wf[net], &bf[net]);
  a.nl = L.n_layers; a.n = n; a.obs_dim = L.obs_dim; a.act_dim = L.act_dim;
  a.o_magic = magic(pad16(L.obs_dim) / 4);
  a.sh = rstride(max_hidden(L));
  a.b_floats = std::max(bf[0], bf[1]);
  a.b_net[0] = bf[0]; a.b_net[1] = bf[1];
  a.params = m->params;
  auto lds = [&](int R) {
    return 4 * (a.b_floats + (size_t)R * (rstride(L.obs_dim) + 2 * a.sh + rstride(L.act_dim) + (L.act_dim + 3) / 4));
  };
  // the tallest tile that still gives every compute unit a workgroup; 64 rows only where two such tiles share one (45:128:128:12,
  // where one does not leave room for the next: 107 us with 32 rows, 143 with 64 for 65536 rows, 17.6 / 20.7 for 8192).
  // us for 16 / 32 / 64 rows: 17:64:64:6 9.1 / 10.4 / 11.5 for 2048, 17.3 / 12.1 / 11.5 for 8192, 97 / 76 / 46 for 65536;
  // 60:256:128:64:8 19.5 / 23.4 / 35 for 2048, 28 / 24 / 35 for 4096, 51 / 34 / 35 for 8192.
  // The weights stream from L2: an LDS copy of them per workgroup took 12.4 us instead of 9.1 (2048 rows of 17:64:64:6), 63
  // instead of 46 (65536).
  int R = 64;
  while (R > 16 && (lds(R) > (R == 64 ? kLdsMax / 2 : kLdsMax) || (n + R - 1) / R < g->cu_count / 2)) R >>= 1;
  if (lds(R) > kLdsMax) return GMI_ERR_UNSUPPORTED;
  a.net0 = do_policy ? 0 : 1;
  a.log_std = m->params + L.logstd_off;
  a.obs = obs;
  a.k0 = (uint32_t)seed; a.k1 = (uint32_t)(seed >> 32); a.step = step; a.env_offset = env_offset;
  a.act = act; a.logp = logp; a.value = value; a.mu_out = mu_out;
  auto go = [&](auto rt) -> int {
    constexpr int RT = decltype(rt)::value;
    static DeviceSet allowed;
    const int rc = allow_lds((const void*)agent_f32_kernel<RT>, kLdsMax, g->device, &allowed);
    if (rc != GMI_OK) return rc;
    ProfScope ps(g, kClsFusedAgent);
    ps.launch(agent_f32_kernel<RT>, dim3((n + R - 1) / R, 2 - a.net0), dim3(kNT), lds(R), a);
    GMI_LAUNCH_CHECK();
    return GMI_OK;
  };
  return R == 16 ? go(std::integral_constant<int, 1>{}) : R == 32 ? go(std::integral_constant<int, 2>{}) : go(std::integral_constant<int, 4>{});
}

int launch_train_f32(gmi_instance* g, gmi_model* m, gmi_buffer* b, const gmi_ppo_hparams* hp, const int32_t* idx, int rows,
                     int cus, int* n_parts) {
  const ModelLayout& L = m->L;
  if (L.dtype != GMI_DTYPE_F32 || L.n_params >= (1ll << 31)) return GMI_ERR_UNSUPPORTED;
  TrainF32Args a;
  int wf[2], bf[2];
  for (int net = 0; net < 2; ++net) fill_net(m, net, &a.net[net], &wf[net], &bf[net]);
  a.b_floats = std::max(bf[0], bf[1]);
  a.b_net[0] = bf[0]; a.b_net[1] = bf[1];
  a.params = m->params;
  // the shortest tile with which a workgroup per net and two compute units holds all rows, else the tallest that
  // fits.  us per minibatch with Adam for 16 / 32 rows (before this form of the kernel with the same rule): 17:64:64:6 21.2 / 21.7
  // (27.9) for 2048 rows, 32 / 23.7 (32) for 4096, with 64 rows 28.6 (37.1) for 8192, 81 (109) for 32768; 45:128:128:12 35.9 / 37.3
  // (49) for 2048, 55 / 42 (55) for 4096, 57 (72) for 8192; 60:256:128:64:8 53 / 62 (79) for 2048, 247 (353) for 16384
  const int most = trainer_groups(cus);
  int R = 16;
  if (train_lds(L, R, a.b_floats) > kLdsMax) return GMI_ERR_UNSUPPORTED;
  while (R < 64 && (rows + R - 1) / R > most && train_lds(L, 2 * R, a.b_floats) <= kLdsMax) R *= 2;
  a.nl = L.n_layers; a.rows = rows; a.obs_dim = L.obs_dim; a.act_dim = L.act_dim;
  a.n_tiles = (rows + R - 1) / R;
  a.sdz = 0;
  int off = 0;
  for (int l = 0; l < L.n_layers; ++l) {
    a.h_off[l] = off;
    off += R * rstride(L.net[0][l].in);
    a.sdz = std::max(a.sdz, rstride(L.net[0][l].out));
  }
  a.h_floats = off;
  a.o_magic = magic(pad16(L.obs_dim) / 4); a.a_magic = magic(L.act_dim);
  a.log_std = m->params + L.logstd_off;
  a.idx = idx;
  a.b_obs = b->d.obs; a.b_act = b->d.act; a.b_logp = b->d.logp; a.b_adv = b->d.adv; a.b_ret = b->d.ret;
  a.n_envs = b->d.n_envs; a.ld_envs = b->d.ld_envs;
  a.clip = hp->clip; a.c_v = hp->c_v;
  a.part = m->grad_part; a.part_stride = L.n_params;
  a.stat_part = m->stat_part;
  const int groups = std::min(a.n_tiles, std::min(most, m->part_rows));
  *n_parts = groups;
  auto go = [&](auto rt) -> int {
    constexpr int RT = decltype(rt)::value;
    static DeviceSet allowed;
    const int rc = allow_lds((const void*)train_f32_kernel<RT>, kLdsMax, g->device, &allowed);
    if (rc != GMI_OK) return rc;
    ProfScope ps(g, kClsChainTrain);
    ps.launch(train_f32_kernel<RT>, dim3(groups, 2), dim3(kNT), train_lds(L, R, a.b_floats), a);
    GMI_LAUNCH_CHECK();
    return GMI_OK;
  };
  return R == 16 ? go(std::integral_constant<int, 1>{}) : R == 32 ? go(std::integral_constant<int, 2>{}) : go(std::integral_constant<int, 4>{});
}

}  // namespace gmi

extern "C" int rollout_collect_f32(gmi_t g, gmi_model_t m, gmi_env_t env, gmi_buffer_t b, float* obs, uint64_t seed,
                                   uint32_t step0, uint32_t env_offset, float* last_value) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect_f32: bad instance");
  if (!valid(m)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect_f32: bad model");
  if (!valid(env)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect_f32: bad env");
  if (!valid(b)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect_f32: bad buffer");
  const ModelLayout& L = m->L;
  const int rc = check_rollout("rollout_collect_f32", m, env, b);
  if (rc != GMI_OK) return rc;
  if (b->d.n_envs == 0 || b->d.horizon == 0) return GMI_OK;
  if (!obs || !last_value) GMI_FAIL(GMI_ERR_INVALID_ARG, "rollout_collect_f32: NULL pointer");
  if (L.dtype != GMI_DTYPE_F32) GMI_FAIL(GMI_ERR_UNSUPPORTED, "rollout_collect_f32: F32 models only; use rollout_collect");
  if (!g->fusion) GMI_FAIL(GMI_ERR_UNSUPPORTED, "rollout_collect_f32: the instance runs one launch per layer");
  RolloutF32Args a;
  fill_rollout_env(m, env, b, obs, seed, step0, env_offset, last_value, &a);
  a.log_std = m->params + L.logstd_off;
  for (int net = 0; net < 2; ++net) fill_net(m, net, &a.net[net], &a.w_floats[net], &a.b_floats[net]);
  a.params = m->params;
  a.nl = L.n_layers;
  a.sh = rstride(max_hidden(L));
  const int O = L.obs_dim, A = L.act_dim, nba = (A + 3) / 4, nbo = a.o4 / 4, npr = nba + nbo + 1;
  auto hid_floats = [&](int R, bool ahead) { return 4 * R * std::max(a.sh, ahead ? 0 : npr); };
  auto lds = [&](int R, bool wl, bool mr, bool ahead) {
    return 4 * ((size_t)(wl ? a.w_floats[0] + a.w_floats[1] : 0) + a.b_floats[0] + a.b_floats[1] + hid_floats(R, ahead) +
                (size_t)R * (rstride(O) + rstride(A) + rstride(1) + 2 * in_stride(O, A) + (ahead ? 8 * npr : 0) + nba + nbo + 1) +
                ((2 * A + 3) & ~3) + (mr ? (size_t)a.o4 * a.ms : 0));
  };
  // 32 envs per workgroup once tiles of 16 are more than the compute units, which hold one workgroup each.  us for 16 steps,
  // 16 / 32 envs (the kernel's first form): 45:128:128:12 289 / 362 for 4096 envs, 569 / 360 for 5000; 60:128:64:8 243 / 301, 475 / 305
  // Height and refusal go by the bytes of the kernel's first form (one state per env, two steps' draws): what was refused stays
  // refused.  Without draws ahead the present form never takes more.
  auto admission = [&](int R) {
    return 4 * ((size_t)a.b_floats[0] + a.b_floats[1] +
                (size_t)R * (rstride(O) + 4 * a.sh + rstride(A) + rstride(1) + a.o4 + 8 * npr + nba + nbo + 1) + ((R * (O + A) + 3) & ~3) +
                ((2 * A + 3) & ~3));
  };
  // layers of at most four feature tiles give each of a net's four waves one tile at most: then the networks in registers and the roles
  // of a step on waves of their own, 16 envs at any number of them.  us for 16 steps, against the other kernel (32 envs beyond 4096): 17:64:64:6 55 / 81 for 4096 envs, 98 /
  // 126 for 8192, 141 / 244 for 9000, 231 / 364 for 20000; 100:64:64:6 112 / 153 for 1000, 320 / 478 for 9000; 8:32:2 29 / 55 for 64, 126 /
  // 206 for 20000.
  const int w0_rows = O <= 64 ? 0 : pad16(L.net[0][0].out), m_floats = a.o4 * a.ms;
  const size_t split_bytes = (size_t)split_lds(O, A, a.sh, w0_rows, 0).floats * 4;
  bool split = L.n_layers <= kPlanLayers && split_bytes <= kLdsMax && admission(16) <= kLdsMax;
  for (int net = 0; net < 2; ++net)
    for (const LayerInfo& li : L.net[net]) split = split && li.out <= 64;
  const int R = !split && (a.n + 15) / 16 > g->cu_count && admission(32) <= kLdsMax ? 32 : 16;
  if (admission(R) > kLdsMax)
    GMI_FAIL(GMI_ERR_UNSUPPORTED, "rollout_collect_f32: a 16-env tile of this model needs %zu bytes of LDS (limit %zu); "
             "use agent_act / env_step / collect_experience", admission(R), kLdsMax);
  a.ahead = lds(R, false, false, true) <= kLdsMax ? 1 : 0;
  a.hid_floats = hid_floats(R, a.ahead != 0);
  typedef void (*kernel_fn)(RolloutF32Args);
  kernel_fn kernel;
  size_t bytes;
  int variant, threads = kNT;
  if (split) {
    a.mr_lds = split_bytes + (size_t)m_floats * 4 <= kLdsMax ? 1 : 0;
    bytes = split_bytes + (a.mr_lds ? (size_t)m_floats * 4 : 0);
    auto pick = [&](auto nl) -> kernel_fn {      // (inputs of at most 64 features: the matrix always fits)
      constexpr int NL = decltype(nl)::value;
      return O <= 64 ? rollout_split_kernel<NL, true, true> : a.mr_lds ? rollout_split_kernel<NL, false, true> : rollout_split_kernel<NL, false, false>;
    };
    kernel = L.n_layers == 2   ? pick(std::integral_constant<int, 2>{})
             : L.n_layers == 3 ? pick(std::integral_constant<int, 3>{})
                               : pick(std::integral_constant<int, 4>{});
    variant = 2 + 3 * (L.n_layers - 2) + (O <= 64 ? 0 : a.mr_lds ? 1 : 2);
    threads = kSplitThreads;
  } else {
    // what stays on chip for all steps: the networks' weights first (read by every layer), then the simulator's matrix
    const bool wl = lds(R, true, false, a.ahead != 0) <= kLdsMax;
    a.mr_lds = lds(R, wl, true, a.ahead != 0) <= kLdsMax ? 1 : 0;
    bytes = lds(R, wl, a.mr_lds != 0, a.ahead != 0);
    kernel = wl ? rollout_f32_kernel<true> : rollout_f32_kernel<false>;
    variant = wl;
  }
  set_rows(&a, R);
  static gmi::DeviceSet allowed[11];
  const int rc2 = gmi::allow_lds((const void*)kernel, kLdsMax, g->device, &allowed[variant]);
  if (rc2 != GMI_OK) return rc2;
  // no more workgroups than the instance's compute units hold at once (see rollout_collect)
  int64_t resident = 1;
  const int rc3 = gmi::resident_groups(g, (const void*)kernel, threads, bytes, &resident);
  if (rc3 != GMI_OK) return rc3;
  const int grid = (int)std::min<int64_t>(a.n_tiles, resident);
  gmi::ProfScope ps(g, gmi::kClsFusedRollout);
  ps.launch(kernel, dim3(grid), dim3(threads), bytes, a);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}
