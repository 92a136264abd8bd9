// Host side of the row-tile kernels (tile_kernel.h): the weight stream in the shadow, its packing kernel and the launches.  The
// kernels themselves are compiled once per model shape, the trainers in tile_p<k>.hip, the forward-only ones in tile_f<k>.hip.
#include <stdlib.h>

#include "tile_kernel.h"

namespace {
using namespace gmi_chain;

// ---------------------------------------------------------------------------------------------------------
// Packing kernel: builds one net's chain stream from the row-major bf16 shadows.  One thread per lane of a
// block (16 bytes).  Lane L of block (tile ft, k step ks) of a segment holds, for output row m = 32 ft + L % 32,
// the 8 contraction indices 16 ks + p(L / 32, j), j = 0..7: p(h, j) = 8 h + j for the first forward layer
// (whose input is loaded from memory in natural order) and p(h, j) = 8 (j / 4) + 4 h + j % 4 for every other
// segment (the order in which the matrix instruction leaves a lane's 8 results of a k step).
struct PackSeg {
  int blk_start;          // first block of the segment in the stream
  int K, F;               // padded contraction / output widths
  int natural;            // 1: first forward layer
  int64_t src;            // byte offset into the shadow of the source matrix, row-major [F, K] bf16
};
struct PackTable {
  int n;
  int total_blocks;
  PackSeg s[2 * (GMI_MAX_HIDDEN + 1)];
};

__global__ __launch_bounds__(256) void chain_pack_kernel(PackTable t0, PackTable t1, const char* __restrict__ shadow,
                                                         char* __restrict__ out0, char* __restrict__ out1) {
  const PackTable& tab = blockIdx.y == 0 ? t0 : t1;
  char* out = blockIdx.y == 0 ? out0 : out1;
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int blk = (int)(gid >> 6), lane = (int)(gid & 63);
  if (blk >= tab.total_blocks) return;
  int si = 0;
  while (si + 1 < tab.n && blk >= tab.s[si + 1].blk_start) ++si;
  const PackSeg& S = tab.s[si];
  const int nft = S.F >> 5, nks = S.K >> 4;
  int lb = blk - S.blk_start;
  // locate the group: full groups of kGroupTiles tiles first, then (2), then (1)
  constexpr int gm = kGroupTiles;
  const int full = nft / gm;
  int tile0, gs;
  if (lb < full * gm * nks) {
    const int gi = lb / (gm * nks);
    tile0 = gm * gi; gs = gm; lb -= gi * gm * nks;
  } else {
    lb -= full * gm * nks;
    tile0 = gm * full;
    if ((nft % gm) >= 2) {
      if (lb < 2 * nks) { gs = 2; }
      else { lb -= 2 * nks; tile0 += 2; gs = 1; }
    } else {
      gs = 1;
    }
  }
  const int ks = lb / gs, t = lb - ks * gs;
  const int m = 32 * (tile0 + t) + (lane & 31), h = lane >> 5;
  const uint16_t* row = reinterpret_cast<const uint16_t*>(shadow + S.src) + (int64_t)m * S.K + 16 * ks;
  uint16_t e[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) e[j] = row[S.natural ? 8 * h + j : 8 * (j >> 2) + 4 * h + (j & 3)];
  uint4 v;
  v.x = e[0] | ((uint32_t)e[1] << 16); v.y = e[2] | ((uint32_t)e[3] << 16);
  v.z = e[4] | ((uint32_t)e[5] << 16); v.w = e[6] | ((uint32_t)e[7] << 16);
  reinterpret_cast<uint4*>(out)[(int64_t)blk * 64 + lane] = v;
}

ChainDims dims_of(const ModelLayout& L) {
  ChainDims D;
  D.nl = L.n_layers;
  for (int l = 0; l < L.n_layers; ++l) { D.d[l] = L.net[0][l].in_pad; D.d[l + 1] = L.net[0][l].out_pad; }
  return D;
}

typedef int (*part_fn)(gmi_instance*, const ModelLayout&, const ChainArgs&, int, int*, double, double);
const part_fn kTileFns[gmi::kTileParts] = {gmi::launch_tile_part0, gmi::launch_tile_part1, gmi::launch_tile_part2,
                                           gmi::launch_tile_part3, gmi::launch_tile_part4, gmi::launch_tile_part5};
const part_fn kTileFwdFns[gmi::kTileFwdParts] = {gmi::launch_tile_fwd_part0, gmi::launch_tile_fwd_part1, gmi::launch_tile_fwd_part2,
                                                 gmi::launch_tile_fwd_part3, gmi::launch_tile_fwd_part4, gmi::launch_tile_fwd_part5};

// True if a trainer kernel is compiled for this model's shape.
bool compiled(const ModelLayout& L) {
  ChainArgs none = {};
  int v = 0;
  for (int p = 0; p < gmi::kTileParts; ++p)
    if (kTileFns[p](nullptr, L, none, 0, &v, 0.0, 0.0) == GMI_OK) return true;
  return false;
}

}  // namespace


namespace gmi {
using namespace gmi_chain;

bool chain_compiled(const ModelLayout& L) { return L.sh_chain_bytes != 0 && compiled(L); }

// Bytes of one net's chain stream (0 if the two nets' padded widths differ, which only a policy head wider
// than 32 outputs can cause: such models have no chain stream).
int64_t chain_stream_bytes(const ModelLayout& L) {
  if (L.dtype != GMI_DTYPE_BF16) return 0;
  for (int l = 0; l < L.n_layers; ++l)
    if (L.net[0][l].in_pad != L.net[1][l].in_pad || L.net[0][l].out_pad != L.net[1][l].out_pad) return 0;
  return (int64_t)cd_nblocks(dims_of(L)) * 1024 + 16 * 1024;      // (the padding keeps the size that shadows always had)
}

// Rebuilds both nets' chain streams from the row-major shadows (W for the forward segments, W^T for the
// input-gradient segments).
int launch_chain_pack(gmi_instance* g, gmi_model* m) {
  const ModelLayout& L = m->L;
  if (L.sh_chain_bytes == 0) return GMI_OK;
  if (!compiled(L)) return GMI_OK;                     // no kernel for this shape: nobody reads the stream
  const ChainDims D = dims_of(L);
  PackTable t[2];
  for (int net = 0; net < 2; ++net) {
    t[net].n = cd_nseg(D);
    int blk = 0;
    for (int s = 0; s < cd_nseg(D); ++s) {
      PackSeg& ps = t[net].s[s];
      const int l = cd_layer(D, s);
      ps.blk_start = blk;
      ps.K = cd_K(D, s);
      ps.F = cd_F(D, s);
      ps.natural = s == 0 ? 1 : 0;
      ps.src = s < D.nl ? L.net[net][l].sh_w : L.net[net][l].sh_wt;
      blk += cd_seg_blocks(D, s);
    }
    t[net].total_blocks = blk;
  }
  const int64_t threads = (int64_t)t[0].total_blocks * 64;
  ProfScope ps(g, kClsShadowTranspose);
  ps.launch(chain_pack_kernel, dim3((unsigned)((threads + 255) / 256), 2), dim3(256), 0, t[0], t[1], (const char*)m->shadow,
            m->shadow + L.sh_chain[0], m->shadow + L.sh_chain[1]);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

void fill_chain_emit(const ModelLayout& L, ChainEmit* ce) {
  ce->gmax = 0;
  ce->n_layers = L.n_layers;
  if (L.sh_chain_bytes == 0) return;
  if (!compiled(L)) return;
  const ChainDims D = dims_of(L);
  ce->gmax = kGroupTiles;
  for (int net = 0; net < 2; ++net) {
    ce->out[net] = L.sh_chain[net];
    for (int l = 0; l < L.n_layers; ++l) ce->l[net * L.n_layers + l] = ChainEmitLayer{0, -1, l == 0 ? 1 : 0};
    int blk = 0;
    for (int s = 0; s < cd_nseg(D); ++s) {
      ChainEmitLayer& e = ce->l[net * L.n_layers + cd_layer(D, s)];
      if (s < D.nl) e.fwd_blk = blk; else e.bwd_blk = blk;
      blk += cd_seg_blocks(D, s);
    }
  }
}

// Gather of the minibatch rows idx[0..rows) of buffer b + forward + loss + input gradients.
// Leaves m->h, m->dz ready for the weight-gradient launch and one row of statistics / log_std partials per
// tile in m->stat_part (*n_stat_rows rows, the layout of the loss kernel's per-workgroup rows).  GMI_ERR_UNSUPPORTED (no message) if
// no kernel is compiled for this shape.
int prepare_obs16(gmi_instance* g, gmi_model* m, gmi_buffer* b, int rows, int cus, bool* ready) {
  const ModelLayout& L = m->L;
  *ready = false;
  if (!b->obs16 || g->fusion < 1 || L.dtype != GMI_DTYPE_BF16 || L.sh_chain_bytes == 0 || L.act_dim > 32 ||
      use_resident(L, rows, cus) || !compiled(L))
    return GMI_OK;
  const int64_t B = (int64_t)b->d.horizon * b->d.n_envs;
  const int rc = launch_gather_to(g, m, b->d.obs, b->d.n_envs, b->d.ld_envs, nullptr, (int)B, nullptr, b->obs16);
  if (rc == GMI_OK) *ready = true;
  return rc;
}

int launch_train_chain(gmi_instance* g, gmi_model* m, gmi_buffer* b, const gmi_ppo_hparams* hp, const int32_t* idx, int rows,
                       int* n_stat_rows, bool obs16_ready) {
  const ModelLayout& L = m->L;
  if (L.dtype != GMI_DTYPE_BF16 || L.sh_chain_bytes == 0 || L.act_dim > 32) return GMI_ERR_UNSUPPORTED;
  // fetch_actions (tile_kernel.h) reads four actions at a time
  if (((int64_t)(b->d.horizon - 1) * b->d.ld_envs + b->d.n_envs) * L.act_dim < 4) return GMI_ERR_UNSUPPORTED;
  ChainArgs a;
  for (int net = 0; net < 2; ++net) {
    a.wstream[net] = m->shadow + L.sh_chain[net];
    for (int l = 0; l < L.n_layers; ++l) {
      a.bias[net][l] = reinterpret_cast<const float*>(m->shadow + L.net[net][l].sh_b);
      a.h[net][l] = (uint16_t*)m->h[net][l];
      a.dz[net][l] = (uint16_t*)m->dz[net][l];
    }
  }
  a.x0 = (uint16_t*)m->x0;
  a.x0b = (uint16_t*)m->x0b;
  a.log_std = reinterpret_cast<const float*>(m->shadow + L.sh_logstd);
  a.idx = idx;
  a.b_obs = b->d.obs; a.b_act = b->d.act; a.b_logp = b->d.logp; a.b_adv = b->d.adv; a.b_ret = b->d.ret;
  a.n_envs = b->d.n_envs; a.ld_envs = b->d.ld_envs; a.obs_dim = L.obs_dim;
  a.x0_ready = (L.obs_dim % 4 == 0 && ((uintptr_t)b->d.obs & 15) == 0) ? 0 : 1;
  a.x16 = b->obs16;
  if (a.x0_ready == 1 && obs16_ready && b->obs16 && idx) a.x0_ready = 2;
  a.stream = beyond_cache(L, rows) ? 1 : 0;
  a.rows = rows; a.act_dim = L.act_dim;
  a.clip = hp->clip; a.c_v = hp->c_v;
  a.stat_part = m->stat_part;
  int tiles = 0, rc;
  if (rows < 1 || rows > m->max_rows) return GMI_ERR_UNSUPPORTED;      // the activation arrays hold max_rows (in whole tiles)
  // algorithmic work at the logical (unpadded) widths: forward products of every layer, input-gradient products
  // of every layer but the first; bytes: the input rows and per-sample scalars read, every hidden activation
  // written once (and read once for ELU': reread), every layer's output gradient written once, the weights read once
  double flops = 0.0, bytes = 0.0;
  a.reread = 0.0;
  for (int net = 0; net < 2; ++net) {
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      flops += 2.0 * rows * (double)li.in * li.out * (l == 0 ? 1.0 : 2.0);
      bytes += 2.0 * li.in * li.out * (l == 0 ? 1.0 : 2.0);                 // bf16 weights, forward (+ transposed)
      bytes += 2.0 * rows * li.out;                                          // gradient at the layer's output
      // fp32 observation rows read and the bf16 copy written (once), or the gathered bf16 rows read, or those read
      // from the copy of all observations and written in minibatch order
      if (l == 0) bytes += net == 0 ? (a.x0_ready == 1 ? 2.0 : (a.x0_ready == 2 ? 4.0 : 6.0)) * rows * li.in : 0.0;
      else bytes += 2.0 * rows * li.in, a.reread += 2.0 * rows * li.in;      // hidden activation
    }
  }
  bytes += 4.0 * rows * (L.act_dim + 3);
  if (!compiled(L)) return GMI_ERR_UNSUPPORTED;
  if (a.x0_ready == 1) {  // unaligned observation rows: the gather kernel converts them
    rc = launch_gather(g, m, b->d.obs, b->d.n_envs, b->d.ld_envs, idx, rows, nullptr);
    if (rc != GMI_OK) return rc;
  }
  rc = GMI_ERR_UNSUPPORTED;
  for (int p = 0; p < kTileParts && rc == GMI_ERR_UNSUPPORTED; ++p) rc = kTileFns[p](g, L, a, rows, &tiles, flops, bytes);
  if (rc != GMI_OK) return rc;
  *n_stat_rows = tiles;
  return GMI_OK;
}

// What the forward-only kernel of the shape answers: 0 its own order of summation, 1 the agent kernel's; -1 if there is none.
static int forward_kind(const ModelLayout& L) {
  if (L.dtype != GMI_DTYPE_BF16 || L.sh_chain_bytes == 0 || L.act_dim > 32) return -1;
  const ChainArgs a = {};
  int kind = 0;
  for (int p = 0; p < kTileFwdParts; ++p)
    if (kTileFwdFns[p](nullptr, L, a, 0, &kind, 0.0, 0.0) == GMI_OK) return kind;
  return -1;
}
bool has_tile_forward(const ModelLayout& L) { return forward_kind(L) == 0; }

// agent_act with the agent kernel / with this one, us:
//   211:512:512:256:128:20 18.4 / 20.3 for 2048 rows, 19.5 / 20.8 for 4096, 27.2 / 20.8 for 4352, 30.2 / 23.7 for 8192, 41.9 / 28.6 for 9216,
//     43.0 / 30.2 for 12032, on 64 compute units 18.3 / 20.3 for 1024, 26.7 / 20.2 for 1088, 39.1 / 25.7 for 2304, on 16 18.2 / 19.9 for
//     256, 26.5 / 20.0 for 272;
//   211:512:512:512:256:20 24.4 / 25.3 for 4096 rows, 33.7 / 27.0 for 4352, 39.1 / 29.2 for 8192, 54.7 / 35.6 for 9216, on 64 compute
//     units 23.1 / 24.4 for 1024, 33.0 / 24.5 for 1088.
// A collection of 16 steps of them: 661 / 676 for 4096 envs, 901 / 781 for 6144, 1319 / 1090 for 12280; 750 / 785, 1024 / 877, 1541 / 1238.
// agent_value alone, the same network pass bit for bit and so the same line: 16.9 / 17.3 and 20.6 / 21.5 from 17 to 32 rows per
// compute unit, 26.8 / 17.3 and 34.0 / 21.6 beyond.  The two add in different orders (error against 64 bits 5.39e-3 and 5.39e-3): a
// row's last bit depends on the side of the line.
// The shapes whose kernel computes in the agent kernel's order are free to choose.  Agent kernel / this one, us:
//   60:256:128:64:8 8.6 / 7.6 for 64 rows, 9.0 / 8.3 for 4096, 11.0 / 8.5 for 8192, 25 / 16 for 32768, 168 / 102 for 262144, on 64 compute
//     units 8.6 / 7.8 for 256, 10.4 / 8.2 for 2048;
//   108:400:200:100:21 11.9 / 13.7 for 512 rows, 12.6 / 14.0 for 4096, 15.7 / 14.2 for 5000, 31 / 19 for 16384, 428 / 262 for 262144, on 64
//     compute units 11.9 / 13.7 for 1024, 15.0 / 13.7 for 2048, on 16 11.8 / 13.3 for 256, 14.9 / 13.7 for 512;
//   23:256:128:64:9, whose rows start at any 4-byte address, 9.1 / 9.3 for 2048, 9.3 / 9.3 for 4096, 10.8 / 9.3 for 5000, 172 / 99 for
//     262144.
// The values of a collection of 108:400:200:100:21 (4096 envs, 32 steps) 128 / 79.
// So: layers of more than 8 feature tiles, which this kernel's 4 waves take 4 at a time and the agent kernel's 8 waves 2, and unaligned
// rows, from the rows on that give the agent kernel more than one workgroup per compute unit (32 rows of one net each); else always.
bool use_tile_forward(const gmi_instance* g, const gmi_model* m, int64_t rows) {
  const ModelLayout& L = m->L;
  const int kind = forward_kind(L);
  if (kind < 0 || L.obs_dim < 4) return false;
  return (cd_maxdim(dims_of(L)) <= 256 && L.obs_dim % 4 == 0) || rows > 16 * (int64_t)g->cu_count;
}

bool forward_chain_reads_x0(const gmi_model* m, const float* obs) {
  return !(m->L.obs_dim % 4 == 0 && ((uintptr_t)obs & 15) == 0);
}

static void fill_forward(const gmi_model* m, ChainArgs* a) {
  const ModelLayout& L = m->L;
  const bool nat = forward_kind(L) == 1;
  for (int net = 0; net < 2; ++net) {
    a->wstream[net] = m->shadow + (nat ? 0 : L.sh_chain[net]);
    for (int l = 0; l < L.n_layers; ++l) {
      a->bias[net][l] = reinterpret_cast<const float*>(m->shadow + L.net[net][l].sh_b);
      a->wf_off[net][l] = (int)L.net[net][l].sh_wf;
    }
  }
  a->x0 = (uint16_t*)m->x0;
  a->log_std = reinterpret_cast<const float*>(m->shadow + L.sh_logstd);
  a->obs_dim = L.obs_dim; a->act_dim = L.act_dim;
  a->T = 1;
}
static int launch_forward(gmi_instance* g, const gmi_model* m, const ChainArgs& a, double out_floats) {
  const ModelLayout& L = m->L;
  const double rows = (double)a.rows * (a.T + (a.val_last ? 1 : 0));
  double flops = 0.0, bytes = 0.0;
  for (int net = a.net0; net < 2; ++net)
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      flops += 2.0 * rows * (double)li.in * li.out;
      bytes += 2.0 * li.in * li.out;
    }
  bytes += (a.x0_ready == 1 ? 2.0 : 4.0) * rows * L.obs_dim * (2 - a.net0) + 4.0 * rows * out_floats;
  int tiles = 0, rc = GMI_ERR_UNSUPPORTED;
  for (int p = 0; p < kTileFwdParts && rc == GMI_ERR_UNSUPPORTED; ++p) rc = kTileFwdFns[p](g, L, a, a.rows, &tiles, flops, bytes);
  return rc;
}

// Inference through the forward-only row-tile kernel.
int launch_forward_chain(gmi_instance* g, gmi_model* m, const float* obs, int n_rows, bool policy, float* mu, float* val,
                         bool x0_valid, const ActionSample* sample) {
  const ModelLayout& L = m->L;
  if (n_rows < 1 || n_rows > m->max_rows || !use_tile_forward(g, m, n_rows)) return GMI_ERR_UNSUPPORTED;
  ChainArgs a = {};
  fill_forward(m, &a);
  a.b_obs = obs;
  a.x0_ready = !forward_chain_reads_x0(m, obs) ? 0 : (x0_valid ? 1 : 3);
  a.rows = n_rows;
  a.net0 = policy ? 0 : 1;
  a.mu_out = mu; a.val_out = val;
  if (sample) {
    a.act_out = sample->act; a.logp_out = sample->logp;
    a.k0 = (uint32_t)sample->seed; a.k1 = (uint32_t)(sample->seed >> 32); a.step = sample->step; a.env_offset = sample->env_offset;
  }
  return launch_forward(g, m, a, (mu ? L.act_dim : 0) + (sample ? L.act_dim + 1 : 0) + 1);
}

int launch_forward_values(gmi_instance* g, gmi_model* m, const float* obs, int T, int n, int64_t ld, float* value, const float* obs_last,
                          float* value_last) {
  const ModelLayout& L = m->L;
  const int64_t slots = T + (value_last ? 1 : 0), tiles = (n + 63) / 64;
  if (forward_kind(L) != 1 || T < 1 || tiles * slots >= (1 << 30) || 3 * (int64_t)n < 2 * 64 * tiles || !use_tile_forward(g, m, slots * n))
    return GMI_ERR_UNSUPPORTED;
  ChainArgs a = {};
  fill_forward(m, &a);
  a.b_obs = obs; a.obs_last = obs_last;
  a.T = T; a.obs_step = ld * L.obs_dim; a.val_step = ld;
  a.val_out = value; a.val_last = value_last;
  a.rows = n;
  a.net0 = 1;
  a.x0_ready = forward_chain_reads_x0(m, obs) || (a.obs_step & 3) != 0 || (value_last && forward_chain_reads_x0(m, obs_last)) ? 3 : 0;
  return launch_forward(g, m, a, 1.0);
}

}  // namespace gmi
