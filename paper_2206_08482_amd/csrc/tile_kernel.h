// Row-tile trainer kernel for the model shapes compiled in tile_p<k>.hip (hidden widths padded to multiples of 32): minibatch gather,
// forward pass, clipped-surrogate / value loss and the whole input-gradient chain of one minibatch (stage (ii)
// of Section 5.1 of the paper, the "DRL Trainer" role of Section 3) in one launch per minibatch.
//
// A workgroup owns 64 samples (4 waves, two workgroups per compute unit) or 128 (8 waves) and keeps their current activations in
// LDS, as the second operands of the 32x32x16 matrix instruction: block (k step ks, row tile rt) = 1 KiB, lane L of it = the 8
// contraction values of sample 32 rt + L % 32 that operand lane L takes.  Every product is computed transposed, H^T = W X^T, and a
// wave owns a slice of the layer's OUTPUT FEATURES for all samples (8 accumulator tiles = 128 registers at most; where there are
// fewer feature tiles than waves, two or four waves share one and split its rows): per k step it fetches its own weight blocks
// straight from the second-level cache into registers (no other wave of the workgroup needs them) and the activation blocks from
// LDS, i.e. 6 KiB of operands for 8 matrix instructions.  (With a wave per 32 samples and the weights in LDS every wave reads every
// weight block: 1 KiB of LDS traffic per matrix instruction, which is the LDS bandwidth of a compute unit.)  The weights come from
// the weight stream (chain_stream.h): its blocks are the first operands of exactly these products, its k order inside a 16-wide step
// is the order in which the matrix instruction leaves its results in a lane, so a lane's 8 results of a k step are written back to
// LDS as one 16-byte piece at its own lane's slot.
//
// A layer is: k loop (all accumulators of the layer live at once) - barrier - epilogue (bias + ELU, or x ELU' of
// the stored activation; conversion; the results into LDS in place of the layer's input; from there they go to memory
// for the weight-gradient kernel) - barrier (variants: TileShapeKeep, late_write).  The next layer's first weight blocks are fetched
// before the epilogue.
//
// Two waves per SIMD: an epilogue is straight-line code that runs once, and a wave gets its instructions at about a byte per cycle,
// half of what the vector unit takes, so one wave alone is bound by them.  In the k loops one wave's fetches ride under the
// other's products, and two workgroups of 64 samples have their barriers, epilogues, loss and start at different times.  What bounds
// the walk now: instructions in the epilogues, and the activations and gradients on their way to memory and back (307 MB for 32768
// samples of 108:400:200:100:21, 540 MB of 211:512:512:256:128:20: 63 and 110 us at the rate of a copy; the matrix unit 19 and 53).
// Forward + loss + gradients of 32768 samples, us: 211:512:512:256:128:20 220 with 4 waves of 128 samples, 178 with 8;
// 108:400:200:100:21 107 with a wave's activations in registers and the weights through LDS, 86 with 8 waves of 128 samples, 79 with 4
// of 64; 60:256:128:64:8 44, 46 and 39.
//
// TileShapeFwd is the same walk cut after the heads (agent_act / agent_value of these models: Section 3, "DRL Agent"):
// nothing is stored for the weight gradients and the heads' results go out as policy means and values.
#pragma once
#include "chain_stream.h"
#include "rng.h"

namespace gmi_tile {
using namespace gmi_chain;

constexpr int kScrBytes = 32 * 33 * 4;      // a loss wave's transposition buffer
constexpr int kHPre = 4;          // tiles whose stored activations are fetched ahead in an input-gradient epilogue

__device__ __forceinline__ intx8 join8(const uint4& a, const uint4& b) {
  const intx8 r = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, (int)b.z, (int)b.w};
  return r;
}

// ROWS: samples per workgroup, 128 (8 waves) or 64 (4 waves).
template <int ROWS, int... DIMS>
struct TileShape {
  static constexpr int rows = ROWS, nrt = ROWS / 32, waves = 2 * nrt, threads = 64 * waves;
  static constexpr int acc_ft = 16 / waves, ring = 8;      // feature tiles of a wave; weight blocks in flight per wave
  static constexpr bool fwd = false;      // TileShapeFwd, TileShapeNat: the forward pass alone (inference)
  static constexpr bool nat = false;      // TileShapeNat, TileShapeFp8
  static constexpr bool fp8 = false;      // TileShapeFp8
  static constexpr bool lp_blocks = false;      // log-densities by blocks of four actions
  static constexpr bool keep = false;      // TileShapeKeep
  static constexpr int store_aux = 17;      // write-through
  // Two waves of the workgroup on a SIMD: the first four take the matrix unit first and are done with the k loop while the others
  // are half way; a layer's results then wait in registers for the barrier behind which they may replace its input, so that the first
  // waves' epilogue runs under the others' products.  (32768 rows of 211:512:512:256:128:20 184 us, 176 so.  With waves of two
  // workgroups on a SIMD, which are at different places anyway, the writes in one piece only cost: 81 and 86 us of 108:400:200:100:21.)
  static constexpr bool late_write = ROWS == 128;
  static constexpr int NL = (int)sizeof...(DIMS) - 1;
  static constexpr ChainDims dims() { return ChainDims{NL, {DIMS...}}; }
  static constexpr int nseg() { return cd_nseg(dims()); }
  static constexpr int maxks() { return cd_maxdim(dims()) / 16; }
  static constexpr int bias_total() {
    int n = 0;
    for (int l = 0; l < NL; ++l) n += dims().d[l + 1];
    return n;
  }
  static constexpr int bias_off(int l) {
    int n = 0;
    for (int i = 0; i < l; ++i) n += dims().d[i + 1];
    return n;
  }
  static constexpr int seg_blk0(int s) {
    int n = 0;
    for (int i = 0; i < s; ++i) n += cd_seg_blocks(dims(), i);
    return n;
  }
  // first block of the activation area that holds layer l's input (TileShapeKeep: an area per layer; TileShapeTurns: two areas; else one)
  static constexpr int area(int) { return 0; }
  // the loss epilogue's per-wave transposition buffers live in the activation area behind the head layer's input
  static constexpr size_t scr_offset() { return (size_t)dims().d[NL - 1] / 16 * nrt * 1024; }
  static constexpr size_t x_bytes() { return (size_t)maxks() * nrt * 1024; }
  static constexpr size_t lds_bytes() { return x_bytes() + (size_t)bias_total() * 4 + (size_t)(nrt * 40 + 64) * 4; }
  static constexpr bool valid() {
    const ChainDims D = dims();
    if (D.d[NL] != 32 || maxks() > 32) return false;
    for (int l = 0; l < NL; ++l)
      if (D.d[l] % 32 != 0) return false;
    return (ROWS == 64 || ROWS == 128) && x_bytes() >= scr_offset() + (size_t)nrt * kScrBytes;
  }
};

// The same with all layers' activations in LDS until the gradient takes their place: the backward epilogues read ELU's inputs there
// (from memory they were 59 of the 219 MB that 32768 rows of 60:256:128:64:8 moved), and a layer's results do not go where its input
// lies, so one barrier per layer is enough.  Area l: layer l's input, then the gradient at it; area NL: the heads' gradient.  The
// first layer's area has no gradient and serves the loss as its transposition buffers.  For shapes of which two workgroups fit a
// compute unit that way (kKeepBytes): with one (108:400:200:100:21) nothing covers a wave's waits.  Agents' kernels that run beside the trainer
// find less LDS free, but lose nothing by it: lag-1 iterations of 60:256:128:64:8, us kept / read from memory, four agents of 4096
// envs (16 steps, four epochs of 32768 rows) unmasked 2609 / 2776, on 32 compute units each 2519 / 2685, apart from the trainer 4769 / 5056; one
// agent 646 / 686, 614 / 642 and 713 / 725.
template <int ROWS, int... DIMS>
struct TileShapeKeep : TileShape<ROWS, DIMS...> {
  using B = TileShape<ROWS, DIMS...>;
  static constexpr bool keep = true;
  static constexpr int area(int l) {
    int n = 0;
    for (int i = 0; i < l; ++i) {
      const int blocks = B::dims().d[i] / 16 * B::nrt, scr = (B::nrt * kScrBytes + 1023) / 1024;
      n += i == 0 && blocks < scr ? scr : blocks;
    }
    return n;
  }
  static constexpr size_t scr_offset() { return 0; }
  static constexpr size_t x_bytes() { return (size_t)(area(B::NL) + 2 * B::nrt) * 1024; }
  static constexpr size_t lds_bytes() { return B::lds_bytes() - B::x_bytes() + x_bytes(); }
};
constexpr size_t kKeepBytes = 80 * 1024;

// The same with streaming stores (write-through either way), for minibatches whose activations no cache holds until they are read
// (beyond_cache, with figures).  Not for the 512-wide shapes (24576 rows of 211:512:512:256:128:20, us per iteration without / with 2730 / 2813),
// whose weight gradients alone stream.
template <class B>
struct TileShapeStream : B {
  static constexpr int store_aux = 19;
};

// The same shape for inference: the walk ends after the heads, nothing is stored for the weight gradients, and the
// heads' results go out as policy means and values (the products and their order are the trainer's forward pass).
template <int ROWS, int... DIMS>
struct TileShapeFwd : TileShape<ROWS, DIMS...> {
  static constexpr bool fwd = true;
};
// The forward pass as the agent kernel computes it (agent_kernel.h), bit for bit: weights from the fragment-major copy in natural k
// order, activations in natural order, the bias added last, log-densities by blocks of four actions.  For the shapes whose
// collection (fused.hip) computes that way.
template <int ROWS, int... DIMS>
struct TileShapeNat : TileShape<ROWS, DIMS...> {
  static constexpr bool fwd = true, nat = true, lp_blocks = true;
};
// The same in fp8 (E4M3): agent_kernel's results for fp8, bit for bit.  A k step is 64 wide and its operands are two blocks: a lane's
// 32 k values of its row, 16 per block.
template <int ROWS, int... DIMS>
struct TileShapeFp8 : TileShape<ROWS, DIMS...> {
  static constexpr bool fwd = true, nat = true, fp8 = true;
  static constexpr int ring = 16;
  static constexpr size_t scr_offset() { return TileShape<ROWS, DIMS...>::scr_offset() / 2; }
  static constexpr size_t x_bytes() { return TileShape<ROWS, DIMS...>::x_bytes() / 2; }
  static constexpr size_t lds_bytes() { return TileShape<ROWS, DIMS...>::lds_bytes() - x_bytes(); }
  static constexpr bool valid() {
    const ChainDims D = TileShape<ROWS, DIMS...>::dims();
    for (int l = 0; l < D.nl; ++l)
      if (D.d[l] % 64 != 0) return false;
    return TileShape<ROWS, DIMS...>::valid() && x_bytes() >= scr_offset() + (size_t)TileShape<ROWS, DIMS...>::nrt * kScrBytes;
  }
};
// A forward-only shape with two activation areas that the layers take in turn: a layer's results do not go where its input lies, so one
// barrier per layer is enough.  The draws wait in the area that is not the heads' input.  For up to 256 wide layers, where a layer is as
// short as its waits, and launches of at most one workgroup per compute unit (turns).  us per decision of 60:256:128:64:8, without / with: 1
// row 7.24 / 6.95, 8192 rows 8.01 / 7.75, fp8 6.72 / 6.56 and 7.13 / 6.97; with more workgroups, which cover each other's waits, the larger
// areas only cost (262144 rows 91.2 / 94.2; 65536 rows of 211:512:512:256:128:20 in fp8 92.4 / 97.5).
template <class B>
struct TileShapeTurns : B {
  static constexpr bool keep = true;
  static constexpr int turn(int parity) {      // blocks of the area of the even or odd layers' inputs
    int n = B::NL % 2 == parity ? (B::nrt * kScrBytes + 1023) / 1024 : 0;
    for (int l = parity; l < B::NL; l += 2) {
      const int blocks = B::dims().d[l] / (B::fp8 ? 32 : 16) * B::nrt;
      n = blocks > n ? blocks : n;
    }
    return n;
  }
  static constexpr int area(int l) { return l % 2 == 0 ? 0 : turn(0); }
  static constexpr size_t scr_offset() { return (size_t)area(B::NL) * 1024; }
  static constexpr size_t x_bytes() { return (size_t)(turn(0) + turn(1)) * 1024; }
  static constexpr size_t lds_bytes() { return B::lds_bytes() - B::x_bytes() + x_bytes(); }
};
template <class B>
using Turns = std::conditional_t<B::maxks() <= 16, TileShapeTurns<B>, B>;
inline bool turns(const ChainArgs& a, int rows, int cus) { return a.T <= 1 && !a.val_last && 2 * ((rows + 63) / 64) <= cus; }
// Segments the kernel runs for shape S.
template <class S>
constexpr int n_run() { return S::fwd ? S::NL : S::nseg(); }

template <class S, int SEG>
struct Seg {
  static constexpr ChainDims D = S::dims();
  static constexpr int K = cd_K(D, SEG), F = cd_F(D, SEG), NKS = K / (S::fp8 ? 64 : 16), NFT = F / 32;
  static constexpr int NP = S::fp8 ? 2 : 1;               // blocks of an operand
  static constexpr bool head = SEG == S::NL - 1;
  static constexpr bool bwd = SEG >= S::NL;
  static constexpr bool last = !S::fwd && SEG == S::nseg() - 1;
  static constexpr int layer = cd_layer(D, SEG);
  // Waves over features, then over rows: a wave has FTW feature tiles (tile_of) and the row tiles (w / NWF) RT ..  One feature tile
  // (the head) is a row tile per wave, by both halves of the workgroup (what the second half computes again is dropped).
  static constexpr int NWF = NFT == 1 ? 1 : (NFT == 2 ? 2 : (NFT <= 4 ? 4 : S::waves));
  static constexpr int FTW = (NFT + NWF - 1) / NWF;       // feature tiles per wave
  static constexpr int RT = NFT == 1 ? 1 : S::nrt * NWF / S::waves;      // row tiles per wave
  static constexpr bool even = NFT == NWF * FTW;          // every wave has FTW tiles of its own
  static constexpr int GS = NFT >= 4 ? 4 : NFT;           // tiles per group of the stream (chain_stream.h) ..
  static constexpr bool one_gs = NFT % 4 == 0 || NFT <= 2;      // .. if all its groups are alike
  static constexpr int DEP = S::ring / (FTW * NP) < NKS ? S::ring / (FTW * NP) : NKS;      // k steps of weight blocks in flight
  static constexpr int XD = FTW >= 2 || S::fp8 ? 1 : 2;             // k steps the activation blocks are read ahead (a k step of
                                                          // fewer products is shorter than an LDS round trip)
  static constexpr int blk0 = S::seg_blk0(SEG);
  static constexpr int in_area = S::area(bwd ? layer + 1 : layer), out_area = S::area(bwd ? layer : layer + 1);
  // The segment's input, which the previous segment's epilogue left in LDS, goes to memory block by block (for the
  // weight-gradient kernel and for ELU') DURING this segment's k loop: h[layer] in a forward segment, dz[layer] in an
  // input-gradient segment.  (Stores issued in the epilogue would all be older than the next k loop's weight
  // fetches, and the memory counter is in order: the loop would wait for every one of them.)  Not for the first
  // segment (the gather stores its rows) nor the first input-gradient segment (the loss epilogue stores the head's).
  static constexpr int HK = NKS > 6 ? NKS - 6 : 0;        // k step at which an input-gradient segment starts to fetch ELU' inputs
  static constexpr bool store_x = !S::fwd && ((SEG >= 1 && SEG <= S::NL - 1) || SEG > S::NL);
  static_assert(!head || NFT == 1, "the head is one 32-wide tile");
  static_assert(FTW <= S::acc_ft, "accumulators of a wave");
};

// The actions of one sample for a lane of the head: features 8 q + 4 hh .. + 3 for q = 0 .. 3, by 16-byte loads (4-byte aligned).  Every
// lane of a load touches a cache line of its own and those take a cycle each, so it is the number of loads that counts: 16
// single ones took a workgroup of train_tile_kernel 9 thousand cycles.  A load that would pass the row's end is moved
// back to end there and its values shifted into place where they are used (lane_actions); with fewer than 4 actions it begins
// in an earlier row, `back` elements before this one, but not before the array's start (the launch sees to 4 elements in all).
__device__ __forceinline__ int actions_back(int64_t slot, int A) {
  return A >= 4 ? 0 : (slot * A < 4 - A ? (int)(slot * A) : 4 - A);
}
__device__ __forceinline__ void fetch_actions(const float* act, int64_t slot, int A, int hh, float (&out)[16]) {
  typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
  const int top = A >= 4 ? A - 4 : 0;
  const float* row = act + slot * A - actions_back(slot, A);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int f0 = 8 * q + 4 * hh;
    const float4u t = *reinterpret_cast<const float4u*>(row + (f0 < top ? f0 : top));
    out[4 * q] = t.x; out[4 * q + 1] = t.y; out[4 * q + 2] = t.z; out[4 * q + 3] = t.w;
  }
}
__device__ __forceinline__ void lane_actions(const float (&in)[16], int A, int back, int q, int hh, float (&out)[4]) {
  const int f0 = 8 * q + 4 * hh;
  const int sh = A >= 4 ? f0 - (A - 4) : back;               // how far back the load began (4 and more: no feature of A)
  const float x0 = in[4 * q], x1 = in[4 * q + 1], x2 = in[4 * q + 2], x3 = in[4 * q + 3];
  const float y = sh == 1 ? x1 : (sh == 2 ? x2 : x3), z = sh == 1 ? x2 : x3;
  out[0] = sh <= 0 ? x0 : y;
  out[1] = sh <= 0 ? x1 : z;
  out[2] = sh <= 0 ? x2 : x3;
  out[3] = x3;
}

template <class S>
struct Ctx {
  floatx16 acc[S::acc_ft][S::nrt];
  uint4 wq[S::ring];                   // weight blocks of k steps g .. g + DEP - 1: block (ks, a) at (ks % DEP) * FTW + a
  uint4 xq[S::fp8 ? 2 : 3][S::nrt][S::fp8 ? 2 : 1];                    // activation blocks of k steps g .. g + XD (ring indexed by k step)
  uint32_t touched;                  // what prefetch_weights loads
  uint4 sx;                          // block of the activation area on its way to memory (store_x)
  uint4 hq[kHPre + 1][2];            // stored activations of the tiles ahead (input-gradient epilogues)
  const uint4* wnet;                 // this net's stream
  uint4* X;                          // activation area
  uint32_t lane16;                   // 16 lane
  uint32_t xo[2];                    // this lane's byte offset in the first 64 KiB of the activation area and behind them
  const float* s_bias;
  float* s_red;
  char* scr;                         // this wave's transposition buffer (loss epilogue only)
  int64_t slot;                      // experience slot of this lane's sample of the head layer
  int l_back;
  float l_act[16], l_lo, l_ad, l_rt;
  int tid, lane, wave, s, hh;
  int row0, net;                     // first row of the workgroup's tile
  float scale;                       // fp8: what the layer's weight codes are multiples of
  const float* obs;                  // inference: the slot's observation rows and values
  float* val_out;
  int tr, rt0;                       // 128-row tile of the stored arrays that it lies in, and its first row tile there
};

// Feature tile `a` of this wave: consecutive tiles where they divide evenly, else every NWF-th one, and beyond the last the last one
// again (its results are written twice, the same).
template <class G, class S>
__device__ __forceinline__ int tile_of(const Ctx<S>& c, int a) {
  if constexpr (G::NFT == 1) return 0;
  const int w = c.wave & (G::NWF - 1);
  if constexpr (G::even) return w * G::FTW + a;
  const int ft = a * G::NWF + w;
  return ft < G::NFT ? ft : G::NFT - 1;
}
template <class G, class S>
__device__ __forceinline__ int first_rt(const Ctx<S>& c) {
  if constexpr (G::NFT == 1) return c.wave & (S::nrt - 1);
  else if constexpr (G::NWF == S::waves) return 0;
  else return c.wave / G::NWF * G::RT;
}

// Where the weight blocks of a wave's feature tiles begin in the stream and how far apart its k steps are, in bytes.
struct WeightPos { int base[4], step[4]; };
template <class S, int SEG>
__device__ __forceinline__ WeightPos seg_weights(const Ctx<S>& c, const ChainArgs& args) {
  using G = Seg<S, SEG>;
  WeightPos p;
  if constexpr (S::nat) {
#pragma unroll
    for (int a = 0; a < G::FTW; ++a) {
      p.base[a] = args.wf_off[c.net][G::layer] + tile_of<G>(c, a) * G::NKS * G::NP * 1024;
      p.step[a] = G::NP * 1024;
    }
    return p;
  }
#pragma unroll
  for (int a = 0; a < G::FTW; ++a) {
    const int ft = tile_of<G>(c, a);
    int t0 = ft & ~3, gs = G::GS;                 // first tile and size of the tile's group: 4, .., 4, (2), (1)
    if constexpr (!G::one_gs) {
      const int left = G::NFT - t0;
      if (left < 4) {
        gs = left == 1 || ft - t0 == 2 ? 1 : 2;
        if (ft - t0 == 2) t0 = ft;
      }
    }
    p.base[a] = (G::blk0 + t0 * G::NKS + ft - t0) * 1024;
    p.step[a] = gs * 1024;
  }
  return p;
}
// This lane's 16 bytes of block (ks, rt) of the area at block `at`.  An LDS instruction's constant reaches 64 KiB: with one offset per half of the area every
// block is a constant away.  (Left to itself the compiler forms an address per block of the upper half, keeps them from one segment
// to the next and spills them: 47 registers, each reload in a k loop behind every fetch and store in flight.)
template <class S>
__device__ __forceinline__ uint4* x_block(const Ctx<S>& c, int at, int ks, int rt) {
  const int blk = at + ks * S::nrt;
  return reinterpret_cast<uint4*>(reinterpret_cast<char*>(c.X) + c.xo[blk / 64] + rt * 1024) + (blk % 64) * 64;
}
template <class S, int SEG, int KS>
__device__ __forceinline__ uint4 weight_block(const Ctx<S>& c, const WeightPos& w, int ta, int p) {
  return gmi::load_uniform(c.wnet, w.base[ta] + KS * w.step[ta] + p * 1024, c.lane16);
}
template <class S, int SEG, int KS>
__device__ __forceinline__ void issue_weights(Ctx<S>& c, const WeightPos& wseg) {
  using G = Seg<S, SEG>;
  if constexpr (KS < G::NKS) {
#pragma unroll
    for (int a = 0; a < G::FTW; ++a)
#pragma unroll
      for (int p = 0; p < G::NP; ++p) c.wq[((KS % G::DEP) * G::FTW + a) * G::NP + p] = weight_block<S, SEG, KS>(c, wseg, a, p);
  }
}
// The first DEP k steps of segment SEG (issued before the previous segment's epilogue).
template <class S, int SEG, int KS = 0>
__device__ __forceinline__ void issue_first_weights(Ctx<S>& c, const ChainArgs& a) {
  if constexpr (SEG < n_run<S>()) {
    if constexpr (KS < Seg<S, SEG>::DEP) {
      issue_weights<S, SEG, KS>(c, seg_weights<S, SEG>(c, a));
      issue_first_weights<S, SEG, KS + 1>(c, a);
    }
  }
}

// Touches segment SEG's weights, one word of every line, so that they are in the die's second-level cache when the k loop asks for
// them: workgroup q of the 32 that a die holds takes every 32nd line.  The workgroups of a die go through the layers nearly in step,
// and what they store and read back pushes the weights out between one round of workgroups and the next: without this every one
// of them waits for the same misses (a workgroup of 211:512:512:256:128:20 191 thousand cycles, now 171).  The one-line shapes' 358 KB
// and the forward kernels, which store next to nothing, gain nothing by it.
template <class S, int SEG>
__device__ __forceinline__ void prefetch_weights(Ctx<S>& c) {
  if constexpr (S::late_write && SEG < n_run<S>()) {
    asm volatile("" ::"v"(c.touched));
    constexpr uint32_t bytes = cd_seg_blocks(S::dims(), SEG) * 1024;
    static_assert(bytes <= 32u * 128 * S::threads, "a line per thread");
    const uint32_t q = (blockIdx.x + gridDim.x * blockIdx.y) >> 3 & 31;
    c.touched = __builtin_amdgcn_raw_buffer_load_b32(
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(c.wnet) + S::seg_blk0(SEG) * 64, 0, bytes, 0x00020000), (q + 32 * c.tid) * 128, 0, 0);
  }
}

template <class S>
constexpr int kXRing = S::fp8 ? 2 : 3;
template <class S, int SEG, int KS>
__device__ __forceinline__ void read_x(Ctx<S>& c) {
  using G = Seg<S, SEG>;
  if constexpr (KS < G::NKS) {
#pragma unroll
    for (int b = 0; b < G::RT; ++b)
#pragma unroll
      for (int p = 0; p < G::NP; ++p) c.xq[KS % kXRing<S>][b][p] = *x_block(c, G::in_area, KS * G::NP + p, first_rt<G>(c) + b);
  }
}

// Block layout of the activation / gradient arrays this kernel leaves for the weight-gradient kernel and for its own
// ELU' factors: exactly the 1 KiB operand blocks of the activation area, workgroup tile after workgroup tile:
// block (k step ks, row tile rt) of the 128 rows of tile tr of an array of NKS k steps starts at 16-byte word
// ((tr * NKS + ks) * 4 + rt) * 64.  (Row-major, a lane's 8 values of a k step are two 8-byte pieces of a row:
// 32 rows x 16 bytes per load or store instruction; as blocks every access is 1 KiB contiguous.)
__device__ __forceinline__ int64_t block_word(int tr, int nks, int ks, int rt) { return (((int64_t)tr * nks + ks) * 4 + rt) * 64; }

// One block to memory for the weight-gradient kernel.
template <class S>
__device__ __forceinline__ void store_block(uint4* blk, uint32_t lane16, const uint4& v, int off = 0) {
  gmi::store_through<S::store_aux>(blk, lane16, v, off);
}

// Streaming loads for them where the weights of the net fill the die's cache (211:512:512:256:128:20, us per iteration without / with: 12450 /
// 12170; 108:400:200:100:21 3108 / 3160).
template <class S>
constexpr int kHAux = S::late_write ? 2 : 0;
// Stored activations h[layer] of tile T = a * RT + b of this wave (input-gradient epilogue of segment SEG): the
// lane's own slots of the blocks (2 ft, b) and (2 ft + 1, b), i.e. the values at the positions of its 16 results.
template <class S, int SEG, int T>
__device__ __forceinline__ void fetch_h(Ctx<S>& c, const ChainArgs& a) {
  using G = Seg<S, SEG>;
  if constexpr (G::bwd && T < G::FTW * G::RT) {
    constexpr int ta = T / G::RT, tb = T % G::RT;
    constexpr int nks = G::D.d[G::layer] / 16;
    const int ft = tile_of<G>(c, ta);
    if constexpr (S::keep) {
      const uint4* x = c.X + (G::out_area + 2 * ft * S::nrt + first_rt<G>(c) + tb) * 64 + c.lane;
      c.hq[T % (kHPre + 1)][0] = x[0];
      c.hq[T % (kHPre + 1)][1] = x[S::nrt * 64];
      return;
    }
    const uint4* p = reinterpret_cast<const uint4*>(a.h[c.net][G::layer]) + block_word(c.tr, nks, 2 * ft, c.rt0 + first_rt<G>(c) + tb);
    c.hq[T % (kHPre + 1)][0] = gmi::load_uniform<kHAux<S>>(p, 0, c.lane16);
    c.hq[T % (kHPre + 1)][1] = gmi::load_uniform<kHAux<S>>(p, 4 * 1024, c.lane16);
  }
}

template <class S, int SEG, int T>
__device__ __forceinline__ void fetch_h_first(Ctx<S>& c, const ChainArgs& a) {
  if constexpr (T < kHPre) {
    fetch_h<S, SEG, T>(c, a);
    fetch_h_first<S, SEG, T + 1>(c, a);
  }
}

// The small operations that ride along with the products of k step KS, by index I: I < RT: the activation block of
// row tile I for k step KS + XD; then, where the segment's input goes to memory (store_x), wave w's share of that move, row tile
// w % nrt of every other k step: I = RT reads a block of the activation area at even k steps, I = RT + 1 stores it at odd ones.
template <class S, int SEG>
__device__ __forceinline__ uint4* store_x_array(const Ctx<S>& c, const ChainArgs& a) {
  using G = Seg<S, SEG>;
  return reinterpret_cast<uint4*>(G::bwd ? a.dz[c.net][G::layer] : a.h[c.net][G::layer]);
}
template <class S, int SEG, int KS, int I>
__device__ __forceinline__ void aux_op(Ctx<S>& c, const ChainArgs& a) {
  using G = Seg<S, SEG>;
  if constexpr (I < G::RT * G::NP) {
    if constexpr (KS + G::XD < G::NKS)
      c.xq[(KS + G::XD) % kXRing<S>][I / G::NP][I % G::NP] = *x_block(c, G::in_area, (KS + G::XD) * G::NP + I % G::NP, first_rt<G>(c) + I / G::NP);
  } else if constexpr (G::store_x) {
    static_assert(G::NKS % 2 == 0, "a wave moves a block every two k steps");
    if constexpr (I == G::RT * G::NP) {
      if constexpr (KS % 2 == 0) c.sx = *x_block(c, G::in_area, KS, c.wave);      // the second half of the waves: k step KS + 1
    } else if constexpr (KS % 2 == 1) {
      store_block<S>(store_x_array<S, SEG>(c, a) + block_word(c.tr, G::NKS, c.wave / S::nrt, c.rt0 + c.wave % S::nrt), c.lane16, c.sx,
                  (KS - 1) * 4096);      // arrays hold whole tiles
    }
  }
}
template <class S, int SEG, int KS, int FIDX, int I>
__device__ __forceinline__ void aux_slot(Ctx<S>& c, const ChainArgs& a) {
  using G = Seg<S, SEG>;
  constexpr int NAUX = G::RT * G::NP + 2, NFREE = G::FTW * (G::RT - 1);
  if constexpr (I < NAUX) {
    if constexpr (I % NFREE == FIDX) aux_op<S, SEG, KS, I>(c, a);
    aux_slot<S, SEG, KS, FIDX, I + 1>(c, a);
  }
}

// Product M = a * RT + b of k step KS and what follows it.  A wave issues in order and a matrix instruction keeps
// its unit busy for 32 cycles: the fetches and address arithmetic of a k step, issued in one block, leave the unit
// idle meanwhile (measured: ~100-170 of a k step's 256 / 512 cycles), one or two of them after every product do not.
// The next weight block of feature tile a follows the last product that reads the present one.
template <class S, int SEG, int KS, int M>
__device__ __forceinline__ void k_products(Ctx<S>& c, const ChainArgs& a, const WeightPos& wseg) {
  using G = Seg<S, SEG>;
  if constexpr (M < G::FTW * G::RT) {
    constexpr int ta = M / G::RT, tb = M % G::RT;
    const uint4* w = c.wq + ((KS % G::DEP) * G::FTW + ta) * G::NP;
    const uint4(&x)[G::NP] = c.xq[KS % kXRing<S>][tb];
    if constexpr (S::fp8)
      c.acc[ta][tb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(join8(w[0], w[1]), join8(x[0], x[1]), c.acc[ta][tb], 0, 0, 0, 0, 0, 0);
    else
      c.acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[0]), __builtin_bit_cast(bf16x8, x[0]),
                                                              c.acc[ta][tb], 0, 0, 0);
    if constexpr (tb == G::RT - 1) {
      if constexpr (KS + G::DEP < G::NKS)
#pragma unroll
        for (int p = 0; p < G::NP; ++p)
          c.wq[((KS % G::DEP) * G::FTW + ta) * G::NP + p] = weight_block<S, SEG, KS + G::DEP>(c, wseg, ta, p);
      if constexpr (G::RT == 1) {                                 // the head: one product per k step
        aux_op<S, SEG, KS, 0>(c, a);
        aux_op<S, SEG, KS, 1>(c, a);
        aux_op<S, SEG, KS, 2>(c, a);
        if constexpr (G::NP > 1) aux_op<S, SEG, KS, 3>(c, a);
      }
    } else {
      aux_slot<S, SEG, KS, ta * (G::RT - 1) + tb, 0>(c, a);
    }
    __builtin_amdgcn_sched_barrier(0);
    k_products<S, SEG, KS, M + 1>(c, a, wseg);
  }
}

template <class S, int SEG, int KS>
__device__ __forceinline__ void k_steps(Ctx<S>& c, const ChainArgs& a, const WeightPos& wseg) {
  using G = Seg<S, SEG>;
  if constexpr (KS < G::NKS) {
    if constexpr (G::bwd && KS == G::HK) {          // the first tiles' stored activations, late enough not to hold up
      fetch_h_first<S, SEG, 0>(c, a);               // the weight fetches behind them, early enough to be there
    }
    k_products<S, SEG, KS, 0>(c, a, wseg);
    k_steps<S, SEG, KS + 1>(c, a, wseg);
  }
}

template <class S, int SEG, int T>
__device__ __forceinline__ void write_tile(const Ctx<S>& c, const uint32_t (&w)[8]) {
  using G = Seg<S, SEG>;
  const int ft = tile_of<G>(c, T / G::RT), rt = first_rt<G>(c) + T % G::RT;
  if constexpr (S::fp8) {      // word q: features 8 q + 4 hh .. of the tile.  The halves of the wave trade words: the lower one gets
                               // quads 0 and 1 of both, the first block's 16 bytes of its row, the upper one quads 2 and 3
    const auto u = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
    const auto v = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
    c.X[(G::out_area + (ft / 2 * 2 + c.hh) * S::nrt + rt) * 64 + c.s + 32 * (ft & 1)] = make_uint4(u[0], u[1], v[0], v[1]);
  } else if constexpr (S::nat) {      // quad q: features 8 (q % 2) + 4 hh .. of k step 2 ft + q / 2
    char* x = reinterpret_cast<char*>(c.X + (G::out_area + (2 * ft) * S::nrt + rt) * 64 + c.s) + 8 * c.hh;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<uint2*>(x + (q / 2) * S::nrt * 1024 + (q % 2) * 512) = make_uint2(w[2 * q], w[2 * q + 1]);
  } else {
    uint4* x = c.X + (G::out_area + (2 * ft) * S::nrt + rt) * 64 + c.lane;
    x[0] = make_uint4(w[0], w[1], w[2], w[3]);
    x[S::nrt * 64] = make_uint4(w[4], w[5], w[6], w[7]);
  }
}
template <class S, int SEG, int T>
__device__ __forceinline__ void write_tiles(const Ctx<S>& c, const uint32_t (&w)[Seg<S, SEG>::FTW * Seg<S, SEG>::RT][8]) {
  if constexpr (T < Seg<S, SEG>::FTW * Seg<S, SEG>::RT) {
    write_tile<S, SEG, T>(c, w[T]);
    write_tiles<S, SEG, T + 1>(c, w);
  }
}

// Epilogue of tile T of a hidden forward layer or of an input-gradient layer: the results as they go into the activation area.
template <class S, int SEG, int T>
__device__ __forceinline__ void tile_results(Ctx<S>& c, const ChainArgs& a, uint32_t (&out)[Seg<S, SEG>::FTW * Seg<S, SEG>::RT][8]) {
  using G = Seg<S, SEG>;
  if constexpr (T < G::FTW * G::RT) {
    constexpr int ta = T / G::RT, tb = T % G::RT;
    const int ft = tile_of<G>(c, ta);
    fetch_h<S, SEG, T + kHPre>(c, a);
    const floatx16& acc = c.acc[ta][tb];
    uint32_t(&w)[8] = out[T];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v0 = acc[4 * q + 0], v1 = acc[4 * q + 1], v2 = acc[4 * q + 2], v3 = acc[4 * q + 3];
      if constexpr (G::bwd) {
        const uint4 hb = c.hq[T % (kHPre + 1)][q / 2];
        const uint32_t h01 = q % 2 == 0 ? hb.x : hb.z, h23 = q % 2 == 0 ? hb.y : hb.w;
        v0 *= elu_grad_f(bf16_lo(h01)); v1 *= elu_grad_f(bf16_hi(h01));
        v2 *= elu_grad_f(bf16_lo(h23)); v3 *= elu_grad_f(bf16_hi(h23));
      } else {
        if constexpr (S::fp8) {
          const float4 b4 = *reinterpret_cast<const float4*>(c.s_bias + S::bias_off(G::layer) + 32 * ft + 8 * q + 4 * c.hh);
          v0 = fmaf(v0, c.scale, b4.x); v1 = fmaf(v1, c.scale, b4.y); v2 = fmaf(v2, c.scale, b4.z); v3 = fmaf(v3, c.scale, b4.w);
        } else if constexpr (S::nat) {
          const float4 b4 = *reinterpret_cast<const float4*>(c.s_bias + S::bias_off(G::layer) + 32 * ft + 8 * q + 4 * c.hh);
          v0 += b4.x; v1 += b4.y; v2 += b4.z; v3 += b4.w;
        }                                                                    // else the bias is in the sums already
        if constexpr (!S::fp8) { v0 = elu_f(v0); v1 = elu_f(v1); v2 = elu_f(v2); v3 = elu_f(v3); }
      }
      if constexpr (S::fp8) {
        w[q] = elu_e4m3x4(v0, v1, v2, v3);
      } else {
        w[2 * q] = pack_bf16(v0, v1);
        w[2 * q + 1] = pack_bf16(v2, v3);
      }
    }
    if constexpr (!S::late_write) write_tile<S, SEG, T>(c, w);
    tile_results<S, SEG, T + 1>(c, a, out);
  }
}
template <class S, int SEG>
__device__ __forceinline__ void layer_epilogue(Ctx<S>& c, const ChainArgs& a) {
  using G = Seg<S, SEG>;
  uint32_t out[G::FTW * G::RT][8];
  if constexpr (!S::keep && !S::late_write) __syncthreads();                       // every wave is done with the layer's input
  tile_results<S, SEG, 0>(c, a, out);
  if constexpr (S::late_write) {
    __syncthreads();                       // every wave is done with the layer's input
    write_tiles<S, SEG, 0>(c, out);
  }
}

// This lane's loss inputs (sample row0 + 32 wave + s): unconditional loads, rows and features past the end read a
// valid neighbour, their results are dropped.
template <class S>
__device__ __forceinline__ void fetch_loss_inputs(Ctx<S>& c, const ChainArgs& a) {
  c.l_lo = a.b_logp[c.slot]; c.l_ad = a.b_adv[c.slot]; c.l_rt = a.b_ret[c.slot];
  c.l_back = actions_back(c.slot, a.act_dim);
  fetch_actions(a.b_act, c.slot, a.act_dim, c.hh, c.l_act);
}

// Sum over the wave, in lane 63.
__device__ __forceinline__ float sum_to_last(float v) {
  auto add = [&](auto ctrl) { v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true)); };
  add(std::integral_constant<int, 0x111>{});      // the lanes of a row of 16, one, two, four and eight up
  add(std::integral_constant<int, 0x112>{});
  add(std::integral_constant<int, 0x114>{});
  add(std::integral_constant<int, 0x118>{});
  add(std::integral_constant<int, 0x142>{});      // a row's last lane to the next row
  add(std::integral_constant<int, 0x143>{});      // lane 31 to the upper half
  return v;
}

// Loss on the wave's 32 samples (row tile `wave` of the workgroup) from the head's accumulators: lane = sample s,
// half hh; register i = feature 8 (i / 4) + 4 hh + i % 4.  Leaves the head gradient as the two k steps of the first
// input-gradient product in the activation area and, as the same blocks, in dz[NL - 1], and the workgroup's
// statistics row.
template <class S>
__device__ __forceinline__ void loss_epilogue(Ctx<S>& c, const ChainArgs& a, const floatx16& acc) {
  constexpr int HB = S::bias_off(S::NL - 1);
  const int A = a.act_dim;
  if (c.wave < S::nrt) {
  const int wrow0 = c.row0 + 32 * c.wave;
  const int row = wrow0 + c.s;
  const bool ok = row < a.rows;
  const float inv_m = 1.0f / (float)a.rows;
  float d[16];
  float* red = c.s_red + c.wave * 40;
  if (c.net == 0) {
    const float* s_ls = c.s_red + S::nrt * 40;      // [f] log_std, [32 + f] exp(-log_std) (0 for f >= A)
    float z[16], isg[16];
    float lp = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) d[i] = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (8 * q >= A) break;                         // no action among these eight features
      const int f0 = 8 * q + 4 * c.hh;
      const float4 ls4 = *reinterpret_cast<const float4*>(s_ls + f0);
      const float4 ig4 = *reinterpret_cast<const float4*>(s_ls + 32 + f0);
      const float4 b4 = *reinterpret_cast<const float4*>(c.s_bias + HB + f0);
      const float lsv[4] = {ls4.x, ls4.y, ls4.z, ls4.w}, igv[4] = {ig4.x, ig4.y, ig4.z, ig4.w};
      const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
      float av[4];
      lane_actions(c.l_act, A, c.l_back, q, c.hh, av);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 4 * q + e;
        const float mu = acc[i] + bv[e];
        isg[i] = igv[e];
        z[i] = f0 + e < A ? (av[e] - mu) * igv[e] : 0.f;      // there av may be what follows the sample (fetch_actions)
        lp += f0 + e < A ? -0.5f * z[i] * z[i] - lsv[e] - 0.918938533204672742f : 0.f;
      }
    }
    lp += __shfl_xor(lp, 32, 64);                   // the other half holds the other 16 features
    float s_pl = 0.f, s_kl = 0.f, s_cf = 0.f, g_lp = 0.f;
    if (ok) {
      const float lo = c.l_lo, ad = c.l_ad;
      const float ratio = expf(lp - lo);
      const float u1 = ratio * ad;
      const float u2 = fminf(fmaxf(ratio, 1.0f - a.clip), 1.0f + a.clip) * ad;
      g_lp = (u1 <= u2) ? -(ad * ratio) * inv_m : 0.f;
      if (c.hh == 0) {                               // each sample counts once
        s_pl = -fminf(u1, u2);
        s_kl = lo - lp;
        s_cf = fabsf(ratio - 1.0f) > a.clip ? 1.f : 0.f;
      }
    }
    // log_std gradient partials g_lp (z^2 - 1): transposed through the wave's buffer as [feature][sample] fp32,
    // then lane (f, half) sums 16 samples of feature f in a fixed order
    float* tp = reinterpret_cast<float*>(c.scr);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (8 * q >= A) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 4 * q + e, f = 8 * q + 4 * c.hh + e;
        d[i] = g_lp * z[i] * isg[i];
        tp[f * 33 + c.s] = g_lp * (z[i] * z[i] - 1.0f);
      }
    }
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += tp[c.s * 33 + 16 * c.hh + k];
    sum += __shfl_xor(sum, 32, 64);
    if (c.lane < A) red[8 + c.lane] = sum;
    s_pl = sum_to_last(s_pl); s_kl = sum_to_last(s_kl); s_cf = sum_to_last(s_cf);
    if (c.lane == 63) { red[0] = s_pl; red[1] = s_kl; red[2] = s_cf; }
  } else {
    float s_vl = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) d[i] = 0.f;
    if (ok && c.hh == 0) {
      const float dv = acc[0] + c.s_bias[HB] - c.l_rt;
      s_vl = dv * dv;
      d[0] = 2.0f * a.c_v * dv * inv_m;
    }
    s_vl = sum_to_last(s_vl);
    if (c.lane == 63) red[0] = s_vl;
  }
  uint32_t w[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) w[q] = pack_bf16(d[2 * q], d[2 * q + 1]);
  c.X[(S::area(S::NL) + c.wave) * 64 + c.lane] = make_uint4(w[0], w[1], w[2], w[3]);
  c.X[(S::area(S::NL) + S::nrt + c.wave) * 64 + c.lane] = make_uint4(w[4], w[5], w[6], w[7]);
  {
    uint4* arr = reinterpret_cast<uint4*>(a.dz[c.net][S::NL - 1]);
    store_block<S>(arr + block_word(c.tr, 2, 0, c.rt0 + c.wave), c.lane16, make_uint4(w[0], w[1], w[2], w[3]));      // arrays hold whole tiles
    store_block<S>(arr + block_word(c.tr, 2, 1, c.rt0 + c.wave), c.lane16, make_uint4(w[4], w[5], w[6], w[7]));
  }
  }
}

// The workgroup's sums -> its row of the statistics partials.
template <class S>
__device__ __forceinline__ void loss_sums(const Ctx<S>& c, const ChainArgs& a) {
  const int A = a.act_dim;
  float* out = a.stat_part + (int64_t)(c.row0 / S::rows) * (gmi::kStatStride + A);
  if (c.net == 0) {
    if (c.tid < 3) {
      float v = 0.f;
      for (int wv = 0; wv < S::nrt; ++wv) v += c.s_red[wv * 40 + c.tid];
      out[c.tid == 0 ? 0 : (c.tid == 1 ? 3 : 4)] = v;
    }
    if (c.tid == 3) {
      float ent = 0.f;
      if (c.row0 == 0)
        for (int j = 0; j < A; ++j) ent += c.s_red[S::nrt * 40 + j] + 1.418938533204672742f;
      out[2] = ent;
      out[5] = out[6] = out[7] = 0.f;
    }
    if (c.tid >= 64 && c.tid < 64 + A) {
      const int j = c.tid - 64;
      float v = 0.f;
      for (int wv = 0; wv < S::nrt; ++wv) v += c.s_red[wv * 40 + 8 + j];
      out[gmi::kStatStride + j] = v;
    }
  } else if (c.tid == 0) {
    float v = 0.f;
    for (int wv = 0; wv < S::nrt; ++wv) v += c.s_red[wv * 40];
    out[1] = v;
  }
}

// Inference: the head's results of row tile `wave` (lane = row, register i = feature 8 (i / 4) + 4 hh + i % 4) plus
// the head's bias go out as policy means [rows, act_dim] or as values [rows], and, where actions are asked for, the decision
// act = mean + exp(log_std) * eps and its log-density: the arithmetic of sample_kernel (model.hip), terms summed in
// its order.  The draws are made beside the head's product by the waves that have no part in it.  (Gather, this kernel and sampling as
// three launches, 16384 rows of 211:512:512:256:128:20: 49 us, now 38.)
template <class S>
__device__ __forceinline__ void head_draws(const Ctx<S>& c, const ChainArgs& a) {
  const int row = c.row0 + 32 * (c.wave & (S::nrt - 1)) + c.s;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (8 * q >= a.act_dim) break;
    float z[4];
    gmi::normal_block(a.env_offset + (uint32_t)row, a.step, gmi::kStreamAction, (uint32_t)(2 * q + c.hh), a.k0, a.k1, z);
    reinterpret_cast<float4*>(c.scr)[q * 64 + c.lane] = make_float4(z[0], z[1], z[2], z[3]);
  }
}
template <class S>
__device__ __forceinline__ void head_outputs(Ctx<S>& c, const ChainArgs& a, const floatx16& acc) {
  constexpr int HB = S::bias_off(S::NL - 1);
  if (c.wave >= S::nrt) return;
  const int row = c.row0 + 32 * c.wave + c.s, A = a.act_dim;
  const bool ok = row < a.rows;
  if (c.net == 1) {
    if (ok && c.hh == 0) c.val_out[row] = S::fp8 ? fmaf(acc[0], c.scale, c.s_bias[HB]) : acc[0] + c.s_bias[HB];
    return;
  }
  typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
  auto store = [&](float* out, int f0, const float (&v)[4]) {
    float* p = out + (int64_t)row * A + f0;
    if (f0 + 4 <= A) {
      const float4u t = {v[0], v[1], v[2], v[3]};
      *reinterpret_cast<float4u*>(p) = t;
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (f0 + e < A) p[e] = v[e];
    }
  };
  const float* s_ls = c.s_red + S::nrt * 40;      // [f] log_std, [32 + f] exp(log_std)
  float lp = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (8 * q >= A) break;
    const int f0 = 8 * q + 4 * c.hh;
    float m[4], act[4], term[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float b = c.s_bias[HB + f0 + e];
      m[e] = S::fp8 ? fmaf(acc[4 * q + e], c.scale, b) : acc[4 * q + e] + b;
    }
    if (a.mu_out && ok) store(a.mu_out, f0, m);
    if (!a.act_out) continue;
    const float4 z4 = reinterpret_cast<const float4*>(c.scr)[q * 64 + c.lane];
    const float z[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float ls = s_ls[f0 + e];
      act[e] = fmaf(s_ls[32 + f0 + e], z[e], m[e]);
      term[e] = -0.5f * z[e] * z[e] - ls - 0.918938533204672742f;
    }
    if (ok) store(a.act_out, f0, act);
    float up[4];                                                             // the upper half's; the lower one's sum goes out
#pragma unroll
    for (int e = 0; e < 4; ++e) up[e] = __shfl_xor(term[e], 32, 64);
    if constexpr (S::lp_blocks) {
      lp += ((term[0] + (8 * q + 1 < A ? term[1] : 0.f)) + (8 * q + 2 < A ? term[2] : 0.f)) + (8 * q + 3 < A ? term[3] : 0.f);
      if (8 * q + 4 < A)
        lp += ((up[0] + (8 * q + 5 < A ? up[1] : 0.f)) + (8 * q + 6 < A ? up[2] : 0.f)) + (8 * q + 7 < A ? up[3] : 0.f);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) lp = 8 * q + e < A ? lp + term[e] : lp;
#pragma unroll
      for (int e = 0; e < 4; ++e) lp = 8 * q + 4 + e < A ? lp + up[e] : lp;
    }
  }
  if (a.act_out && ok && c.hh == 0) a.logp_out[row] = lp;
}

template <class S, int SEG>
__device__ __forceinline__ void run_segment(Ctx<S>& c, const ChainArgs& a) {
  if constexpr (SEG < n_run<S>()) {
    using G = Seg<S, SEG>;
    const WeightPos wseg = seg_weights<S, SEG>(c, a);
    if constexpr (S::fp8) c.scale = a.scale[c.net * S::NL + G::layer];
    if constexpr (!G::bwd && !G::head && !S::nat) {
      // the accumulators start at the bias (register i of a lane = feature 8 (i / 4) + 4 hh + i % 4 of the tile)
      constexpr int boff = S::bias_off(G::layer);
#pragma unroll
      for (int ta = 0; ta < G::FTW; ++ta) {
        const float* bp = c.s_bias + boff + 32 * tile_of<G>(c, ta) + 4 * c.hh;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 b4 = *reinterpret_cast<const float4*>(bp + 8 * q);
#pragma unroll
          for (int tb = 0; tb < G::RT; ++tb) {
            c.acc[ta][tb][4 * q + 0] = b4.x; c.acc[ta][tb][4 * q + 1] = b4.y;
            c.acc[ta][tb][4 * q + 2] = b4.z; c.acc[ta][tb][4 * q + 3] = b4.w;
          }
        }
      }
    } else {
#pragma unroll
      for (int ta = 0; ta < G::FTW; ++ta)
#pragma unroll
        for (int tb = 0; tb < G::RT; ++tb)
#pragma unroll
          for (int v = 0; v < 16; ++v) c.acc[ta][tb][v] = 0.f;
    }
    read_x<S, SEG, 0>(c);
    if constexpr (G::XD > 1) read_x<S, SEG, 1>(c);
    if constexpr (G::head && S::fwd) {
      if (c.wave < S::nrt) k_steps<S, SEG, 0>(c, a, wseg);
      else if (c.net == 0 && a.act_out) head_draws<S>(c, a);
    } else {
      k_steps<S, SEG, 0>(c, a, wseg);
    }
    issue_first_weights<S, SEG + 1>(c, a);
    prefetch_weights<S, SEG + 1>(c);
    if constexpr ((!S::keep || S::fwd) && G::head) __syncthreads();      // every wave is done with the layer's input, or has made its draws
    // this lane's loss inputs: cold loads, issued where a long stretch of arithmetic follows and no younger load is
    // waited for (the memory counter is in order)
    if constexpr (!S::fwd && SEG == (S::NL >= 3 ? S::NL - 3 : 0)) fetch_loss_inputs<S>(c, a);
    if constexpr (G::head && S::fwd) {
      head_outputs<S>(c, a, c.acc[0][0]);
    } else if constexpr (G::head) {
      loss_epilogue<S>(c, a, c.acc[0][0]);
    } else {
      layer_epilogue<S, SEG>(c, a);
    }
    __syncthreads();
    if constexpr (G::head && !S::fwd) loss_sums<S>(c, a);
    if constexpr (G::last) {
      // nothing consumes the last results on chip: the activation area goes to dz[layer - 1] block by block, the way a k
      // loop moves its input
      uint4* arr = reinterpret_cast<uint4*>(a.dz[c.net][G::layer - 1]) +
                   block_word(c.tr, G::F / 16, c.wave / S::nrt, c.rt0 + c.wave % S::nrt);
#pragma unroll 8
      for (int k2 = 0; k2 < G::F / 16; k2 += 2) {
        store_block<S>(arr, c.lane16, c.X[(G::out_area + k2 * S::nrt + c.wave) * 64 + c.lane], k2 * 4096);      // arrays hold whole tiles
      }
    }
    run_segment<S, SEG + 1>(c, a);
  }
}

// Floats f0 .. f0 + 3 of a row of O (>= 4) floats at any 4-byte address, zero beyond it; `ragged`: whether f0 + 3 may lie beyond.
__device__ __forceinline__ void row_quad(const float* row, int f0, int O, bool ragged, float (&f)[4]) {
  typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
  const int back = ragged ? f0 - (f0 < O - 4 ? f0 : O - 4) : 0;
  const float4u t = *reinterpret_cast<const float4u*>(row + f0 - back);
  f[0] = back == 0 ? t.x : back == 1 ? t.y : back == 2 ? t.z : back == 3 ? t.w : 0.f;
  f[1] = back == 0 ? t.y : back == 1 ? t.z : back == 2 ? t.w : 0.f;
  f[2] = back == 0 ? t.z : back == 1 ? t.w : 0.f;
  f[3] = back == 0 ? t.w : 0.f;
}

template <class S>
__device__ __forceinline__ void row_tile(const ChainArgs& a, int item, unsigned char* smem_raw) {
  static_assert(S::valid(), "shape not supported by the row-tile trainer kernel");
  constexpr ChainDims D = S::dims();
  Ctx<S> c;
  c.tid = threadIdx.x;
  c.lane = c.tid & 63;
  c.wave = __builtin_amdgcn_readfirstlane(c.tid >> 6);
  c.s = c.lane & 31;
  c.hh = c.lane >> 5;
  c.net = S::fwd ? (int)blockIdx.y + a.net0 : (S::late_write ? (int)blockIdx.x >> 2 & 1 : (int)blockIdx.y);
  if constexpr (S::fwd) {
    const int t = item / a.slot_tiles;
    c.row0 = (item - t * a.slot_tiles) * S::rows;
    c.obs = t < a.T ? a.b_obs + t * a.obs_step : a.obs_last;
    c.val_out = t < a.T ? a.val_out + t * a.val_step : a.val_last;
  } else {
    c.row0 = item * S::rows;
  }
  c.tr = c.row0 / 128;
  c.rt0 = c.row0 / 32 & 3;
  c.X = reinterpret_cast<uint4*>(smem_raw);
  c.lane16 = c.lane * 16;
  c.xo[0] = c.lane16;
  c.xo[1] = c.lane16 + 65536;
  asm volatile("" : "+v"(c.xo[1]));
  float* s_bias = reinterpret_cast<float*>(smem_raw + S::x_bytes());
  c.s_bias = s_bias;
  c.s_red = s_bias + S::bias_total();
  c.scr = reinterpret_cast<char*>(smem_raw) + S::scr_offset() + (c.wave & (S::nrt - 1)) * kScrBytes;
  c.wnet = reinterpret_cast<const uint4*>(a.wstream[c.net]);

  // Everything a workgroup starts from is requested before anything is waited for, in the order in which it is needed: the memory
  // counter is in order.  (Indices, biases and scales loaded and stored one after another behind the first weights: 17 thousand
  // cycles up to the first product, of 170.)
  constexpr int NG = S::rows / 16 / S::waves;
  const int rr = c.lane & 15, jj = c.lane >> 4;
  int sm[NG], srow[NG], hrow = 0, hsm = 0;
  const void* ixp = a.idx ? (const void*)a.idx : (const void*)a.log_std;      // no index: rows in order
  const auto ix = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ixp), 0, 0xFFFFFFFFu, 0x00020000);
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    const int row = c.row0 + 16 * (c.wave + S::waves * gi) + rr;
    srow[gi] = row < a.rows ? row : a.rows - 1;
    if constexpr (!S::fwd) sm[gi] = __builtin_amdgcn_raw_buffer_load_b32(ix, a.idx ? srow[gi] * 4 : 0, 0, 0);
  }
  if constexpr (!S::fwd) {
    // this lane's sample of the head layer (rows past the batch take the last sample, the waves without a part in the loss one
    // sample for all lanes; their results are dropped)
    const int row = c.row0 + (c.wave < S::nrt ? 32 * c.wave + c.s : 0);
    hrow = row < a.rows ? row : a.rows - 1;
    hsm = __builtin_amdgcn_raw_buffer_load_b32(ix, a.idx ? hrow * 4 : 0, 0, 0);
  }
  float bv[S::NL][(S::maxks() * 16 + S::waves * 64 - 1) / (S::waves * 64)];
#pragma unroll
  for (int l = 0; l < S::NL; ++l)
#pragma unroll
    for (int i = 0; i * S::waves * 64 < D.d[l + 1]; ++i) {
      const int f = c.tid + i * S::waves * 64;
      bv[l][i] = a.bias[c.net][l][f < D.d[l + 1] ? f : D.d[l + 1] - 1];
    }
  const float ls = a.log_std[c.tid < a.act_dim ? c.tid : a.act_dim - 1];
  {
    // The gather: the workgroup's observation rows as the first layer's operand blocks in natural k order (lane
    // (s, h) of block (ks, rt) holds features 16 ks + 8 h .. + 7 of sample 32 rt + s), zero padded.  A lane takes
    // 16-byte piece jj + 4 it of row 16 g + rr: 16 lanes write 256 consecutive bytes of LDS, 4 lanes read 64
    // consecutive bytes of a row.  The policy net's workgroups also leave the same blocks in x0b for the
    // weight-gradient kernel.  All loads unconditional (clamped addresses, selected values).
    constexpr int NP = D.d[0] / (S::fp8 ? 16 : 8);       // 16-byte pieces of a row
    const int O = a.obs_dim;
    constexpr int NI = (NP + 3) / 4;
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) sm[gi] = !S::fwd && a.idx ? sm[gi] : srow[gi];
    uint4 v[NG][NI];
    if constexpr (S::fp8) {
#pragma unroll
      for (int it = 0; it < NI; ++it) {
        uint32_t e[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float f[4];
          row_quad(c.obs + (int64_t)sm[0] * O, 16 * (4 * it + jj) + 4 * q, O, it == NI - 1, f);
          e[q] = to_e4m3x4(f[0], f[1], f[2], f[3]);
        }
        v[0][it] = make_uint4(e[0], e[1], e[2], e[3]);
      }
    } else if (S::fwd && a.x0_ready == 3) {                     // workgroup-uniform; no branch around a single load
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        const float* orow = c.obs + (int64_t)sm[gi] * O;
#pragma unroll
        for (int it = 0; it < NI; ++it) {
          const int j = 4 * it + jj;
          float f[8];
#pragma unroll
          for (int q = 0; q < 2; ++q) row_quad(orow, 8 * j + 4 * q, O, it == NI - 1, reinterpret_cast<float(&)[4]>(f[4 * q]));
          v[gi][it] = make_uint4(pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7]));
        }
      }
    } else if (a.x0_ready != 0) {
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        const int row = c.row0 + 16 * (c.wave + S::waves * gi) + rr;
        const uint16_t* src = a.x0_ready == 1 ? a.x0 + (int64_t)row * D.d[0] : a.x16 + (int64_t)sm[gi] * D.d[0];
#pragma unroll
        for (int it = 0; it < NI; ++it) {
          const int j = 4 * it + jj;
          v[gi][it] = *reinterpret_cast<const uint4*>(src + 8 * (j < NP ? j : NP - 1));
        }
      }
    } else {
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        const float* orow;
        if constexpr (S::fwd) orow = c.obs + (int64_t)sm[gi] * O;
        else orow = a.b_obs + ((int64_t)(sm[gi] / a.n_envs) * a.ld_envs + (sm[gi] % a.n_envs)) * O;
#pragma unroll
        for (int it = 0; it < NI; ++it) {
          const int j = 4 * it + jj;
          const int jc = j < NP ? j : NP - 1;
          float f[8];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int f0 = 8 * jc + 4 * q;                  // O % 4 == 0: a piece is inside the row or past it
            const float4 t = *reinterpret_cast<const float4*>(orow + (f0 < O ? f0 : O - 4));
            f[4 * q + 0] = f0 < O ? t.x : 0.f; f[4 * q + 1] = f0 < O ? t.y : 0.f;
            f[4 * q + 2] = f0 < O ? t.z : 0.f; f[4 * q + 3] = f0 < O ? t.w : 0.f;
          }
          v[gi][it] = make_uint4(pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7]));
        }
      }
    }
    issue_first_weights<S, 0>(c, a);
    c.touched = 0;
    prefetch_weights<S, 0>(c);
    {
      int off = 0;
#pragma unroll
      for (int l = 0; l < S::NL; ++l) {
#pragma unroll
        for (int i = 0; i * S::waves * 64 < D.d[l + 1]; ++i) {
          const int f = c.tid + i * S::waves * 64;
          if (f < D.d[l + 1]) s_bias[off + f] = bv[l][i];
        }
        off += D.d[l + 1];
      }
      if (c.tid < S::nrt * 40) c.s_red[c.tid] = 0.f;
      if (c.tid < 32) {                      // per-feature constants of the Gaussian log-prob (policy net)
        c.s_red[S::nrt * 40 + c.tid] = ls;
        c.s_red[S::nrt * 40 + 32 + c.tid] = c.tid < a.act_dim ? expf(S::fwd ? ls : -ls) : 0.f;
      }
      if constexpr (!S::fwd) {
        hsm = a.idx ? hsm : hrow;
        c.slot = (int64_t)(hsm / a.n_envs) * a.ld_envs + (hsm % a.n_envs);
      }
    }
    uint4* xb = reinterpret_cast<uint4*>(a.x0b) + block_word(c.tr, D.d[0] / 16, 0, c.rt0);
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      const int r = 16 * (c.wave + S::waves * gi) + rr;
#pragma unroll
      for (int it = 0; it < NI; ++it) {
        const int j = 4 * it + jj;
        if constexpr (S::fp8) {      // piece j: k step j / 4, half j / 2 % 2 of the lanes, block j % 2
          if (j < NP) c.X[(((j >> 2) * 2 + (j & 1)) * S::nrt + (r >> 5)) * 64 + (r & 31) + 32 * ((j >> 1) & 1)] = v[gi][it];
        } else if (j < NP) {
          const int w = (r >> 5) * 64 + (r & 31) + 32 * (j & 1);
          c.X[(j >> 1) * S::nrt * 64 + w] = v[gi][it];
          if (!S::fwd && c.net == 0) xb[(j >> 1) * 256 + w] = v[gi][it];      // arrays hold whole tiles
        }
      }
    }
  }
  __syncthreads();
  if constexpr (S::late_write) { if (c.wave < 4) __builtin_amdgcn_s_setprio(1); }
  run_segment<S, 0>(c, a);
}

template <class S>
__global__ __launch_bounds__(S::threads, 2) void train_tile_kernel(ChainArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  if constexpr (!S::late_write) {
    row_tile<S>(a, blockIdx.x, smem_raw);
  } else {
    // half of the dies (ids go round-robin over 8) take the policy net, the others the value net: a die's second-level cache holds the
    // weights of one net over both rounds of workgroups (32768 rows of 211:512:512:256:128:20 175 us, 170 so; the narrower shapes, whose
    // nets both fit, 84 and 87)
    const int item = (int)(blockIdx.x >> 3) * 4 + (blockIdx.x & 3);
    if (item < a.items) row_tile<S>(a, item, smem_raw);
  }
}
// Items one after the other: a launch that its compute units cannot hold keeps kernels of other streams waiting.  The arguments are
// read again for every item: kept over the loop, they and what follows from them spilled 170 scalar registers.
template <class S>
__global__ __launch_bounds__(S::threads, 2) void tile_items_kernel(ChainArgs) {
  typedef const __attribute__((address_space(4))) ChainArgs KernelArgs;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  KernelArgs* p = (KernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const int items = p->items;
  for (int item = blockIdx.x; item < items; item += gridDim.x) {
    asm volatile("" : "+s"(p));
    row_tile<S>(*(const ChainArgs*)p, item, smem_raw);
    __syncthreads();
  }
}

template <class S>
bool shape_matches(const ModelLayout& L) {
  constexpr ChainDims D = S::dims();
  if (L.n_layers != D.nl) return false;
  auto pad = [](int x) { return S::fp8 ? (x + 63) & ~63 : x; };
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < D.nl; ++l)
      if (pad(L.net[net][l].in_pad) != D.d[l] || (l == D.nl - 1 ? L.net[net][l].out_pad : pad(L.net[net][l].out_pad)) != D.d[l + 1])
        return false;
  return true;
}

// The widest shapes: 128 samples per workgroup, which read the weights half as often, where the last round of such workgroups (one per
// compute unit) is at least five eighths full (the only one: three quarters), or where on most of the card two full rounds come before
// it; else 64, of which two share a compute unit.  A minibatch with its weight gradients and update, us, 64 / 128 rows, of 211:512:512:256:128:20: 8192 rows 96 /
// 106, 9216 122 / 126, 10240 120 / 115 and 127 / 130 (two boxes), 12288 127 / 125, 16384 155 / 147, 18432 201 / 225, 20000 199 / 207, 22528 231 / 242, 24576 224 / 225, 26624 267 /
// 257, 28000 262 / 251, 32768 298 / 274, 34816 364 / 347, 40960 363 / 350, 49152 428 / 401, 65536 564 / 522; on 192 compute units
// 18432 210 / 226, 20480 241 / 237, 27648 323 / 317, 30720 342 / 330; on 128 4096 95 / 110, 5120 117 / 114, 12288 175 / 195, 13312 201 / 198,
// 18432 263 / 275, 20480 277 / 282, 32768 398 / 371; on 64 2048 122 / 137, 2560 145 / 143, 4096 153 / 151, 6144 193 / 211, 6656 219 / 214,
// 8192 229 / 224, 10240 270 / 285, 16384 395 / 379.  Of 211:512:512:512:256:20: 8192 128 / 138, 10240 161 / 150 and 169 / 167, 16384 221 / 193, 18432 270 / 289,
// 20000 277 / 266 (at this size and at 10240 the rule takes the side that is 4 and 1 to 7 % slower), 24576 311 / 302, 26624 361 / 322,
// 34816 466 / 444, 65536 757 / 662; on 64 6144 256 / 273, 6656 290 / 274, 10240 365 / 376.
inline bool wide_rows(int rows, int cus) {
  const int n = 2 * ((rows + 127) / 128), last = (n - 1) % cus + 1;      // workgroups, of the last round
  return n <= cus ? 4 * last >= 3 * cus : 8 * last >= 5 * cus || (n > 2 * cus && cus >= 192);
}

template <class S>
int launch_shape(gmi_instance* g, ChainArgs a, int rows, int* tiles_out, double flops, double bytes) {
  static gmi::DeviceSet allowed;
  const size_t lds = S::lds_bytes();
  int tiles = (rows + S::rows - 1) / S::rows;
  *tiles_out = tiles;
  if (!S::fwd && tiles > gmi::kStatRowsMax) return GMI_ERR_UNSUPPORTED;      // one statistics row per tile
  if (a.x0_ready == 3 && (!S::fwd || a.obs_dim < 4 || a.obs_dim <= S::dims().d[0] - (S::fp8 ? 64 : 32))) return GMI_ERR_UNSUPPORTED;
  if (a.x0_ready == 0 && (a.obs_dim % 4 != 0 || a.obs_dim < 4)) return GMI_ERR_UNSUPPORTED;
  int rc = gmi::allow_lds((const void*)train_tile_kernel<S>, lds, g->device, &allowed);
  if (rc != GMI_OK) return rc;
  gmi::ProfScope ps(g, S::fwd ? gmi::kClsFusedAgent : gmi::kClsChainTrain);
  ps.work(flops, bytes + (S::fwd || S::keep ? 0.0 : a.reread));
  if constexpr (S::fwd) {
    a.slot_tiles = tiles;
    a.items = tiles * (a.T + (a.val_last ? 1 : 0));
    tiles = a.items;
  } else {
    a.items = tiles;
  }
  if constexpr (S::nat && !S::fp8) {
    if (a.T > 1 || a.val_last) {
      static gmi::DeviceSet allowed_items;
      rc = gmi::allow_lds((const void*)tile_items_kernel<S>, lds, g->device, &allowed_items);
      if (rc != GMI_OK) return rc;
      int64_t resident = 1;
      rc = gmi::resident_groups(g, (const void*)tile_items_kernel<S>, S::threads, lds, &resident);
      if (rc != GMI_OK) return rc;
      const int64_t rounds = (a.items + resident - 1) / resident;
      ps.launch(tile_items_kernel<S>, dim3((unsigned)((a.items + rounds - 1) / rounds)), dim3(S::threads), lds, a);
      GMI_LAUNCH_CHECK();
      return GMI_OK;
    }
  }
  ps.launch(train_tile_kernel<S>, S::late_write ? dim3((tiles + 3) / 4 * 8) : dim3(tiles, S::fwd ? 2 - a.net0 : 2), dim3(S::threads), lds, a);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

}  // namespace gmi_tile

namespace gmi {
// One function per shape compiled for the row-tile kernel (trainers tile_p<k>.hip, forward-only kernels tile_f<k>.hip, fp8
// tile_q<k>.hip): launches it if the model has exactly that shape, GMI_ERR_UNSUPPORTED otherwise; rows == 0 only asks (a
// forward-only kernel's answer: 1 if it computes as the agent kernel does).
constexpr int kTileParts = 6;
constexpr int kTileFwdParts = 6, kTileFp8Parts = 5;
#define GMI_TILE_PART_DECL(k)                                                                              \
  int launch_tile_part##k(gmi_instance* g, const ModelLayout& L, const gmi_chain::ChainArgs& a, int rows, \
                          int* tiles_out, double flops, double bytes)
GMI_TILE_PART_DECL(0); GMI_TILE_PART_DECL(1); GMI_TILE_PART_DECL(2); GMI_TILE_PART_DECL(3); GMI_TILE_PART_DECL(4); GMI_TILE_PART_DECL(5);
#define GMI_TILE_FWD_PART_DECL(k)                                                                              \
  int launch_tile_fwd_part##k(gmi_instance* g, const ModelLayout& L, const gmi_chain::ChainArgs& a, int rows, \
                              int* tiles_out, double flops, double bytes)
GMI_TILE_FWD_PART_DECL(0); GMI_TILE_FWD_PART_DECL(1); GMI_TILE_FWD_PART_DECL(2); GMI_TILE_FWD_PART_DECL(3);
GMI_TILE_FWD_PART_DECL(4); GMI_TILE_FWD_PART_DECL(5);
#define GMI_TILE_FP8_PART_DECL(k) \
  int launch_tile_fp8_part##k(gmi_instance* g, const ModelLayout& L, const gmi_chain::ChainArgs& a, int rows)
GMI_TILE_FP8_PART_DECL(0); GMI_TILE_FP8_PART_DECL(1); GMI_TILE_FP8_PART_DECL(2); GMI_TILE_FP8_PART_DECL(3); GMI_TILE_FP8_PART_DECL(4);
#define GMI_TILE_FP8_PART_DEFINE(k, ...)                                                          \
  GMI_TILE_FP8_PART_DECL(k) {                                                                     \
    using S = gmi_tile::TileShapeFp8<64, __VA_ARGS__>;                                            \
    if (!gmi_tile::shape_matches<S>(L)) return GMI_ERR_UNSUPPORTED;                               \
    int tiles = 0;                                                                                \
    if (rows == 0) return GMI_OK;                                                                 \
    if (gmi_tile::turns(a, rows, g->cu_count))                                                    \
      return gmi_tile::launch_shape<gmi_tile::Turns<S>>(g, a, rows, &tiles, 0.0, 0.0);            \
    return gmi_tile::launch_shape<S>(g, a, rows, &tiles, 0.0, 0.0);                               \
  }
#define GMI_TILE_FWD_PART_DEFINE(k, SHAPE, ...)                                                   \
  GMI_TILE_FWD_PART_DECL(k) {                                                                     \
    using S = gmi_tile::SHAPE<64, __VA_ARGS__>;                                                   \
    if (!gmi_tile::shape_matches<S>(L)) return GMI_ERR_UNSUPPORTED;                               \
    *tiles_out = S::nat ? 1 : 0;                                                                  \
    if (rows == 0) return GMI_OK;                                                                 \
    if (gmi_tile::turns(a, rows, g->cu_count))                                                    \
      return gmi_tile::launch_shape<gmi_tile::Turns<S>>(g, a, rows, tiles_out, flops, bytes);     \
    return gmi_tile::launch_shape<S>(g, a, rows, tiles_out, flops, bytes);                        \
  }
#define GMI_TILE_PART_DEFINE(k, ...)                                                              \
  GMI_TILE_PART_DECL(k) {                                                                         \
    using K = gmi_tile::TileShapeKeep<64, __VA_ARGS__>;                                           \
    using S = std::conditional_t<K::lds_bytes() <= gmi_tile::kKeepBytes, K, gmi_tile::TileShape<64, __VA_ARGS__>>; \
    if (!gmi_tile::shape_matches<S>(L)) return GMI_ERR_UNSUPPORTED;                               \
    if (rows == 0) return GMI_OK;                                                                 \
    if (a.stream) return gmi_tile::launch_shape<gmi_tile::TileShapeStream<S>>(g, a, rows, tiles_out, flops, bytes); \
    return gmi_tile::launch_shape<S>(g, a, rows, tiles_out, flops, bytes);                        \
  }
#define GMI_TILE_WIDE_PART_DEFINE(k, ...)                                                         \
  GMI_TILE_PART_DECL(k) {                                                                         \
    using S = gmi_tile::TileShape<64, __VA_ARGS__>;                                               \
    using W = gmi_tile::TileShape<128, __VA_ARGS__>;                                              \
    if (!gmi_tile::shape_matches<S>(L)) return GMI_ERR_UNSUPPORTED;                               \
    if (rows == 0) return GMI_OK;                                                                 \
    if (gmi_tile::wide_rows(rows, g->cu_count))                                                   \
      return gmi_tile::launch_shape<W>(g, a, rows, tiles_out, flops, bytes);                      \
    return gmi_tile::launch_shape<S>(g, a, rows, tiles_out, flops, bytes);                        \
  }
}  // namespace gmi
