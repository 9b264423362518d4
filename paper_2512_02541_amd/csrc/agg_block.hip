// The parts of a global-attention block around the attention itself (AVGGT Sec. 4.2: a
// block is converted or subsampled with all its other components unchanged):
// LayerNorm, the Q/K/V projections, the output projection with bias and residual.
// They are a few percent of a block's time next to attention over 10^5..10^6 tokens and
// follow the MFMA conventions of the attention kernel.
#include "agg_internal.h"
#include "agg_lds_copy.h"
#include "agg_linear_plan.h"

namespace agg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

namespace {

union Frag {
  u32x4 u;
  bf16x8 h;
};

__device__ inline uint32_t pack2(float lo, float hi) {
  f32x2 p = {lo, hi};
  bf16x2 h = __builtin_convertvector(p, bf16x2);
  return __builtin_bit_cast(uint32_t, h);
}
__device__ inline float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float hi16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

}  // namespace

// ---------------------------------------------------------------------------
// LayerNorm over the channel dimension: one wavefront per token row, fp32 statistics
// (mean, then variance of the centred values), bf16 in and out.  C must be a multiple
// of 8; a lane owns 16-byte chunks lane, lane+64, ...
// ---------------------------------------------------------------------------
constexpr int kLnThreads = 256;
constexpr int kLnMaxChunks = 8;  // per lane: supports C <= 64*8*8 = 4096

// kChunks = 16-byte chunks per lane (4 up to 2048 channels, else 8): the row lives in registers,
// and the narrower instance keeps enough wavefronts resident to run at the memory rate
template <int kChunks>
__global__ __launch_bounds__(kLnThreads) void layernorm_kernel(const uint16_t* __restrict__ x,
                                                               const float* __restrict__ gamma,
                                                               const float* __restrict__ beta,
                                                               uint16_t* __restrict__ y, int64_t rows,
                                                               int C, float eps) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (kLnThreads / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int nchunk = C / 8;
  const uint16_t* xr = x + row * C;
  float v[kChunks][8];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int ch = lane + 64 * c;
    if (ch < nchunk) {
      u32x4 raw = *reinterpret_cast<const u32x4*>(xr + ch * 8);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[c][2 * i] = lo16(raw[i]);
        v[c][2 * i + 1] = hi16(raw[i]);
        sum += v[c][2 * i] + v[c][2 * i + 1];
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
  const float mean = sum / (float)C;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int ch = lane + 64 * c;
    if (ch < nchunk) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float d = v[c][i] - mean;
        sq += d * d;
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off);
  const float rstd = rsqrtf(sq / (float)C + eps);
  uint16_t* yr = y + row * C;
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int ch = lane + 64 * c;
    if (ch < nchunk) {
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        o[i] = (v[c][i] - mean) * rstd * gamma[ch * 8 + i] + beta[ch * 8 + i];
      u32x4 w = {pack2(o[0], o[1]), pack2(o[2], o[3]), pack2(o[4], o[5]), pack2(o[6], o[7])};
      *reinterpret_cast<u32x4*>(yr + ch * 8) = w;
    }
  }
}

// ---------------------------------------------------------------------------
// Linear layer  Y[m, n] = sum_k A[m, k] W[n, k] + bias[n] (+ R[m, n]),  bf16 in/out,
// fp32 accumulation on v_mfma_f32_16x16x32_bf16.  A: [rows, K] row-major; W: [N, K]
// row-major (one row per output channel), so both operands are contiguous along k.
// Requires K % 64 == 0 and N % 64 == 0.
//
// One workgroup (8 wavefronts) walks a list of 256 x 256 tiles, alone on its CU, or of 128 x 128
// tiles, two to a CU (launch_linear chooses); in a large tile a wavefront owns 64 tokens x 128
// channels, so that twelve fragment reads feed 32 MFMAs.
// k advances 64 at a time: whole 128-byte lines are fetched (with 32 the copies took twice the
// requests and bounded the kernel: 970 us without a single LDS read).  The operands go global ->
// LDS without passing through registers, into five slots used in turn by A(0) W(0) A(1) W(1) ...:
// a step works on two of them while the next W and the next two A are on their way, which is as
// deep as 160 KiB allows; the tokens, which come from HBM, get the longer lead.  The list goes on over tile
// borders: the next tile's operands are under way during a tile's last steps, and its stores drain
// under the next tile's first.
// LDS rows are 128 bytes with the 16-byte chunk number XOR-ed by bits 1..3 of the row, which
// spreads the 16 rows of a fragment read over all 64 banks.
// W's rows are copied into LDS in an order that leaves a lane with eight consecutive channels of
// a token: bias and residual are added in float before the one rounding, and a store instruction
// writes four 256-byte runs.
//
// One launch serves up to three weight matrices applied to the same input (the Q, K and V
// projections): their output tiles of one token tile are neighbours in an XCD's list, so that a
// token tile is fetched from HBM once and then served by that XCD's L2 to all of them.
//
// Measured at 137 400 rows, C = 1024 (us for Q/K/V and for the output projection): 1060 + 420
// before (256 x 256 tiles through registers, one workgroup per tile); 1040 + 400 with 256 x 128
// tiles, two to a CU, 32-wide k; 855 + 360 persistent with two 64 KiB stages; 817 + 325 as it is
// (1.06 PFLOP/s); on other boxes 797 + 324 and 840 + 328, on the last of which the library's products
// without residual take 786 + 272.  Without its copies it takes 610, without copies and stores 552, the products
// alone 480; spreading a step's copies over its products, grouping token tiles, touching lines
// ahead of the copies and streaming stores made it no faster or slower.
// ---------------------------------------------------------------------------
constexpr int kGemmThreads = 512;
constexpr int kTK = 64;
constexpr int kSlots = 5;

// kEdge: 256 or 128, the tile's tokens and channels
template <int kEdge, bool kResidual>
__global__ __launch_bounds__(kGemmThreads, kEdge == 256 ? 2 : 4) void linear_kernel(
    const uint16_t* __restrict__ A, LinearOuts outs, const uint16_t* __restrict__ R, int64_t rows,
    int N, int K, int gm, int gn) {
  constexpr int kMT = kEdge / 64;              // 16-token tiles of a wavefront; also copies per slot of A
  constexpr int kNT = kEdge / 32;              // its 16-channel tiles
  constexpr int kSlotBytes = kEdge * kTK * 2;  // one step's rows of A or of W
  constexpr int kCopies = kEdge / 64;          // copies of a wavefront per slot
  constexpr int kRows = kEdge / 8;             // LDS rows of a slot that a wavefront copies
  constexpr int kTileStores = 4 * kMT;         // store instructions of a wavefront per tile
  __shared__ __align__(16) char sm[kSlots * kSlotBytes];
  const int xcd = blockIdx.x % kGemmXcds;
  const int per_m = gn * outs.count;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15;
  const int G = lane >> 4;
  const int wm = (wave & 3) * (16 * kMT);  // this wavefront's tokens inside the tile
  const int wn = (wave >> 2) * (16 * kNT); // and its output channels
  const int nk = K / kTK;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)sm;
  const lds_char* lds = (const lds_char*)sm;

  // All output tiles of one token tile, then of the next: every XCD takes an equal, contiguous run
  // of that list, and workgroup j of an XCD positions j, j + stride, ... of its run.
  struct Tile {
    int64_t m0;
    int which, n0;
  };
  const int64_t total = (int64_t)gm * per_m;
  const int64_t first = total * xcd / kGemmXcds;
  const int count = (int)(total * (xcd + 1) / kGemmXcds - first);
  const int stride = gridDim.x / kGemmXcds;
  auto tile_at = [&](int seq) {
    Tile t;
    const int64_t mt = (first + seq) / per_m;
    const int nt = (int)((first + seq) - mt * per_m);
    t.m0 = mt * kEdge;
    t.which = nt / gn;
    t.n0 = (nt % gn) * kEdge;
    return t;
  };
  int seq = blockIdx.x / kGemmXcds;
  if (seq >= count) return;  // uniform for the workgroup, before any barrier

  // Copies: an instruction lands 8 LDS rows; a wavefront owns kRows token rows and W rows.  The
  // chunk swizzle of rows 8 i .. 8 i + 7 differs from that of the first eight by bit 2 for odd i.
  // W's LDS row 16 ct + i of a wavefront's run of channels is channel kNT i + ct.
  const uint32_t k2 = (uint32_t)K * 2;
  const uint32_t lrow = lane >> 3, lchunk = ((lane & 7) ^ (lane >> 4)) * 16u;
  // where the next slot of A and of W is fetched from: position in the list, k, first row
  int a_seq = seq, a_k = 0, w_seq = seq, w_k = 0;
  const uint16_t *abase, *wbase;
  uint32_t alast;   // last token row that exists, counted from this wavefront's first
  int64_t wodd;     // elements from a W row to the one 8 kNT channels on (0 where that does not exist)
  auto aim_a = [&]() {
    const int64_t m = tile_at(a_seq).m0 + wave * kRows;
    alast = (uint32_t)max(min(rows - 1 - m, (int64_t)kRows - 1), (int64_t)0);
    abase = uniform_ptr(A + min(m, rows - 1) * K);
  };
  auto aim_w = [&]() {
    const Tile t = tile_at(w_seq);
    const int n = t.n0 + wn;
    wbase = uniform_ptr(outs.W[t.which] + (int64_t)(min(n, N - 64) + (wave & 3) * (kNT / 4)) * K);
    wodd = n + 8 * kNT < N ? (int64_t)(8 * kNT) * K : 0;
  };
  // token rows past the end repeat the last one, channels past the end others; never stored
  // (the lane's place is made opaque so that the offsets are worked out here and not held)
  auto copy_a = [&](int slot) {
    uint32_t lr = lrow;
    asm volatile("" : "+v"(lr));
#pragma unroll
    for (int i = 0; i < kCopies; ++i)
      dma16(abase, __umul24(min(i * 8 + lr, alast), k2) + (lchunk ^ ((i & 1) * 64u)),
            lds0 + slot * kSlotBytes + (wave * kRows + i * 8) * 128);
    if (++a_k < nk) {
      abase += kTK;
    } else {
      a_k = 0;
      a_seq += stride;
      if (a_seq < count) aim_a();
    }
  };
  auto copy_w = [&](int slot) {
    uint32_t lr = lrow;
    asm volatile("" : "+v"(lr));
#pragma unroll
    for (int i = 0; i < kCopies; ++i)
      dma16(wbase + (i >> 1) * K + ((i & 1) ? wodd : 0), (__umul24(lr, kNT * k2) + lchunk) ^ ((i & 1) * 64u),
            lds0 + slot * kSlotBytes + (wave * kRows + i * 8) * 128);
    if (++w_k < nk) {
      wbase += kTK;
    } else {
      w_k = 0;
      w_seq += stride;
      if (w_seq < count) aim_w();
    }
  };
  int slot = 0;                // of this step's A; W's is the next, and so on in turn
  bool ahead = false;          // the youngest copies are an A that the coming step does not need
  auto ring = [](int s) { return s >= kSlots ? s - kSlots : s; };
  // the copies that go out in a step: the next step's W, then the A after the next
  auto fetch = [&](int at) {
    if (w_seq < count) copy_w(ring(at + 3));
    ahead = a_seq < count;
    if (ahead) copy_a(ring(at + 4));
  };

  // byte offsets of this lane's fragment chunks inside a slot, for the two 32-wide halves of k
  const int f0 = c * 128 + ((G ^ ((c >> 1) & 7)) * 16), f1 = f0 ^ 64;

  aim_a();
  aim_w();
  copy_a(0);
  copy_w(1);
  if (a_seq < count) copy_a(2);
  wait_vm0();
  lds_barrier();
  fetch(0);
  bool stores_behind = false;  // exactly kTileStores stores are younger than the first step's fetch
  for (;;) {
    const Tile cur = tile_at(seq);
    f32x4 acc[kMT][kNT];  // [token tile][channel tile]
#pragma unroll
    for (int t = 0; t < kMT; ++t)
#pragma unroll
      for (int a = 0; a < kNT; ++a) acc[t][a] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < nk; ++k) {
      if (k > 0) {  // (a tile's first step is waited for, and its fetch sent, before the last one's stores)
        if (!ahead) wait_vm0();
        else if (k == 1 && stores_behind) wait_vm<kCopies + kTileStores>();
        else wait_vm<kCopies>();
        lds_barrier();  // everybody's copies of this step are in, and the last step's slots are free
        fetch(slot);
      }
      const lds_char* at_a = lds + slot * kSlotBytes + wm * 128;
      const lds_char* at_w = lds + ring(slot + 1) * kSlotBytes + wn * 128;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        Frag fa[kMT], fw[kNT];
#pragma unroll
        for (int a = 0; a < kNT; ++a)
          fw[a].u = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(
              at_w + (h ? f1 : f0) + a * 16 * 128);
#pragma unroll
        for (int t = 0; t < kMT; ++t)
          fa[t].u = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(
              at_a + (h ? f1 : f0) + t * 16 * 128);
#pragma unroll
        for (int t = 0; t < kMT; ++t)
#pragma unroll
          for (int a = 0; a < kNT; ++a)
            acc[t][a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[t].h, fw[a].h, acc[t][a], 0, 0, 0);
      }
      slot = ring(slot + 2);
    }

    // Epilogue: a lane holds channels n .. n + kNT - 1 of token m for every (token tile, r).  What
    // it reads is waited for together with the next step's operands; then that step's fetch goes
    // out ahead of the stores, which have two steps to drain before a copy is awaited behind them.
    // (The lane's place is made opaque here: otherwise its store addresses are worked out before
    // the loops and held in registers that the products need.)
    typedef uint32_t Run __attribute__((ext_vector_type(kNT / 2)));  // kNT channels of a token
    int ec = c, eg = 4 * G;
    asm("" : "+v"(ec), "+v"(eg));
    const float* __restrict__ bias = outs.bias[cur.which];
    const int n = cur.n0 + wn + ec * kNT;
    const bool channels = n < N;
    const int64_t corner = (cur.m0 + wm) * N + cur.n0 + wn;  // of this wavefront's part, uniform
    const int mleft = (int)min(rows - cur.m0 - wm, (int64_t)kEdge) - eg;  // tokens from this lane's first on
    const uint32_t lane_at = (uint32_t)(eg * N + ec * kNT) * 2u;
    float bv[kNT];
    Run rr[kMT][4];
#pragma unroll
    for (int a = 0; a < kNT; ++a) bv[a] = (bias && channels) ? bias[n + a] : 0.f;
    if (kResidual) {
#pragma unroll
      for (int t = 0; t < kMT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          rr[t][r] = Run(0u);
          if (channels && t * 16 + r < mleft)
            rr[t][r] = *reinterpret_cast<const Run*>(
                reinterpret_cast<const char*>(R + corner + (int64_t)(t * 16 + r) * N) + lane_at);
        }
    }
    wait_vm0();
    const bool more = seq + stride < count;
    if (more) {
      lds_barrier();
      fetch(slot);
    }
    auto store = [&](int t, int r) {
      Run w;
#pragma unroll
      for (int i = 0; i < kNT / 2; ++i) {
        float lo = acc[t][2 * i][r] + bv[2 * i], hi = acc[t][2 * i + 1][r] + bv[2 * i + 1];
        if (kResidual) {
          lo += lo16(rr[t][r][i]);
          hi += hi16(rr[t][r][i]);
        }
        w[i] = pack2(lo, hi);
      }
      *reinterpret_cast<Run*>(
          reinterpret_cast<char*>(outs.Y[cur.which] + corner + (int64_t)(t * 16 + r) * N) + lane_at) = w;
    };
    const bool full = cur.m0 + kEdge <= rows && cur.n0 + kEdge <= N;
    if (full) {
#pragma unroll
      for (int t = 0; t < kMT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) store(t, r);
    } else {
#pragma unroll
      for (int t = 0; t < kMT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (channels && t * 16 + r < mleft) store(t, r);
    }
    if (!more) break;
    // a partial tile's stores are not counted: its successor waits for everything
    stores_behind = full;
    if (!full) ahead = false;
    seq += stride;
  }
}

// ---------------------------------------------------------------------------
// The same layer for few tokens: 64 x 64 tiles, one per workgroup of eight wavefronts (16 tokens x 32
// channels each), k 64 at a time through a ring of four steps of A and W.  With at most two tiles per
// CU a launch is one chain of steps, and what counts is how little each of them waits: three steps are
// under way, and a step's fragments are read while the one before is multiplied.  The tiles of a run of
// channels follow each other, so that an XCD fetches an eighth of W instead of most of it.
// Sums are in the order of linear_kernel: the same bits.
//
// Measured, Q/K/V + output projection, us, tiles of 128 / these: 261 rows of 1024 channels 13.5 + 13.3 /
// 7.9 + 6.7; 522 rows 13.7 + 13.3 / 10.9 + 6.8; 522 rows of 512 channels 8.7 + 8.3 / 5.7 + 4.8.  At 522 rows the
// output projection's launch and epilogue are 3.4 of 6.8, its copies alone 2.7 and its products, bound by LDS reads,
// 2.6.  No faster: five or nine steps, fragments read in their own step (7.2), four wavefronts of
// 32 x 32 (8.1), k shared between two groups of wavefronts (7.3), 32 x 64 or 128 x 64 tiles (7.2, 9.1); W read
// straight into registers is twice as slow (13.8 and more).
// ---------------------------------------------------------------------------
constexpr int kFewSteps = 4;                      // of the ring
constexpr int kFewStepBytes = 2 * kFewEdge * kTK * 2;  // A's rows, then W's
constexpr int kFewCopies = kFewStepBytes / 1024 / (kGemmThreads / 64);  // of a wavefront per step
static_assert(kFewCopies == 2, "one eight-row copy of A and one of W per wavefront");

// waits until the step `ahead` steps before the youngest one that was requested is in (ahead <= kMost)
template <int kMost>
__device__ __forceinline__ void wait_steps(int ahead) {
  if (ahead >= kMost) wait_vm<kMost * kFewCopies>();
  else if constexpr (kMost > 0) wait_steps<kMost - 1>(ahead);
}

template <bool kResidual>
__global__ __launch_bounds__(kGemmThreads, 4) void linear_few_kernel(
    const uint16_t* __restrict__ A, LinearOuts outs, const uint16_t* __restrict__ R, int64_t rows,
    int N, int K, int gm, int gn) {
  __shared__ __align__(16) char sm[kFewSteps * kFewStepBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, G = lane >> 4;
  const int wm = (wave & 3) * 16, wn = (wave >> 2) * 32;  // this wavefront's tokens and channels in the tile
  const int nk = K / kTK;

  // the tiles, all of one run of channels, then of the next; every XCD takes an equal run of that list
  const int total = gm * gn * outs.count;  // (at most two per CU)
  const int xcd = blockIdx.x % kGemmXcds;
  const int at = total * xcd / kGemmXcds + (int)(blockIdx.x / kGemmXcds);
  if (at >= total * (xcd + 1) / kGemmXcds) return;  // uniform for the workgroup, before any barrier
  const int nt = at / gm;
  const int64_t m0 = (int64_t)(at - nt * gm) * kFewEdge;
  const int which = nt / gn, n0 = (nt - which * gn) * kFewEdge;

  // Copies: wavefront w lands rows 8 w .. 8 w + 7 of A and of W (LDS layout and channel order as in
  // linear_kernel: W's LDS row 16 ct + i of a wavefront's 32 channels is channel 2 i + ct).  Token rows
  // past the end repeat the last one; never stored.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)sm + wave * 1024u;
  const uint32_t lrow = lane >> 3, k2 = (uint32_t)K * 2;
  const uint32_t chunk = ((lane & 7) ^ (lane >> 4) ^ (4 * (wave & 1))) * 16u;
  const int64_t m = min(m0 + 8 * wave, rows - 1);
  const uint16_t* abase = uniform_ptr(A + m * K);
  const uint16_t* wbase = uniform_ptr(
      outs.W[which] + (int64_t)(n0 + (wave >> 2) * 32 + (wave & 1) * 16 + ((wave >> 1) & 1)) * K);
  const uint32_t aoff = __umul24((uint32_t)min((int64_t)lrow, rows - 1 - m), k2) + chunk;
  const uint32_t woff = __umul24(lrow, 2 * k2) + chunk;
  auto fetch = [&](int slot) {
    dma16(abase, aoff, lds0 + slot * kFewStepBytes);
    dma16(wbase, woff, lds0 + slot * kFewStepBytes + kFewStepBytes / 2);
    abase += kTK;
    wbase += kTK;
  };

  // what the epilogue adds, requested first: channels n, n + 1 of tokens mw .. mw + 3
  const float* __restrict__ bias = outs.bias[which];
  const int n = n0 + wn + 2 * c;
  const int64_t mw = m0 + wm + 4 * G;
  const float b0 = bias ? bias[n] : 0.f, b1 = bias ? bias[n + 1] : 0.f;
  uint32_t rr[4] = {0u, 0u, 0u, 0u};
  if (kResidual) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (mw + r < rows) rr[r] = *reinterpret_cast<const uint32_t*>(R + (mw + r) * N + n);
  }

#pragma unroll
  for (int s = 0; s < kFewSteps - 1; ++s)
    if (s < nk) fetch(s);
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  struct Step { Frag a[2], w[2][2]; };  // [half of k], [channel tile]
  const int f0 = c * 128 + ((G ^ ((c >> 1) & 7)) * 16);
  auto read = [&](Step& f, int slot) {
    const lds_char* s = (const lds_char*)sm + slot * kFewStepBytes;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int fh = f0 ^ (64 * h);
#pragma unroll
      for (int a = 0; a < 2; ++a)
        f.w[h][a].u = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(
            s + kFewStepBytes / 2 + (wn + 16 * a) * 128 + fh);
      f.a[h].u = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(s + wm * 128 + fh);
    }
  };
  int slot = 0;  // of the step whose fragments were read last
  wait_steps<kFewSteps - 2>(nk - 1);
  lds_barrier();
  Step even, odd;
  read(even, 0);
  auto step = [&](int k, const Step& now, Step& then) {
    if (k + 1 < nk) {
      wait_steps<kFewSteps - 3>(nk - 2 - k);
      lds_barrier();  // everybody's copies of step k + 1 are in, and the slot of step k - 1 is free
      if (k + kFewSteps - 1 < nk) fetch((slot + kFewSteps - 1) % kFewSteps);
      slot = (slot + 1) % kFewSteps;
      read(then, slot);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int a = 0; a < 2; ++a)
        acc[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(now.a[h].h, now.w[h][a].h, acc[a], 0, 0, 0);
  };
  for (int k = 0;; ++k) {
    step(k, even, odd);
    if (++k >= nk) break;
    step(k, odd, even);
    if (k + 1 >= nk) break;
  }

#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (mw + r < rows) {
      float lo = acc[0][r] + b0, hi = acc[1][r] + b1;
      if (kResidual) {
        lo += lo16(rr[r]);
        hi += hi16(rr[r]);
      }
      *reinterpret_cast<uint32_t*>(outs.Y[which] + (mw + r) * N + n) = pack2(lo, hi);
    }
}

hipError_t launch_layernorm(const void* x, const float* gamma, const float* beta, void* y,
                            int64_t rows, int C, float eps, hipStream_t st) {
  if (C % 8 != 0 || C > 64 * 8 * kLnMaxChunks) return hipErrorInvalidValue;
  const int64_t groups = (rows + (kLnThreads / 64) - 1) / (kLnThreads / 64);
  if (groups > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
  (void)hipGetLastError();
  if (C <= 64 * 8 * 4)
    hipLaunchKernelGGL(layernorm_kernel<4>, dim3((unsigned)groups), dim3(kLnThreads), 0, st,
                       (const uint16_t*)x, gamma, beta, (uint16_t*)y, rows, C, eps);
  else
    hipLaunchKernelGGL(layernorm_kernel<kLnMaxChunks>, dim3((unsigned)groups), dim3(kLnThreads), 0,
                       st, (const uint16_t*)x, gamma, beta, (uint16_t*)y, rows, C, eps);
  return hipGetLastError();
}

template <int kEdge>
static hipError_t launch_linear_tiles(const uint16_t* A, const LinearOuts& outs, const uint16_t* R,
                                      int64_t rows, int N, int K, hipStream_t st) {
  const int64_t gm = (rows + kEdge - 1) / kEdge;
  const int gn = (N + kEdge - 1) / kEdge;
  const int64_t per_xcd = (gm * gn * outs.count + kGemmXcds - 1) / kGemmXcds;
  if (gm > 0x7FFFFFFF || per_xcd > 0x3FFFFFFF) return hipErrorInvalidConfiguration;
  constexpr int64_t kMost = kEdge == 256 ? kGemmCus : 2 * kGemmCus;  // workgroups resident at once
  const int64_t groups = per_xcd * kGemmXcds;
  const dim3 grid((unsigned)(groups < kMost ? groups : kMost));
  if (R)
    hipLaunchKernelGGL((linear_kernel<kEdge, true>), grid, dim3(kGemmThreads), 0, st, A, outs, R, rows,
                       N, K, (int)gm, gn);
  else
    hipLaunchKernelGGL((linear_kernel<kEdge, false>), grid, dim3(kGemmThreads), 0, st, A, outs, R, rows,
                       N, K, (int)gm, gn);
  return hipGetLastError();
}

static hipError_t launch_linear_few(const uint16_t* A, const LinearOuts& outs, const uint16_t* R,
                                    int64_t rows, int N, int K, hipStream_t st) {
  const int gm = (int)((rows + kFewEdge - 1) / kFewEdge), gn = N / kFewEdge;
  const int tiles = (int)few_tiles(rows, N, outs.count);
  const dim3 grid((unsigned)((tiles + kGemmXcds - 1) / kGemmXcds * kGemmXcds));
  if (R)
    hipLaunchKernelGGL(linear_few_kernel<true>, grid, dim3(kGemmThreads), 0, st, A, outs, R, rows, N, K, gm, gn);
  else
    hipLaunchKernelGGL(linear_few_kernel<false>, grid, dim3(kGemmThreads), 0, st, A, outs, R, rows, N, K, gm, gn);
  return hipGetLastError();
}

static hipError_t launch_linear_edge(int edge, const uint16_t* A, const LinearOuts& outs, const uint16_t* R,
                                     int64_t rows, int N, int K, hipStream_t st) {
  if (edge == kFewEdge) return launch_linear_few(A, outs, R, rows, N, K, st);
  if (edge == kSmallEdge) return launch_linear_tiles<kSmallEdge>(A, outs, R, rows, N, K, st);
  return launch_linear_tiles<kLargeEdge>(A, outs, R, rows, N, K, st);
}

hipError_t launch_linear(const void* A, const LinearOuts& outs, const void* R, int64_t rows, int N,
                         int K, hipStream_t st) {
  if (K % 64 != 0 || N % 64 != 0 || outs.count < 1 || outs.count > 3) return hipErrorInvalidValue;
  (void)hipGetLastError();
  const uint16_t* a = (const uint16_t*)A;
  const uint16_t* r = (const uint16_t*)R;
  const LinearPlan plan = plan_linear(rows, N, K, outs.count, r != nullptr);
  if (plan.split == 0) return launch_linear_edge(plan.edge, a, outs, r, rows, N, K, st);
  const hipError_t e = launch_linear_edge(kLargeEdge, a, outs, r, plan.split, N, K, st);
  if (e != hipSuccess) return e;
  LinearOuts rest = outs;
  for (int i = 0; i < outs.count; ++i) rest.Y[i] += plan.split * N;
  return launch_linear_edge(plan.edge, a + plan.split * K, rest, r ? r + plan.split * N : nullptr,
                            rows - plan.split, N, K, st);
}

}  // namespace agg
