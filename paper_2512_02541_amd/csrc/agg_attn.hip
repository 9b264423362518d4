// Flash-style forward kernel for subsampled global attention (AVGGT Sec. 4.3):
// every query attends to the compacted key/value set, plus -- inside the same
// softmax -- its own key/value when its token was dropped and the mean pair of
// all dropped patches.  With an un-subsampled compacted set and no extras the
// same kernel is ordinary global attention (Sec. 4.2).
//
// Mapping to gfx950
//   * One workgroup = 4 wavefronts; a wavefront owns kQB blocks of 16 kJ queries (2 x 32 at full
//     width) for the whole key loop and keeps Q and the output accumulator in registers.  The
//     last workgroups of a launch may be narrower (plan_tiles).
//   * Both products run on v_mfma_f32_16x16x32_bf16, which accumulates 32 products per pass
//     through its four accumulator registers: half the accumulator traffic per flop of the
//     32x32x16 shape, and the part is power-limited on this kernel (measured on hashed
//     operands, MFMAs alone: 1.94 against 1.74 PFLOP/s).
//   * The score tile is computed transposed, S^T = K * Q^T: a lane then holds keys of ONE
//     query (four per 16-key tile), so row sums are in-register plus a reduction over the four
//     lanes c, c+16, c+32, c+48, and the exponentiated tiles are already the B operand of the
//     second product O^T += V^T * P^T.  P never touches LDS.  A 32-key block is scored as two
//     16-key tiles whose rows are assigned to the block's keys such that the eight probabilities
//     of a lane belong to exactly one 16-byte chunk of the compacted V tile (row_key below).
//     On the fast path the row sums are a ninth product of the same shape per query tile, a
//     row of ones against P^T (+12.5 % MFMAs): the vector ALU, which has to issue twice as
//     many MFMAs as with the larger shape, then does nothing per score but exponentiate and
//     convert.
//   * K/V arrive in "fragment order" (agg.h): a 64-key tile is a linear 8 KiB
//     copy into LDS and every MFMA A operand is one conflict-free 16-byte read.
//     Three tiles are resident: the one in use, the next one and the one being
//     filled.  Tiles go global -> LDS without passing through registers
//     (global_load_lds_dwordx4 with a scalar base, so advancing a tile costs two
//     scalar adds); a wavefront waits for its own copies before the barrier that
//     ends an iteration.  The tile loop is unrolled over the three buffers, so every
//     LDS read uses an immediate offset: the loop spends no vector instruction on
//     addresses.
//   * At head dimension 64 the vector ALU is as loaded as the matrix core (one
//     exponential per 256 MFMA flops) and a wavefront issues in order, so the key
//     loop is a software pipeline over "units" (32 keys x 16 kJ queries).  Step u
//     exponentiates unit u on the vector ALU while the matrix core computes the
//     scores of unit u + kQB - 1 and then P V of unit u - 1.  K fragments of a
//     32-key block are fetched from LDS once per kQB units, V fragments likewise.
//   * Fast path: Q is pre-multiplied by scale*log2(e) and the probabilities are
//     exp2 of the raw base-2 logits, with NO reference subtracted: softmax is
//     invariant to the reference, float/bf16 exponents cover 2^+-126, and the
//     per-score work shrinks to exp + convert.  A row whose sum leaves
//     [2^-90, 2^90] (logits beyond about +-60 nats) makes the whole workgroup
//     redo its rows in the general path (in place, or by a second kernel behind this
//     one, see redo_in_place); ordinary attention logits never get there.  The
//     sums are checked every few tiles, so an overflow ends the fast pass early.
//   * General path: the same pipeline with a per-row reference.  The score MFMAs start from
//     an accumulator holding minus the reference instead of zero, so the scores come out
//     relative to it and the vector ALU does no more per score than on the fast path.  The
//     reference starts at the largest of the extras and the first 32 keys and is raised
//     lazily: a unit's row sums show when a score exceeds it by more than 2^100; only then
//     (a rare, wavefront-uniform branch) is the unit's maximum taken, the accumulator
//     rescaled and the unit redone.  No running maximum is computed otherwise.
//   * A launch with at most one workgroup per CU runs eight wavefronts in each: two groups of four
//     that take half the key tiles each and add their sums and accumulators at the end (attend).
//   * The zero-padded rows of the last tile are masked there (the last tile is
//     peeled), nowhere else.
//   * The extras enter as the initial state (sum, accumulator) of either path, so
//     the three parts share one normalisation by construction.
//   * Workgroups are numbered so that the 8 XCDs each stream a different
//     (batch, head): all workgroups resident on one XCD read the same K/V
//     stream and share it through that XCD's L2.
#include "agg_attn_plan.h"
#include "agg_internal.h"
#include "agg_lds_copy.h"

namespace agg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kAttnThreads = 64 * kWaves;
constexpr int kBlocksPerCu = 2;         // two wavefronts per SIMD
constexpr int kXcds = 8;
constexpr int kLdsTiles = 3;
constexpr int kEpiStride = kHeadDim + 8;  // bf16 per query row of the epilogue's LDS tile (padded)
constexpr int kChunks = kTileElems / 8;  // 16-byte chunks per K or V tile (512)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kSumHi = 1.2379400392853803e27f;   // 2^90
constexpr float kSumLo = 8.077935669463161e-28f;   // 2^-90
constexpr float kLazy = 60.0f;  // general path: a unit may exceed the row's reference by 2^60
constexpr float kUnitHi = 1.2676506002282294e30f;  // 2^100: a unit's row sum that forces a look

union Frag {
  u32x4 u;
  bf16x8 h;
};

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2 p = {lo, hi};
  bf16x2 h = __builtin_convertvector(p, bf16x2);  // round to nearest even
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Exchange between lanes l and l ^ 32.  v_permlane32_swap exchanges the upper 32 lanes of its
// first operand with the lower 32 of its second; fed the same value twice it returns
// (own, partner) in one order or the other, and both uses below are symmetric.
__device__ __forceinline__ float pair_max(float x) {
  const uint32_t b = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  const uint32_t b = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

#define AGG_MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16((a).h, (b).h, (c), 0, 0, 0)

// Lane geometry of v_mfma_f32_16x16x32_bf16: c = lane & 15 is the row of the A operand, the
// column of the B operand and of the result; G = lane >> 4 selects eight of the 32 contraction
// elements (8 G .. 8 G + 7) in A and B, and result rows 4 G .. 4 G + 3.
//
// A 32-key block is scored as two 16-key tiles.  Tile kt takes the block's keys
//     row i  ->  key (i & 7) + 16 (i >> 3) + 8 kt          (tile 0: 0-7, 16-23; tile 1: 8-15, 24-31)
// so that the eight probabilities a lane holds after both tiles (rows 4 G .. 4 G + 3 of each) are
// exactly the eight keys of ONE 16-byte chunk of the compacted V tile (agg.h: chunk (t, g) holds
// keys 16 t + 4 g + {0..3, 8..11}; here t = 2 kb + (G >> 1), g = G & 1): the exponentiated scores
// are the B operand of O^T += V^T P^T as they stand, and V fragments are plain 16-byte reads.
__device__ __forceinline__ int row_key(int i) { return (i & 7) + 16 * (i >> 3); }

// sum / maximum over the four lanes c, c + 16, c + 32, c + 48 that share a query
__device__ __forceinline__ float quad_sum(float x) {
  x += __shfl_xor(x, 16);
  return pair_sum(x);
}
__device__ __forceinline__ float quad_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return pair_max(x);
}

// LDS words through which wavefronts tell each other of rows that the fast path cannot handle: four
// for the check inside the key loop, four for the one behind it.
constexpr int kVoteWords = 2 * kWaves;

// Whether x holds in any lane of the workgroup's first kWaves wavefronts (`mine`: this is one of them).
// Passes one barrier.  (The library's workgroup-wide "or" passes three and reduces through LDS: a layer
// of two frames of 16x16 14.55 us with it and 14.3 without, its block 43.5 / 43.1, index-driven, 40
// frames, 2700 / 2684; longer calls alike.)
__device__ __forceinline__ bool vote(bool x, uint32_t* words, int wave, int lane, bool mine) {
  const bool any = __builtin_amdgcn_ballot_w64(x) != 0;
  if (mine && lane == 0) words[wave] = any ? 1u : 0u;
  __syncthreads();
  const u32x4 all = *reinterpret_cast<const u32x4*>(words);
  return __builtin_amdgcn_readfirstlane(all[0] | all[1] | all[2] | all[3]) != 0;
}

// zero-padded rows of the last tile: key index inside the tile >= valid -> -inf
template <int kJ>
__device__ __forceinline__ void mask_unit(f32x4 (&S)[2 * kJ], int kb, int valid, int G) {
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int km = 32 * kb + 8 * kt + row_key(4 * G + r);
      if (km >= valid) {
#pragma unroll
        for (int j = 0; j < kJ; ++j) S[kJ * kt + j][r] = -INFINITY;
      }
    }
}

// Everything a wavefront keeps in registers across the key loop.  qb = query block, j = its
// 16-query tile, kt = 16-key tile of a key block, h = half of the channel range, dt = 16-channel
// tile of the output.
template <int kQB, int kJ>
struct Wave {
  Frag Qf[kQB][2 * kJ];    // [qb][2 j + h]: B operand of S^T = K Q^T, pre-multiplied by scale*log2(e)
  f32x4 O[kQB][kJ][4];     // [qb][j][dt]: O^T accumulator; channel = 16 dt + 4 G + r, query = c
  f32x4 S[kQB][2 * kJ];    // [qb][kJ kt + j]: score tiles in flight; key = row_key(4 G + r) + 8 kt
  f32x4 L[kQB][kJ];        // [qb][j]: fast path: element 0 of the lanes G = 0 is the row sum, kept by the matrix core
  float la[kQB][kJ];       // [qb][j]: general path: this lane's part of the row sum
  float mref[kQB][kJ];     // general path: the row's reference (base-2 logit)
  Frag a[4];               // [2 kt + h]: K fragments of the block whose scores are being computed
  Frag v[4];               // [dt]: V fragments of the block whose P V is being accumulated
  Frag P[kJ];              // [j]: probabilities of the previous unit
  Frag ones;               // A operand of the row sums: row 0 ones, the others zeros
};

// Probabilities of the 8 kJ base-2 logits a lane holds for a unit, packed as the B operands of
// the PV MFMAs: for query tile j, contraction elements 8 G .. 8 G + 7 are key tile 0's rows, then
// key tile 1's.  The query tiles alternate in the instruction stream.
template <int kJ>
__device__ __forceinline__ void exp_unit(const f32x4 (&S)[2 * kJ], Frag (&P)[kJ]) {
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < kJ; ++j)
        P[j].u[2 * kt + i] = pack_bf16(fast_exp2(S[kJ * kt + j][2 * i]), fast_exp2(S[kJ * kt + j][2 * i + 1]));
}

// General path: the same, and the sums of each query tile's part (there the vector ALU keeps
// the sums: the unit's own sum is what tells that a score has run away from the row's reference,
// and it is needed before the probabilities reach the matrix core)
template <int kJ>
__device__ __forceinline__ void exp_unit_sum(const f32x4 (&S)[2 * kJ], Frag (&P)[kJ], float (&l)[kJ]) {
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < kJ; ++j) {
        const float e0 = fast_exp2(S[kJ * kt + j][2 * i]);
        const float e1 = fast_exp2(S[kJ * kt + j][2 * i + 1]);
        P[j].u[2 * kt + i] = pack_bf16(e0, e1);
        l[j] += e0;
        l[j] += e1;
      }
}

// Where the key/value tiles come from.
//   kSrcCompact: the fragment-order compacted tensors of agg_kv_subsample: a tile is a linear
//                8 KiB copy and already in MFMA operand order.
//   kSrcRows:    consecutive rows of the token-major K and V themselves (ordinary and per-frame
//                attention: every token is a key), no compacted copy.
//   kSrcIndexed: rows of K and V picked through a list of token ids (Sec. 4.3 restricts keys
//                and values to a subset of the tokens; here the subset is read in place).
// In the two row modes a tile lies in LDS row-major, 128 bytes per key, with the 16-byte chunk
// number XOR-ed by a function of the row so that the fragment reads spread over all 64 banks:
// K fragments (eight channels of one key per lane) are plain 16-byte reads; V fragments (eight
// keys of one channel per lane) come from the transposing read ds_read_b64_tr_b16, which hands
// lane i of a 16-lane group the i-th 16-bit column of the four 8-byte rows the group's lanes
// 4j .. 4j+3 point at.
enum { kSrcCompact = 0, kSrcRows = 1, kSrcIndexed = 2 };

typedef short s16x4 __attribute__((ext_vector_type(4)));

// chunk swizzle of a K row in the row modes: the 16 rows a lane group reads (i, i + 16 for eight
// consecutive i) must fall on 16 different 16-byte slots of the 256-byte bank period
__device__ __forceinline__ uint32_t k_swizzle(uint32_t row) {
  return ((row >> 1) & 3u) | (((row >> 4) & 1u) << 2);
}

// per-lane LDS byte offsets of the fragment reads (row modes) or chunk numbers (compact mode)
struct FragAddr {
  int lane;
  int kc[2];             // compact: chunk of tile kt inside a (key block, channel half) run
  int vc;                // compact: chunk inside a key block's V run (plus 16 dt)
  uint32_t k[4];         // rows: K fragment [2 kt + h]
  uint32_t v[4];         // rows: V fragment of channel tile dt (first four keys; +8 rows: the others)
};

__device__ __forceinline__ FragAddr frag_addr(int lane) {
  FragAddr f;
  const int c = lane & 15, G = lane >> 4;
  f.lane = lane;
  // compact K tile in LDS: [kb][h][G][32 keys], a key at position (key with bits 3 and 4
  // exchanged): tile kt's sixteen keys are then consecutive
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) f.kc[kt] = G * 32 + 16 * kt + c;
  f.vc = G * 64 + c;
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t row = (uint32_t)(row_key(c) + 8 * kt);
      f.k[2 * kt + h] = row * 128u + (((uint32_t)(4 * h + G) ^ k_swizzle(row)) * 16u);
    }
  // V: the lanes 4 i' .. 4 i' + 3 of a 16-lane group point at row i' of the group's first four
  // keys (16 (G >> 1) + 4 (G & 1) + i'), each at 8 of the 32 bytes of channels 16 dt .. 16 dt + 15;
  // chunk bit 2 is flipped on rows 2, 3 mod 4
  const int row = 16 * (G >> 1) + 4 * (G & 1) + (c >> 2);
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) {
    const int chunk = (2 * dt + ((c & 3) >> 1)) ^ (4 * ((row >> 1) & 1));
    f.v[dt] = (uint32_t)(row * 128 + chunk * 16 + (c & 1) * 8);
  }
  return f;
}

template <int kSrc>
__device__ __forceinline__ void load_k_frags(const u32x4* __restrict__ lds, int buf, int kb,
                                             const FragAddr& f, Frag (&a)[4]) {
  if (kSrc == kSrcCompact) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        a[2 * kt + h].u = lds[buf * kChunks + kb * 256 + h * 128 + f.kc[kt]];
  } else {
    const lds_char* base = (const lds_char*)lds + buf * (kChunks * 16) + kb * (32 * 128);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a[i].u = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(base + f.k[i]);
  }
}
template <int kSrc>
__device__ __forceinline__ void load_v_frags(const u32x4* __restrict__ lds, int buf, int kb,
                                             const FragAddr& f, Frag (&v)[4]) {
  if (kSrc == kSrcCompact) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      v[dt].u = lds[(kLdsTiles + buf) * kChunks + kb * 256 + dt * 16 + f.vc];
  } else {
    lds_char* base = (lds_char*)lds + (kLdsTiles + buf) * (kChunks * 16) + kb * (32 * 128);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      // the group's first four keys, then the four that lie eight rows further on: the order
      // the P operand has
      lds_char* at = base + f.v[dt];
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4*)at);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4*)(at + 8 * 128));
      const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
      v[dt].u = u32x4{l2[0], l2[1], h2[0], h2[1]};
    }
  }
}

// What a workgroup needs to know about its key/value source.
struct KvSource {
  const uint16_t *k, *v;   // compact: tile 0 of this (batch, head); rows: token 0's row of this head
  const int32_t* list;     // indexed: the batch element's token ids
  int64_t rows;            // number of keys (M, or the sequence length)
  uint32_t row_bytes;      // rows: distance between consecutive tokens' rows (H * 128)
  uint32_t max_token;      // indexed: largest valid token id (N*L - 1)
};

// Issues the asynchronous copy of tile t into LDS buffer `buf`.  Every wavefront lands 64
// consecutive 16-byte LDS slots per instruction; which global chunk a lane fetches for its slot
// is what differs between the modes.
template <int kSrc>
struct TileCopier {
  KvSource src;
  const uint16_t *knext, *vnext;  // compact, rows: where the next tile to be copied starts
  int64_t tnext;                  // its number (tiles are copied in order)
  uint32_t wbase;          // LDS byte address of this wavefront's first slot in buffer 0
  // byte offset of this lane's first chunk from the tile's (rows, compact) or the row's (indexed)
  // start, for K and for V; the second lies half a tile (32 rows, whose swizzle is that of the first 32)
  // further on
  uint32_t vk, vv;
  uint32_t row;            // row of the tile this lane's first slot belongs to (rows)
  // Indexed: an instruction's eight rows and a tile's two instructions make 16 ids per wavefront.
  // Lane l holds the id of row l % 16 of them; byte offsets are worked out once per row and handed
  // to the eight lanes that fetch it, a tile ahead of their use.  (Every lane reading and scaling
  // its own two ids cost 17 vector instructions a tile instead of 8, in a loop that the vector ALU
  // bounds: 40 frames 2768 us against 2658, 100 frames 32.4 ms against 31.7, 8 frames 158 against 143.)
  uint32_t lane;           // of the wavefront
  uint32_t list_at;        // byte offset of this lane's id for the tile after the next
  uint32_t id;             // its id for the tile after the next to be copied
  uint32_t from[2];        // next tile to be copied: byte offset of the rows this lane fetches

  __device__ __forceinline__ void init(const KvSource& s, const u32x4* lds, int tid, int wave) {
    src = s;
    knext = s.k;
    vnext = s.v;
    tnext = 0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_char*)lds);
    wbase = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)wave * 1024u);
    const uint32_t slot = (uint32_t)tid;  // 0 .. 255, and 256 more
    row = slot >> 3;
    const uint32_t c = slot & 7;
    const uint32_t ck = (c ^ k_swizzle(row)) * 16u;
    const uint32_t cv = (c ^ (4u * ((row >> 1) & 1))) * 16u;
    if (kSrc == kSrcCompact) {
      // K: the LDS slot of a key has bits 3 and 4 of the key number exchanged (frag_addr)
      const uint32_t key = slot & 31u;
      const uint32_t swapped = (key & 7u) | ((key & 8u) << 1) | ((key & 16u) >> 1);
      vk = ((slot & ~31u) | swapped) * 16u;
      vv = slot * 16u;
    } else if (kSrc == kSrcRows) {
      vk = row * s.row_bytes + ck;
      vv = row * s.row_bytes + cv;
    } else {
      vk = ck;
      vv = cv;
    }
    if (kSrc == kSrcIndexed) {
      lane = tid & 63;
      const uint32_t l = lane & 15;
      list_at = ((l & 8) * 4u + wave * 8u + (l & 7)) * 4u;
      fetch_ids();
      spread_ids();
      fetch_ids();
    }
  }
  __device__ __forceinline__ void fetch_ids() {  // rows past the end repeat the last one; masked later
    const uint32_t at = min(list_at, ((uint32_t)src.rows - 1u) * 4u);
    id = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(src.list) + at);
    list_at += kTileRows * 4u;
  }
  __device__ __forceinline__ void spread_ids() {
    // an id outside the sequence cannot leave it
    const int base = (int)__umul24(min(id, src.max_token), src.row_bytes);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
      from[hh] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane >> 3) + 8 * hh) * 4, base);
  }
  // copies tile tnext into LDS buffer `buf`
  __device__ __forceinline__ void issue(int buf) {
    const uint32_t mk = wbase + (uint32_t)buf * (kChunks * 16);
    const uint32_t mv = wbase + (uint32_t)(kLdsTiles + buf) * (kChunks * 16);
    static_assert(2 * kAttnThreads == kChunks, "two copies per thread and tile");
    if (kSrc == kSrcCompact) {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        dma16(knext + hh * (kTileElems / 2), vk, mk + hh * kAttnThreads * 16);
        dma16(vnext + hh * (kTileElems / 2), vv, mv + hh * kAttnThreads * 16);
      }
      knext += kTileElems;
      vnext += kTileElems;
    } else if (kSrc == kSrcRows) {
      // the tile's rows follow each other in memory
      const size_t half = (size_t)(kTileRows / 2) * (src.row_bytes / 2);
      if ((tnext + 1) * kTileRows <= src.rows) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          dma16(knext + hh * half, vk, mk + hh * kAttnThreads * 16);
          dma16(vnext + hh * half, vv, mv + hh * kAttnThreads * 16);
        }
      } else {  // last, partial tile: rows past the end repeat the last one; masked later
        const uint32_t last = (uint32_t)(src.rows - 1 - tnext * kTileRows);
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const uint32_t r = row + hh * (kTileRows / 2);
          const uint32_t at = (min(r, last) - row) * src.row_bytes;  // (wraps where the row is before this lane's)
          dma16(knext, vk + at, mk + hh * kAttnThreads * 16);
          dma16(vnext, vv + at, mv + hh * kAttnThreads * 16);
        }
      }
      knext += 2 * half;
      vnext += 2 * half;
    } else {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        dma16(src.k, from[hh] + vk, mk + hh * kAttnThreads * 16);
        dma16(src.v, from[hh] + vv, mv + hh * kAttnThreads * 16);
      }
      spread_ids();  // the next tile's offsets; its ids came with the last wait
      fetch_ids();                   // and the ids after those
    }
    ++tnext;
  }
};

// Query tile of product i: 0 .. kJ-1, then back, so that consecutive products always have an operand
// in common.  Measured pass by pass against plain order on two boxes: layers of 100 and 800 frames take 0.1 to
// 0.3 % less (29.05 ms instead of 29.13), calls under 6 ms the same.  With the row of ones (pv_unit) it is 0.8 to
// 1.0 %; of 0.9 % under the counters 0.5 +- 0.2 were cycles and 0.4 +- 0.2 the clock, so less power is a part of it
// at most.
template <int kJ>
constexpr int there_and_back(int i) {
  return (i / kJ) % 2 ? kJ - 1 - i % kJ : i % kJ;
}

// Scores of one unit: the 32 keys of block fragments `a` against the 16 kJ queries of block tq.
// General path: the accumulator starts at minus the row's reference instead of zero, so the
// scores come out relative to it at no cost (the reference is a float, nothing is split).
template <bool kGen, int kQB, int kJ>
__device__ __forceinline__ void score_unit(const Wave<kQB, kJ>& w, int tq, f32x4 (&Sn)[2 * kJ]) {
  f32x4 init[kJ];
#pragma unroll
  for (int j = 0; j < kJ; ++j) {
    const float m = kGen ? -w.mref[tq][j] : 0.f;
    init[j] = f32x4{m, m, m, m};
  }
#pragma unroll
  for (int i = 0; i < 2 * kJ; ++i) {
    const int kt = i / kJ, j = there_and_back<kJ>(i);
    Sn[kJ * kt + j] = AGG_MFMA16(w.a[2 * kt], w.Qf[tq][2 * j], init[j]);
  }
#pragma unroll
  for (int i = 0; i < 2 * kJ; ++i) {
    const int kt = i / kJ, j = there_and_back<kJ>(i);
    Sn[kJ * kt + j] = AGG_MFMA16(w.a[2 * kt + 1], w.Qf[tq][2 * j + 1], Sn[kJ * kt + j]);
  }
}
// O^T += V^T P^T for the unit whose probabilities are in w.P.  Fast path: the row sums are one
// more product, a row of ones and fifteen of zeros against P^T: row 0 of that 16 x 16 result, in
// the lanes G = 0, is the sum of the unit's 32 probabilities of a query, and the vector ALU adds
// nothing.  (Sixteen rows of ones leave the sum in every lane but take 0.7 % longer: the layer of 100
// frames 29.25 ms instead of 29.05, ordinary attention, 24 frames, 1448 us instead of 1440; 0.3 to 0.7 % elsewhere.)
template <bool kGen, int kQB, int kJ>
__device__ __forceinline__ void pv_unit(Wave<kQB, kJ>& w, int pq) {
#pragma unroll
  for (int i = 0; i < 4 * kJ; ++i) {
    const int dt = i / kJ, j = there_and_back<kJ>(i);
    w.O[pq][j][dt] = AGG_MFMA16(w.v[dt], w.P[j], w.O[pq][j][dt]);
  }
  if (!kGen) {
#pragma unroll
    for (int j = 0; j < kJ; ++j) w.L[pq][j] = AGG_MFMA16(w.ones, w.P[j], w.L[pq][j]);
  }
}

// One step of the pipeline inside tile `cur` (see the file header).  kLast: the tile is the
// last one (`valid` of its 64 rows exist, nothing follows).  kGen: general path.
template <int kSrc, bool kLast, bool kGen, int kQB, int kJ>
__device__ __forceinline__ void tile_steps(Wave<kQB, kJ>& w, const u32x4* __restrict__ lds, int cur, int nxt,
                                           int valid, const FragAddr& fa, int G) {
#pragma unroll
  for (int sg = 0; sg < 2 * kQB; ++sg) {
    // A last tile of up to 32 keys: its second block is padding throughout.  (Left out from here on; a
    // separate body for such tiles spilled 80 registers.  Per-frame attention over 1374 keys, 90 frames, 663 /
    // 651 us; layer of 2 frames of 16x16 14.3 / 14.0; 9.5 ms calls alike.)
    if (kLast && sg == kQB && valid <= kTileRows / 2) break;
    const int kb = sg / kQB, qb = sg % kQB;
    const int un = sg + kQB - 1;              // unit whose scores start now
    const int tq = un % kQB;                  // its query block
    const bool beyond = un >= 2 * kQB;        // it belongs to the next tile
    const int pq = (qb + kQB - 1) % kQB;      // query block of the previous unit

    // ---- matrix core, part 1: scores of unit `un` ----
    const bool do_qk = !(kLast && beyond);
    f32x4 Sn[2 * kJ];
    if (do_qk) score_unit<kGen, kQB, kJ>(w, tq, Sn);
    if (tq == kQB - 1) {  // that was the block's last unit: fragments of the following block
      if (un / kQB == 0) load_k_frags<kSrc>(lds, cur, 1, fa, w.a);
      else if (!kLast) load_k_frags<kSrc>(lds, nxt, 0, fa, w.a);
    }

    // ---- vector ALU: probabilities of unit sg ----
    Frag Pn[kJ];
    float unit_sum[kJ];  // general path: the unit's own row sums
#pragma unroll
    for (int j = 0; j < kJ; ++j) unit_sum[j] = 0.f;
    {
      f32x4 (&S)[2 * kJ] = w.S[qb];
      if (kLast && valid < kTileRows) mask_unit<kJ>(S, kb, valid, G);
      if (!kGen) {
        exp_unit<kJ>(S, Pn);
      } else {
        // the scores are already relative to the row's reference; whether it still holds is
        // looked at below, behind the step's last MFMA
        exp_unit_sum<kJ>(S, Pn, unit_sum);
      }
    }
    if (do_qk) {
#pragma unroll
      for (int i = 0; i < 2 * kJ; ++i) w.S[tq][i] = Sn[i];
    }

    // ---- matrix core, part 2: P V of unit sg - 1 ----
    pv_unit<kGen, kQB, kJ>(w, pq);
    if (qb == 0) load_v_frags<kSrc>(lds, cur, kb, fa, w.v);  // the previous block is done with them
#pragma unroll
    for (int j = 0; j < kJ; ++j) w.P[j] = Pn[j];
    // Issue order inside the step: MFMAs and exponentials alternate one by one, a conversion
    // after every second pair (general path: pairs of MFMAs, then their share of the vector work,
    // which there includes the additions).  Left to itself the scheduler bunches the MFMAs, and
    // the wavefront then stalls on the matrix pipe with vector work still to issue.
    if (!kGen) {
      __builtin_amdgcn_sched_group_barrier(0x008, kJ, 0);  // the row-sum products of the last unit
#pragma unroll
      for (int i = 0; i < 4 * kJ; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);  // transcendental
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);  // the pair's conversion
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4 * kJ; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // conversion and two additions
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (kGen) {
      // The unit's sums tell whether the reference still holds: a score more than 2^100 above it
      // cannot hide in them.  Rare, wavefront-uniform: raise the reference of the rows that need
      // it (the others keep theirs: shift 0, factor 1), scale what they have accumulated, and
      // redo the unit's probabilities (its scores are untouched until the next step).
      float all = unit_sum[0];
#pragma unroll
      for (int j = 1; j < kJ; ++j) all += unit_sum[j];
      if (__builtin_amdgcn_ballot_w64(!(all < kUnitHi)) != 0) {
        f32x4 (&S)[2 * kJ] = w.S[qb];
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
          float mx = S[j][0];
#pragma unroll
          for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, S[kJ * kt + j][r]);
          mx = quad_max(mx);  // the four lanes of a row agree
          const float old = w.mref[qb][j];
          if (mx > kLazy) w.mref[qb][j] = old + mx;
          const float d = w.mref[qb][j] - old;
          const float f = fast_exp2(-d);
#pragma unroll
          for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[kJ * kt + j][r] -= d;
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 4; ++r) w.O[qb][j][dt][r] *= f;
          w.la[qb][j] *= f;
        }
#pragma unroll
        for (int j = 0; j < kJ; ++j) unit_sum[j] = 0.f;
        exp_unit_sum<kJ>(S, w.P, unit_sum);
      }
#pragma unroll
      for (int j = 0; j < kJ; ++j) w.la[qb][j] += unit_sum[j];
    }
  }
}

// The key loop of one path.  `first_tile` runs once tile 0 is resident and its first K fragments
// are loaded (the general path takes its reference there).  Returns false when the fast path
// found a row sum it cannot trust.
// kSplit: the workgroup's other wavefronts walk other tiles, perhaps one fewer: no early check, whose
// barriers would not match (the sums are looked at when the loops are done).
template <int kSrc, bool kGen, bool kSplit, int kQB, int kJ, class FirstTile>
__device__ __forceinline__ bool key_loop(Wave<kQB, kJ>& w, u32x4* __restrict__ lds, uint32_t* votes,
                                         const KvSource& src, int ntiles, int last_valid, int tid, int wave,
                                         const FragAddr& fa, int G, FirstTile&& first_tile) {
  TileCopier<kSrc> copy;
  copy.init(src, lds, tid, wave);
  copy.issue(0);
  if (ntiles > 1) copy.issue(1);
  wait_vm0();
  lds_barrier();

  // fill: scores of units 0 .. kQB-2; nothing to multiply by V yet
  load_k_frags<kSrc>(lds, 0, 0, fa, w.a);
  first_tile();
#pragma unroll
  for (int i = 0; i < 4; ++i) w.v[i].u = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int j = 0; j < kJ; ++j) w.P[j].u = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int qb = 0; qb + 1 < kQB; ++qb) score_unit<kGen, kQB, kJ>(w, qb, w.S[qb]);

  int t = 0, cur = 0;
  bool ok = true;
  // one iteration = three tiles, so that the LDS buffer of every access is a constant
  for (int round = 0;; ++round) {
#define AGG_TILE(CUR)                                                                       \
  if (t + 1 >= ntiles) {                                                                    \
    cur = CUR;                                                                              \
    break;                                                                                  \
  }                                                                                         \
  if (t + 2 < ntiles) copy.issue((CUR + 2) % kLdsTiles);                                    \
  tile_steps<kSrc, false, kGen, kQB, kJ>(w, lds, CUR, (CUR + 1) % kLdsTiles, kTileRows, fa, G);      \
  wait_vm0();                                                                               \
  lds_barrier();                                                                            \
  ++t;
    AGG_TILE(0)
    AGG_TILE(1)
    AGG_TILE(2)
#undef AGG_TILE
    if (!kGen && !kSplit && (round & 7) == 7) {  // an overflowing row ends the fast pass early
      bool bad = false;
#pragma unroll
      for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
        for (int j = 0; j < kJ; ++j) bad = bad || !(w.L[qb][j][0] < kSumHi);
      if (vote(bad, votes, wave, tid & 63, true)) {
        ok = false;
        break;
      }
    }
  }
  if (!ok) return false;
  // last tile (runtime buffer number), then the P V of its last unit
  tile_steps<kSrc, true, kGen, kQB, kJ>(w, lds, cur, 0, last_valid, fa, G);
  pv_unit<kGen, kQB, kJ>(w, kQB - 1);
  return true;
}

// Kernel arguments.
struct AttnArgs {
  Geom g;
  uint32_t flags;
  float qscale, mean_bias2;  // scale*log2(e), mean_logit_bias*log2(e)
  const uint16_t *Q, *K, *V, *Kc, *Vc;
  const float *kmean, *vmean;
  uint16_t* O;
  float* lse;
  int npairs;
  TilePlan plan;
  const uint32_t* kept_bits;
  const int32_t* nd_dev;
  const int32_t* list;   // kSrcIndexed: token ids of the keys, [list_stride] per batch element
  int64_t list_stride;   // 0 when every batch element uses the same list
};

constexpr int kTileLds = 2 * kLdsTiles * kTileElems;  // elements: K tiles, then V tiles

// One workgroup's queries q_begin .. q_end - 1 (at most what four wavefronts hold) by one of the
// two paths.  Returns false, without storing anything, when the fast path met a row it cannot
// handle.
// tiles: kTileLds elements of LDS per four wavefronts; votes: kVoteWords words.
// kMode:
//   kAlone      four wavefronts.
//   kSplitKeys  (fast path) eight: the first four take the extras and the first half of the key
//               tiles, the others the second half.  Without a reference the two halves' sums and
//               accumulators just add: the second group's go through LDS to the first, which
//               finishes the rows.
//   kTwin       eight: both groups do the same (so that their barriers match), the first stores.
enum { kAlone, kSplitKeys, kTwin };
template <int kSrc, bool kGen, int kQB, int kJ, int kMode = kAlone>
__device__ __forceinline__ bool attend(const AttnArgs& p, uint16_t* tiles, uint32_t* votes, int b, int h,
                                       int64_t q_begin, int64_t q_end) {
  constexpr bool kSplit = kMode == kSplitKeys;
  static_assert(!(kGen && kSplit), "the general path's halves would need a common reference");
  constexpr int kWaveQ = wave_queries(kQB, kJ);
  const Geom& g = p.g;
  // The general path starts from an opaque thread number, so that the addresses it has in common
  // with a fast pass ahead of it in the same kernel are worked out again: held across the fast
  // key loop they spilled (sga_attn_kernel).
  int thread = threadIdx.x;
  if (kGen) asm volatile("" : "+v"(thread));
  const int group = kMode != kAlone ? __builtin_amdgcn_readfirstlane(thread / kAttnThreads) : 0;
  uint16_t* smem = tiles + group * kTileLds;
  u32x4* lds = reinterpret_cast<u32x4*>(smem);
  const int tid = thread - group * kAttnThreads;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int c = lane & 15;
  const int G = lane >> 4;
  const FragAddr fa = frag_addr(lane);

  // this group's key tiles: first_tile_no .. first_tile_no + ntiles - 1
  const int all_tiles = (int)(g.M_pad / kTileRows);
  const int half = kSplit ? (all_tiles + 1) / 2 : all_tiles;
  const int skip = kSplit && group ? half : 0;
  const int ntiles = kSplit && group ? all_tiles - half : half;
  const int64_t rows_here = min(g.M - (int64_t)skip * kTileRows, (int64_t)ntiles * kTileRows);
  const int last_valid = (int)(rows_here - (int64_t)(ntiles - 1) * kTileRows);  // 1..64
  KvSource src;
  src.rows = rows_here;
  src.row_bytes = (uint32_t)g.H * (kHeadDim * 2);
  src.max_token = (uint32_t)(g.NQ - 1);
  if (kSrc == kSrcCompact) {
    const int64_t bh_off = (((int64_t)b * g.H + h) * g.M_pad + (int64_t)skip * kTileRows) * kHeadDim;
    src.k = uniform_ptr(p.Kc + bh_off);
    src.v = uniform_ptr(p.Vc + bh_off);
    src.list = nullptr;
  } else {
    const int64_t first_row = (int64_t)b * g.NQ + (kSrc == kSrcRows ? (int64_t)skip * kTileRows : 0);
    const int64_t bh_off = (first_row * g.H + h) * kHeadDim;
    src.k = uniform_ptr(p.K + bh_off);
    src.v = uniform_ptr(p.V + bh_off);
    src.list = kSrc == kSrcIndexed
                   ? p.list + (int64_t)b * p.list_stride + (int64_t)skip * kTileRows
                   : nullptr;
  }

  Wave<kQB, kJ> w;
  const uint32_t one = c == 0 ? 0x3F803F80u : 0u;
  w.ones.u = u32x4{one, one, one, one};
  bool dropped[kQB][kJ];
  float l_self[kQB][kJ], l_mean[kQB][kJ];  // base-2 logits of the extras (-inf when absent)
  // caller's list: membership comes from a bitmap, the dropped count from device memory
  const int64_t n_drop = p.nd_dev ? (int64_t)p.nd_dev[b] : g.n_dropped;
  // ordinary and per-frame attention have no extras; where that is known at compile time the fast
  // path's code is a third shorter (the general path's would spill: 363 to 532 registers instead of 9
  // or 10 in the second launch, 64 to 271 instead of none where rows are redone in place)
  constexpr bool kExtras = kSrc != kSrcRows || kGen;
  const bool takes = kExtras && !(kSplit && group);
  const bool use_mean = takes && (p.flags & AGG_MEAN) && n_drop > 0;
  const bool use_diag = takes && (p.flags & AGG_DIAG) && (p.kept_bits != nullptr || n_drop > 0);
  const uint32_t* kbits = p.kept_bits ? p.kept_bits + (int64_t)b * ((g.NQ + 31) / 32) : nullptr;
  const int64_t q_wave = q_begin + wave * kWaveQ;
  // first element of query (qb, j, c)'s row of this head in Q, K, V and O
  auto row_base = [&](int qb, int j) {
    const int64_t q = q_wave + (qb * kJ + j) * 16 + c;
    const int64_t qc = q < q_end ? q : q_end - 1;  // tail rows recompute the last query, never stored
    return (((int64_t)b * g.NQ + qc) * g.H + h) * kHeadDim;
  };
  // this lane's channels 16 dt + 4 G .. + 3 of the query's own value and of the mean value
  auto load_own_v = [&](int qb, int j, int dt) {
    return *reinterpret_cast<const u32x2*>(p.V + row_base(qb, j) + 16 * dt + 4 * G);
  };
  auto load_mean_v = [&](int dt) {
    const float* vm = p.vmean + ((int64_t)b * g.H + h) * kHeadDim;
    return *reinterpret_cast<const f32x4*>(vm + 16 * dt + 4 * G);
  };

  // ---- Q fragments and the logits of the extras ----
  // A lane holds channels 32 h + 8 G .. + 7 (h = 0, 1) of its query: the four lanes c + 16 G
  // share the channel range.  Everything is requested before anything is used, and one lane per
  // query works out whether that was dropped: with a tile's loads behind the previous tile's
  // arithmetic, and every lane dividing for each of its tiles, a workgroup spent 14 us here before its
  // first key in a layer of 10 frames (now 8.5; 363 us a call instead of 370), 3.8 in one of two frames of
  // 16x16 (2.6; 14.5 instead of 15.1).
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
    for (int j = 0; j < kJ; ++j)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
        w.Qf[qb][2 * j + hh].u = *reinterpret_cast<const u32x4*>(p.Q + row_base(qb, j) + hh * 32 + G * 8);
  uint64_t drop_mask = 0;  // bit i: query q_wave + i was dropped
  if (use_diag) {
    const int64_t q = q_wave + lane;
    bool d = false;
    if (lane < kWaveQ && q < q_end)
      d = kbits ? ((kbits[q >> 5] >> (q & 31)) & 1u) == 0u : (bool)token_is_dropped(g, q);
    drop_mask = __builtin_amdgcn_ballot_w64(d);
  }
  // the query's own key and value, the mean pair (general path: the values only once the row's
  // reference is known, its registers being scarcer)
  u32x4 own_k[kQB][kJ][2];
  u32x2 own_v[kQB][kJ][4];
  f32x4 mean_k[4], mean_v[4];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
      dropped[qb][j] = (drop_mask >> (16 * (qb * kJ + j) + c)) & 1u;
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) own_k[qb][j][hh] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) own_v[qb][j][dt] = u32x2{0u, 0u};
      if (kExtras && dropped[qb][j]) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
          own_k[qb][j][hh] = *reinterpret_cast<const u32x4*>(p.K + row_base(qb, j) + hh * 32 + G * 8);
        if (!kGen) {
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) own_v[qb][j][dt] = load_own_v(qb, j, dt);
        }
      }
    }
  if (kExtras && use_mean) {
    const float* km = p.kmean + ((int64_t)b * g.H + h) * kHeadDim;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mean_k[i] = *reinterpret_cast<const f32x4*>(km + (i >> 1) * 32 + G * 8 + 4 * (i & 1));
      if (!kGen) mean_v[i] = load_mean_v(i);
    }
  }
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const u32x4 raw = w.Qf[qb][2 * j + hh].u;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          w.Qf[qb][2 * j + hh].u[i] =
              pack_bf16(bf16_lo(raw[i]) * p.qscale, bf16_hi(raw[i]) * p.qscale);
      }
      float dot_self = 0.f, dot_mean = 0.f;
      if (use_mean || use_diag) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          float qv[8];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            qv[2 * i] = bf16_lo(w.Qf[qb][2 * j + hh].u[i]);
            qv[2 * i + 1] = bf16_hi(w.Qf[qb][2 * j + hh].u[i]);
          }
          if (use_mean) {
#pragma unroll
            for (int i = 0; i < 4; ++i) dot_mean += qv[i] * mean_k[2 * hh][i] + qv[4 + i] * mean_k[2 * hh + 1][i];
          }
          if (use_diag) {
            const u32x4 kr = own_k[qb][j][hh];
#pragma unroll
            for (int i = 0; i < 4; ++i)
              dot_self += qv[2 * i] * bf16_lo(kr[i]) + qv[2 * i + 1] * bf16_hi(kr[i]);
          }
        }
      }
      dot_self = quad_sum(dot_self);
      dot_mean = quad_sum(dot_mean);
      l_self[qb][j] = dropped[qb][j] ? dot_self : -INFINITY;
      l_mean[qb][j] = use_mean ? dot_mean + p.mean_bias2 : -INFINITY;
    }

  // Initial state = extras weighted by exp2(logit - m0):  O0[d] = w_self v_i[d] + w_mean vmean[d]
  auto init_extras = [&](int qb, int j, float m0) {
    const float w_self = dropped[qb][j] ? fast_exp2(l_self[qb][j] - m0) : 0.f;
    const float w_mean = use_mean ? fast_exp2(l_mean[qb][j] - m0) : 0.f;
    const float l0 = w_self + w_mean;
    if (kGen) w.la[qb][j] = (G == 0) ? l0 : 0.f;  // four lanes split a row's sum
    else w.L[qb][j] = f32x4{l0, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      if (use_mean) acc = (kGen ? load_mean_v(dt) : mean_v[dt]) * w_mean;
      if (dropped[qb][j]) {
        const u32x2 vr = kGen ? load_own_v(qb, j, dt) : own_v[qb][j][dt];
        acc[0] += w_self * bf16_lo(vr[0]);
        acc[1] += w_self * bf16_hi(vr[0]);
        acc[2] += w_self * bf16_lo(vr[1]);
        acc[3] += w_self * bf16_hi(vr[1]);
      }
      w.O[qb][j][dt] = acc;
    }
  };

  if (!kGen) {
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
      for (int j = 0; j < kJ; ++j) {
        w.mref[qb][j] = 0.f;
        init_extras(qb, j, 0.f);
      }
  }
  // general path: the reference is the largest of the extras and of the first 32 keys (row 0
  // always exists); taken when the first tile's K fragments are in registers
  auto first_tile = [&]() {
    if (!kGen) return;
    const int valid0 = ntiles == 1 ? last_valid : kTileRows;
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
#pragma unroll
      for (int j = 0; j < kJ; ++j) w.mref[qb][j] = 0.f;
      f32x4 s[2 * kJ];
      score_unit<kGen, kQB, kJ>(w, qb, s);
      if (valid0 < 32) mask_unit<kJ>(s, 0, valid0, G);
#pragma unroll
      for (int j = 0; j < kJ; ++j) {
        float mx = s[j][0];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[kJ * kt + j][r]);
        mx = quad_max(mx);
        mx = fmaxf(mx, fmaxf(l_self[qb][j], l_mean[qb][j]));
        // a NaN or infinite score cannot serve as reference; the row's result is NaN anyway
        if (!(fabsf(mx) < 3.0e38f)) mx = 0.f;
        w.mref[qb][j] = mx;
        init_extras(qb, j, mx);
      }
    }
  };

  const bool done = key_loop<kSrc, kGen, kSplit, kQB, kJ>(w, lds, votes, src, ntiles, last_valid, tid,
                                                          wave, fa, G, first_tile);
  if (kSplit) {
    // a loop passes one barrier per tile: the shorter one makes up for its missing tile
    if (ntiles < half) lds_barrier();
    __syncthreads();  // both groups are done with their tiles
    // [register][wavefront][lane], over the second group's tiles
    f32x4* over = reinterpret_cast<f32x4*>(tiles + kTileLds) + tid;
    float* over_l = reinterpret_cast<float*>(tiles + kTileLds) + kQB * kJ * 4 * 4 * kAttnThreads + tid;
    static_assert(!kSplit || kQB * kJ * (4 * 16 + 4) * kAttnThreads <= kTileLds * 2, "fits the group's LDS");
    if (group) {
#pragma unroll
      for (int i = 0; i < kQB * kJ; ++i) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) over[(4 * i + dt) * kAttnThreads] = w.O[i / kJ][i % kJ][dt];
        over_l[i * kAttnThreads] = w.L[i / kJ][i % kJ][0];
      }
    }
    __syncthreads();
    if (!group) {
#pragma unroll
      for (int i = 0; i < kQB * kJ; ++i) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) w.O[i / kJ][i % kJ][dt] += over[(4 * i + dt) * kAttnThreads];
        w.L[i / kJ][i % kJ][0] += over_l[i * kAttnThreads];
      }
    }
  }
  float l_fin[kQB][kJ];
  bool unsafe = false;
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
      l_fin[qb][j] = kGen ? quad_sum(w.la[qb][j]) : __shfl(w.L[qb][j][0], c);  // every lane knows its query's
      // a sum outside [2^-90, 2^90] (or NaN): the unreferenced exponentials were not safe
      unsafe = unsafe || (group == 0 && (!(l_fin[qb][j] < kSumHi) || !(l_fin[qb][j] > kSumLo)));
    }
  if (!kGen) {
    if (!done) return false;  // uniform: decided by a workgroup-wide vote inside the loop
    if (vote(unsafe, votes + kWaves, wave, lane, group == 0)) return false;
  }

  // ---- normalise and store ----
  // A lane holds four consecutive channels of one query per accumulator tile: stored from there,
  // every instruction would scatter 8-byte pieces over 16 rows that lie 2*H*64 bytes apart.
  // Each wavefront instead turns its tile, a query block at a time, through a private part of the
  // (now idle) K/V LDS and writes whole 128-byte (query, head) rows, eight per instruction.
  // every wavefront is done with the K/V tiles (fast path: the vote's barrier has seen to that)
  if (kGen) __syncthreads();
  if (group) return true;
  // (The thread number is made opaque here, so that this part's lane numbers and addresses are worked
  // out again: held across the key loop they take 6 to 14 registers more, and the narrow index-driven
  // kernels have none left.)
  int here = tid;
  asm volatile("" : "+v"(here));
  const int elane = here & 63, ec = here & 15, eG = elane >> 4;
  uint16_t* epi = smem + wave * (16 * kJ * kEpiStride);
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    const int64_t q0 = q_wave + qb * kJ * 16;
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
      const float l = l_fin[qb][j];
      const float inv = 1.0f / l;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const int d0 = 16 * dt + 4 * eG;
        u32x2 o2;
        o2[0] = pack_bf16(w.O[qb][j][dt][0] * inv, w.O[qb][j][dt][1] * inv);
        o2[1] = pack_bf16(w.O[qb][j][dt][2] * inv, w.O[qb][j][dt][3] * inv);
        *reinterpret_cast<u32x2*>(epi + (16 * j + ec) * kEpiStride + d0) = o2;
      }
      if (p.lse && eG == 0 && q0 + 16 * j + ec < q_end)
        p.lse[((int64_t)b * g.H + h) * g.NQ + q0 + 16 * j + ec] =
            ((kGen ? w.mref[qb][j] : 0.f) + log2f(l)) * kLn2;
    }
    // the wavefront's own writes, read back by other lanes of the same wavefront
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
#pragma unroll
    for (int i = 0; i < 2 * kJ; ++i) {
      const int row = i * 8 + (elane >> 3);
      const int64_t q = q0 + row;
      const u32x4 o4 = *reinterpret_cast<const u32x4*>(epi + row * kEpiStride + (elane & 7) * 8);
      if (q < q_end)
        *reinterpret_cast<u32x4*>(p.O + (((int64_t)b * g.NQ + q) * g.H + h) * kHeadDim +
                                  (elane & 7) * 8) = o4;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  }
  return true;
}

// position in a launch list of n tiles per pair -> (pair, tile of the pair).  Consecutive ids go
// to consecutive XCDs.  Whole pairs are dealt out one per XCD, so that an XCD streams one
// key/value set at a time through its own L2; the npairs % 8 pairs that are left share the XCDs
// between them, each XCD taking an equal, contiguous run of their tiles.  (Dealing those out whole
// as well left XCDs idle: ordinary attention over 24 frames of 28x37 patches with 12 heads took
// 2.12 ms, with the shared run 1.52.)
struct TileList {
  int n;         // tiles per pair
  int whole;     // tiles of an XCD's whole pairs
  int rest;      // tiles of an XCD's run over the remaining pairs
  int groups;    // workgroups of the list
};
__host__ __device__ inline TileList tile_list(int npairs, int n) {
  TileList l;
  l.n = n;
  l.whole = npairs / kXcds * n;
  l.rest = (npairs % kXcds * n + kXcds - 1) / kXcds;
  l.groups = kXcds * (l.whole + l.rest);
  return l;
}
__device__ __forceinline__ bool list_tile(const TileList& l, int npairs, int bid, int& pair, int& i) {
  const int xcd = bid % kXcds;
  const int seq = bid / kXcds;
  if (seq < l.whole) {
    pair = (seq / l.n) * kXcds + xcd;
    i = seq % l.n;
  } else {
    const int u = seq - l.whole + xcd * l.rest;
    if (u >= npairs % kXcds * l.n) return false;  // uniform for the whole workgroup
    pair = npairs / kXcds * kXcds + u / l.n;
    i = u % l.n;
  }
  return true;
}
__host__ __device__ inline TileList first_list(const TilePlan& t, int npairs) {
  return tile_list(npairs, t.n_full + (t.tails_last ? 0 : t.n_tail));
}
__host__ __device__ inline TileList second_list(const TilePlan& t, int npairs) {
  return tile_list(npairs, t.tails_last ? t.n_tail : 0);
}

// What a workgroup does: queries q_begin .. q_end - 1 of batch element b, head h.
struct Work {
  int b, h;
  int64_t q_begin, q_end;
  bool tail;
};
__device__ __forceinline__ bool workgroup_work(const AttnArgs& p, Work& w) {
  const TilePlan& t = p.plan;
  const TileList first = first_list(t, p.npairs);
  int pair, i;
  if ((int)blockIdx.x < first.groups) {
    if (!list_tile(first, p.npairs, blockIdx.x, pair, i)) return false;
  } else {
    if (!list_tile(second_list(t, p.npairs), p.npairs, blockIdx.x - first.groups, pair, i)) return false;
    i += t.n_full;
  }
  w.b = pair / p.g.H;
  w.h = pair % p.g.H;
  w.tail = i >= t.n_full;
  w.q_begin = w.tail ? (int64_t)t.n_full * kQTile + (int64_t)(i - t.n_full) * t.tail_q
                     : (int64_t)i * kQTile;
  w.q_end = min(p.g.NQ, w.q_begin + (w.tail ? t.tail_q : kQTile));
  return true;
}

// A workgroup whose fast pass failed leaves this pattern (four bf16 NaNs with distinct payloads)
// in the first four channels of its first output row and stores nothing else; the second kernel
// redoes exactly the workgroups that carry it.  Should a correct result ever equal the pattern,
// the second kernel recomputes that workgroup, which is harmless.
constexpr uint64_t kRedoMark = 0x7F997FC37FA57FC1ull;

__device__ __forceinline__ uint64_t* redo_slot(const AttnArgs& p, const Work& w) {
  return reinterpret_cast<uint64_t*>(p.O + (((int64_t)w.b * p.g.NQ + w.q_begin) * p.g.H + w.h) * kHeadDim);
}

// The kernel's arguments (its only parameter, at the start of its argument memory), to be read again
// from here on: what one path derives from them is then not held for another.
__device__ __forceinline__ const AttnArgs& args_again() {
  typedef const __attribute__((address_space(4))) AttnArgs* KernelArgs;
  KernelArgs args = (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  return *(const AttnArgs*)args;
}

// blocks (of one 16-query tile) of a narrow workgroup's wavefront
constexpr int tail_blocks(int tail_q) { return tail_q == 192 ? 3 : 2; }

// kTailQ: queries of the launch's narrow workgroups (0: it has none).
// kRedo: a workgroup redoes its own rows by the general path, 128 queries at a time, instead of
// leaving the mark for a second launch.  At that width the general path needs no more registers
// than the fast one, provided that nothing is held for it meanwhile: it starts from an opaque
// thread number (attend) and reads the kernel's arguments again.  So no instance spills, which a
// build test checks, and each uses within 2 registers what it uses without kRedo (234 to 248).  Sharing
// both with the fast path spills 4 registers (compacted), 14 (rows) and 25 (indexed) at full width.
template <int kSrc, int kTailQ, bool kRedo>
__global__ __launch_bounds__(kAttnThreads, kBlocksPerCu) void sga_attn_kernel(AttnArgs p) {
  __shared__ __align__(16) uint16_t tiles[kTileLds];
  __shared__ __align__(16) uint32_t votes[kVoteWords];
  Work w;
  if (!workgroup_work(p, w)) return;
  bool done;
  if (kTailQ != 0 && w.tail)
    done = attend<kSrc, false, tail_blocks(kTailQ), 1>(p, tiles, votes, w.b, w.h, w.q_begin, w.q_end);
  else
    done = attend<kSrc, false, 2, 2>(p, tiles, votes, w.b, w.h, w.q_begin, w.q_end);
  if (done) return;
  if (!kRedo) {
    if (threadIdx.x == 0) *redo_slot(p, w) = kRedoMark;
    return;
  }
  const AttnArgs& again = args_again();
#pragma unroll 1
  for (int64_t q = w.q_begin; q < w.q_end; q += kWaves * wave_queries(2, 1)) {
    __syncthreads();  // the LDS is free
    attend<kSrc, true, 2, 1>(again, tiles, votes, w.b, w.h, q, min(w.q_end, q + kWaves * wave_queries(2, 1)));
  }
}

// A launch of few workgroups: 128 queries each, eight wavefronts.  Rows that leave the fast path's
// range are redone here by the general path, which at this width needs no more registers: an idle
// second launch would be a fifth of a small call's time.
template <int kSrc>
__global__ __launch_bounds__(2 * kAttnThreads, 2) void sga_attn_split_kernel(AttnArgs p) {
  __shared__ __align__(16) uint16_t tiles[2 * kTileLds];
  __shared__ __align__(16) uint32_t votes[kVoteWords];
  Work w;
  if (!workgroup_work(p, w)) return;
  if (attend<kSrc, false, 2, 1, kSplitKeys>(p, tiles, votes, w.b, w.h, w.q_begin, w.q_end)) return;
  __syncthreads();
  attend<kSrc, true, 2, 1, kTwin>(p, tiles, votes, w.b, w.h, w.q_begin, w.q_end);
}

// The general path is a kernel of its own, launched behind the first on the same stream: it is
// rarely needed, starts over from the workgroup's inputs, and this way does not weigh on the
// register allocation of the fast path.  Workgroups without the mark leave at once; narrow ones are
// redone at their own width.  (At full width, with the queries beyond their own left out, calls of
// which every workgroup is redone took, us, then / now, and with full-width workgroups alone in both
// launches: ordinary attention, 12 frames of 37x37 2013 / 1610, 1835; 10 frames of 28x37, 8 heads
// 398 / 301, 398; compacted, 25 frames 2927 / 2739, 2990.)
template <int kSrc, int kTailQ>
__global__ __launch_bounds__(kAttnThreads, kBlocksPerCu) void sga_attn_general_kernel(AttnArgs p) {
  __shared__ __align__(16) uint16_t tiles[kTileLds];
  __shared__ __align__(16) uint32_t votes[kVoteWords];
  Work w;
  if (!workgroup_work(p, w)) return;
  if (*redo_slot(p, w) != kRedoMark) return;  // same value in every lane
  __syncthreads();  // every wavefront has read the mark before any of them overwrites it
  if (kTailQ != 0 && w.tail)
    attend<kSrc, true, tail_blocks(kTailQ), 1>(args_again(), tiles, votes, w.b, w.h, w.q_begin, w.q_end);
  else
    attend<kSrc, true, 2, 2>(p, tiles, votes, w.b, w.h, w.q_begin, w.q_end);
}

template <int kSrc, int kTailQ>
static void launch_both(const AttnArgs& p, dim3 grid, hipStream_t st) {
  const dim3 block(kAttnThreads);
  if (redo_in_place(p.g.M_pad / kTileRows)) {
    hipLaunchKernelGGL((sga_attn_kernel<kSrc, kTailQ, true>), grid, block, 0, st, p);
  } else {
    hipLaunchKernelGGL((sga_attn_kernel<kSrc, kTailQ, false>), grid, block, 0, st, p);
    hipLaunchKernelGGL((sga_attn_general_kernel<kSrc, kTailQ>), grid, block, 0, st, p);
  }
}

template <int kSrc>
static void launch_source(const AttnArgs& p, hipStream_t st) {
  const dim3 grid((unsigned)(first_list(p.plan, p.npairs).groups + second_list(p.plan, p.npairs).groups));
  const int tail_q = p.plan.n_tail ? p.plan.tail_q : 0;
  if (p.plan.split) hipLaunchKernelGGL(sga_attn_split_kernel<kSrc>, grid, dim3(2 * kAttnThreads), 0, st, p);
  else if (tail_q == 0) launch_both<kSrc, 0>(p, grid, st);
  else if (tail_q == 192) launch_both<kSrc, 192>(p, grid, st);
  else launch_both<kSrc, 128>(p, grid, st);
}

hipError_t launch_attn(const Geom& g, uint32_t flags, float scale, float mean_bias, const void* Q,
                       const void* K, const void* V, const void* Kc, const void* Vc,
                       const float* kmean, const float* vmean, void* O, float* lse, hipStream_t st,
                       const uint32_t* kept_bits, const int32_t* nd_dev, int src_mode,
                       const int32_t* list, int64_t list_stride) {
  const int npairs = g.B * g.H;
  // the bound on the grid, with whole pairs per XCD throughout (narrow workgroups: plan_tiles)
  if ((int64_t)((npairs + kXcds - 1) / kXcds) * kXcds * ((g.NQ + kQTile - 1) / kQTile) > 0x7FFFFFFF)
    return hipErrorInvalidConfiguration;
  // indexed rows are addressed with 32-bit byte offsets from the (batch, head) base, formed by
  // a 24-bit multiplication of token id and row length
  if (src_mode == kSrcIndexed && ((uint64_t)g.NQ * g.H * (kHeadDim * 2) > 0xFFFFFFFFull ||
                                  g.NQ > 0xFFFFFF || (uint64_t)g.H * (kHeadDim * 2) > 0xFFFFFF))
    return hipErrorInvalidValue;
  (void)hipGetLastError();  // drop any stale error so the check below is this launch's
  AttnArgs p;
  p.g = g;
  p.flags = flags;
  p.qscale = scale * kLog2e;
  p.mean_bias2 = mean_bias * kLog2e;
  p.Q = (const uint16_t*)Q;
  p.K = (const uint16_t*)K;
  p.V = (const uint16_t*)V;
  p.Kc = (const uint16_t*)Kc;
  p.Vc = (const uint16_t*)Vc;
  p.kmean = kmean;
  p.vmean = vmean;
  p.O = (uint16_t*)O;
  p.lse = lse;
  p.npairs = npairs;
  p.plan = plan_tiles(g.NQ, npairs, g.M_pad / kTileRows);
  p.kept_bits = kept_bits;
  p.nd_dev = nd_dev;
  p.list = list;
  p.list_stride = list_stride;
  if (src_mode == kSrcCompact) launch_source<kSrcCompact>(p, st);
  else if (src_mode == kSrcRows) launch_source<kSrcRows>(p, st);
  else launch_source<kSrcIndexed>(p, st);
  return hipGetLastError();
}

}  // namespace agg
