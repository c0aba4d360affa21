// prefill_attn_kernels.hip -- sink + window causal attention of one prefill
// chunk on bf16 or binary16 MFMA (gfx950).
//
// Query token t of the chunk [p0, p1), query head q of KV head h = q / G,
// attends over R(t + 1) restricted to [0, t]: positions s <= t with s < S or
// s >= t + 1 - w (every s <= t for a full unit) -- the windowed attention of
// the paper's conditional attention equations with the sink prefix of its
// StreamingLLM control.  Keys below p0 come from the cache as it stands
// before the chunk is materialised (sinks, plus the ring for a finite unit,
// whose residency at length p0 covers every s >= p0 + 1 - w); keys in
// [p0, t] come from the chunk's own K/V.
//
// The calibration replay (replay_attn, below) uses the same tiles, operand
// layouts and softmax on a traced history, for every candidate in one pass.
//
// Formulation.  A workgroup owns one KV head and 32 * NW consecutive
// (token, q-head) columns of that head (column c = token * G + g), one
// 32-column block per wavefront.  Per block of 32 key positions it computes
//     S^T = K Q^T           (v_mfma_f32_32x32x16_bf16, K from LDS, Q^T held
//                            in registers for the whole kernel)
//     O^T += V^T P^T        (V^T from LDS by transposing reads, P^T straight
//                            from the S^T accumulator registers)
// In the 32x32 accumulator layout a lane owns one column and 16 key rows, so
// the softmax max and sum are in-lane plus one swap between the two lane
// halves.  The P^T operand needs 8 keys per lane in MFMA k order; instead of
// moving P, the keys of each 16-key step are permuted (k index 8*half + j is
// key 16*step + 8*(j/4) + 4*half + j%4, exactly the rows a lane already
// holds), and the V^T operand is read in that key order.
//
// Schedule (prefill_attn).  A tile is two such blocks (one at head_dim 256),
// and a wavefront's tile takes two phases: the products -- S^T of tile i
// alternating with V^T P^T of tile i - 1 -- and the softmax of tile i.  The
// eight wavefronts are two groups, one of each on every SIMD, that run the
// phases in turn, a barrier apart: while one keeps the matrix cores busy the
// other has the vector ALU.  (With every wavefront in the same phase, as the
// barrier per tile of a plain loop leaves them, the two units take turns.)
// Measured on one chip, before -> after, 8K tokens at 120K of context, head_dim
// 256, windows {2K, 8K, 32K, full}: 7.34 -> 6.89 ms, 1,168 -> 1,245 TFLOP/s (7.06 to
// 7.34 -> 6.64 to 7.07 over several; the matrix cores busy 0.575 -> 0.667 of 14.2 ->
// 12.3 million cycles, at a clock that falls with the load); 4K tokens at 12K,
// head_dim 64, binary16: 508 -> 319 us, bound by the exponentials and the
// arithmetic around them.  The softmax phase also
// issues the loads of tile i + 2 into the fourth stage of LDS; tile addresses
// are kept as runs (issue_loads), since a lane's address worked out per tile
// cost as much as a third of the softmax.
//
// Split keys.  A launch of few column blocks (a short chunk over a long
// context), or with most of its keys in one head, leaves CUs idle: the host
// then splits the key tiles of every block over several workgroups
// (tiles_per_split), whose partials prefill_merge adds up.  512 tokens at 48K
// of context, head_dim 128: 1,718 -> 143 us with both changes (206 by this
// one); 1,999 tokens at 30K over fp8, head_dim 256: 1,451 -> 677 (801).
// A split is made only where it also pays for the merge launch, and where the
// caller gives room for the partials.  The weights are rounded to 16 bits under a
// split's own shift, so a split call's outputs differ from the unsplit one's by up
// to 2e-3 of their norm (bf16), as far from 64-bit results as they (1.7e-3).
//
// Short launches (a few tiles) are bound by the latency of the chain before
// the first tile, its mask and the output: the arguments come in two rounds of
// scalar loads, q and the first two tiles' loads are in flight together, a
// partly visible tile is masked by bits (keep_rows), the rows go out through
// LDS (store_rows; few columns directly), and one to two tiles run without the
// phase shift.  Against a loop without phases a launch of one block of columns
// (8 heads, head_dim 64 / 128 / 256, us in a replayed graph) takes: 16 tokens into an
// empty sequence, group 1, 4.1 / 4.5 / 5.5 -> 5.0 / 5.4 / 6.5; 64 tokens, group 4,
// 6.1 / 9.0 / 15.5 -> 6.6 / 9.5 / 14.7; 256 tokens 11.1 / 15.2 / 24.4 -> 10.5 / 15.0 /
// 22.8; 512 tokens 17.7 / 23.1 / 38.8 -> 15.4 / 20.4 / 33.0.  (Issuing a call takes the
// host 9 us.)  What the shortest lose is the last phase, whose S^T goes unused, a
// second block of keys, and barriers; leaving out the barrier after the softmax
// where the second group has no columns changed nothing.
//
// Data movement.  K and V tiles go from global memory straight into LDS
// (buffer_load_dwordx4 ... lds: lane i of an instruction fills bytes
// [16i, 16i + 16) of the instruction's LDS block; each lane picks its own
// source), in four stages, no staging
// registers.  Both are stored as rows of one 16-byte channel chunk for the 32
// keys of a block (512 B), two rows per load instruction; in odd rows key k sits at
// position k ^ 4.  Lane L of every load then fetches key (L % 32) ^
// (4 (L / 32)) -- one key per lane and tile, so its cache slot and row
// addresses are worked out once per tile -- at chunk 2n + L / 32.
//   K tile: rows contiguous.  The S^T operand (a lane's key, 8 channels of
//           one chunk) is one 16-byte read; a half-wave reads a whole row.
//   V tile: row pairs spaced 1 KiB + 128 B apart.  ds_read_b64_tr_b16 over
//           a 16-lane group turns 4 keys x 16 channels of V into 4 keys of
//           one channel per lane -- the V^T operand.  A half-wave (two
//           16-lane groups: the same 4 keys, adjacent 16-channel pieces)
//           touches four 64-byte pieces that the odd-row swizzle and the pair
//           pad place on disjoint banks of the 256-byte-wide LDS.
// Every operand address is a per-lane base plus a compile-time offset.
// Keys past the tile's range lie past the buffer's span, so they read as zeros
// (and are masked).
//
// Binary16 caches (prefill_attn<.., true>): the same tiles, loads and
// layouts (both formats are 2-byte elements), on v_mfma_f32_32x32x16_f16.
// The keys and values enter as stored; q (bf16) is converted to binary16
// after scaling by a power of two 2^sh common to the wavefront that puts the
// wavefront's largest |q| in [2^14, 2^15), which is exact for every
// component within a factor 2^31 of it, and the logit scale takes 2^-sh back.
// The softmax weights enter the value product as binary16 with a 2^7 bias
// (they are at most 2^8 before it, so at most 2^15 after), which keeps the
// small ones clear of binary16's subnormal range; the running sum carries the
// same bias, so the quotient is unchanged.
//
// Online softmax in base 2 with a lazy rescale: the running shift m only
// moves when a tile's maximum exceeds it by more than 8 (log2 units), so the
// O^T accumulators are rescaled rarely; any shift gives the same quotient
// and terms stay below 2^8.  Tiles no column of a wavefront can see are
// skipped by that wavefront; tiles every column sees whole skip the mask.
#include <type_traits>

#include "hwkv_internal.h"

namespace hwkv {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int kKeys = 32;                  // keys per product block
constexpr int kPipe = 2;                   // operand reads ahead of their products

__device__ __forceinline__ u32x4_t ld16(const uint16_t *p) {
  return *reinterpret_cast<const u32x4_t *>(p);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const f32x2_t f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ uint32_t pack_f16(float lo, float hi) {
  const f32x2_t f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, f16x2_t));
}

// 32x32x16 MFMA on 2-byte operands: binary16 (F16) or bf16
template <bool F16>
__device__ __forceinline__ f32x16_t mfma16(u32x4_t a, u32x4_t b, f32x16_t c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a),
                                                  __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// 16 bytes from global memory into the LDS block of the issuing instruction, at
// a scalar base and unsigned 32-bit byte offsets (lane's and uniform).  The
// descriptor spans kRowSpan bytes, as many as the largest unit's K or V (the bf16
// image of an fp8 unit) has; an access is out of range, and reads as zero, where
// the lane's offset is at or past the span less the uniform offset, so an offset
// past the span always is.
constexpr uint32_t kNoRow = 0xfffff000u;
static_assert(kNoRow >= kRowSpan, "no row lies there");
typedef u32x4_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void *base) {
  const uint64_t u = (uint64_t)base;
  return rsrc_t{(uint32_t)u, (uint32_t)(u >> 32) & 0xffffu, kRowSpan, 0x00020000u};
}
__device__ __forceinline__ const uint8_t *scalar_ptr(const void *p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (const uint8_t *)(((uint64_t)hi << 32) | lo);
}
// The load has no destination register, and the kernel waits for it itself
// (wait_loads, then a barrier).  As a builtin it would make the compiler wait
// for every load in flight before each transposing read of LDS, the next
// tiles' loads among them, which are to stay in flight.
__device__ __forceinline__ void b2lds(rsrc_t r, uint8_t *lds_block, uint32_t voffset,
                                      uint32_t soffset) {
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(
          (uint32_t)(uintptr_t)(lds_void_t *)lds_block),
      "v"(voffset), "s"(r), "s"(soffset)
      : "memory", "m0");
}

// The larger of two numbers, NaN if either is: pairs of these are one
// v_maximum3_f32, where fmaxf first quiets every operand with an instruction
// of its own (a product's result is not known to be a quiet number).
__device__ __forceinline__ float max_of(float x, float y) {
  return __builtin_elementwise_maximum(x, y);
}

// The lane index, worked out where it is used: what follows from it does not
// stay live in vector registers between uses.
__device__ __forceinline__ int lane_now() {
  int x = threadIdx.x & 63;
  asm volatile("" : "+v"(x));
  return x;
}

// no instruction moves across this point
__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }

// at most LEFT vector loads of the wave are still in flight
template <int LEFT = 0>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(LEFT) : "memory");
}

// -inf for the logits of a block whose bit is clear: row r of st holds key e +
// cr of the lane, cr = 8 (r / 4) + r % 4, and word has bit cr for it.  Two
// instructions a logit (a comparison for each bound takes three to eight).
__device__ __forceinline__ void keep_rows(f32x16_t &st, uint32_t word) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t keep =
        (uint32_t)__builtin_amdgcn_sbfe((int)word, (r >> 2) * 8 + (r & 3), 1);
    const float x = st[r];
    st[r] = __builtin_bit_cast(float,
                               (__builtin_bit_cast(uint32_t, x) & keep) | (0xff800000u & ~keep));
  }
}

// x / G, inv = 2^24 / G + 1, for x < G + 255 (a block's columns, from its first
// token's first): exact, since x * inv < 2^32 and its error, at most x G, stays
// below 2^24.  A division takes some hundred cycles, and a launch of one tile
// waits for six of them.
__device__ __forceinline__ int token_of(int x, uint32_t inv) {
  return (int)(((uint32_t)x * inv) >> 24);
}

// bits [0, x), for x of any value; bit 31 stays clear
__device__ __forceinline__ uint32_t below(int x) { return (1u << min(max(x, 0), 31)) - 1; }

// LDS accesses of a wave's lanes stay in order across this point
__device__ __forceinline__ void wave_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// x of lane l and x of lane l ^ 32 in both lanes (VALU lane swap)
__device__ __forceinline__ void halves(float x, float *a, float *b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, x),
                                                  __builtin_bit_cast(int, x), false, false);
  *a = __builtin_bit_cast(float, (int)r[0]);      // x of the lower-half lane
  *b = __builtin_bit_cast(float, (int)r[1]);      // x of the upper-half lane
}


template <int D, int NW>
struct Prefill {
  static constexpr int DC = D / 8;                 // 16-byte channel chunks
  static constexpr int KS = D / 16;                // k-steps of S^T
  static constexpr int DB = D / 32;                // 32-channel blocks of O^T
  static constexpr int NINST = DC / 2;             // loads per tile (K or V), 2 rows each
  static constexpr int KBYTES = NINST * 1024;      // K tile
  static constexpr int VPAIR = 1024 + 128;         // bytes per V row pair (padded)
  static constexpr int VBYTES = NINST * VPAIR;     // V tile
  static constexpr int STAGE = KBYTES + VBYTES;
  static constexpr int IPW = (NINST + NW - 1) / NW;   // per wave and tile, each of K, V
};

// The V^T operand of 16-key step s of a block at 32-channel block db (vl: the
// block's V with the lane's offset).
template <typename P>
__device__ __forceinline__ u32x4_t read_values(const uint8_t *vl, int s, int db) {
  i16x4_t v2[2];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
    v2[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4_t *)(vl + 2 * db * P::VPAIR + (16 * s + 8 * hh) * 16));
  return __builtin_bit_cast(u32x4_t,
                            __builtin_shufflevector(v2[0], v2[1], 0, 1, 2, 3, 4, 5, 6, 7));
}

// The products of a phase: S^T of a tile of U blocks of 32 keys (K at kl) and,
// if VALUES, O^T += V^T P^T of the one before it (its blocks' V at vl and vl1; 16
// keys a step, two steps a block).  They alternate, and so do the blocks of S^T: a product that
// adds to the one before it would wait out that one's latency.  The order of
// operand reads and products is pinned, reads kPipe products of their kind
// ahead: left to itself the scheduler reads each operand just before its
// product and waits out the LDS latency every time.
template <int D, int NW, bool F16, int U, bool VALUES>
__device__ __forceinline__ void tile_products(f32x16_t (&o)[D / 32], f32x16_t (&st)[U],
                                              const u32x4_t (&pb)[2 * U], const u32x4_t (&qv)[D / 16],
                                              const uint8_t *kl, const uint8_t *vl,
                                              const uint8_t *vl1) {
  using P = Prefill<D, NW>;
  constexpr int KS = P::KS, DB = P::DB;
  constexpr int N = U * KS;                      // products of each kind
  static_assert(N == 2 * U * DB, "as many products of both kinds");
  constexpr int A = VALUES ? kPipe : 2 * kPipe;
  u32x4_t kx[A], va[A];
  auto read_k = [&](int i) {
    kx[i % A] = *reinterpret_cast<const u32x4_t *>(kl + (i % U) * P::STAGE + (i / U) * 1024);
  };
  auto read_v = [&](int i) {
    const int s = i / DB, db = i % DB;
    va[i % A] = read_values<P>(s / 2 == 0 ? vl : vl1, s % 2, db);
  };
#pragma unroll
  for (int i = 0; i < A; ++i) {
    read_k(i);
    if constexpr (VALUES) read_v(i);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i < U)
#pragma unroll
      for (int r = 0; r < 16; ++r) st[i % U][r] = 0.0f;
    pin();
    st[i % U] = mfma16<F16>(kx[i % A], qv[i / U], st[i % U]);
    pin();
    if (i + A < N) read_k(i + A);
    if constexpr (VALUES) {
      pin();
      o[i % DB] = mfma16<F16>(va[i % A], pb[i / DB], o[i % DB]);
      pin();
      if (i + A < N) read_v(i + A);
    }
  }
  pin();
}

// The weights 2^(st c2 - mc) of a tile, packed for the value product, and their
// sum added to l.  Every weight comes before the sums and the packing, which
// would otherwise each wait for its exponential.
template <int U, bool F16>
__device__ __forceinline__ void tile_weights(f32x16_t (&st)[U], u32x4_t (&pb)[2 * U], float &l,
                                             float c2, float mc) {
#pragma unroll
  for (int r = 0; r < 16 * U; ++r)
    st[r / 16][r % 16] = __builtin_fmaf(st[r / 16][r % 16], c2, -mc);
  pin();
#pragma unroll
  for (int r = 0; r < 16 * U; ++r) st[r / 16][r % 16] = __builtin_amdgcn_exp2f(st[r / 16][r % 16]);
  pin();
  float ls[4] = {l, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int r = 0; r < 16 * U; r += 2) {
    const float w0 = st[r / 16][r % 16], w1 = st[r / 16][r % 16 + 1];
    ls[r % 4] += w0;
    ls[r % 4 + 1] += w1;
    pb[r / 8][r % 8 / 2] = F16 ? pack_f16(w0, w1) : pack_bf16(w0, w1);
  }
  l = (ls[0] + ls[1]) + (ls[2] + ls[3]);
}

// The largest of a tile's logits, in both lanes of a column.
template <int U>
__device__ __forceinline__ float tile_max(const f32x16_t (&st)[U]) {
  float mx = max_of(st[0][0], st[0][1]), lo, hi;
#pragma unroll
  for (int r = 2; r < 16 * U; r += 2)
    mx = max_of(max_of(mx, st[r / 16][r % 16]), st[r / 16][r % 16 + 1]);
  halves(mx, &lo, &hi);
  return max_of(lo, hi);
}

// Writes a wave's columns, O^T times inv, as rows of D floats: column c's row
// (in the lane c and c + 32) at dst + row * stride, for columns up to last.
// Through LDS (area: 128 CH bytes of the wave's own): a lane holds 4
// channels in 8 of its column, and written from there an instruction would
// touch 32 rows, 32 bytes each; a workgroup's rows took 5,000 cycles at
// head_dim 128.  CH channels a pass, 16-byte chunks swizzled by the column.
template <int D, int CH>
__device__ __forceinline__ void store_rows(const f32x16_t (&o)[D / 32], float inv, float *dst,
                                           int stride, uint32_t row, int last, uint8_t *area) {
  constexpr int NC = CH / 4, RPI = 64 / NC;
  const int ln = lane_now();
  auto at = [&](int col, int chunk) {
    return reinterpret_cast<float4 *>(area + (col * NC + (chunk ^ (col & (NC - 1)))) * 16);
  };
#pragma unroll
  for (int p = 0; p < D / CH; ++p) {
#pragma unroll
    for (int x = 0; x < NC / 2; ++x) {             // chunk 2x + half of the pass
      const int db = (p * CH + 8 * x) / 32, rq = (p * CH + 8 * x) / 8 % 4;
      *at(ln & 31, 2 * x + (ln >> 5)) =
          make_float4(o[db][4 * rq + 0] * inv, o[db][4 * rq + 1] * inv, o[db][4 * rq + 2] * inv,
                      o[db][4 * rq + 3] * inv);
    }
    wave_order();
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
      const int col = i * RPI + ln / NC, chunk = ln % NC;
      const float4 v = *at(col, chunk);
      const uint32_t rw = (uint32_t)__shfl((int)row, col);
      if (col <= last)
        *reinterpret_cast<float4 *>(dst + (size_t)rw * stride + p * CH + chunk * 4) = v;
    }
    wave_order();
  }
}

// Every wave's LDS reads are done, and the loads it waited for are in LDS.
__device__ __forceinline__ void phase_end() {
  asm volatile("" ::: "memory");
  pin();
  __builtin_amdgcn_s_barrier();
  pin();
  asm volatile("" ::: "memory");
}

template <int D, int NW, bool F16>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
void prefill_attn(const PrefillAttnArgs a) {
  using P = Prefill<D, NW>;
  constexpr int KS = P::KS, DB = P::DB;
  constexpr int KT = prefill_keys(D);               // keys per tile
  constexpr int U = KT / kKeys;                     // blocks of 32 keys per tile
  constexpr int NH = NW / U;                        // waves loading each block
  constexpr int IPW = P::NINST / NH;                // loads per wave and tile, each of K, V
  constexpr int STAGES = 4;
  static_assert(NW == 8 && P::NINST % NH == 0, "two groups of waves; tile loads");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[STAGES * U * P::STAGE];

  // Every argument that does not depend on the head, in one round of scalar
  // loads; then the head's.
  asm volatile("" ::"s"(a.cache), "s"(a.page_table), "s"(a.pool_off), "s"(a.q), "s"(a.k), "s"(a.v),
               "s"(a.p0), "s"(a.n_tokens), "s"(a.n_kv_heads), "s"(a.group), "s"(a.n_sinks),
               "s"(a.n_col_blocks), "s"(a.scale_log2), "s"(a.split), "s"(a.tiles_per_split), "s"(a.group_inv));
  const int nb = a.n_col_blocks;
  const int blk = blockIdx.x;
  // The head: heads have nb workgroups each, or where keys are split the head
  // is the number of those that begin at or before this workgroup.
  int rank;
  if (a.split)
    rank = __builtin_amdgcn_readfirstlane(
        __popcll(__ballot(a.head[threadIdx.x & 63].wg_begin <= blk)) - 1);
  else
    rank = blk / nb;
  const PrefillAttnHead &hd = a.head[rank];
  asm volatile("" ::"s"(hd.k_off), "s"(hd.v_off), "s"(hd.window), "s"(hd.pto), "s"(hd.k_scale),
               "s"(hd.v_scale), "s"(hd.h), "s"(hd.wg_begin));
  const int h = hd.h, pto = hd.pto;
  const int run0 = blk - hd.wg_begin;
  const int split = a.split ? run0 / nb : 0;
  const int cb = nb - 1 - (run0 - split * nb);      // later tokens first
  const int G = a.group;
  const int Hq = a.n_kv_heads * G;
  const int ncols = a.n_tokens * G;
  const int c_first = cb * 32 * NW;
  const int c_last = min(c_first + 32 * NW, ncols) - 1;
  // positions and slots fit in 32 bits (max_ctx < 2^24).  Query row r sits
  // at position p0 + r.
  const int p0 = a.p0;
  auto pos = [&](int r) -> int { return p0 + r; };
  const int S = a.n_sinks;
  const int W = hd.window;                          // 0 = full
  // A column's token: one division for the block's first column, the others
  // from there by the reciprocal (exact: token_of).
  const int t0 = c_first / G, r0 = c_first - t0 * G;
  auto token = [&](int c) -> int { return t0 + token_of(r0 + c - c_first, a.group_inv); };
  const int ta = pos(t0), tb = pos(token(c_last));

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // uniform across the wavefront: keeps the per-wave tile tests and the LDS
  // block of every load in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, cl = lane & 31;

  // this wavefront's columns and this lane's column
  const int wc0 = c_first + 32 * wave;
  const bool wave_live = wc0 <= c_last;
  const int wc_last = min(wc0 + 31, c_last);
  const int t_lo = pos(token(min(wc0, c_last))), t_hi = pos(token(wc_last));
  const int cc = min(wc0 + cl, c_last);
  const int tl = token(cc), g = cc - tl * G;
  const size_t q_row = ((size_t)tl * Hq + (size_t)h * G + g) * D;

  // key ranges: [0, ra1) then [rb0, rb1)
  const int lo = (W == 0) ? 0 : max(0, ta + 1 - W);
  int ra1, rb0 = 0, rb1 = 0;
  if (lo <= S) {
    ra1 = tb + 1;
  } else {
    ra1 = S;
    rb0 = lo;
    rb1 = tb + 1;
  }
  const int na = (ra1 + KT - 1) / KT;
  const int ntiles = na + (rb1 - rb0 + KT - 1) / KT;   // prefill_tiles(ta, tb, S, W)
  // this split's tiles (uniform; a shorter block has fewer splits)
  const int i_lo = split * a.tiles_per_split;
  if (i_lo >= ntiles) return;
  const int n_it = min(ntiles - i_lo, a.tiles_per_split);

  u32x4_t qv[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qv[ks] = ld16(a.q + q_row + 16 * ks + 8 * half);   // past the last column: its copy

  const uint16_t *kc = a.cache + hd.k_off;
  const uint16_t *vc = a.cache + hd.v_off;
  const size_t in_stride = (size_t)a.n_kv_heads * D;
  const uint16_t *kin = a.k + (size_t)h * D;
  const uint16_t *vin = a.v + (size_t)h * D;

  auto tile_range = [na, ra1, rb0, rb1](int i, int *s0, int *se) {
    const bool first = i < na;
    *s0 = first ? i * KT : rb0 + (i - na) * KT;
    *se = first ? ra1 : rb1;
  };

  // Wave w loads block w % U of every tile; lkey is the key of the block this
  // lane loads.
  const int lblk = wave % U, ln = wave / U;
  // Tile loads go by runs: consecutive tiles whose keys follow one another in
  // the chunk's rows or in cache slots, so that a tile costs two additions to
  // scalar bases.  K and V bases of the next tile of the run, their steps to
  // the tile after it (K steps alternate between kstep and kper - kstep: a
  // 32-key tile is half a 64-slot K tile), the lane's byte offsets (of even and
  // odd tiles for K) and the bytes from one load's K rows to the next's.
  int run = 0;                                      // tiles left in the run
  const uint8_t *run_k = nullptr, *run_v = nullptr;
  int kstep = 0, kper = 0, vstep = 0, kn = 0;
  int ko = 0, ko2 = 0, vo = 0;
  constexpr int TB = kTile * D * 2;                 // bytes of a K tile
  auto put = [&](const uint8_t *kb, const uint8_t *vb, uint32_t ko, uint32_t vo, int kn, uint8_t *stage) {
    const rsrc_t kr = make_rsrc(scalar_ptr(kb)), vr = make_rsrc(scalar_ptr(vb));
    kn = __builtin_amdgcn_readfirstlane(kn);
    uint8_t *kl = stage + lblk * P::STAGE + ln * 1024;
    uint8_t *vl = stage + lblk * P::STAGE + P::KBYTES + ln * P::VPAIR;
#pragma unroll
    for (int j = 0; j < IPW; ++j) {                 // chunk rows 2n, 2n + 1, n = ln + j NH
      b2lds(kr, kl + j * NH * 1024, ko, (ln + j * NH) * kn);
      b2lds(vr, vl + j * NH * P::VPAIR, vo, (ln + j * NH) * 32);
    }
  };
  const uint8_t *const kcb = reinterpret_cast<const uint8_t *>(kc);
  const uint8_t *const vcb = reinterpret_cast<const uint8_t *>(vc);
  // the page of position s0 of a paged unit (scalar loads: the table does not
  // change under the kernel)
  auto page_of = [&](int s0) -> const uint8_t * {
    const int pg = ((const __attribute__((address_space(4))) int32_t *)
                        a.page_table)[__builtin_amdgcn_readfirstlane(pto + (s0 >> 8))];
    return reinterpret_cast<const uint8_t *>(a.cache + a.pool_off + (int64_t)pg * 2 * kPageTokens * D);
  };
  auto issue_loads = [&](int it, uint8_t *stage) {
    if (run == 0) {
      const int half = lane_now() >> 5, lkey = (lane_now() & 31) ^ (4 * half);
      int s0, se;
      tile_range(i_lo + it, &s0, &se);
      s0 += kKeys * lblk;                           // the block's first key
      const int ce = min(p0, se);                   // keys [s0, ce) are cached
      int sl0 = s0, len = 0;                        // first slot and slots in a row
      const uint8_t *kb = kcb, *vb = vcb;
      if (s0 >= p0) {
        len = se - s0;
      } else if (W == 0) {
        len = ce - s0;
        if (pto >= 0) {
          kb = page_of(s0);
          vb = kb + kPageTokens * D * 2;
          sl0 = s0 & (kPageTokens - 1);
          len = min(len, kPageTokens - sl0);
        }
      } else if (s0 >= S) {
        const int rb = (s0 - S) % W;
        sl0 = S + rb;
        len = min(ce - s0, W - rb);
      }
      if (len >= kKeys) {
        run = __builtin_amdgcn_readfirstlane((len - kKeys) / KT + 1);
        if (s0 >= p0) {
          const size_t at = (size_t)(s0 - p0) * in_stride;
          run_k = scalar_ptr(kin + at);
          run_v = scalar_ptr(vin + at);
          vstep = kstep = __builtin_amdgcn_readfirstlane(KT * (int)in_stride * 2);
          kper = 2 * kstep;
          ko = ko2 = vo = lkey * (int)in_stride * 2 + half * 16;
          kn = 32;
        } else {
          // slots sl0 + lkey: K tile and slot within it by the lane, tiles
          // 64 slots apart
          run_k = scalar_ptr(kb + (size_t)(sl0 >> 6) * TB);
          run_v = scalar_ptr(vb + (size_t)sl0 * (D * 2));
          const int x = (sl0 & 63) + lkey, y = x + (KT & 63);
          ko = (x >> 6) * TB + (x & 63) * 16 + half * 1024;
          ko2 = (y >> 6) * TB + (y & 63) * 16 + half * 1024;
          kstep = KT < kTile ? 0 : TB;
          kper = KT < kTile ? TB : 2 * TB;
          vstep = KT * D * 2;
          vo = lkey * D * 2 + half * 16;
          kn = 2048;
        }
      } else {
        // a block that is not one run, key by key: keys below p0 (and, as
        // zeros, those past the range) from the cache, the others from the
        // chunk
        const int s = s0 + lkey;
        const bool own = s >= p0 && s < se;
        if (s0 + kKeys > p0 && s0 < se) {
          const int c0 = max(s0, p0);
          const size_t at = (size_t)(c0 - p0) * in_stride;
          const int off = (s - c0) * (int)in_stride * 2 + half * 16;
          if (own)
            put(reinterpret_cast<const uint8_t *>(kin + at),
                reinterpret_cast<const uint8_t *>(vin + at), off, off, 32, stage);
        }
        int sl = cached_slot(s, S, W);
        if (pto >= 0) {
          sl &= kPageTokens - 1;
          if (s0 >= ce) kb = kcb;                   // no cached key: nothing is read
        }
        const bool cached = s < ce;
        if (!own)
          put(kb, vb, cached ? cached_k(D, sl) + half * 1024 : kNoRow,
              cached ? cached_v(D, sl) + half * 16 : kNoRow, 2048, stage);
        return;
      }
    }
    put(run_k, run_v, ko, vo, kn, stage);
    --run;
    run_k = scalar_ptr(run_k + kstep);
    run_v = scalar_ptr(run_v + vstep);
    kstep = __builtin_amdgcn_readfirstlane(kper - kstep);
    if constexpr (KT < kTile) {
      const int x = ko;
      ko = ko2;
      ko2 = x;
    }
  };

  // logit scale, base 2, with the stored keys' scale (1 but for fp8 caches);
  // uniform, so kept in a scalar register (the 256-channel kernel has no
  // vector register to spare for it)
  float c2 = __builtin_bit_cast(
      float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, a.scale_log2 * hd.k_scale)));
  float v_scale = hd.v_scale;
  asm volatile("" : "+s"(v_scale));              // loaded here, not after the loop
  if constexpr (F16) {
    // q to binary16 under the wavefront's power of two 2^sh; c2 takes 2^-sh
    // (sh is capped so that c2 stays a normal number)
    float mx = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x0 = __builtin_bit_cast(float, qv[ks][j] << 16);
        const float x1 = __builtin_bit_cast(float, qv[ks][j] & 0xffff0000u);
        mx = fmaxf(mx, fmaxf(fabsf(x0), fabsf(x1)));
      }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    mx = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, mx)));
    int ex, ec;
    (void)frexpf(mx, &ex);                      // mx in [2^(ex-1), 2^ex)
    (void)frexpf(c2, &ec);
    int sh = mx > 0.0f ? 15 - ex : 0;
    sh = min(sh, ec + 120);
    sh = __builtin_amdgcn_readfirstlane(sh);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x0 = __builtin_bit_cast(float, qv[ks][j] << 16);
        const float x1 = __builtin_bit_cast(float, qv[ks][j] & 0xffff0000u);
        qv[ks][j] = pack_f16(ldexpf(x0, sh), ldexpf(x1, sh));
      }
    c2 = ldexpf(c2, -sh);
  }
  const float tau = 8.0f / c2;                  // lazy-rescale slack (raw units)
  constexpr float pbias = F16 ? 7.0f : 0.0f;    // log2 of the weights' bias
  float m = -1e30f;                              // running shift (raw units)
  float l = 0.0f;                                // this lane's partial sum
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.0f;

  // S^T operand: key cl of chunk row 2ks + half (odd rows swizzled).
  int klane = half * 512 + (cl ^ (4 * half)) * 16;
  // V^T operand: 16-lane group gq = lane / 16, local lane mq.  For k-step s
  // and half hh of its 8 keys, lane (gq, mq) reads 8 bytes of key
  // 16s + 8hh + 4(gq / 2) + mq / 4 at channel 32db + 16(gq % 2) + 4(mq % 4),
  // i.e. in chunk row 4db + 2(gq % 2) + (mq % 4) / 2 of parity (mq / 2) % 2.
  const int gq = lane >> 4, mq = lane & 15;
  const int vpar = (mq >> 1) & 1;
  const int vkey0 = 4 * (gq >> 1) + (mq >> 2);
  int vlane = P::KBYTES + (gq & 1) * P::VPAIR + vpar * 512 + (vkey0 ^ (4 * vpar)) * 16 +
              (mq & 1) * 8;
  // one register each, not the terms of their sums (the 256-channel kernel
  // has none to spare)
  asm volatile("" : "+v"(klane), "+v"(vlane));

  // masks the tile of keys [s0, min(s0 + KT, se))
  auto mask = [&](f32x16_t (&st)[U], int s0, int se) {
    const int tm = pos(token(min(wc0 + (lane_now() & 31), c_last)));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = s0 + kKeys * u + 4 * (lane_now() >> 5);
      uint32_t vis = below(min(se, tm + 1) - e);
      if (W != 0) vis &= below(S - e) | ~below(tm + 1 - W - e);
      keep_rows(st[u], vis);
    }
  };
  // raises the shift (and rescales the sums) where a tile's maximum exceeds it
  // by more than 8 in base 2
  auto raise = [&](float mx) {
    if (__any(mx > m + tau)) {
      const float mn = fmaxf(m, mx);
      const float alpha = __builtin_amdgcn_exp2f((m - mn) * c2);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    }
  };
  auto products = [&](auto values, f32x16_t (&st)[U], const u32x4_t (&pb)[2 * U], const uint8_t *kl,
                      const uint8_t *vl, const uint8_t *vl1) {
    tile_products<D, NW, F16, U, decltype(values)::value>(o, st, pb, qv, kl, vl, vl1);
  };
  // Tiles [f0, f0 + fn) of this split are seen whole by every column of the
  // wave.
  int f0, f1;
  {
    const int base = lo <= S ? 0 : rb0, tile0 = lo <= S ? 0 : na;   // of the range holding t_lo
    f1 = tile0 + max(0, t_lo + 1 - base) / KT;
    f0 = tile0 + (W == 0 ? 0 : (max(0, t_hi + 1 - W - base) + KT - 1) / KT);
    f0 = max(f0 - i_lo, 0);
    f1 = wave_live ? f1 - i_lo : f0;
  }
  const uint32_t fn = (uint32_t)max(f1 - f0, 0);
  // whether any column of this wave sees a key of tile it
  auto visible = [&](int it) {
    int s0, se;
    tile_range(i_lo + it, &s0, &se);
    const int slast = min(s0 + KT, se) - 1;
    return wave_live && s0 <= t_hi && !(W != 0 && s0 >= S && slast < t_lo + 1 - W);
  };
  constexpr int SB = U * P::STAGE;               // bytes of a stage
#pragma unroll 1
  for (int it = 0; it < min(n_it, 2); ++it) issue_loads(it, smem + it * SB);
  if (n_it > 1)
    wait_loads<2 * IPW>();
  else
    wait_loads();
  // q has arrived before the loop: a wait for it inside would wait for the
  // tiles' loads too
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qv[ks]));
  phase_end();
  // the second group (together with the first where there is little to overlap)
  const bool late = wave >= NW / 2 && n_it > 2;
  if (late) phase_end();

  f32x16_t st[U];                                // S^T of the tile
  u32x4_t pb[2 * U];                             // the weights of the tile, packed
  bool held = false;                             // pb holds weights to add
  int so = 0;                                    // LDS offset of tile it
  int sv = 0, dv = 0;                            // and of the values pb weighs: first block, second
  for (int it = 0;; ++it) {
    // ---- products: S^T of tile it, then V^T P^T of tile it - 1
    const bool whole = (uint32_t)(it - f0) < fn;
    const bool vis = it < n_it && (whole || visible(it));
    __builtin_amdgcn_s_waitcnt(0xc07f);          // no scalar load outstanding: LDS waits can count
    const uint8_t *kl = smem + so + klane, *vl = smem + sv + vlane, *vl1 = vl + dv;
    if (held)                                    // (S^T goes unused where !vis)
      products(std::true_type{}, st, pb, kl, vl, vl1);
    else if (vis)
      products(std::false_type{}, st, pb, kl, vl, vl1);
    wait_loads();                                // tile it + 1, issued a phase ago
    if (it == n_it) break;
    phase_end();
    // ---- softmax of tile it
    if (it + 2 < n_it) issue_loads(it + 2, smem + (so >= 2 * SB ? so - 2 * SB : so + 2 * SB));
    held = vis;
    sv = so;
    dv = P::STAGE;
    if (vis) {
      if (!whole) {
        int s0, se;
        tile_range(i_lo + it, &s0, &se);
        mask(st, s0, se);
        // A block that no column of the wave sees (of a tile that it sees: the second
        // past its tokens, or the first below its windows) has zero weights only;
        // they meet the other block's values, so that what is not finite in it
        // stays out.
        if (U > 1 && s0 + kKeys > t_hi) {
          dv = 0;
        } else if (U > 1 && W != 0 && s0 >= S && s0 + kKeys <= t_lo + 1 - W) {
          sv = so + P::STAGE;
          dv = 0;
        }
      }
      raise(tile_max(st));
      tile_weights<U, F16>(st, pb, l, c2, m * c2 - pbias);
    }
    so = so == (STAGES - 1) * SB ? 0 : so + SB;
    phase_end();
  }
  if (!late) phase_end();
  if (!wave_live) return;                          // no column to write

  float l_lo, l_hi;
  halves(l, &l_lo, &l_hi);
  const float lt = l_lo + l_hi;
  // The lane's column and its output row, recomputed rather than kept live
  // through the loop.
  const int c_out = wc0 + (lane_now() & 31);
  float inv = 1.0f;
  float *dst = a.out;
  uint32_t row;                                    // of D floats
  if (n_it == ntiles) {
    inv = v_scale / lt;                            // the stored values' scale (fp8)
    const int tl_o = token(min(c_out, c_last));
    row = (uint32_t)tl_o * (Hq - G) + h * G + c_out;
  } else {
    dst = a.part_acc;
    row = (uint32_t)blk * (32 * NW) + (c_out - c_first);
    if (c_out <= c_last && lane_now() < 32)
      *reinterpret_cast<float2 *>(a.part_ml + (size_t)row * 2) =
          make_float2(fmaxf(m * c2, -3e38f), lt);
  }
  constexpr int CH = D > 64 ? 64 : 32, AREA = 128 * CH;
  static_assert(NW / 2 * AREA <= SB && STAGES >= 4, "two stages hold every wave's area");
  // two stages that the other group's last products do not read
  // Few columns (two waves' at most) go straight from the registers: 64 columns
  // over four tiles, head_dim 256, 10.4 -> 9.7 us, but 128 columns 9.4 -> 10.5.  (At
  // head_dim 64 the second path costs longer launches more, 2 %.)
  if (D > 64 && c_last - c_first < 64) {
    if (c_out <= c_last)
#pragma unroll
      for (int x = 0; x < 4 * DB; ++x)
        *reinterpret_cast<float4 *>(dst + (size_t)row * D + 8 * x + 4 * (lane_now() >> 5)) =
            make_float4(o[x / 4][4 * (x % 4) + 0] * inv, o[x / 4][4 * (x % 4) + 1] * inv,
                        o[x / 4][4 * (x % 4) + 2] * inv, o[x / 4][4 * (x % 4) + 3] * inv);
    return;
  }
  const int stage = so + (wave < NW / 2 ? SB : 2 * SB);
  store_rows<D, CH>(o, inv, dst, D, row, c_last - wc0,
                smem + (stage >= STAGES * SB ? stage - STAGES * SB : stage) +
                    wave % (NW / 2) * AREA);
}

// Merge of the split partials: one row of D / 4 lanes per column, a lane
// owning 4 channels.  A column block of more than tiles_per_split tiles has
// one partial per split; out = sum acc_j 2^(m_j - M) / sum l_j 2^(m_j - M),
// M = max m_j (a split in which the column sees no key has m = -1e30 logit
// units and zero sums), times the V scale.  Bound by reading the partials.
constexpr int kMergeUnroll = 4;
template <int D, int NW>
__global__ __launch_bounds__(256) void prefill_merge(const PrefillAttnArgs a) {
  constexpr int LPC = D / 4;                       // lanes per column
  constexpr int CPW = 256 / LPC;                   // columns per workgroup
  constexpr int COLS = 32 * NW;                    // columns per block
  constexpr int PER = COLS / CPW;                  // workgroups per block
  const int nb = a.n_col_blocks;
  const int rank = blockIdx.x / (nb * PER);
  const int x = blockIdx.x % (nb * PER);
  const int cb = x / PER;
  const int G = a.group, Hq = a.n_kv_heads * G;
  const int c_first = cb * COLS;
  const int c_last = min(c_first + COLS, a.n_tokens * G) - 1;
  const PrefillAttnHead &hd = a.head[rank];
  const int h = hd.h;
  const int T = a.tiles_per_split;
  const int nt = prefill_tiles(prefill_keys(D), a.p0 + c_first / G, a.p0 + c_last / G, a.n_sinks,
                               hd.window);
  if (nt <= T) return;                             // uniform: written by its one split
  const int ns = (nt + T - 1) / T;
  const int col = x % PER * CPW + threadIdx.x / LPC;   // column of the block
  const int c = c_first + col;
  if (c > c_last) return;
  const int ch = threadIdx.x % LPC * 4;
  // split j's workgroup is w0 + j nb
  const size_t w0 = (size_t)hd.wg_begin + (nb - 1 - cb);
  const float *acc = a.part_acc + (w0 * COLS + col) * D + ch;
  const float *ml = a.part_ml + (w0 * COLS + col) * 2;
  const size_t step = (size_t)nb * COLS;
  float M = -INFINITY, L = 0.0f;
  float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int j0 = 0; j0 < ns; j0 += kMergeUnroll) {
    float2 s[kMergeUnroll];
    float4 v[kMergeUnroll];
#pragma unroll
    for (int u = 0; u < kMergeUnroll; ++u) {       // every load of the round in flight
      const size_t j = (size_t)min(j0 + u, ns - 1);
      s[u] = *reinterpret_cast<const float2 *>(ml + j * step * 2);
      v[u] = *reinterpret_cast<const float4 *>(acc + j * step * D);
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < kMergeUnroll; ++u) {
      if (j0 + u >= ns) s[u] = make_float2(-INFINITY, 0.0f);
      Mn = fmaxf(Mn, s[u].x);
    }
    const float f = __builtin_amdgcn_exp2f(M - Mn);
    L *= f;
    A.x *= f;
    A.y *= f;
    A.z *= f;
    A.w *= f;
#pragma unroll
    for (int u = 0; u < kMergeUnroll; ++u) {
      if (j0 + u >= ns) break;                     // uniform
      const float e = __builtin_amdgcn_exp2f(s[u].x - Mn);
      L += s[u].y * e;
      A.x += v[u].x * e;
      A.y += v[u].y * e;
      A.z += v[u].z * e;
      A.w += v[u].w * e;
    }
    M = Mn;
  }
  const float inv = hd.v_scale / L;
  const int tl = c / G, g = c - tl * G;
  *reinterpret_cast<float4 *>(a.out + ((size_t)tl * Hq + (size_t)h * G + g) * D + ch) =
      make_float4(A.x * inv, A.y * inv, A.z * inv, A.w * inv);
}

// Calibration replay in one pass.  Workgroups, columns and phases as in
// prefill_attn (column c = row * G + g of one KV head, row r at position
// rows[r]; tiles of 32 keys); the keys are the traced history, each candidate
// window w holds the sinks [0, S) and the suffix [max(S, t + 1 - w), t] of row
// position t, and the full candidate holds every s <= t.  The suffixes are
// nested, so a column walks its keys once, from the top tile down: when the walk
// has added every key at or above a window's edge t + 1 - w, the running
// (m, l, acc) is that window's share of the split, written out there.  A tile
// holding an edge is added on its own, in the softmax phase, in up to two
// passes of the V^T P^T product per edge: the keys at or above the edge, then
// the rest.  Split y < n_splits covers key tiles [y tps, (y + 1) tps) of
// [0, t_last] without the sinks; split n_splits adds the sinks alone.
// replay_merge assembles each candidate.
//
// Where the sampled rows lie far apart nearly every tile of the top splits
// holds an edge of some row, and these passes, which the barriers make every
// wave wait for, are most of the time: a row's edges in tiles of their own
// take a pass each.  Their masks by bits (keep_rows) rather than by two
// comparisons a logit, and the last rows written through LDS, took a 20,011-key
// fp8 trace's replay (101 rows, head_dim 128) from 291 to 269 us; 256 rows of a
// 128K trace at head_dim 256, where few tiles hold an edge, stay at 819.
template <int D, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
void replay_attn(const ReplayAttnArgs a) {
  using P = Prefill<D, NW>;
  constexpr int KS = P::KS, DB = P::DB;
  constexpr int STAGES = 4;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[STAGES * P::STAGE];
  __shared__ int swin[kMaxWindows];

  const int nb = a.n_col_blocks;
  const int h = blockIdx.x / nb;
  const int cb = nb - 1 - (int)(blockIdx.x % nb);   // later rows first
  const int G = a.group;
  const int Hq = a.n_kv_heads * G;
  const int ncols = a.n_rows * G;
  const int c_first = cb * 32 * NW;
  const int c_last = min(c_first + 32 * NW, ncols) - 1;
  const int32_t *rows = a.rows;
  const int S = a.n_sinks;
  const int K = a.n_windows;
  const int tb = rows[c_last / G];                  // the block's last position

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, cl = lane & 31;
  const int wc0 = c_first + 32 * wave;
  const bool wave_live = wc0 <= c_last;
  const int wc_last = min(wc0 + 31, c_last);
  const int t_lo = rows[min(wc0, c_last) / G], t_hi = rows[wc_last / G];
  const size_t n_cols = (size_t)a.n_rows * Hq;
  // the lane's column (the last one where it has none) and its id (row * Hq +
  // h * G + g), recomputed where they are needed rather than kept live
  // through the tile loop
  auto column = [&]() { return min(wc0 + (lane_now() & 31), c_last); };
  auto column_id = [&]() -> size_t {
    const int ccx = column(), tx = ccx / G;
    return (size_t)tx * Hq + (size_t)h * G + (size_t)(ccx - tx * G);
  };
  const int t = rows[column() / G];

  // this workgroup's key tiles
  const int ntiles = tb / kKeys + 1;
  const bool sink_pass = (int)blockIdx.y == a.n_splits;
  int i_lo, i_hi;
  if (sink_pass) {
    i_lo = 0;
    i_hi = min(ntiles, (S + kKeys - 1) / kKeys);
  } else {
    i_lo = blockIdx.y * a.tiles_per_split;
    i_hi = min(ntiles, i_lo + a.tiles_per_split);
  }
  if (i_lo >= i_hi) {                               // uniform: an empty split
    if (wc0 + cl <= c_last && half == 0) {
      float *pp = a.part + ((size_t)blockIdx.y * n_cols + column_id()) * (D + 4);
      pp[0] = -1e30f;
      pp[1] = 0.0f;
    }
    return;
  }
  for (int i = tid; i < K; i += NW * 64) swin[i] = a.windows[i];

  u32x4_t qv[KS];
  {
    const uint16_t *qr = a.q + column_id() * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qv[ks] = ld16(qr + 16 * ks);
  }

  // Tile loads: chunk rows 2n, 2n + 1 by wave n % NW (see prefill_attn), from
  // the top tile down; keys past the block's last position read as zeros.
  const size_t in_stride = (size_t)a.n_kv_heads * D;
  const int n_it = i_hi - i_lo;
  const uint8_t *run_k = scalar_ptr(a.k + (size_t)(i_hi - 1) * kKeys * in_stride + (size_t)h * D);
  const uint8_t *run_v = scalar_ptr(a.v + (size_t)(i_hi - 1) * kKeys * in_stride + (size_t)h * D);
  const int tile_bytes = kKeys * (int)in_stride * 2;
  int vo = (cl ^ (4 * half)) * (int)in_stride * 2 + half * 16;
  auto issue_loads = [&](uint8_t *stage, int off) {
    const rsrc_t kr = make_rsrc(run_k), vr = make_rsrc(run_v);
#pragma unroll
    for (int j = 0; j < P::IPW; ++j) {
      const int n = wave + j * NW;
      if (P::NINST % NW != 0 && n >= P::NINST) break;   // uniform per wave
      b2lds(kr, stage + n * 1024, off, n * 32);
      b2lds(vr, stage + P::KBYTES + n * P::VPAIR, off, n * 32);
    }
    run_k = scalar_ptr(run_k - tile_bytes);
    run_v = scalar_ptr(run_v - tile_bytes);
  };

  // logit scale, base 2, with the keys' scale; uniform (scalar register)
  const float c2 = __builtin_bit_cast(
      float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, a.scale_log2 * a.k_scale[h])));
  float m = -1e30f;                              // running shift (raw units)
  float l = 0.0f;                                // this lane's partial sum
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.0f;

  int klane = half * 512 + (cl ^ (4 * half)) * 16;
  const int gq = lane >> 4, mq = lane & 15;
  const int vpar = (mq >> 1) & 1;
  const int vkey0 = 4 * (gq >> 1) + (mq >> 2);
  int vlane = P::KBYTES + (gq & 1) * P::VPAIR + vpar * 512 + (vkey0 ^ (4 * vpar)) * 16 +
              (mq & 1) * 8;
  asm volatile("" : "+v"(klane), "+v"(vlane), "+v"(vo));
#pragma unroll 1
  for (int it = 0; it < min(n_it, 2); ++it) {
    const bool past = it == 0 && (i_hi - 1) * kKeys + (cl ^ (4 * half)) > tb;
    issue_loads(smem + it * P::STAGE, past ? kNoRow : vo);
  }
  if (P::NINST % NW == 0 && n_it > 1)
    wait_loads<2 * P::IPW>();                    // the first tile has landed
  else
    wait_loads();
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qv[ks]));
  __syncthreads();                               // swin too
  // The lane's next window: the first whose edge lies below this split's top
  // (windows with an edge at or above it have no key here).  An edge at or
  // below S means the window holds every key: it is the full candidate.
  const int top = i_hi * kKeys;
  int kn = 0;
  int edge = INT_MIN;
  auto edge_of = [&](int k) {
    return (k < K && t + 1 - swin[k] > S) ? t + 1 - swin[k] : INT_MIN;
  };
  if (!sink_pass) {
    while (kn < K && t + 1 - swin[kn] >= top) ++kn;
    edge = edge_of(kn);
  }
  phase_end();
  // the second group (together with the first where there is little to overlap)
  const bool late = wave >= NW / 2 && n_it > 2;
  if (late) phase_end();

  f32x16_t st[1];                                // S^T of the tile
  u32x4_t pb[2];                                 // the weights of the tile, packed
  bool held = false;                             // pb holds weights to add
  int so = 0, so1 = 0;                           // LDS offsets of tiles it, it - 1
  for (int it = 0;; ++it) {
    // ---- products: S^T of tile it, then V^T P^T of tile it - 1
    const int s0 = (i_hi - 1 - it) * kKeys;      // tiles from the top down
    const bool vis = it < n_it && wave_live && s0 <= t_hi &&
                     (sink_pass ? s0 < S : s0 + kKeys > S);
    const uint8_t *kl = smem + so + klane, *vl = smem + so1 + vlane;
    // One pass, or for a tile that holds window edges one per edge and the rest:
    // first the keys at or above a lane's next edge (the whole tile where it
    // has none), whose state is then the window's partial, then those below
    // the last edge taken; the logits are formed again for each.  (One call of
    // the products for all of them: a second place that adds to o would take
    // a second set of its registers.)
    bool act = false;                            // the lane's edge is in this pass
    int lo = s0, cut = s0 + kKeys;               // its keys: [lo, cut)
    for (bool first = true;; first = false) {
      __builtin_amdgcn_s_waitcnt(0xc07f);        // as in prefill_attn
      if (held)
        tile_products<D, NW, false, 1, true>(o, st, pb, qv, kl, vl, vl);
      else if (vis)
        tile_products<D, NW, false, 1, false>(o, st, pb, qv, kl, vl, vl);
      held = false;
      if (first) {
        wait_loads();                            // tile it + 1, issued a phase ago
        if (it == n_it) break;
        phase_end();
        // ---- softmax of tile it
        if (it + 2 < n_it)
          issue_loads(smem + (so >= 2 * P::STAGE ? so - 2 * P::STAGE : so + 2 * P::STAGE), vo);
        if (!vis) break;
      } else {
        // the windows' partials, for the lanes whose edge this pass reached
        float l_lo, l_hi;
        halves(l, &l_lo, &l_hi);
        if (act && wc0 + (lane_now() & 31) <= c_last) {
          const int hf = lane_now() >> 5;
          const size_t col_id = column_id();
          float *wa = a.win_acc + ((size_t)kn * n_cols + col_id) * D;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
              *reinterpret_cast<float4 *>(wa + 32 * db + 8 * rq + 4 * hf) =
                  make_float4(o[db][4 * rq + 0], o[db][4 * rq + 1], o[db][4 * rq + 2],
                              o[db][4 * rq + 3]);
          if (hf == 0)
            *reinterpret_cast<float2 *>(a.win_ml + ((size_t)kn * n_cols + col_id) * 2) =
                make_float2(m, l_lo + l_hi);
        }
        if (act) {
          ++kn;
          edge = edge_of(kn);
        }
        cut = lo;
        if (!__any(cut > s0)) break;
      }
      // visible keys: s <= t, and s < S in the sink pass, s >= S otherwise
      if (!(s0 + kKeys - 1 <= t_lo && (sink_pass ? s0 + kKeys <= S : s0 >= S))) {
        const int e = s0 + 4 * (lane_now() >> 5);
        const uint32_t sinks = below(S - e);
        keep_rows(st[0], below(t + 1 - e) & (sink_pass ? sinks : ~sinks));
      }
      if (first) {
        const float mx = tile_max(st);
        if (__any((mx - m) * c2 > 8.0f)) {       // lazy rescale: shift moves by > 8
          const float mn = fmaxf(m, mx);
          const float alpha = __builtin_amdgcn_exp2f((m - mn) * c2);
          m = mn;
          l *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        }
      }
      held = true;                               // added with the next products
      act = edge >= s0;
      const bool edges = __any(act);             // uniform; rare
      if (first && !edges) {
        tile_weights<1, false>(st, pb, l, c2, m * c2);
        break;
      }
      lo = act ? edge : s0;
      const float mc = m * c2;
      const int e = s0 + 4 * (lane_now() >> 5);
      keep_rows(st[0], below(cut - e) & ~below(lo - e));
      float ls = 0.0f;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r0 = 8 * s + 2 * j, r1 = r0 + 1;
          const float w0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[0][r0], c2, -mc));
          const float w1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[0][r1], c2, -mc));
          ls += w0 + w1;
          pb[s][j] = pack_bf16(w0, w1);
        }
      l += ls;
      if (!edges) break;
      vl = smem + so + vlane;                    // this tile's values, now
    }
    if (it == n_it) break;
    so1 = so;
    so = so == (STAGES - 1) * P::STAGE ? 0 : so + P::STAGE;
    phase_end();
  }
  if (!late) phase_end();

  float l_lo, l_hi;
  halves(l, &l_lo, &l_hi);
  const uint32_t row = (uint32_t)(blockIdx.y * n_cols + column_id());
  float *pp = a.part + (size_t)row * (D + 4);
  if (lane_now() < 32 && wc0 + lane_now() <= c_last) {
    pp[0] = m;
    pp[1] = l_lo + l_hi;
  }
  constexpr int SB = P::STAGE, CH = D / 4, AREA = 128 * CH;
  static_assert(NW / 2 * AREA <= SB && STAGES >= 4, "two stages hold every wave's area");
  const int stage = so + (wave < NW / 2 ? SB : 2 * SB);   // as in prefill_attn
  store_rows<D, CH>(o, 1.0f, a.part + 4, D + 4, row, c_last - wc0,
                smem + (stage >= STAGES * SB ? stage - STAGES * SB : stage) +
                    wave % (NW / 2) * AREA);
}

}  // namespace

int prefill_attn_columns_per_block() { return 32 * kPrefillWaves; }

hipError_t launch_prefill_attn(int D, bool f16, const PrefillAttnArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)a.n_wgs);
  const dim3 block(kPrefillWaves * 64);
#define HWKV_PA(DD, FF) \
  hipLaunchKernelGGL((prefill_attn<DD, kPrefillWaves, FF>), grid, block, 0, s, a)
  switch (D) {
    case 64: if (f16) HWKV_PA(64, true); else HWKV_PA(64, false); break;
    case 128: if (f16) HWKV_PA(128, true); else HWKV_PA(128, false); break;
    case 256: if (f16) HWKV_PA(256, true); else HWKV_PA(256, false); break;
    default: return hipErrorInvalidValue;
  }
#undef HWKV_PA
  return hipGetLastError();
}

hipError_t launch_prefill_merge(int D, const PrefillAttnArgs &a, hipStream_t s) {
  const int per = 32 * kPrefillWaves / (256 / (D / 4));   // workgroups per column block
  const dim3 grid((unsigned)(a.n_col_blocks * a.n_kv_heads * per)), block(256);
  switch (D) {
    case 64: hipLaunchKernelGGL((prefill_merge<64, kPrefillWaves>), grid, block, 0, s, a); break;
    case 128: hipLaunchKernelGGL((prefill_merge<128, kPrefillWaves>), grid, block, 0, s, a); break;
    case 256: hipLaunchKernelGGL((prefill_merge<256, kPrefillWaves>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_replay_attn(int D, const ReplayAttnArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)(a.n_col_blocks * a.n_kv_heads),
                  (unsigned)(a.n_splits + (a.n_sinks > 0 ? 1 : 0)));
  const dim3 block(kPrefillWaves * 64);
  switch (D) {
    case 64: hipLaunchKernelGGL((replay_attn<64, kPrefillWaves>), grid, block, 0, s, a); break;
    case 128: hipLaunchKernelGGL((replay_attn<128, kPrefillWaves>), grid, block, 0, s, a); break;
    case 256: hipLaunchKernelGGL((replay_attn<256, kPrefillWaves>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace hwkv
