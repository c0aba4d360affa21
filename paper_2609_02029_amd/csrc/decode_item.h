// decode_item.h -- decode attention with one workgroup per (sequence, KV
// head) item (gfx950, wave64, VALU), for every cache format; the counterpart
// of the split kernels (decode_split.h, decode_mfma.h) where the items are
// short, or many and alike: no partials leave the workgroup, so there is no
// merge launch, and one launch takes every item of up to 192 sequences.  Items
// longer than a share of the CUs are split all the same, and then merged
// (item_merge).
//
// NW = 16 or 8 waves: wave w takes the item's 64-slot tiles w, w + NW, ... whole,
// with an online softmax of its own (base 2), and the waves' (m, l, acc) are
// merged exactly in LDS at the end.  Per tile, one stream of chunk loads per
// lane with PF in flight, running on into the wave's next tile, as in
// decode_split: q.k with one lane per slot (q from LDS, one address for every
// lane; bf16 pairs in v_dot2_f32_bf16 -- fp8 codes widen to bf16 exactly -- and
// binary16 pairs in v_dot2_f32_f16; four partial logits a head over 16-bit keys),
// p.v with a lane on 8 channels of a row and fp32 weights.  Against 64 bits its rms
// error is 1.02 times decode_split's on average (0.88 to 1.18 over 42 shapes; 1.29
// with one chain of products a logit), and 0.09 times decode_mfma's over fp8.
//
// What bounds it: launch and latency for short items; for long ones what one
// CU can stream.  Figures stand at the rule that chooses it (hwkv_api.hip).
#pragma once

// Included by decode_split.h after its helpers.

namespace hwkv {
namespace {

// Orders the wave's LDS writes before its later LDS reads (the hardware keeps
// a wave's LDS operations in order).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <int D, int G>
struct ItemSmem {
  static constexpr int PST = G == 6 ? 8 : G;     // weights per slot (fp32)
  static constexpr int NW = decode_item_waves(D, G);
  union {
    float p[NW][64 * PST];               // a wave's weights of its tile
    __attribute__((aligned(16))) float acc[NW][G * D];   // epilogue
  } u;
  __attribute__((aligned(16))) uint32_t q[G * D / 2];   // pairs, head-major
  float qsc[G];                                  // logit scale of each head
  float m[NW][G], l[NW][G];
};

template <int D, int G, int F>
__global__ __launch_bounds__(decode_item_waves(D, G) * 64) void decode_item(ItemArgs a) {
  using Chunk = typename KvFormat<F>::Chunk;
  constexpr int EB = KvFormat<F>::kBytes;
  constexpr int LB = 8 * EB;                     // bytes per chunk
  constexpr int NC = D / 8;                      // chunks per row
  constexpr int RPS = 64 / NC;                   // rows per V step
  constexpr int PIECES = 2 * NC;                 // loads per tile: K chunks, V steps
  constexpr int NW = decode_item_waves(D, G);
  constexpr int PF = NW == 8 && D * G < 2048 ? 16 : 8;   // loads in flight
  constexpr int PST = ItemSmem<D, G>::PST;
  static_assert(RPS * D * EB == 64 * LB, "K chunks and V steps are equally long");
  __shared__ ItemSmem<D, G> sm;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // heads by capacity, sequences by length, longest first; the head is the
  // number of heads that begin at or before this workgroup's run of sequences
  const int run = blockIdx.x / a.n_seqs;
  const int rank = __builtin_amdgcn_readfirstlane(__popcll(__ballot(a.wg_begin[lane] <= run)) - 1);
  const int h = a.head_order[rank];
  const int split = run - a.wg_begin[rank];
  int si = blockIdx.x - run * a.n_seqs;
  if (a.rotate) {                                // by one from run to run
    si -= run % a.n_seqs;
    si += si < 0 ? a.n_seqs : 0;
  }
  const int b = a.seq[si];
  const int n = a.len[si];
  const ItemHead &hd = a.head[h];
  const int nv = min(n, hd.cap);                 // occupied slots attended
  const int all_tiles = (nv + 63) / 64;
  const int t_lo = split * a.tiles_per_wg;       // this workgroup's tiles [t_lo, n_tiles)
  if (t_lo >= all_tiles) return;                 // uniform: a shorter item
  const int n_tiles = min(all_tiles - t_lo, a.tiles_per_wg) + t_lo;
  const int pto = hd.page0 >= 0 ? hd.page0 + b * a.max_pages : -1;
  const int64_t seq_at = (int64_t)b * hd.cap_pad * D;
  uint8_t *const kbase = static_cast<uint8_t *>(a.cache) + (pto >= 0 ? a.pool_off : hd.k_off + seq_at) * EB;
  uint8_t *const vbase =
      static_cast<uint8_t *>(a.cache) + (pto >= 0 ? a.pool_off + kPageTokens * D : hd.v_off + seq_at) * EB;
  const size_t q_row = ((size_t)b * a.n_kv_heads + h) * G;
  auto page_of = [&](int t) -> int {
    return pto >= 0 ? ((const __attribute__((address_space(4))) int32_t *)
                           a.page_table)[pto + t / (kPageTokens / 64)]
                    : 0;
  };
  // byte offset of tile t (page pg of a paged unit); K and V alike
  auto tile_at = [&](int t, int pg) -> size_t {
    if (pto >= 0)
      return (size_t)pg * 2 * kPageTokens * D * EB + (size_t)(t % (kPageTokens / 64)) * 64 * D * EB;
    return (size_t)t * 64 * D * EB;
  };

  // fused append: the new token goes to its slot, by the workgroup that reads
  // the slot, before any of its waves does
  const int pos = n - 1;
  const int slot = (hd.window == 0 || pos < a.n_sinks)
                       ? pos
                       : a.n_sinks + (pos - a.n_sinks) % hd.window;
  if (a.k_new && slot / 64 >= t_lo && slot / 64 < n_tiles && threadIdx.x < 2 * NC) {
    const size_t t0 = tile_at(slot / 64, page_of(slot / 64));
    const size_t src = ((size_t)b * a.n_kv_heads + h) * D;
    if (threadIdx.x < NC) {
      const int g = threadIdx.x;
      store_chunk<F>(kbase + t0 + ((size_t)g * 64 + slot % 64) * LB,
                     encode8<F>(*reinterpret_cast<const uint4 *>(a.k_new + src + g * 8), hd.k_scale));
    } else {
      const int g = threadIdx.x - NC;
      store_chunk<F>(vbase + t0 + (size_t)(slot % 64) * D * EB + g * LB,
                     encode8<F>(*reinterpret_cast<const uint4 *>(a.v_new + src + g * 8), hd.v_scale));
    }
  }
  // q to LDS: as it is, or (binary16 keys) as binary16 with head g scaled by
  // the power of two that puts its largest |q| in [2^14, 2^15), which the head's
  // logit scale takes back (as in decode_split)
  const float zscale = a.scale_log2 * hd.k_scale;
  if (wave < G) {
    const uint32_t *qh = reinterpret_cast<const uint32_t *>(a.q + (q_row + wave) * D);
    constexpr int QN = (D / 2 + 63) / 64;
    uint32_t w[QN];
    float mx = 0.0f;
#pragma unroll
    for (int r = 0; r < QN; ++r) {
      w[r] = qh[min(64 * r + lane, D / 2 - 1)];
      mx = fmaxf(mx, fmaxf(fabsf(bf_lo(w[r])), fabsf(bf_hi(w[r]))));
    }
    int sh = 0;
    if constexpr (F == HWKV_KV_F16) {
      int ex, ez;
      (void)frexpf(wave_max(mx), &ex);
      (void)frexpf(zscale, &ez);
      sh = __builtin_amdgcn_readfirstlane(min(wave_max(mx) > 0.0f ? 15 - ex : 0, ez + 120));
    }
#pragma unroll
    for (int r = 0; r < QN; ++r) {
      if constexpr (F == HWKV_KV_F16) {
        const f16x2_t x = {(_Float16)ldexpf(bf_lo(w[r]), sh), (_Float16)ldexpf(bf_hi(w[r]), sh)};
        w[r] = __builtin_bit_cast(uint32_t, x);
      }
      if (64 * r + lane < D / 2) sm.q[wave * (D / 2) + 64 * r + lane] = w[r];
    }
    if (lane == 0) sm.qsc[wave] = ldexpf(zscale, -sh);
  }
  // only this workgroup reads the new slot in this launch (see decode_split)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

  // m starts at a finite number, so that a tile whose logits are all -inf has zero
  // weights (decode_split's workgroups take a tile together, and the later ones
  // meet a finite shift; here every wave has a first tile of its own)
  float m[G], l[G], acc[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -3e38f;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
  }
  const int c8 = lane % NC, rsub = lane / NC;
  const int kl = lane * LB;                      // K: lane = slot
  const int vl = rsub * D * EB + c8 * LB;        // V: row rsub of the step, 8 channels
  float *const pl = sm.u.p[wave];
  // descriptors of tile t's K (whole) and V (rows below nv; the others read as
  // zero); a tile that does not exist gets empty ones, so that every tile's
  // loads are issued the same way
  auto rsrc = [&](const uint8_t *base, int t, int pg, int rows) {
    return make_rsrc(base + tile_at(t, pg), (uint32_t)(rows * D * EB));
  };
  auto ld = [&](__amdgpu_buffer_rsrc_t kr, __amdgpu_buffer_rsrc_t vr, auto qc) -> Chunk {
    constexpr int q = decltype(qc)::value;
    return q < NC ? bload_chunk<F>(kr, kl, q * 64 * LB) : bload_chunk<F>(vr, vl, (q - NC) * 64 * LB);
  };

  int t = t_lo + wave;
  if (t < n_tiles) {
    int pg = page_of(t);
    __amdgpu_buffer_rsrc_t kr = rsrc(kbase, t, pg, 64), vr = rsrc(vbase, t, pg, min(64, nv - 64 * t));
    Chunk buf[PF];
    static_for<PF>([&](auto jc) { buf[jc.value] = ld(kr, vr, jc); });
    for (;;) {
      const bool more = t + NW < n_tiles;
      const int tn = more ? t + NW : t;
      const int pgn = more ? page_of(tn) : 0;
      const __amdgpu_buffer_rsrc_t krn = rsrc(kbase, tn, pgn, more ? 64 : 0);
      const __amdgpu_buffer_rsrc_t vrn = rsrc(vbase, tn, pgn, more ? min(64, nv - 64 * tn) : 0);
      auto issue = [&](auto qc) {                // the load PF pieces on
        constexpr int qn = decltype(qc)::value + PF;
        if constexpr (qn < PIECES)
          buf[qn % PF] = ld(kr, vr, std::integral_constant<int, qn>{});
        else
          buf[qn % PF] = ld(krn, vrn, std::integral_constant<int, qn - PIECES>{});
      };
      // q is read from LDS in every tile (opaque: kept in registers from tile to
      // tile it would take them from the loads in flight)
      int q0 = 0;
      asm volatile("" : "+v"(q0));
      // a head's logit is the sum of four partial ones, of a quarter of the channels
      // each, as decode_split's waves hold them: one chain over all channels has
      // about twice their rounding error (both opaque in every step, below)
      float s[G], zsum[G];
#pragma unroll
      for (int g = 0; g < G; ++g) s[g] = zsum[g] = 0.f;
      static_for<NC>([&](auto jc) {
        constexpr int q = decltype(jc)::value;
        if constexpr (F != HWKV_KV_FP8_E4M3 && q > 0 && q % (NC / 4) == 0) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            zsum[g] += s[g];
            s[g] = 0.f;
          }
        }
        // (opaque at each step, so that each issues its own loads: the
        // compiler would otherwise hoist a tile's loads and spill)
#pragma unroll
        for (int g = 0; g < G; ++g) asm volatile("" : "+v"(s[g]), "+v"(zsum[g]));
        const Chunk x = buf[q % PF];
        issue(jc);
        const u32x4_t *q4 = reinterpret_cast<const u32x4_t *>(sm.q + q0) + q;
        if constexpr (F == HWKV_KV_F16) {
          const f16x8_t kv = __builtin_bit_cast(f16x8_t, u32x4_t{x.x, x.y, x.z, x.w});
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const f16x8_t qv = __builtin_bit_cast(f16x8_t, q4[g * NC]);
            s[g] = __builtin_amdgcn_fdot2(__builtin_shufflevector(qv, qv, 0, 1),
                                          __builtin_shufflevector(kv, kv, 0, 1), s[g], false);
            s[g] = __builtin_amdgcn_fdot2(__builtin_shufflevector(qv, qv, 2, 3),
                                          __builtin_shufflevector(kv, kv, 2, 3), s[g], false);
            s[g] = __builtin_amdgcn_fdot2(__builtin_shufflevector(qv, qv, 4, 5),
                                          __builtin_shufflevector(kv, kv, 4, 5), s[g], false);
            s[g] = __builtin_amdgcn_fdot2(__builtin_shufflevector(qv, qv, 6, 7),
                                          __builtin_shufflevector(kv, kv, 6, 7), s[g], false);
          }
        } else {
          uint32_t kx[4];
          if constexpr (F == HWKV_KV_FP8_E4M3) {
            kx[0] = fp8x2_bf16x2<false>(x.x);
            kx[1] = fp8x2_bf16x2<true>(x.x);
            kx[2] = fp8x2_bf16x2<false>(x.y);
            kx[3] = fp8x2_bf16x2<true>(x.y);
          } else {
            kx[0] = x.x;
            kx[1] = x.y;
            kx[2] = x.z;
            kx[3] = x.w;
          }
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const u32x4_t qv = q4[g * NC];
            s[g] = dot2(qv.x, kx[0], s[g]);
            s[g] = dot2(qv.y, kx[1], s[g]);
            s[g] = dot2(qv.z, kx[2], s[g]);
            s[g] = dot2(qv.w, kx[3], s[g]);
          }
        }
      });
      const bool valid = 64 * t + lane < nv;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float x = zsum[g] + s[g], c = sm.qsc[g];
        const float mn = fmaxf(m[g], wave_max(valid ? x * c : -INFINITY));
        if (mn > m[g]) {                         // uniform
          const float alpha = exp2f(m[g] - mn);
          l[g] *= alpha;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[g][e] *= alpha;
          m[g] = mn;
        }
        // the logit enters unrounded: half an ulp of it is as much as the sums' error
        const float p = valid ? exp2f(fmaf(x, c, -mn)) : 0.f;
        l[g] += p;
        pl[lane * PST + g] = p;
      }
      wave_lds_order();
      static_for<NC>([&](auto jc) {
        constexpr int i = decltype(jc)::value;
        constexpr int q = NC + i;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < 8; e += 2)
            asm volatile("" : "+v"(acc[g][e]), "+v"(acc[g][e + 1]));
        const Chunk x = buf[q % PF];
        issue(std::integral_constant<int, q>{});
        float vf[8];
        if constexpr (F == HWKV_KV_FP8_E4M3) {
          const uint32_t w[4] = {fp8x2_bf16x2<false>(x.x), fp8x2_bf16x2<true>(x.x),
                                 fp8x2_bf16x2<false>(x.y), fp8x2_bf16x2<true>(x.y)};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vf[2 * e] = bf_lo(w[e]);
            vf[2 * e + 1] = bf_hi(w[e]);
          }
        } else {
          widen8<F>(x, vf);
        }
        const float *pr = pl + (i * RPS + rsub) * PST;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float p = pr[g];
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[g][e] = fmaf(p, vf[e], acc[g][e]);
        }
      });
      wave_lds_order();                          // the weights are read before the next tile's
      if (!more) break;
      t = tn;
      pg = pgn;
      kr = krn;
      vr = vrn;
    }
  }

  // ---- merge: the lanes that share a channel chunk, then the waves
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float lg = wave_sum(l[g]);
    if (lane == 0) {
      sm.m[wave][g] = m[g];
      sm.l[wave][g] = lg;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int off = 32; off >= NC; off >>= 1) acc[g][e] += __shfl_xor(acc[g][e], off);
  }
  __syncthreads();                               // every wave's weights are read
  if (lane < NC) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < 8; e += 4)
        *reinterpret_cast<float4 *>(&sm.u.acc[wave][g * D + c8 * 8 + e]) =
            make_float4(acc[g][e], acc[g][e + 1], acc[g][e + 2], acc[g][e + 3]);
  }
  __syncthreads();
  const int waves = min(NW, n_tiles - t_lo);     // those that had a tile
  const bool whole = n_tiles - t_lo == all_tiles;
  for (int i = threadIdx.x; i < G * D / 4; i += NW * 64) {
    const int g = i / (D / 4), c = (i % (D / 4)) * 4;
    float M = sm.m[0][g];
    for (int w = 1; w < waves; ++w) M = fmaxf(M, sm.m[w][g]);
    float L = 0.f;
    float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int w = 0; w < waves; ++w) {
      const float f = exp2f(sm.m[w][g] - M);
      const float4 x = *reinterpret_cast<const float4 *>(&sm.u.acc[w][g * D + c]);
      L += sm.l[w][g] * f;
      A.x += x.x * f;
      A.y += x.y * f;
      A.z += x.z * f;
      A.w += x.w * f;
    }
    const float inv = whole ? hd.v_scale / L : 1.0f;
    const size_t part = (size_t)(a.part_begin[rank] + split * a.part_seqs[rank] + si) * G + g;
    float *const to = whole ? a.out + (q_row + g) * D : a.part_acc + part * D;
    __builtin_nontemporal_store(f32x4_t{A.x * inv, A.y * inv, A.z * inv, A.w * inv},
                                reinterpret_cast<f32x4_t *>(to + c));
    if (!whole && c == 0)
      __builtin_nontemporal_store(f32x2_t{M, L}, reinterpret_cast<f32x2_t *>(a.part_ml + part * 2));
  }
}

// Merge of split items: one row of D / 4 lanes per (item, q head), a lane
// owning 4 channels; items of one split are written already.
template <int D, int G>
__global__ __launch_bounds__(256) void item_merge(ItemArgs a) {
  constexpr int LPR = D / 4;
  constexpr int RPW = 256 / LPR;                 // rows per workgroup
  const int row = blockIdx.x * RPW + threadIdx.x / LPR;   // (rank, sequence, q head)
  const int c = threadIdx.x % LPR * 4;
  const int rank = row / (a.n_seqs * G);
  if (rank >= a.n_kv_heads) return;
  const int si = row / G % a.n_seqs, g = row % G;
  const int h = a.head_order[rank], b = a.seq[si];
  const ItemHead &hd = a.head[h];
  const int tiles = (min(a.len[si], hd.cap) + 63) / 64;
  if (tiles <= a.tiles_per_wg) return;
  const int ns = (tiles + a.tiles_per_wg - 1) / a.tiles_per_wg;
  const size_t p0 = (size_t)(a.part_begin[rank] + si) * G + g;
  const size_t step = (size_t)a.part_seqs[rank] * G;   // the next split's partial
  float M = -INFINITY, L = 0.f;
  float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
  constexpr int U = 4;                           // splits per round, loads in flight
  for (int j0 = 0; j0 < ns; j0 += U) {
    float2 ml[U];
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t p = p0 + (size_t)min(j0 + u, ns - 1) * step;
      ml[u] = *reinterpret_cast<const float2 *>(a.part_ml + p * 2);
      x[u] = *reinterpret_cast<const float4 *>(a.part_acc + p * D + c);
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (j0 + u >= ns) ml[u].x = -INFINITY;
      Mn = fmaxf(Mn, ml[u].x);
    }
    const float f = exp2f(M - Mn);
    L *= f;
    A.x *= f;
    A.y *= f;
    A.z *= f;
    A.w *= f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float e = exp2f(ml[u].x - Mn);
      L += ml[u].y * e;
      A.x += x[u].x * e;
      A.y += x[u].y * e;
      A.z += x[u].z * e;
      A.w += x[u].w * e;
    }
    M = Mn;
  }
  const float inv = hd.v_scale / L;
  *reinterpret_cast<float4 *>(a.out + (((size_t)b * a.n_kv_heads + h) * G + g) * D + c) =
      make_float4(A.x * inv, A.y * inv, A.z * inv, A.w * inv);
}

}  // namespace
}  // namespace hwkv
