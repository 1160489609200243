// Decode attention over compressed K/V on the matrix cores (gfx950): both
// contractions of Algorithm 1 are MFMAs whose operands the lanes expand from the
// packed values in registers, four channels (a nibble of the bitmap) at a time.
//
// One wave per token segment, blocks of NB = 64 / T tokens (64 tiles, one per
// lane in the metadata steps). A nibble's kept values are at most four
// consecutive packed ones; two LDS dwords hold them (every LDS array of values
// is a sliding one, dword p = values p and p + 1, so a nibble may start at any
// value), and a 16-entry table gives the byte selectors with which two byte
// permutes put them in their channels, zeros elsewhere. Nothing is scattered,
// cleared or masked:
//   * keys: lane t of a tile loads its tile's values (16-byte pieces, each tile
//     starts at one) and writes them to a column of LDS rows, so that the reads
//     of different tiles never share a bank. Lane (token r, quad q) expands the
//     16 T channels of quad q of token r, eight at a time, which are the A
//     operand of v_mfma_f32_16x16x32_f16 (16 tokens x 32 channels); q is the B
//     operand (head columns), held in registers for the whole segment;
//   * softmax on the result layout (lane = head r, tokens 4 q + e): the scores
//     become the A operand of the second product in place (row = head);
//   * values: the block's run goes to LDS as it is; lane (quad q, column r)
//     expands channels 4 T r .. of its tokens 4 q + e and transposes them with
//     byte permutes into B operands (32 tokens x 16 channels).
// A block of 32 tokens at d = 128 costs about 380 vector and 100 LDS instructions
// (550 LDS cycles of the CU, bank conflicts included) at any number of query heads
// per kv-head; the walks spend 560 to 850 vector ones, and the kernel that scattered
// the values into dense tiles before its MFMAs spent 660. What bounds it is the LDS
// and, below about 6 blocks a wave, the latency of one block (1.5 us alone). 32
// streams of 16K tokens (70/70, warm): 30.6 us with 4 heads (walks 46.9) and 32.1
// with 8 (57.7 before), 3.7 TB/s of needed bytes with 4 heads (2.4); 512 streams of 32K at
// K 50% / V 70%: 750 us (822), 5.95 TB/s. Tried and left out: half the key columns
// at a time (12 waves a CU instead of 9 or 11: +10%), values in 8-byte loads
// (conflict-free LDS writes: even, +7% at 50%), the metadata loaded before the
// stream's count is known (even).
#include "attn_mfma.h"

namespace mf {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The probabilities enter the p.V product as fp16 with this exponent bias: the
// largest is 2^15 (inside fp16), and the small ones keep 15 more binades before they
// flush to zero. The running maximum is kept unscaled and subtracted before the
// scaling: the difference is zero for the largest score, whatever its size. (Against
// the rounded product max * scale the exponent of a large score's p came out up to
// half an ulp of that product above the bias, and p infinite.) The partial's l and
// o are scaled back, exactly.
constexpr float kMfmaPBias = 15.f;
constexpr float kMfmaPUnit = 0x1p-15f;

// Byte selectors of nibble n: channel c (kept) takes packed value popc(n below c)
// of the four at hand (bytes 2 pos, 2 pos + 1), a dropped one zero (selector 12).
__device__ __forceinline__ u32x2 nibble_selectors(uint32_t n) {
  uint32_t s[2] = {0u, 0u}, pos = 0u;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const bool kept = (n >> c) & 1u;
    const uint32_t h = kept ? (2u * pos + 1u) << 8 | 2u * pos : 0x0c0cu;
    s[c >> 1] |= h << (16 * (c & 1));
    pos += kept ? 1u : 0u;
  }
  return (u32x2){s[0], s[1]};
}

// The four channels of a nibble: t = 8 n, the packed values from dword address a
// on, dword stride STRIDE bytes (dwords p and p + 2 of a sliding array).
struct Nibble {
  uint32_t v0, v1;
  u32x2 sel;
};

template <uint32_t STRIDE>
__device__ __forceinline__ Nibble nibble_load(uint32_t t, uint32_t a) {
  Nibble x;
  x.v0 = lds_load<uint32_t>(a);
  x.v1 = lds_load<uint32_t>(a + 2u * STRIDE);
  x.sel = lds_load<u32x2>(t);  // the table is at LDS address 0
  return x;
}

__device__ __forceinline__ u32x2 nibble_expand(const Nibble& x) {
  return (u32x2){__builtin_amdgcn_perm(x.v1, x.v0, x.sel.x), __builtin_amdgcn_perm(x.v1, x.v0, x.sel.y)};
}

__device__ __forceinline__ half8_t as_h8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const u32x4 w = {a, b, c, d};
  return __builtin_bit_cast(half8_t, w);
}

// Wait states between a chain of MFMAs and the first vector use of its result
// (11 for these products). The compiler inserts them within a block only: where
// a branch follows the chain, its target would read the result too early.
template <int N>
__device__ __forceinline__ void mfma_settle(f32x4 (&r)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(r[i]));
  asm volatile("s_nop 15" : "+v"(r[0]));
}

// Even and odd nibbles of a word, each times 8 in a byte of its own.
// (Opaque results: the compiler would otherwise shift and mask the word again
// for every nibble instead of extracting a byte.)
__device__ __forceinline__ uint32_t even_nibbles8(uint32_t x) {
  uint32_t r = (x << 3) & 0x78787878u;
  asm("" : "+v"(r));
  return r;
}
__device__ __forceinline__ uint32_t odd_nibbles8(uint32_t x) {
  uint32_t r = (x >> 1) & 0x78787878u;
  asm("" : "+v"(r));
  return r;
}

// The values that follow w0 of every lane: the next lane's w0, for lane 63 the
// next piece's first (next: any lane's register of that piece).
__device__ __forceinline__ uint32_t lane_next(uint32_t w0, uint32_t next) {
  return (uint32_t)__builtin_amdgcn_update_dpp(__builtin_amdgcn_readfirstlane((int)next), (int)w0, 0x130, 0xf, 0xf,
                                               false);  // wave_shl:1
}

template <int T, int G, int KP, int VC>
__device__ __forceinline__ void sparse_body_mfma(const AttnArgs& a, const MfmaLds& L, int seg, int bh,
                                                 float& m_run, float& l_run,
                                                 f32x4 (&o)[MfmaGeom<T>::NO]) {
  using Geo = MfmaGeom<T>;
  constexpr int d = kTile * T;
  constexpr int NB = Geo::NB, NG = Geo::NG, NC = Geo::NC, NO = Geo::NO;
  const uint32_t lane = lane_id();
  const uint32_t r16 = lane % 16, q4 = lane / 16;

  const int j0 = seg * a.sparse_seg_tokens;
  const int j1 = min(j0 + a.sparse_seg_tokens, stream_tokens(a, bh));
  if (j0 >= j1) return;  // past this stream's tokens: an empty partial
  const int64_t kt0 = (int64_t)bh * a.K.cap_tokens * T;
  const int64_t vt0 = (int64_t)bh * a.V.cap_tokens * T;
  const uint16_t* kv = a.K.values + (int64_t)bh * a.K.val_stride;
  const uint16_t* vv = a.V.values + (int64_t)bh * a.V.val_stride;
  int nb = min(NB, j1 - j0);
  TileMeta cur = load_meta<T>(a, kt0, vt0, j0, nb, lane);
  RunPos pos = segment_start<T>(a, kt0, vt0, j0);

  // q as the B operand: column r16 = head (zero past G), k = 8 q4 + i = channel
  // 16 T quad + 8 c + i, where quad q4 owns the 16 T channels 16 T quad .. (at
  // T = 2 in the order tile 0 lower half, tile 1 lower, tile 0 upper, tile 1
  // upper: the 32 lanes of an LDS pass then read 32 different tiles' columns).
  const uint32_t quad = T == 2 ? (q4 & 1u) * 2u + (q4 >> 1) : q4;
  half8_t qb[NC];
  {
    const uint16_t* qsrc = a.q + ((int64_t)bh * G + (r16 < (uint32_t)G ? r16 : 0u)) * d + 16 * T * quad;
    const uint32_t keep = r16 < (uint32_t)G ? 0xffffffffu : 0u;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const u32x4 w = *reinterpret_cast<const u32x4*>(qsrc + 8 * c);
      qb[c] = as_h8(w.x & keep, w.y & keep, w.z & keep, w.w & keep);
    }
  }
  if (lane < 16u) lds_store<u32x2>(8u * lane, nibble_selectors(lane));

  // Per-lane constants of the key expansion: the tile of quad q4 (as a lane
  // of the metadata steps, group 0) and what of the tile lies below its channels.
  const uint32_t ktile = r16 * T + (T == 4 ? q4 : T == 2 ? q4 & 1u : 0u);
  const uint32_t kcol = L.kv + 4u * ktile;
  const uint32_t vent = L.ent + 4u * q4 * kEntRow + 4u * r16;

  Runs rn = runs_of(cur, pos);
  u32x4 ks[KP], vs[VC];
  // Key pieces: 16-byte piece c of this lane's tile. A lane whose tile ends before
  // reads what follows it (never used, and in the cache for that tile's lane;
  // cached loads, as a line's pieces are taken by several loads: non-temporal
  // ones took 5% longer). Past the run the descriptor returns zeros. Unconditional
  // loads: skipping the pieces that no lane needs took 2% longer at 50% sparsity.
  auto issue_keys = [&](const TileMeta& m, const Runs& r) {
    const __amdgpu_buffer_rsrc_t rk = run_rsrc(kv + r.kstart, r.kn);
#pragma unroll
    for (int c = 0; c < KP; ++c) ks[c] = __builtin_amdgcn_raw_buffer_load_b128(rk, 2u * m.ko + 16u * c, 0, 0);
  };
  auto issue_values = [&](const Runs& r) {
    const __amdgpu_buffer_rsrc_t rv = run_rsrc(vv + r.vstart, r.vn);
#pragma unroll
    for (int c = 0; c < VC; ++c)
      vs[c] = __builtin_amdgcn_raw_buffer_load_b128(rv, 16u * lane, 2u * kChunk * (uint32_t)c, kLoadNT);
  };
  issue_keys(cur, rn);
  issue_values(rn);
  int nb_next = min(NB, j1 - (j0 + NB));
  TileMeta nxt = {0ull, 0ull, 0u, 0u};
  if (nb_next > 0) nxt = load_meta<T>(a, kt0, vt0, j0 + NB, nb_next, lane);

  for (int b0 = j0; b0 < j1; b0 += NB) {
    const int nb_next2 = min(NB, j1 - (b0 + 2 * NB));
    // Keys to their columns: row 8 c + i of a tile's column holds its values
    // 8 c + i and 8 c + i + 1.
    {
      const uint32_t n = (uint32_t)__popcll(cur.kb);
      const uint32_t col = L.kv + 4u * lane;
#pragma unroll
      for (int c = 0; c < KP; ++c) {
        if (c > 0 && !ballot(n > 8u * c)) break;
        const uint32_t w[5] = {ks[c].x, ks[c].y, ks[c].z, ks[c].w, c + 1 < KP ? ks[c + 1 < KP ? c + 1 : c].x : 0u};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          lds_store<uint32_t>(col + (8u * c + 2u * i) * kColRow, w[i]);
          lds_store<uint32_t>(col + (8u * c + 2u * i + 1u) * kColRow, __builtin_amdgcn_alignbit(w[i + 1], w[i], 16u));
        }
      }
    }
    Runs rnext = {0u, 0u, 0u, 0u};
    if (nb_next > 0) rnext = runs_of(nxt, pos);
    issue_keys(nxt, rnext);

    // Scores: S[group g][token 4 q4 + e][head r16].
    f32x4 sc[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      sc[g] = (f32x4){0.f, 0.f, 0.f, 0.f};
      const int src = (int)(4u * (ktile + 16u * T * g));
      const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)cur.kb);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)(cur.kb >> 32));
      const uint32_t col = kcol + 4u * 16u * T * g;
      uint32_t rank, word[T == 4 ? 2 : 1];
      if constexpr (T == 1) {
        const uint32_t lo16 = __popc(lo & 0xffffu), nlo = __popc(lo), hi16 = nlo + __popc(hi & 0xffffu);
        word[0] = ((q4 & 2u) ? hi : lo) >> (16u * (q4 & 1u)) & 0xffffu;
        rank = (q4 & 2u) ? ((q4 & 1u) ? hi16 : nlo) : ((q4 & 1u) ? lo16 : 0u);
      } else if constexpr (T == 2) {
        word[0] = (q4 & 2u) ? hi : lo;
        rank = (q4 & 2u) ? (uint32_t)__popc(lo) : 0u;
      } else {
        word[0] = lo;
        word[T == 4 ? 1 : 0] = hi;
        rank = 0u;
      }
      // Up to eight nibbles' LDS loads in flight before the first is used.
      constexpr int CB = NC < 4 ? NC : 4;
      uint32_t ev = 0u, od = 0u;
#pragma unroll
      for (int c0 = 0; c0 < NC; c0 += CB) {
        Nibble nib[2 * CB];
#pragma unroll
        for (int c = c0; c < c0 + CB; ++c) {
          if (c % 4 == 0) {
            ev = even_nibbles8(word[c / 4]);
            od = odd_nibbles8(word[c / 4]);
          }
          const uint32_t t0 = ev >> (8 * (c % 4)) & 0xffu, t1 = od >> (8 * (c % 4)) & 0xffu;
          nib[2 * (c - c0)] = nibble_load<kColRow>(t0, col + kColRow * rank);
          rank += __popc(t0);
          nib[2 * (c - c0) + 1] = nibble_load<kColRow>(t1, col + kColRow * rank);
          rank += __popc(t1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = c0; c < c0 + CB; ++c) {
          const u32x2 e0 = nibble_expand(nib[2 * (c - c0)]), e1 = nibble_expand(nib[2 * (c - c0) + 1]);
          sc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(e0.x, e0.y, e1.x, e1.y), qb[c], sc[g], 0, 0, 0);
        }
      }
    }

    mfma_settle(sc);

    // Online softmax per head (lanes with the same r16 share a head); tokens past
    // the block end score -inf.
    if (nb < NB) {
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (16 * g + 4 * (int)q4 + e >= nb) sc[g][e] = -INFINITY;
    }
    float bmax = -INFINITY;
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) bmax = fmaxf(bmax, sc[g][e]);
    if (ballot(bmax > m_run)) {
      bmax = fmaxf(bmax, __shfl_xor(bmax, 16, kWave));
      bmax = fmaxf(bmax, __shfl_xor(bmax, 32, kWave));
      const float mnew = fmaxf(m_run, bmax);
      const float alpha = __builtin_amdgcn_exp2f((m_run - mnew) * a.scale_log2);  // the scale is positive
      m_run = mnew;
      l_run *= alpha;
      // Row 4 q4 + e of every O tile is head 4 q4 + e.
      float ar[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) ar[e] = __shfl(alpha, (int)(4u * q4) + e, kWave);
#pragma unroll
      for (int c = 0; c < NO; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[c][e] *= ar[e];
    }
    // p = exp2((s - max) scale + kMfmaPBias) in fp16 (at most 2^15); the sum is taken
    // over the same rounded p that the p.V product multiplies (per lane, reduced
    // at the segment's end).
    half4_t pa[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
#pragma unroll
      for (int e = 0; e < 4; ++e) pa[g][e] = (_Float16)__builtin_amdgcn_exp2f(fmaf(sc[g][e] - m_run, a.scale_log2, kMfmaPBias));
      const half2_t one = {(_Float16)1.f, (_Float16)1.f};
      l_run = __builtin_amdgcn_fdot2((half2_t){pa[g][0], pa[g][1]}, one, l_run, false);
      l_run = __builtin_amdgcn_fdot2((half2_t){pa[g][2], pa[g][3]}, one, l_run, false);
    }

    // Values over the consumed keys: dword p = values p and p + 1 of the run.
    {
#pragma unroll
      for (int c = 0; c < VC; ++c) {
        if (kChunk * c >= rn.vn) break;
        const uint32_t w4 = lane_next(vs[c].x, c + 1 < VC ? vs[c + 1 < VC ? c + 1 : c].x : 0u);
        const uint32_t w[5] = {vs[c].x, vs[c].y, vs[c].z, vs[c].w, w4};
        uint32_t od[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) od[i] = __builtin_amdgcn_alignbit(w[i + 1], w[i], 16u);
        const uint32_t dst = L.kv + 4u * kChunk * c + 32u * lane;
        lds_store<u32x4>(dst, (u32x4){w[0], od[0], w[1], od[1]});
        lds_store<u32x4>(dst + 16u, (u32x4){w[2], od[2], w[3], od[3]});
      }
    }
    // Entries: lane (token j, tile t) gives every column of its tile the dword
    // address of its first value (high half) and its nibbles (low half).
    {
      const uint32_t j = lane / T, t = lane % T;
      uint32_t row = L.ent + j * kEntRow + t * (64u / T);
      uint32_t r = cur.vo + L.kv / 4u;  // dword index of the next value
      const uint32_t w[2] = {(uint32_t)cur.vb, (uint32_t)(cur.vb >> 32)};
      uint32_t ent[16 / T], ev = 0u, od = 0u;
#pragma unroll
      for (int i = 0; i < 16 / T; ++i) {
        if (T < 4 && i % (8 / T) == 0) {
          ev = even_nibbles8(w[i * T / 8]);
          od = odd_nibbles8(w[i * T / 8]);
        }
        uint32_t bits;
        if constexpr (T == 1)
          bits = ((i & 1) ? od : ev) >> (8 * (i % 8 / 2)) & 0xffu;
        else if constexpr (T == 2)
          bits = __builtin_amdgcn_perm(od, ev, 0x0c0c0400u + 0x0101u * (uint32_t)(i % 4));
        else
          bits = w[i / 2] >> (16 * (i % 2)) & 0xffffu;
        ent[i] = r << 18 | bits;
        r += __popc(bits);
      }
#pragma unroll
      for (int i = 0; i < 16 / T; i += 4)
        lds_store<u32x4>(row + 4u * i, (u32x4){ent[i], ent[i + 1], ent[i + 2], ent[i + 3]});
    }
    issue_values(rnext);
    TileMeta nxt2 = {0ull, 0ull, 0u, 0u};
    if (nb_next2 > 0) nxt2 = load_meta<T>(a, kt0, vt0, b0 + 2 * NB, nb_next2, lane);

    // p.V: O[head][channel NO r16 + c] += P[head][32 tokens] . V. Steps of 32
    // tokens (two score groups; 16 at T = 4): token i of this lane is 4 q4 + i of
    // the first group, then of the second.
    constexpr int TS = NG >= 2 ? 8 : 4;          // tokens per lane and step
#pragma unroll
    for (int st = 0; st < (NG >= 2 ? NG / 2 : 1); ++st) {
      uint32_t ent[TS], ad[TS];
#pragma unroll
      for (int i = 0; i < TS; ++i) {
        ent[i] = lds_load<uint32_t>(vent + (32u * st + (i < 4 ? i : 12 + i)) * kEntRow);
        ad[i] = ent[i] >> 16;
      }
#pragma unroll
      for (int n = 0; n < T; ++n) {              // nibbles of the column
        Nibble nib[TS];
#pragma unroll
        for (int i = 0; i < TS; ++i) {
          const uint32_t t = T == 4 ? (n == 0 ? ent[i] << 3 : ent[i] >> (4 * n - 3)) & 0x78u : ent[i] >> (8 * n) & 0xffu;
          nib[i] = nibble_load<4u>(t, ad[i]);
          ad[i] += 4u * __popc(t);
        }
        __builtin_amdgcn_sched_barrier(0);
        u32x2 x[TS];
#pragma unroll
        for (int i = 0; i < TS; ++i) x[i] = nibble_expand(nib[i]);
        // Transpose: channel c of the nibble for the lane's tokens, in pairs.
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          uint32_t y[TS / 2];
#pragma unroll
          for (int i = 0; i < TS / 2; ++i)
            y[i] = __builtin_amdgcn_perm(x[2 * i + 1][c >> 1], x[2 * i][c >> 1], (c & 1) ? 0x07060302u : 0x05040100u);
          if constexpr (TS == 8) {
            const half4_t p0 = pa[2 * st], p1 = pa[2 * st + 1 < NG ? 2 * st + 1 : 0];
            const half8_t pv = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
            o[4 * n + c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pv, as_h8(y[0], y[1], y[TS / 2 - 2], y[TS / 2 - 1]),
                                                                  o[4 * n + c], 0, 0, 0);
          } else {
            const u32x2 yy = {y[0], y[1]};
            o[4 * n + c] = __builtin_amdgcn_mfma_f32_16x16x16f16(pa[0], __builtin_bit_cast(half4_t, yy), o[4 * n + c], 0, 0, 0);
          }
        }
      }
    }
    cur = nxt;
    rn = rnext;
    nxt = nxt2;
    nb = nb_next;
    nb_next = nb_next2;
  }
  mfma_settle(o);
  l_run += __shfl_xor(l_run, 16, kWave);
  l_run += __shfl_xor(l_run, 32, kWave);
}

// Sparse call on the matrix cores: grid (n_sparse_segs + n_dense_segs, BHkv).
template <int T, int G, int KP, int VC>
__global__ __launch_bounds__(64, mfma_waves(T, KP)) void k_sparse_attn_mfma(AttnArgs a, MfmaLds L) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int seg = blockIdx.x, bh = blockIdx.y;
  if (seg >= a.n_sparse_segs) {
    float m_run[G], l_run[G], od[G][T];
    init_state<T, G>(m_run, l_run, od);
    dense_body<T, G>(a, seg - a.n_sparse_segs, bh, smem, m_run, l_run, od);
    write_partial<T, G>(a, seg, bh, m_run, l_run, od);
    return;
  }
  using Geo = MfmaGeom<T>;
  constexpr int d = kTile * T;
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o[Geo::NO];
#pragma unroll
  for (int c = 0; c < Geo::NO; ++c) o[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
  sparse_body_mfma<T, G, KP, VC>(a, L, seg, bh, m_run, l_run, o);
  m_run *= a.scale_log2;  // -inf stays -inf for an empty segment
  l_run *= kMfmaPUnit;

  const uint32_t lane = lane_id();
  const uint32_t r16 = lane % 16, q4 = lane / 16;
  const int64_t row0 = (int64_t)seg * a.BHq + (int64_t)bh * G;
  if (q4 == 0 && r16 < (uint32_t)G) a.ws_ml[row0 + r16] = make_float2(m_run, l_run);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t h = 4u * q4 + (uint32_t)e;
    if (h < (uint32_t)G) {
      f32x4* dst = reinterpret_cast<f32x4*>(a.ws_o + (row0 + h) * d + Geo::NO * r16);
#pragma unroll
      for (int n = 0; n < T; ++n) dst[n] = (f32x4){o[4 * n][e], o[4 * n + 1][e], o[4 * n + 2][e], o[4 * n + 3][e]} * kMfmaPUnit;
    }
  }
}

template <int T, int G, int KP, int VC>
static hipError_t mfma_launch(const AttnShape& sh, const AttnArgs& a, int kpieces, int vchunks, hipStream_t s) {
  const MfmaLds L = mfma_lds_layout<T>(kpieces, vchunks);
  size_t lds = L.total;
  if (sh.n_dense_segs > 0 && dense_lds_bytes(T, G) > lds) lds = dense_lds_bytes(T, G);
  hipLaunchKernelGGL((k_sparse_attn_mfma<T, G, KP, VC>), dim3(sh.n_sparse_segs + sh.n_dense_segs, sh.BHkv),
                     dim3(kWave), lds, s, a, L);
  return hipGetLastError();
}

template <int T, int G>
static hipError_t mfma_stage(const AttnShape& sh, const AttnArgs& a, hipStream_t s) {
  int kp, vc;
  mfma_staging(T, a.K, a.V, &kp, &vc);
  if (kp <= 5 && vc <= 3) return mfma_launch<T, G, 5, 3>(sh, a, kp, vc, s);
  if (vc <= 3) return mfma_launch<T, G, 8, 3>(sh, a, kp, vc, s);
  if (vc <= 5) return mfma_launch<T, G, 8, 5>(sh, a, kp, vc, s);
  return mfma_launch<T, G, 8, 8>(sh, a, kp, vc, s);
}

template <int T>
static hipError_t mfma_T(const AttnShape& sh, const AttnArgs& a, hipStream_t s) {
  switch (sh.G) {
    case 1: return mfma_stage<T, 1>(sh, a, s);
    case 2: return mfma_stage<T, 2>(sh, a, s);
    case 4: return mfma_stage<T, 4>(sh, a, s);
    case 8: return mfma_stage<T, 8>(sh, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_sparse_mfma(const AttnShape& sh, const AttnArgs& a, hipStream_t s) {
  switch (sh.T) {
    case 1: return mfma_T<1>(sh, a, s);
    case 2: return mfma_T<2>(sh, a, s);
    case 4: return mfma_T<4>(sh, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mf
