// Backward pass of the value-distillation loss through the maps 128 -> 256 -> 256 (the paper's default widths, Tab. "phi", P = 2),
// gfx950 only.  Mathematics and notation: ha_grad.hip.
//
//   back256_kernel      per 32 tokens and wave, all in registers: h = relu(W1 x + b1), the activations t of W2 h + b2, dphi = M u rs + wz z,
//                       du, dpre = (W2^T du) [h > 0].  What the products over the tokens need leaves as bf16 register images (layout:
//                       ha_wide.hip): h, du, dpre, over the queries phi_q / den, and x where it has to be rounded.
//   contract256_kernel  the sums over the tokens [dW2 | db2] = du [h | 1]^T, [dW1 | db1] = dpre [x | 1]^T and, over the queries,
//                       [dS | dz] = (phi_q / den) [g | dden den]^T, each from partial tiles per range of tokens
//   reduce256_kernel    fixed-order sum of the partial tiles; dS as operand fragments for the key side
//   prep256_kernel      weight fragments of both maps, W2^T and S as fragments, in one launch
// (the layer-by-layer passes of ha_wide_grad.hip, 14 launches more, took 1520 us behind the forward at 480p / 81 frames, 12 heads, R = 4; these
// take 875.  H = 1, N = 200, R = 2: the whole step 208 -> 146 us; B = 2, H = 8, N = 2000, R = 8: 381 -> 240.)
#include <type_traits>

#include "ha_mlp256.h"
#include "ha_plan.h"

namespace ha {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

struct Back256Args {
  const void *x;                      // q or k rows (io dtype, strided)
  const void *u;                      // queries: sign tensor, bf16 dense [B*H][N][D]; keys: v rows (io dtype, strided)
  const float *rs, *wp;               // queries: [B*H][N]
  const bf16x8 *w1f, *w2f, *w2tf;     // per head
  const float *b1, *b2;               // per head, may be null
  const bf16x8 *m_hi, *m_lo;          // [B*H][F*D/8]: natural-order fragments of S (queries) or dS (keys)
  const float *zvec;                  // [B*H][F]
  bf16x8 *h_img, *du_img, *dpre_img;  // [B*H][n_tb][8][2][64]
  bf16x8 *phi_img;                    // queries: phi_q / den
  __bf16 *x_img;                      // fp32 io: x in bf16, dense rows [B*H][32 n_tb][128]
  int H, N, n_tok, n_tb, R, G, P, act;
  int n_tiles, total, run;            // tiles of 128 tokens per (batch, head), overall, and per workgroup
  int64_t sb, sh, sn;
};

// ------------------------------------------------------------------------------------------------
// back256_kernel: persistent, two workgroups of four waves per CU, a wave has 32 tokens of a 128-token tile.  Everything between the rows
// and the images stays in registers; W1, W2, M (S or dS, hi + lo) and W2^T, 448 KiB per head, stream through an LDS ring of three slabs that
// runs ahead across tiles and heads: a hidden block of the map per step (24 KiB, see ha_mlp256.h), then a block of 32 features or hidden
// units per step (16 KiB).  The softmax's Jacobian needs the sum of t dt over all channels before the first du: t (128 registers) and dphi
// (128) do not fit a wave at two waves per SIMD, so M meets the rows twice, once for the sum.
// Bound: matrix and vector instructions of a SIMD together, 704 products of 32 cycles per wave and tile (42 % of the cycles at 2.0 GHz) and 2800
// vector instructions (30 %).  Among these, and not counted as work: some 220 scalar registers that are spilled to lanes of vector registers (addresses
// of slabs and images; 292 v_readlane and 220 v_writelane in the body of the measured instance, 134 null checks of the LDS pointers that the
// requests cast), in the fp32 query instances two vector registers in scratch as well.  With its image stores left out it takes 272 us of 310; eight waves of one workgroup (256 tokens, ring of four
// slabs) took 304 and four waves with a SIMD each 379.
// Measured at 480p / 81 frames, 12 heads: queries 310 us, linear keys (R = 4) 240; as the three passes it replaces (the layers run again,
// dphi, W2^T du), which passed pre-activations, du and h through HBM, 555 and 417.
// PC: the degree (it divides 256), 0: any (not with the softmax, ACT0).
template <bool F32, bool QUERY, bool ACT0, int PC>
__global__ __launch_bounds__(256, 2) void back256_kernel(Back256Args a) {
  constexpr int D = 128, HD = 256, F = 256, KS = D / 16, HB = HD / 32, FB = F / 32, NW = 4;
  constexpr int NBUF = 3, SLOT = kSlabChunks * 64;        // slabs of up to 24 KiB
  constexpr int STEP_A = HB, STEP_B = STEP_A + (ACT0 ? FB : 0), STEP_C = STEP_B + FB, STEPS = STEP_C + HB;
  constexpr int NW1 = HD * D / 8, NW2 = F * HD / 8, NST = D * F / 8;
  __shared__ bf16x8 ring[NBUF * SLOT];
  __shared__ __align__(16) float vecs[HD + 2 * F];        // b1, b2, z
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwg = gridDim.x;                              // a multiple of 8
  const int wg = (blockIdx.x & 7) * (nwg >> 3) + (blockIdx.x >> 3);
  const int t_lo = wg * a.run, t_hi = min(t_lo + a.run, a.total);
  if (t_lo >= t_hi) return;

  // slab `s` of a tile of (batch, head) bh -> ring slot; chunks are dealt round-robin to the waves
  const unsigned lane_off = lane * 16;
  auto request = [&](int bh, int s, int slot) {
    const int h = bh % a.H;
    auto dma = [&](const bf16x8 *gp, int c) {
      const unsigned l = __builtin_amdgcn_readfirstlane(
          (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)(&ring[slot * SLOT + c * 64]));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(gp) : "memory");
    };
    if (s < STEP_A) {
#pragma unroll
      for (int i = 0; i < kSlabChunks / NW; ++i) {
        const int c = i * NW + w;
        dma(slab_chunk(a.w1f + (int64_t)h * NW1, a.w2f + (int64_t)h * NW2, s, c), c);
      }
    } else if (s < STEP_C) {                              // M of a feature block: 8 fragments of the hi part, 8 of the lo part
      const int fb = (s - STEP_A) & (FB - 1);
#pragma unroll
      for (int i = 0; i < 16 / NW; ++i) {
        const int c = i * NW + w;
        dma((c < 8 ? a.m_hi : a.m_lo) + (int64_t)bh * NST + (fb * KS + (c & 7)) * 64, c);
      }
    } else {                                              // W2^T of a hidden block
#pragma unroll
      for (int i = 0; i < 16 / NW; ++i) {
        const int c = i * NW + w;
        dma(a.w2tf + (int64_t)h * NW2 + ((s - STEP_C) * 16 + c) * 64, c);
      }
    }
  };
  // Barrier ahead of a slab: this wave's share of it has landed and so has everybody's, and everybody is done with the slab
  // before it, whose slot takes the request NBUF - 1 slabs ahead.  What a wave has issued since it requested the slab may stay in
  // flight (loads and stores retire in order): the request of the newer slab and the stores of the last two steps, which every
  // wave makes (one whose tokens are past the end writes a block that nobody reads).  The steps of the hidden layer count no
  // more than their own kind, and none in front of a workgroup's first tile.
  static_assert(NBUF == 3, "one newer slab, two steps");
  constexpr auto n_req = [](int s) { return (s % STEPS < STEP_A ? kSlabChunks : 16) / NW; };
  constexpr auto n_st = [](int s) { return s < STEP_A ? 2 : s < STEP_B ? 0 : s < STEP_C ? (QUERY ? 4 : 2) : 2; };
  int slot = 0;
  int bh = t_lo / a.n_tiles, bh_next = bh;
  auto advance = [&](auto step_c, int step, bool stored) {
    constexpr int SC = decltype(step_c)::value;           // the step where it is known, -1 in the hidden layer
    constexpr int REQ = SC < 0 ? n_req(STEP_A) : n_req(SC + 1);
    constexpr int FLY = REQ + (SC < 0 ? 2 * n_st(0) : n_st(SC - 2) + n_st(SC - 1));
    static_assert(FLY < 63, "vmcnt immediate too large");
    if (SC < 0 && !stored) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(REQ) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FLY) : "memory");
    __syncthreads();
    const int s = step + NBUF - 1;
    request(s < STEPS ? bh : bh_next, s < STEPS ? s : s - STEPS, slot == 0 ? NBUF - 1 : slot - 1);   // (past the last tile: slabs nobody reads)
    const lds_frag_ptr sl = (lds_frag_ptr)&ring[slot * SLOT];
    slot = slot == NBUF - 1 ? 0 : slot + 1;
    return sl;
  };
  const LinearMap lmap(a.R, a.G);
  auto token_of = [&](int i) {                            // rows past the end repeat the last token
    const int at = min(i, a.n_tok - 1);
    return QUERY ? at : lmap.token(at);
  };
  auto base_of = [&](int b) { return (int64_t)(b / a.H) * a.sb + (int64_t)(b % a.H) * a.sh; };
  bf16x8 xf[KS];
  auto load_x = [&](int t) {
    const int b = t / a.n_tiles;
    const int tok = token_of((t - b * a.n_tiles) * 32 * NW + 32 * w + r);
    const int64_t base = base_of(b) + (int64_t)tok * a.sn + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xf[ks] = load8<F32>(a.x, base + 16 * ks);
  };
  load_x(t_lo);
#pragma unroll
  for (int s = 0; s < NBUF - 1; ++s) request(bh, s, s);
  const float *b1 = &vecs[0], *b2 = &vecs[HD], *zz = &vecs[HD + F];

  // A chain of 16 products from a slab; a fragment is requested NF - 1 products ahead of its own.
  auto chain = [&](auto nf_c, lds_frag_ptr sl, auto frag_of, auto operand, f32x16 &acc) {
    constexpr int NF = decltype(nf_c)::value;
    bf16x8 fr[NF];
#pragma unroll
    for (int f = 0; f < NF - 1; ++f) fr[f] = frag_at(sl, frag_of(f), lane);
#pragma unroll
    for (int f = 0; f < 16; ++f) {
      if (f + NF - 1 < 16) fr[(f + NF - 1) % NF] = frag_at(sl, frag_of(f + NF - 1), lane);
      if (f % 2 == 0) HA_FENCE();
      acc = mfma32(fr[f % NF], operand(f), acc);
    }
    HA_FENCE();
  };

  auto each8 = [](auto f) {
    static_assert(FB == 8 && HB == 8 && (PC != 0 || !ACT0), "eight blocks; the softmax with its degree compiled in");
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
    f(std::integral_constant<int, 4>{});
    f(std::integral_constant<int, 5>{});
    f(std::integral_constant<int, 6>{});
    f(std::integral_constant<int, 7>{});
  };
  // (scalar base, lane offset: per-lane pointers to four images would not fit the registers)
  auto store_piece = [&](bf16x8 *image, int64_t at, const u32x4 &v) {
    *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(image + at) + lane_off) = v;
  };
  int bh_vecs = -1;
  for (int t = t_lo; t < t_hi; ++t) {
    bh_next = t + 1 < t_hi ? (t + 1) / a.n_tiles : bh;
    if (bh != bh_vecs) {                                  // workgroup-uniform: the first tile, or the head changes
      const int h = bh % a.H;
      __syncthreads();                                    // every wave is done with the previous head's vectors
      for (int i = tid; i < HD; i += 64 * NW) vecs[i] = a.b1 ? a.b1[(int64_t)h * HD + i] : 0.f;
      for (int i = tid; i < F; i += 64 * NW) vecs[HD + i] = a.b2 ? a.b2[(int64_t)h * F + i] : 0.f;
      for (int i = tid; i < F; i += 64 * NW) vecs[HD + F + i] = a.zvec[(int64_t)bh * F + i];
      bh_vecs = bh;
      __syncthreads();
    }
    const int tb = (t - bh * a.n_tiles) * NW + w;
    const bool live = tb < a.n_tb, valid = 32 * tb + r < a.n_tok;
    const int64_t img = (live ? (int64_t)bh * a.n_tb + tb : (int64_t)(a.total / a.n_tiles) * a.n_tb) * (FB * 128);   // (past the end: the block behind the images)
    if constexpr (F32) {
      if (live)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          *reinterpret_cast<bf16x8 *>(a.x_img + ((int64_t)(bh * a.n_tb + tb) * 32 + r) * D + 16 * ks + 8 * g) = xf[ks];
    }
    // ---------------- the map: u = W2 relu(W1 x + b1) + b2, one hidden block per slab; the ReLU gate as one bit per hidden unit
    // (word i of a block's eight: bits i and 16 + i, the second block of a pair 8 further up)
    f32x16 u[FB];
    unsigned gate[HB / 2];
#pragma unroll
    for (int i = 0; i < HB / 2; ++i) gate[i] = 0u;
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) u[fb] = column_tile(b2, fb, g);
#pragma unroll 1
    for (int hp = 0; hp < HB / 2; ++hp) {
      unsigned bits = 0u;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int hb = 2 * hp + e;
        const lds_frag_ptr sl = advance(std::integral_constant<int, -1>{}, hb, t > t_lo || hp > 0);
        u32x4 h_hi[2], h_lo[2];
        hidden_block(sl, b1, hb, xf, lane, g, h_hi, h_lo);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          store_piece(a.h_img, img + (2 * hb + s) * 64, h_hi[s]);
#pragma unroll
          for (int i = 0; i < 4; ++i)                     // h >= 0: positive unless its bf16 pattern is a zero
            bits |= __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(u16x2, h_hi[s][i] & 0x7fff7fffu), u16x2{1, 1})) << (8 * e + 4 * s + i);
        }
        hidden_to_outputs<8>(sl + 8 * 64, __builtin_bit_cast(bf16x8, h_hi[0]), __builtin_bit_cast(bf16x8, h_hi[1]),
                             __builtin_bit_cast(bf16x8, h_lo[0]), __builtin_bit_cast(bf16x8, h_lo[1]), lane, u);
      }
#pragma unroll
      for (int i = 0; i + 1 < HB / 2; ++i) gate[i] = gate[i + 1];
      gate[HB / 2 - 1] = bits;
    }
    // ---------------- the rows that M meets, and their factors; they travel under the output stage
    bf16x8 uf[KS];
    float rs_ = 1.f, wp_ = 1.f;
    {
      const int tok = token_of(32 * tb + r);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if constexpr (QUERY) uf[ks] = static_cast<const bf16x8 *>(a.u)[((int64_t)bh * a.N + tok) * (D / 8) + 2 * ks + g];
        else uf[ks] = load8<F32>(a.u, base_of(bh) + (int64_t)tok * a.sn + 16 * ks + 8 * g);
      }
      if constexpr (QUERY) {
        rs_ = a.rs[(int64_t)bh * a.N + tok];
        wp_ = a.wp[(int64_t)bh * a.N + tok];
      }
    }
    // ---------------- the positive activation t = inv u, before the slice powers (u: of the softmax the exponentials)
    float inv = 1.f;
    if constexpr (ACT0) {
      float m = -INFINITY;
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int x = 0; x < 16; ++x) m = fmaxf(m, u[fb][x]);
      const float off = -xhalf_max(m) * kLog2e;
      float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          u[fb][x] = fast_exp2(__builtin_fmaf(u[fb][x], kLog2e, off));
          sum[x & 3] += u[fb][x];
        }
      inv = 1.0f / xhalf_sum((sum[0] + sum[1]) + (sum[2] + sum[3]));
    } else {
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int x = 0; x < 16; ++x) u[fb][x] = a.act == 1 ? fast_exp2(u[fb][x] * kLog2e) : relu(u[fb][x]);
    }
    // (the compiler's wait for these rows falls here, and not behind a newer request of slabs, which it does not know of)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(uf[ks]));
    asm volatile("" : "+v"(rs_), "+v"(wp_));
    rs_ = valid ? rs_ : 0.f;                              // rows past the end contribute nothing
    // t^e and its factor in the derivative, e + 1, for register group q of tile fb (channels 32 fb + 8 q ..: wave-uniform)
    // (any degree: through a value the compiler cannot see through, so that no exponent is kept across the tile)
    auto extra_of = [&](int fb, int q) { return PC ? (32 * fb + 8 * q) * PC / F : ((32 * fb + 8 * q) * (a.P + opaque_zero())) / F; };
    auto power = [&](float v, int e) {
      const float v2 = v * v;
      float p = (e & 1) ? v : 1.f;
      p = (e & 2) ? p * v2 : p;
      return (e & 4) ? p * (v2 * v2) : p;
    };
    // dphi / rs = M u + wp z of feature block fb: the lo part's products first
    auto dphi = [&](lds_frag_ptr sl, int fb, f32x16 &acc) {
      acc = column_tile(zz, fb, g);
#pragma unroll
      for (int x = 0; x < 16; ++x) acc[x] *= wp_;
      chain(std::integral_constant<int, 6>{}, sl, [](int f) { return (f & 1) * -8 + 8 + (f >> 1); }, [&](int f) { return uf[f >> 1]; }, acc);
    };
    auto put = [&](u32x4 (&half)[2], int q, const float (&v)[4]) {   // register group q of a tile
      half[q >> 1][2 * (q & 1)] = pack_bf16(v[0], v[1]);
      half[q >> 1][2 * (q & 1) + 1] = pack_bf16(v[2], v[3]);
    };
    auto store_tile = [&](bf16x8 *image, int tile, const u32x4 (&v)[2]) {
#pragma unroll
      for (int c = 0; c < 2; ++c) store_piece(image, img + (2 * tile + c) * 64, v[c]);
    };
    // ---------------- the sum of t dt over the channels (the softmax's Jacobian); dphi is formed again below: it has no room beside t
    // (slices are summed apart, so that inv^p meets a sum and not every term)
    float ip[PC ? PC : 1], dot = 0.f;                     // inv^1 ..
    ip[0] = inv;
#pragma unroll
    for (int i = 1; i < PC; ++i) ip[i] = ip[i - 1] * inv;
    if constexpr (ACT0) {
      float part[PC ? PC : 1];
#pragma unroll
      for (int i = 0; i < PC; ++i) part[i] = 0.f;
      each8([&](auto ic) {
        constexpr int fb = decltype(ic)::value;
        const lds_frag_ptr sl = advance(std::integral_constant<int, STEP_A + fb>{}, STEP_A + fb, true);
        f32x16 acc;
        dphi(sl, fb, acc);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int ex = extra_of(fb, q);
#pragma unroll
          for (int x = 4 * q; x < 4 * q + 4; ++x) part[ex] = __builtin_fmaf(ex ? u[fb][x] * power(u[fb][x], ex) : u[fb][x], acc[x], part[ex]);
        }
      });
#pragma unroll
      for (int i = 0; i < PC; ++i) dot = __builtin_fmaf((float)(i + 1) * ip[i], part[i], dot);
      dot = inv * rs_ * xhalf_sum(dot);                   // (with the factor inv that its product with t has)
    }
    // (the powers are formed again below: kept from here they would be spilled)
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) asm volatile("" : "+v"(u[fb]));
    // ---------------- du (and phi_q / den), a feature block per slab
    u32x4 du[FB][2];
    each8([&](auto ic) {
      constexpr int fb = decltype(ic)::value;
      const lds_frag_ptr sl = advance(std::integral_constant<int, STEP_B + fb>{}, STEP_B + fb, true);
      f32x16 acc;
      dphi(sl, fb, acc);
      u32x4 ph[2];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ex = extra_of(fb, q);
        const float rp = rs_ * ip[PC ? ex : 0], c = rp * (float)(ex + 1);
        float d[4], p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float tv = u[fb][4 * q + j], pw = power(tv, ex);
          const float dt = c * (ex ? pw * acc[4 * q + j] : acc[4 * q + j]);
          if constexpr (ACT0) d[j] = tv * (dt - dot);
          else d[j] = a.act == 1 ? tv * dt : (tv > 0.f ? dt : 0.f);
          p[j] = rp * (ex ? pw * tv : tv);
        }
        put(du[fb], q, d);
        if constexpr (QUERY) put(ph, q, p);
      }
      store_tile(a.du_img, fb, du[fb]);
      if constexpr (QUERY) store_tile(a.phi_img, fb, ph);
    });
    load_x(t + 1 < t_hi ? t + 1 : t);                     // the next tile's rows travel under the products below
    // ---------------- dpre = (W2^T du) [h > 0], a hidden block per slab
    each8([&](auto ic) {
      constexpr int hb = decltype(ic)::value;
      const lds_frag_ptr sl = advance(std::integral_constant<int, STEP_C + hb>{}, STEP_C + hb, true);
      f32x16 acc;
#pragma unroll
      for (int x = 0; x < 16; ++x) acc[x] = 0.f;
      chain(std::integral_constant<int, 12>{}, sl, [](int f) { return f; }, [&](int f) { return __builtin_bit_cast(bf16x8, du[f >> 1][f & 1]); }, acc);
      u32x4 dp[2];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const u16x2 open = u16x2{0, 0} - __builtin_bit_cast(u16x2, (gate[hb >> 1] >> (8 * (hb & 1) + i)) & 0x00010001u);
        dp[i >> 2][i & 3] = pack_bf16(acc[2 * i], acc[2 * i + 1]) & __builtin_bit_cast(unsigned, open);
      }
      store_tile(a.dpre_img, hb, dp);
    });
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(xf[ks]));   // (likewise: ahead of the next tile's requests)
    bh = bh_next;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // nothing may still be on its way into this workgroup's LDS
}


// ------------------------------------------------------------------------------------------------
// contract256_kernel: 8 waves, one workgroup per (product, batch and head, range of 128-token tiles).  Both operands go straight from
// HBM into a ring of NST blocks in LDS (direct-to-LDS loads, one barrier per block) in the images' own order (a 1 KiB chunk is 16 channels
// of 32 tokens, 16 bytes per token and lane group) or as rows.  The token-contiguous fragments come out through transposing reads: four
// consecutive channels of a token are 8 contiguous bytes in both.  Lane slot r of an image's chunk holds token r ^ 4 g ^ 8 (chunk % 2), so that the 32 lanes of
// half a read fall on all banks.
// Bound: HBM, every image once (1.0 GB over the queries at 480p / 81 frames, 12 heads: 197 us, three launches of wide_contract_kernel took 300;
// linear keys 102 and 162).  256 x 256 or 256 x 128 outputs per workgroup, so that no operand is read twice.  The tiles are taken in the order
// that finds the last written ones in the 256 MB memory-side cache: 250 -> 236 and 127 -> 118 us against ascending order, and
// read non-temporally, so that what has been used makes no room at the cost of what has not (ONCE): 197 and 102 us, 5.2 TB/s.  All fragments of a
// block requested at once, whole rows per request and an uneven offset between the images changed nothing.
struct Contract256Args {
  const bf16x8 *du, *h, *dpre, *phi;  // images [B*H][n_tb][8][2][64]
  const __bf16 *x_img;                // x in bf16 [B*H][32 n_tb][128], or null:
  const __bf16 *x;                    // rows of q or k
  const __bf16 *gsign;                // [B*H][N][128]
  const float *wp;                    // [B*H][N]
  float *part;
  int H, BH, N, n_tok, n_tb, R, G;
  int n_tiles, run;                   // of back256_kernel
  int nc[3];                          // ranges per (batch, head) of the three products
  int64_t sb, sh, sn;
};
// Tiles per (batch, head) and range: eight row blocks of 256 / 32 (P1) or 128 / 32 (P2, P3) column blocks and an extra one.
constexpr int kTilesP1 = 8 * 9, kTilesP23 = 8 * 5;
static __host__ __device__ inline int64_t part256_base(const int (&nc)[3], int BH, int product) {   // in tiles
  int64_t at = 0;
  if (product > 0) at += (int64_t)BH * nc[0] * kTilesP1;
  if (product > 1) at += (int64_t)BH * nc[1] * kTilesP23;
  if (product > 2) at += (int64_t)BH * nc[2] * kTilesP23;
  return at;
}

// PRODUCT 0: du x [h | 1], wave = 64 rows x 128 columns; 1: dpre x [x | 1], 2: phi x [g | wp], wave = 32 rows x 128 columns.
template <int PRODUCT, bool ONCE>
static __device__ __forceinline__ void contract256(const Contract256Args &a, bf16x8 *ring, float *wcol, int bh, int range) {
  constexpr int NST = 4, ACH = 16, BCH = PRODUCT == 0 ? 16 : 8, STG = (ACH + BCH) * 64;
  constexpr int NRB = PRODUCT == 0 ? 2 : 1, PER = (ACH + BCH) / 8;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // This workgroup's tiles, as back256_kernel numbers them over all heads, and the order they are taken in: those that were written last come
  // first (a tile is number t % run of its writer), while they are still in the memory-side cache.
  const int t_lo = bh * a.n_tiles + (int)((int64_t)range * a.n_tiles / a.nc[PRODUCT]), t_hi = bh * a.n_tiles + (int)((int64_t)(range + 1) * a.n_tiles / a.nc[PRODUCT]);
  int turn = a.run - 1;                                   // next request: block `sub` of tile t, which is number `turn` of its writer
  auto first_of = [&](int n) { return t_lo + (n + a.run - t_lo % a.run) % a.run; };
  int t = first_of(turn), sub = 0;
  auto settle = [&]() {                                   // past the last tile of a turn: on to the one before
    while (t >= t_hi && turn > 0) t = first_of(--turn);
  };
  settle();
  int last = 0;                                           // (past the end: the last block again, which nobody reads)
  auto next_block = [&]() {
    if (t < t_hi) {
      last = (t - bh * a.n_tiles) * 4 + sub;
      if (++sub == 4 || last + 1 == a.n_tb) {
        sub = 0;
        t += a.run;
        settle();
      }
    }
    return last;
  };
  const int n_blocks = min((t_hi - bh * a.n_tiles) * 4, a.n_tb) - (t_lo - bh * a.n_tiles) * 4;
  const bf16x8 *a_img = (PRODUCT == 0 ? a.du : PRODUCT == 1 ? a.dpre : a.phi) + (int64_t)bh * a.n_tb * 1024;
  const LinearMap lmap(a.R, a.G);
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  auto dma = [&](const void *gp, unsigned voff, bf16x8 *to) {
    const unsigned l = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)to);
    if constexpr (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(l), "v"(voff), "s"(gp) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(voff), "s"(gp) : "memory");
  };
  // chunk c of a block: lane slot (g, r) takes the piece of token r ^ 4 g ^ 8 (c % 2)
  const unsigned img_off[2] = {(unsigned)(32 * g + (r ^ (4 * g))) * 16, (unsigned)(32 * g + (r ^ (4 * g) ^ 8)) * 16};
  auto request = [&](int b, int slot) {
    bf16x8 *st = ring + slot * STG;
#pragma unroll
    for (int i = 0; i < ACH / 8; ++i) {
      const int c = 8 * i + w;                            // c % 2 = w % 2
      dma(a_img + ((int64_t)b * ACH + c) * 64, img_off[w & 1], st + c * 64);
    }
    bf16x8 *sb = st + ACH * 64;
    if constexpr (PRODUCT == 0) {
#pragma unroll
      for (int i = 0; i < BCH / 8; ++i) {
        const int c = 8 * i + w;
        dma(a.h + ((int64_t)bh * a.n_tb + b) * 1024 + c * 64, img_off[w & 1], sb + c * 64);
      }
    } else {
      // whole rows: four tokens of 256 bytes per instruction, the 16-byte pieces of a row swizzled by the row (per-lane addresses:
      // a tensor of any stride)
      const int tok = 4 * w + (lane >> 4), i = min(32 * b + tok, a.n_tok - 1);
      const __bf16 *row;
      if constexpr (PRODUCT == 2) row = a.gsign + ((int64_t)bh * a.N + i) * 128;
      else if (a.x_img) row = a.x_img + ((int64_t)bh * a.n_tb * 32 + i) * 128;
      else row = a.x + base + (int64_t)lmap.token(i) * a.sn;
      const __bf16 *piece = row + 8 * ((lane & 15) ^ RowTile<128>::sw(tok));
      const unsigned l = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)(sb + w * 64));
      if constexpr (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(l), "v"(piece) : "memory");
      else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(l), "v"(piece) : "memory");
      if constexpr (PRODUCT == 2) {
        if (w == 0) {                                     // the extra column's 32 values (twice)
          const float *src = a.wp + (int64_t)bh * a.N + min(32 * b + r, a.n_tok - 1);
          const unsigned lw = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)(wcol + slot * 64));
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lw), "v"(src) : "memory");
        }
      }
    }
  };
  // transposing reads (see ds_read_tr): lane = (group tm, row ti, columns ta); tokens 16 kk + 8 tg + 4 jj + ti, channels 16 c + 4 ta .. + 3.  In an
  // image these are 8 bytes at 512 (ta % 2) + 8 (ta / 2) of chunk c, in rows half of piece 2 c + ta / 2.
  const int tm = lane >> 4, ti = (lane >> 2) & 3, ta = lane & 3, tg = tm >> 1, ch = tm & 1;
  int off_a[2][2], off_r[4];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
      off_a[kk][jj] = 1024 * ch + 512 * (ta & 1) + (((16 * kk + 8 * tg + 4 * jj + ti) ^ (4 * (ta & 1)) ^ (8 * ch)) << 4) + 8 * (ta >> 1);
#pragma unroll
  for (int i = 0; i < 4; ++i)                             // (the swizzle depends on ti alone)
    off_r[i] = (8 * tg + ti) * 256 + (((4 * i + 2 * ch + (ta >> 1)) ^ RowTile<128>::sw(ti)) << 4) + 8 * (ta & 1);
  const int row0 = PRODUCT == 0 ? 2 * (w & 3) : w, col0 = PRODUCT == 0 ? 4 * (w >> 2) : 0;
  const bool extra = PRODUCT != 0 || w < 4;               // who sums the extra column
  f32x16 acc[NRB][5];
#pragma unroll
  for (int e = 0; e < NRB; ++e)
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
      for (int x = 0; x < 16; ++x) acc[e][i][x] = 0.f;
  const __bf16 one = static_cast<__bf16>(r == 0 ? 1.0f : 0.0f);
  const bf16x8 ones = bf16x8{one, one, one, one, one, one, one, one};
  constexpr int FLY = (NST - 2) * PER;                    // requests of the newer blocks that may stay in flight
  if (n_blocks > 0) {
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) request(next_block(), s);
    int slot = 0;
    for (int n = 0; n < n_blocks; ++n) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FLY) : "memory");
      __syncthreads();                                    // the block is in place, the one before has been read
      request(next_block(), (slot + NST - 1) & (NST - 1));
      const char *at_ = reinterpret_cast<const char *>(ring + slot * STG), *bt = at_ + ACH * 1024;
      // all fragments of the block ahead of its products: one LDS round trip per block
      bf16x8 af[2][NRB], bf[2][4], ex[2] = {ones, ones};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int e = 0; e < NRB; ++e)
          af[kk][e] = join(ds_read_tr(at_, off_a[kk][0] + (row0 + e) * 2048), ds_read_tr(at_, off_a[kk][1] + (row0 + e) * 2048));
#pragma unroll
        for (int i = 0; i < 4; ++i)
          bf[kk][i] = PRODUCT == 0 ? join(ds_read_tr(bt, off_a[kk][0] + (col0 + i) * 2048), ds_read_tr(bt, off_a[kk][1] + (col0 + i) * 2048))
                                   : join(ds_read_tr(bt, off_r[i] + 16 * kk * 256), ds_read_tr(bt, off_r[i] + (16 * kk + 4) * 256));
        if constexpr (PRODUCT == 2) {                     // columns 0 and 1: the hi and lo parts of the factor
          const f32x4 *src = reinterpret_cast<const f32x4 *>(wcol + slot * 64 + 16 * kk + 8 * g);
          const f32x4 w0 = src[0], w1 = src[1];
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const float v = t < 4 ? w0[t & 3] : w1[t & 3];
            const __bf16 hi = static_cast<__bf16>(v);
            ex[kk][t] = r == 0 ? hi : static_cast<__bf16>(r == 1 ? v - static_cast<float>(hi) : 0.f);
          }
        }
      }
      HA_FENCE();
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int e = 0; e < NRB; ++e) acc[e][i] = mfma32(af[kk][e], bf[kk][i], acc[e][i]);
        if (extra)
#pragma unroll
          for (int e = 0; e < NRB; ++e) acc[e][4] = mfma32(af[kk][e], ex[kk], acc[e][4]);
      }
      slot = (slot + 1) & (NST - 1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing may still be on its way into this workgroup's LDS
  }
  constexpr int NCB = PRODUCT == 0 ? 9 : 5, TILES = 8 * NCB;
  float *dst = a.part + (part256_base(a.nc, a.BH, PRODUCT) + ((int64_t)bh * a.nc[PRODUCT] + range) * TILES) * 1024;
#pragma unroll
  for (int e = 0; e < NRB; ++e)
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      if (i == 4 && !extra) continue;
      float *tile = dst + (int64_t)((row0 + e) * NCB + (i < 4 ? col0 + i : NCB - 1)) * 1024;
#pragma unroll
      for (int x = 0; x < 16; ++x) tile[x * 64 + lane] = acc[e][i][x];
    }
}

template <bool ONCE>
__global__ __launch_bounds__(512, 2) void contract256_kernel(Contract256Args a) {
  __shared__ bf16x8 ring[4 * 32 * 64];
  __shared__ __align__(16) float wcol[4 * 64];
  const int per = a.nc[0] + a.nc[1] + a.nc[2];
  const int bh = blockIdx.x / per, j = blockIdx.x % per;
  if (j < a.nc[0]) contract256<0, ONCE>(a, ring, wcol, bh, j);
  else if (j < a.nc[0] + a.nc[1]) contract256<1, ONCE>(a, ring, wcol, bh, j - a.nc[0]);
  else contract256<2, ONCE>(a, ring, wcol, bh, j - a.nc[0] - a.nc[1]);
}

// ------------------------------------------------------------------------------------------------
// reduce256_kernel: grid (4 (72 + 40 [+ 40]), max(H, [B*H])), a thread per element of the partial tiles.  dW, db: sums over the ranges of
// every batch entry of head blockIdx.y; dS, dz: of (batch, head) blockIdx.y.
struct Reduce256Args {
  const float *part;
  float *w2, *b2, *w1, *b1;
  __bf16 *ds_hi, *ds_lo;
  float *dz;
  int B, H;
  int nc[3];
};
__global__ __launch_bounds__(256) void reduce256_kernel(Reduce256Args a) {
  int e = blockIdx.x * 256 + threadIdx.x;
  const int product = e < kTilesP1 * 1024 ? 0 : e < (kTilesP1 + kTilesP23) * 1024 ? 1 : 2;
  if (product > 0) e -= kTilesP1 * 1024;
  if (product > 1) e -= kTilesP23 * 1024;
  const int ncb = product == 0 ? 9 : 5, tiles = 8 * ncb, nc = a.nc[product];
  const int tile = e >> 10, x = (e >> 6) & 15, r = e & 31, g = (e >> 5) & 1;
  const int row = 32 * (tile / ncb) + crow(x, g), cb = tile % ncb;
  const bool is_extra = cb == ncb - 1;
  if (is_extra && r != 0) return;
  const int y = blockIdx.y, n_sum = product == 2 ? 1 : a.B;
  if (product != 2 && y >= a.H) return;
  const bool two = is_extra && product == 2;             // the hi and the lo part
  float sum = 0.f;
  for (int b = 0; b < n_sum; ++b) {
    const float *src = a.part + (part256_base(a.nc, a.B * a.H, product) + (int64_t)(product == 2 ? y : b * a.H + y) * nc * tiles) * 1024 + e;
    int c = 0;
    for (; c + 4 <= nc; c += 4) {                         // four loads in flight, added in order
      float v[4], u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = src[(int64_t)(c + i) * tiles * 1024];
        u[i] = two ? src[(int64_t)(c + i) * tiles * 1024 + 1] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) sum += v[i] + u[i];
    }
    for (; c < nc; ++c) sum += src[(int64_t)c * tiles * 1024] + (two ? src[(int64_t)c * tiles * 1024 + 1] : 0.f);
  }
  const int col = 32 * cb + r;
  if (product == 0) {
    if (is_extra) a.b2[y * 256 + row] = sum;
    else a.w2[((int64_t)y * 256 + row) * 256 + col] = sum;
  } else if (product == 1) {
    if (is_extra) a.b1[y * 256 + row] = sum;
    else a.w1[((int64_t)y * 256 + row) * 128 + col] = sum;
  } else if (is_extra) {
    a.dz[y * 256 + row] = sum;
  } else {                                                // natural order: [row block][16-column step][lane][8]
    const int64_t at = (int64_t)y * 256 * 128 + ((((row >> 5) * 8 + (col >> 4)) * 64 + 32 * ((col >> 3) & 1) + (row & 31)) << 3) + (col & 7);
    const __bf16 hi = static_cast<__bf16>(sum);
    a.ds_hi[at] = hi;
    a.ds_lo[at] = static_cast<__bf16>(sum - static_cast<float>(hi));
  }
}

// ------------------------------------------------------------------------------------------------
// prep256_kernel: 2 H + B*H rows of 32 blocks, in one dimension (they may be more than a second one takes), a thread per 16-byte piece.  Rows 0 .. 2 H - 1: one head's map (queries first) as fragments of W1 (4096 pieces),
// W2 (8192) and W2^T; the rest: S as hi + lo fragments in natural order.
struct Prep256Args {
  const void *w1[2], *w2[2];
  bf16x8 *w1f[2], *w2f[2], *w2tf[2];
  const float *S;
  bf16x8 *s_hi, *s_lo;
  int H;
};
template <bool F32>
__global__ __launch_bounds__(256) void prep256_kernel(Prep256Args a) {
  const int y = blockIdx.x >> 5, p = (blockIdx.x & 31) * 256 + threadIdx.x;
  if (y < 2 * a.H) {
    const int side = y >= a.H, h = side ? y - a.H : y;
    if (p < 4096) a.w1f[side][(int64_t)h * 4096 + p] = weight_piece<F32, false>(a.w1[side], (int64_t)h * 256 * 128, 128, p);
    if (p < 8192) a.w2f[side][(int64_t)h * 8192 + p] = weight_piece<F32, true>(a.w2[side], (int64_t)h * 256 * 256, 256, p);
    // W2^T: [hidden block][feature block][s][lane][t] = W2[32 fb + crow(8 s + t, g)][32 hb + r]
    if (p < 8192) {
      const int lane = p & 63, r = lane & 31, g = lane >> 5, s = (p >> 6) & 1, fb = (p >> 7) & 7, hb = p >> 10;
      bf16x8 v;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int64_t at = ((int64_t)h * 256 + 32 * fb + crow(8 * s + t, g)) * 256 + 32 * hb + r;
        if constexpr (F32) v[t] = static_cast<__bf16>(static_cast<const float *>(a.w2[side])[at]);
        else v[t] = static_cast<const __bf16 *>(a.w2[side])[at];
      }
      a.w2tf[side][(int64_t)h * 8192 + p] = v;
    }
  } else if (p < 4096) {
    const int bh = y - 2 * a.H, lane = p & 63, r = lane & 31, g = lane >> 5, ks = (p >> 6) & 7, rb = p >> 9;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(a.S + ((int64_t)bh * 256 + 32 * rb + r) * 128 + 16 * ks + 8 * g);
    const f32x4 s0 = src[0], s1 = src[1];
    bf16x8 hi, lo;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float v = t < 4 ? s0[t & 3] : s1[t & 3];
      hi[t] = static_cast<__bf16>(v);
      lo[t] = static_cast<__bf16>(v - static_cast<float>(hi[t]));
    }
    a.s_hi[(int64_t)bh * 4096 + p] = hi;
    a.s_lo[(int64_t)bh * 4096 + p] = lo;
  }
}

// ------------------------------------------------------------------------------------------------
// host side

template <typename T>
static inline T *ws_ptr(void *ws, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(ws) + off); }

void make_grad256_plan(const Plan &pl, size_t base_off, Grad256Plan &gp) {
  const size_t BH = (size_t)pl.B * pl.H, F = 256, D = 128;
  gp.n_tb[0] = (pl.N + 31) / 32;
  gp.n_tb[1] = (pl.NL + 31) / 32;
  // Ranges of the products: 256 workgroups shared in proportion to the bytes per token (image pairs 1024, image and rows 768), at least one
  // tile of 128 tokens each
  size_t part = 0;
  for (int side = 0; side < 2; ++side) {
    const int bytes[3] = {4, 3, side == 0 ? 3 : 0};
    int (&nc)[3] = gp.nc[side];
    int left = 256 / (int)BH;
    const int most = (gp.n_tb[side] + 3) / 4;
    for (int p = 0; p < 3; ++p) nc[p] = bytes[p] ? 1 : 0;
    left -= side == 0 ? 3 : 2;
    while (left-- > 0) {
      int worst = -1;
      for (int p = 0; p < 3; ++p)
        if (bytes[p] && nc[p] < most && (worst < 0 || bytes[p] * nc[worst] > bytes[worst] * nc[p])) worst = p;
      if (worst < 0) break;
      ++nc[worst];
    }
    const size_t bytes_side = (size_t)part256_base(nc, (int)BH, 3) * 4096;
    if (bytes_side > part) part = bytes_side;
  }
  // The partial tiles take the workspace from its start: the forward's part of it (S and z last, in the query side's pass) and the
  // query side's operands are spent when the first product is formed.  Behind these only what does not fit there, so that the whole is never more
  // than the layer-by-layer passes asked for (B = H = 1, N = 64: 2.02 of 2.24 MiB, 2.61 with a place of their own; 12 heads, 32760 tokens: 1.14 of 2.16 GiB).
  size_t off = base_off;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~static_cast<size_t>(255); return o; };
  gp.off_part = 0;
  for (int side = 0; side < 2; ++side) {
    gp.off_w1[side] = take((size_t)pl.H * F * D * 2);
    gp.off_w2[side] = take((size_t)pl.H * F * F * 2);
    gp.off_w2t[side] = take((size_t)pl.H * F * F * 2);
    gp.off_mhi[side] = take(BH * F * D * 2);
    gp.off_mlo[side] = take(BH * F * D * 2);
    if (side == 0 && off < part) off = part;              // (whole tiles of 4 KiB)
  }
  gp.off_dz = take(BH * F * 4);
  gp.off_gsign = take(BH * pl.N * D * 2);
  gp.off_rs = take(BH * pl.N * 4);
  gp.off_wp = take(BH * pl.N * 4);
  const size_t image = (BH * gp.n_tb[0] + 1) * 32 * F * 2;           // (the key side has no more blocks; one more that nobody reads)
  gp.off_h = take(image);
  gp.off_du = take(image);
  gp.off_dpre = take(image);
  gp.off_phi = take(image);
  gp.off_x = take(pl.f32 ? image / 2 : 0);
  gp.total = off;
}

hipError_t launch_value_distill_backward256(const Plan &pl, const Grad256Plan &gp, const void *q, const void *k, const void *v,
                                            const ha_feature_map &phi_q, const ha_feature_map &phi_k, const void *y_teacher,
                                            const void *y_student, const float *row_den, const ha_feature_map_grad &gq,
                                            const ha_feature_map_grad &gk, void *ws, hipStream_t st, double *l1_partial, double *loss) {
  const int BH = pl.B * pl.H;
  hipError_t e;
  if ((e = launch_vd_rows(pl, y_teacher, y_student, row_den, ws_ptr<void>(ws, gp.off_gsign), ws_ptr<float>(ws, gp.off_rs),
                          ws_ptr<float>(ws, gp.off_wp), st, l1_partial, loss)) != hipSuccess)
    return e;
  Prep256Args pa;
  for (int side = 0; side < 2; ++side) {
    pa.w1[side] = side == 0 ? phi_q.w1 : phi_k.w1;
    pa.w2[side] = side == 0 ? phi_q.w2 : phi_k.w2;
    pa.w1f[side] = ws_ptr<bf16x8>(ws, gp.off_w1[side]);
    pa.w2f[side] = ws_ptr<bf16x8>(ws, gp.off_w2[side]);
    pa.w2tf[side] = ws_ptr<bf16x8>(ws, gp.off_w2t[side]);
  }
  pa.S = ws_ptr<float>(ws, pl.off_S);
  pa.s_hi = ws_ptr<bf16x8>(ws, gp.off_mhi[0]);
  pa.s_lo = ws_ptr<bf16x8>(ws, gp.off_mlo[0]);
  pa.H = pl.H;
  if (pl.f32) prep256_kernel<true><<<32 * (2 * pl.H + BH), 256, 0, st>>>(pa);
  else prep256_kernel<false><<<32 * (2 * pl.H + BH), 256, 0, st>>>(pa);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int side = 0; side < 2; ++side) {
    const bool is_query = side == 0;
    const ha_feature_map &fm = is_query ? phi_q : phi_k;
    const ha_feature_map_grad &gm = is_query ? gq : gk;
    const int n_tok = is_query ? pl.N : pl.NL;
    Back256Args a;
    a.x = is_query ? q : k;
    a.u = is_query ? ws_ptr<void>(ws, gp.off_gsign) : v;
    a.rs = ws_ptr<float>(ws, gp.off_rs);
    a.wp = ws_ptr<float>(ws, gp.off_wp);
    a.w1f = ws_ptr<bf16x8>(ws, gp.off_w1[side]);
    a.w2f = ws_ptr<bf16x8>(ws, gp.off_w2[side]);
    a.w2tf = ws_ptr<bf16x8>(ws, gp.off_w2t[side]);
    a.b1 = fm.b1;
    a.b2 = fm.b2;
    a.m_hi = ws_ptr<bf16x8>(ws, gp.off_mhi[side]);
    a.m_lo = ws_ptr<bf16x8>(ws, gp.off_mlo[side]);
    a.zvec = is_query ? ws_ptr<float>(ws, pl.off_z) : ws_ptr<float>(ws, gp.off_dz);
    a.h_img = ws_ptr<bf16x8>(ws, gp.off_h);
    a.du_img = ws_ptr<bf16x8>(ws, gp.off_du);
    a.dpre_img = ws_ptr<bf16x8>(ws, gp.off_dpre);
    a.phi_img = ws_ptr<bf16x8>(ws, gp.off_phi);
    a.x_img = ws_ptr<__bf16>(ws, gp.off_x);
    a.H = pl.H; a.N = pl.N; a.n_tok = n_tok; a.n_tb = gp.n_tb[side]; a.R = is_query ? 0 : pl.R; a.G = pl.G; a.P = pl.P;
    a.act = is_query ? pl.act_q : pl.act_k;
    a.sb = pl.sb; a.sh = pl.sh; a.sn = pl.sn;
    a.n_tiles = (n_tok + 127) / 128;
    a.total = a.n_tiles * BH;
    a.run = (a.total + 511) / 512;                        // two workgroups per CU
    const int nwg = ((a.total + a.run - 1) / a.run + 7) / 8 * 8;
#define HA_BACK256(F32, QUERY, ACT0, PC) back256_kernel<F32, QUERY, ACT0, PC><<<nwg, 256, 0, st>>>(a)
#define HA_BACK256_MAP(F32, QUERY) \
  do { \
    if (a.act != HA_ACT_SOFTMAX) HA_BACK256(F32, QUERY, false, 0); \
    else if (pl.P == 1) HA_BACK256(F32, QUERY, true, 1); \
    else if (pl.P == 2) HA_BACK256(F32, QUERY, true, 2); \
    else if (pl.P == 4) HA_BACK256(F32, QUERY, true, 4); \
    else HA_BACK256(F32, QUERY, true, 8); \
  } while (0)
    if (is_query) { if (pl.f32) HA_BACK256_MAP(true, true); else HA_BACK256_MAP(false, true); }
    else { if (pl.f32) HA_BACK256_MAP(true, false); else HA_BACK256_MAP(false, false); }
#undef HA_BACK256_MAP
#undef HA_BACK256
    if ((e = hipGetLastError()) != hipSuccess) return e;
    Contract256Args c;
    c.du = a.du_img; c.h = a.h_img; c.dpre = a.dpre_img; c.phi = a.phi_img;
    c.x_img = pl.f32 ? a.x_img : nullptr;
    c.x = static_cast<const __bf16 *>(a.x);
    c.gsign = ws_ptr<__bf16>(ws, gp.off_gsign);
    c.wp = a.wp;
    c.part = ws_ptr<float>(ws, gp.off_part);
    c.H = pl.H; c.BH = BH; c.N = pl.N; c.n_tok = n_tok; c.n_tb = a.n_tb; c.n_tiles = a.n_tiles; c.run = a.run; c.R = a.R; c.G = a.G;
    c.sb = pl.sb; c.sh = pl.sh; c.sn = pl.sn;
    for (int p = 0; p < 3; ++p) c.nc[p] = gp.nc[side][p];
    // Images of more than a quarter of the memory-side cache are read non-temporally.  12 heads, both forms in turn, the whole step:
    // 38 MB of them over the queries 208 us (non-temporal 213), 123 MB 348 (342), 1.0 GB 2702 (2665).
    const int64_t image_bytes = (int64_t)BH * a.n_tb * 32 * 512 * (is_query ? 4 : 3);
    const dim3 grid(BH * (c.nc[0] + c.nc[1] + c.nc[2]));
    if (image_bytes > kMemorySideCache / 4) contract256_kernel<true><<<grid, 512, 0, st>>>(c);
    else contract256_kernel<false><<<grid, 512, 0, st>>>(c);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    Reduce256Args ra;
    ra.part = c.part;
    ra.w2 = gm.w2; ra.b2 = gm.b2; ra.w1 = gm.w1; ra.b1 = gm.b1;
    ra.ds_hi = ws_ptr<__bf16>(ws, gp.off_mhi[1]);
    ra.ds_lo = ws_ptr<__bf16>(ws, gp.off_mlo[1]);
    ra.dz = ws_ptr<float>(ws, gp.off_dz);
    ra.B = pl.B; ra.H = pl.H;
    for (int p = 0; p < 3; ++p) ra.nc[p] = c.nc[p];
    reduce256_kernel<<<dim3(4 * (kTilesP1 + kTilesP23 * (is_query ? 2 : 1)), is_query ? BH : pl.H), 256, 0, st>>>(ra);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ha
